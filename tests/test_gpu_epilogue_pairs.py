"""QKV and gate/up epilogues that store two items of a wave together: four and six feature tiles per wave (pairs that begin on the wave's first
and on its third tile), query, key and value heads of 64 and 128 features, biases, padding tiles, ragged rows; against the oracle."""
import pytest

from paper_2507_02620_amd import synth

pytestmark = pytest.mark.gpu


# the QKV kernels: rows and tiles per wave are the last arguments but one and two
_BLOCK16, _BLOCK12, _WIDE = "block_gemm_kernel<0, false, 2, 4, 8, 4, 4>", "block_gemm_kernel<0, false, 4, 2, 4, 6, 4>", "wide_gemm_kernel<0, false, 8, 4, 4, false>"
_STREAM6A, _STREAM6B, _STREAM4 = "stream_gemm_kernel<0, false, 2, 1, 2, 2, 6, 6>", "stream_gemm_kernel<0, false, 2, 1, 2, 4, 6, 4>", "stream_gemm_kernel<0, false, 4, 1, 2, 2, 4, 6>"


@pytest.mark.parametrize("heads,kv,hd,rows,block,bias,qkv", [
    (6, 3, 64, 385, 1, True, _BLOCK16), (6, 3, 64, 385, 2, True, _BLOCK12),        # 256-row blocks of 16 tiles, four per wave, and of 12, six
    (5, 1, 128, 400, 1, False, _BLOCK16), (5, 1, 128, 400, 2, True, _BLOCK12),
    (6, 3, 64, 385, 0, True, _WIDE), (3, 3, 128, 513, 0, False, _WIDE),            # 128-row blocks, four tiles per wave
    (192, 48, 64, 40, -1, True, _STREAM6A), (96, 24, 128, 100, -1, False, _STREAM6B), (192, 192, 64, 50, -1, True, _STREAM6A),   # streamed, six
    (20, 10, 128, 90, -1, True, _STREAM4),                                         # streamed, four
])
def test_two_items_in_one_store(heads, kv, hd, rows, block, bias, qkv, monkeypatch):
    from tests.gpu_util import TOL, Pair, kernel_names, max_rel_err, to_dev
    if block >= 0:
        monkeypatch.setenv("FLOWSPEC_BLOCK_GEMM", str(block))
    cfg = synth.StageConfig(f"pairs-{heads}x{hd}-{rows}", "bf16", 2, 64, heads, kv, hd, 1120, 0, 37, rows + 3, rows, 6, 3, qkv_bias=bias)
    print(f"[case] {cfg}", flush=True)
    pair = Pair(cfg, seed=rows)
    tree = synth.config_tree(cfg, seed=rows)
    hid = synth.hidden(cfg, tree.size, 0, rows)
    o, g = pair.verify_tree(tree.parent, hid, rows)
    L = cfg.l_glo + tree.size
    got = pair.kv[:, :, :, cfg.l_glo:L].float().cpu().numpy()
    err = max_rel_err(g, o)
    kv_err = max(max_rel_err(got[l, c], pair.orc.kv[l, c, :, cfg.l_glo:L]) for l in range(2) for c in range(2))
    print(f"  hidden {err:.2e}, K/V {kv_err:.2e}", flush=True)
    assert err < TOL["bf16"] and kv_err < TOL["bf16"]
    x = to_dev(hid[:rows], pair.tdtype)
    names = kernel_names(lambda: pair.gpu.tree_verify_stage(pair.kv, cfg.l_glo, cfg.l_glo, x, 0, tree.parent[:rows]))
    assert any(qkv in n for n in names), names
