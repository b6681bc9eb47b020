"""QKV of up to 16 rows with a value tile beside every rotary pair, against the oracle: head counts on either side of the rule, one wave to
eight, odd numbers of k-tiles, biases, both element types, weights in groups of two and of four tiles, row-major and fragment-major rows."""
import pytest

from paper_2507_02620_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,heads,kv,hd,max_seg,rows,bias,taken", [
    ("bf16", 32, 43, 43, 64, 16, 16, True, True),      # 172 pairs: the first number whose groups of two need a second round; one wave
    ("bf16", 64, 42, 42, 64, 16, 16, False, False),    # 168: one round of groups of two
    ("bf16", 96, 22, 22, 128, 16, 1, False, True),     # one row, three waves
    ("bf16", 544, 32, 32, 128, 16, 5, True, True),     # 256 pairs, 17 k-tiles: a wave with one more than the others
    ("bf16", 64, 33, 33, 128, 16, 16, False, False),   # 264 pairs: more than a round of three tiles
    ("bf16", 64, 64, 64, 64, 64, 16, True, True),      # groups of four tiles
    ("bf16", 64, 43, 43, 128, 64, 9, False, True),     # the same, two rounds
    ("bf16", 64, 60, 60, 128, 64, 16, False, False),   # 480 pairs
    ("bf16", 64, 32, 16, 128, 16, 16, False, False),   # fewer value tiles than pairs
    ("bf16", 64, 32, 32, 128, 16, 17, False, False),   # two row tiles
    ("f32", 48, 24, 24, 128, 16, 16, True, True),
    ("f32", 272, 50, 50, 64, 64, 7, False, True),      # 200 pairs, 17 k-tiles
])
def test_value_tile_beside_every_pair(dtype, d, heads, kv, hd, max_seg, rows, bias, taken):
    from tests.gpu_util import TOL, Pair, kernel_names, max_rel_err, to_dev
    cfg = synth.StageConfig(f"qkv-{heads}x{hd}", dtype, 2, d, heads, kv, hd, 256, 0, 37, rows + 3, rows, 6, 3, qkv_bias=bias)
    print(f"[case] {cfg}", flush=True)
    pair = Pair(cfg, seed=rows, max_seg=max(max_seg, rows))
    tree = synth.config_tree(cfg, seed=rows)
    hid = synth.hidden(cfg, tree.size, 0, rows)
    o, g = pair.verify_tree(tree.parent, hid, rows)     # one segment of `rows` rows, then the rest
    L = cfg.l_glo + tree.size
    err = max_rel_err(g, o)
    kv_err = max_rel_err(pair.kv[:, :, :, cfg.l_glo:L].float().cpu().numpy(), pair.orc.kv[:, :, :, cfg.l_glo:L])
    print(f"  hidden {err:.2e}, K/V {kv_err:.2e}", flush=True)
    assert err < TOL[dtype] and kv_err < TOL[dtype]
    x = to_dev(hid[:rows], pair.tdtype)
    names = kernel_names(lambda: pair.gpu.tree_verify_stage(pair.kv, cfg.l_glo, cfg.l_glo, x, 0, tree.parent[:rows]))
    assert any("skinny_qkv_kernel" in n for n in names) == taken, names
    if not taken:   # the QKV form (0) of the kernels in groups of tiles
        assert any("skinny_gemm_kernel" in n and (", 0>(" in n or "Li0EEv" in n) or "stream_gemm_kernel<0," in n for n in names), names
