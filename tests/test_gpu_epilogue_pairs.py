"""QKV and gate/up epilogues that store two items of a wave together: four and six feature tiles per wave (pairs that begin on the wave's first
and on its third tile), query, key and value heads of 64 and 128 features, biases, padding tiles, ragged rows; against the oracle."""
import pytest

from paper_2507_02620_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,kv,hd,rows,block,bias", [
    (6, 3, 64, 385, 1, True), (6, 3, 64, 385, 2, True), (5, 1, 128, 400, 1, False), (5, 1, 128, 400, 2, True),   # 256-row blocks of 16 and 12 tiles
    (6, 3, 64, 385, 0, True), (3, 3, 128, 513, 0, False),                                                        # 128-row blocks, four tiles per wave
    (192, 48, 64, 40, -1, True), (96, 24, 128, 100, -1, False),   # streamed, six tiles per wave
    (192, 192, 64, 50, -1, True), (20, 10, 128, 90, -1, True),    # streamed, four tiles per wave
])
def test_two_items_in_one_store(heads, kv, hd, rows, block, bias, monkeypatch):
    from tests.gpu_util import TOL, Pair, max_rel_err
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
