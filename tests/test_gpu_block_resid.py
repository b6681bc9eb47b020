"""Residual projections of many rows in 256-row blocks with K slices, against the oracle: slices of unequal length, feature counts that leave the
last block partly filled, one to four row blocks, the sums of squares that the next projection takes."""
import pytest

from paper_2507_02620_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,ffn,rows,taken", [
    (512, 1536, 400, True),     # 48 k-tiles in two slices; two feature blocks, two row blocks
    (672, 2336, 513, True),     # 73 k-tiles in three slices of 24, 24 and 25; 42 feature tiles; a third row block of one row
    (1056, 1600, 1000, True),   # 50 k-tiles; five feature blocks over the XCDs
    (256, 6176, 385, True),     # one feature block, 193 k-tiles in eight slices
    (512, 1504, 400, False),    # 47 k-tiles: no slices of 24
])
def test_residual_projection_in_256_row_blocks(d, ffn, rows, taken, monkeypatch):
    from tests.gpu_util import TOL, Pair, kernel_names, max_rel_err, to_dev
    monkeypatch.setenv("FLOWSPEC_BLOCK_GEMM", "1")   # without the estimates, which choose it for larger matrices
    cfg = synth.StageConfig(f"block-resid-{d}-{rows}", "bf16", 2, d, 4, 2, 64, ffn, 0, 20, rows, rows, 6, 3)
    print(f"[case] {cfg}", flush=True)
    pair = Pair(cfg, seed=rows)
    tree = synth.config_tree(cfg, seed=rows)
    hid = synth.hidden(cfg, tree.size, 0, rows)
    o, g = pair.verify_tree(tree.parent, hid, rows)
    err = max_rel_err(g, o)
    kv_err = max_rel_err(pair.kv[1, :, :, 20:20 + rows].float().cpu().numpy(), pair.orc.kv[1, :, :, 20:20 + rows])
    print(f"  hidden {err:.2e}, K/V of the second layer {kv_err:.2e}", flush=True)
    assert err < TOL["bf16"] and kv_err < TOL["bf16"]
    x = to_dev(hid, pair.tdtype)
    names = kernel_names(lambda: pair.gpu.tree_verify_stage(pair.kv, 20, 20, x, 0, tree.parent))
    assert any("block_gemm_kernel<1" in n or "block_gemm_kernelILi1" in n for n in names) == taken, names
    if not taken:   # the same projections in 128-row blocks with K slices
        assert any("wide_gemm_kernel<1, true" in n or "wide_gemm_kernelILi1ELb1" in n for n in names), names
