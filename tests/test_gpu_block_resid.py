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


@pytest.mark.parametrize("d,ffn,rows,taken", [
    (4608, 256, 769, 0), (4608, 256, 850, 0),   # output projection in 504 128-row blocks of 36 k-tiles: two rounds that overlap
    (4608, 256, 960, 1),                        # in 144
    (4608, 12288, 900, 2),                      # the same, and the down projection in 432 blocks of 128 k-tiles
])
def test_residual_projection_takes_the_shorter_form(d, ffn, rows, taken):
    """Which of the layer's two residual projections go into 256-row blocks by the estimates."""
    import numpy as np
    import torch
    from paper_2507_02620_amd import flowspec as fs
    from tests.gpu_util import kernel_names
    w = lambda n, k: torch.randn(n, k, device="cuda").mul_(0.02).bfloat16()  # noqa: E731
    ones = torch.ones(d, dtype=torch.bfloat16, device="cuda")
    layer = dict(rms_attn=ones, rms_ffn=ones, wq=w(d, d), wk=w(128, d), wv=w(128, d), wo=w(d, d), w_gate=w(ffn, d), w_up=w(ffn, d), w_down=w(d, ffn))
    st = fs.Stage(n_layers=1, d_model=d, n_q_heads=d // 128, n_kv_heads=1, head_dim=128, d_ffn=ffn, vocab=0, dtype=fs.FS_BF16, rms_eps=1e-5, rope_theta=1e4,
                  kv_capacity=rows, max_tree=rows, max_seg=rows, layers=[layer])
    kv, x, out = st.new_kv_cache(), w(rows, d), torch.empty(rows, d, dtype=torch.bfloat16, device="cuda")
    parent = np.arange(-1, rows - 1, dtype=np.int32)
    print(f"[case] {d} x {ffn}, {rows} rows", flush=True)
    names = kernel_names(lambda: st.tree_verify_stage(kv, 0, 0, x, 0, parent, out))
    assert sum("block_gemm_kernel<1" in n or "block_gemm_kernelILi1" in n for n in names) == taken, names
    st.close()
