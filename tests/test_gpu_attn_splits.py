"""Tree attention of few KV heads at the ends of the rule on how many KV splits a context goes into, against the oracle; the plan's own numbers
are checked in test_launch_rules.py."""
import pytest

from paper_2507_02620_amd import synth
from tests.test_gpu_parity import _check_stage

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,kv,hd,rows", [(8, 4, 128, 16), (4, 4, 64, 5), (6, 2, 128, 7), (16, 4, 128, 16), (32, 8, 128, 13), (16, 4, 128, 12)])
@pytest.mark.parametrize("slots", [28 * 64, 28 * 64 + 1, 33 * 64 - 1, 65 * 64, 128 * 64, 128 * 64 + 1])
def test_splits_of_few_kv_heads(heads, kv, hd, rows, slots):
    """28 and 29 tiles, an odd number of them, more than 64 (32 splits of several), 128 and 129; (2 KV heads: the rule does not apply;
    four row tiles of 4 and 8 KV heads: the direct-to-LDS kernel in that range, three: not)."""
    from tests.gpu_util import kernel_names
    cfg = synth.StageConfig(f"splits-{hd}-{slots}", "bf16", 1, 128, heads, kv, hd, 256, 0, slots - rows, rows, rows, 6, 3)
    names = kernel_names(lambda: _check_stage(cfg, slots, rows))
    dma = hd == 128 and kv >= 4 and 48 < heads // kv * rows <= 64 and 28 * 64 < slots <= 128 * 64
    assert any("tree_attn_dma_kernel<2," in n or "tree_attn_dma_kernelILi2E" in n for n in names) == dma, names
    assert any("tree_attn_kernel" in n for n in names) != dma and any("attn_merge_kernel" in n for n in names), names


@pytest.mark.parametrize("heads,kv,specs", [
    # (context, tree, depth, branching, offset of the segment, its rows): 6 and 8 KV heads with the requests, four row tiles and fewer; the
    # shorter requests have splits without a tile
    (8, 2, [(7000, 20, 5, 3, 4, 16), (300, 20, 5, 3, 0, 13), (3011, 20, 5, 3, 3, 5)]),
    (8, 2, [(64, 20, 5, 3, 0, 16), (2500, 24, 5, 3, 8, 16), (5, 20, 5, 3, 0, 1), (1999, 20, 5, 3, 4, 16)]),
])
def test_few_kv_heads_in_a_ragged_batch(heads, kv, specs):
    from tests.gpu_util import TOL, kernel_names, max_rel_err
    from tests.test_gpu_batch import _run_batch
    cfg = synth.StageConfig(f"splits-b-{len(specs)}", "bf16", 1, 128, heads, kv, 128, 256, 0, max(s[0] for s in specs), 32, 64, 5, 3)
    print(f"[case] {cfg.name}: {specs}", flush=True)
    runs = []
    names = kernel_names(lambda: runs.append(_run_batch(cfg, specs, seed=5)))
    got, want, _, _ = runs[-1]
    row = 0
    for w in want:
        assert max_rel_err(got[row:row + w.shape[0]], w) < TOL["bf16"]
        row += w.shape[0]
    assert any("tree_attn_dma_kernel<2," in n or "tree_attn_dma_kernelILi2E" in n for n in names), names
