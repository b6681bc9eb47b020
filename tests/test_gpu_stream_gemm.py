"""The projection kernel for 17 to 128 rows (both operands streamed through LDS) against the oracle: row counts at the edges of its
row blocks, K ranges of an odd number of k-tiles and shorter than the ring of stage buffers, K slices, feature counts that leave
the last block partly filled, row-major and fragment-major activations."""
import numpy as np
import pytest

from paper_2507_02620_amd import synth

pytestmark = pytest.mark.gpu


def _check(cfg, rows):
    import torch
    from tests.gpu_util import TOL, Pair, max_rel_err, to_dev
    print(f"[case] {cfg.name}", flush=True)
    pair = Pair(cfg, seed=rows, head=True)
    tree = synth.config_tree(cfg, seed=rows)
    hid = synth.hidden(cfg, tree.size, 0, rows)
    o, g = pair.verify_tree(tree.parent, hid, rows)     # one segment of `rows` rows, then 3 rows
    L = cfg.l_glo + tree.size
    err = max_rel_err(g, o)
    kerr = max_rel_err(pair.kv[:, :, :, cfg.l_glo:L].float().cpu().numpy(), pair.orc.kv[:, :, :, cfg.l_glo:L])
    x = synth.storage(cfg, o[:rows].astype(np.float32))
    lo, _ = pair.orc.logits(x.astype(np.float64))
    lg, _ = pair.gpu.tree_logits(to_dev(x, torch.bfloat16))
    lerr = max_rel_err(lg.cpu().numpy(), lo)
    print(f"  hidden {err:.2e}, K/V {kerr:.2e}, logits {lerr:.2e}", flush=True)
    assert err < TOL["bf16"] and kerr < TOL["bf16"] and lerr < TOL["bf16"]


@pytest.mark.parametrize("rows", [17, 33, 64, 65, 81, 113, 128])
@pytest.mark.parametrize("d,hq,hkv,f,vocab", [
    # blocks of 6 feature tiles: QKV of 1152, gate/up of 1092 tiles (ragged last block), LM head of 1100; the down projection's 273
    # k-tiles and the attention output's 384 take blocks of 8 tiles from 65 rows on (one wave group, one k-tile per stage, 8 buffers), in K
    # slices, the last one shorter; 2 k-tiles elsewhere: fewer stages than buffers
    (64, 96, 24, 8736, 17600),
    # blocks of 8 feature tiles: up to 64 rows gate/up of 1644 tiles (from 33 rows on), LM head of 1600; from 65 rows on gate/up of 3136 tiles;
    # 3 k-tiles, an odd last stage
    (96, 3, 3, 13152, 25600), (96, 3, 3, 25088, 40),
])
def test_blocks_of_six_and_eight_feature_tiles(rows, d, hq, hkv, f, vocab):
    _check(synth.StageConfig(f"stream-wide-{d}-{rows}", "bf16", 2, d, hq, hkv, 128, f, vocab, 37, rows + 3, rows, 6, 3), rows)


@pytest.mark.parametrize("d,hq,hkv,f,rows", [
    # QKV of 1728 tiles: streamed, in 128-row blocks from 65 rows on; gate/up of 1792 tiles: few-row kernel, 64-row, 128-row blocks
    *[(64, 72, 72, 14336, rows) for rows in (32, 33, 64, 65, 128)],
    # QKV of 3072 tiles: few-row kernel, streamed, 128-row blocks; gate/up of 4096 tiles: as above; 1024 k-tiles of the down projection in
    # blocks of 8 feature tiles from 33 rows on
    *[(64, 128, 128, 32768, rows) for rows in (32, 33, 64, 65, 128)],
    (2080, 1, 1, 14336, 17),  # gate/up of 1792 tiles and 65 k-tiles: one 64-row block of 32 rows
    (32, 8, 8, 512, 33), (64, 16, 16, 1056, 64),  # residual projections of 32 and 33 k-tiles: few-row kernel and K slices
])
def test_projections_that_take_another_kernel_at_some_row_counts(d, hq, hkv, f, rows):
    _check(synth.StageConfig(f"mid-{d}-{f}-{rows}", "bf16", 1, d, hq, hkv, 128, f, 40, 37, rows + 3, rows, 6, 3), rows)


@pytest.mark.parametrize("rows", [17, 32, 33, 64, 65, 113, 128])
@pytest.mark.parametrize("d,hq,hkv,hd,f,vocab,bias", [
    (480, 6, 3, 64, 1056, 1000, True),      # 15 and 33 k-tiles (an odd last stage), ragged feature blocks everywhere
    (64, 1, 1, 64, 96, 40, False),          # 2 k-tiles: fewer stages than buffers
    (1024, 64, 2, 128, 6400, 4000, False),  # QKV of 544 tiles through the kernel, gate/up of 800 tiles, several K slices
])
def test_rows_between_one_tile_and_a_block(rows, d, hq, hkv, hd, f, vocab, bias):
    _check(synth.StageConfig(f"stream-{d}-{rows}", "bf16", 2, d, hq, hkv, hd, f, vocab, 37, rows + 3, rows, 6, 3, qkv_bias=bias), rows)
