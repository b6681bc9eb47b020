"""HIP path with 4-bit group weights (W4A16, the paper's 13B setting, Sec. IV-A) against the oracle run on the plain
matrices the codes stand for.  Same tolerance as the dense bf16 path: only activations, KV and outputs are rounded to
bf16; the weights are identical on both sides."""
import numpy as np
import pytest

from paper_2507_02620_amd import synth

pytestmark = pytest.mark.gpu

SMALL = synth.StageConfig("w4-small", "bf16", 2, 512, 4, 2, 128, 1408, 1000, 96, 40, 16, 5, 3, qkv_bias=True)


@pytest.mark.parametrize("seg", [16, 7, 24, 40])
def test_w4_small_stage(seg):
    import torch
    from tests.gpu_util import TOL, Pair, max_rel_err, to_dev
    cfg = SMALL.with_(seg_len=seg)
    print(f"case w4 small seg={seg}", flush=True)
    pair = Pair(cfg, seed=11, head=True, w4=True)
    tree = synth.config_tree(cfg, seed=11)
    hid = synth.hidden(cfg, cfg.tree_size, 0, 11)
    o, g = pair.verify_tree(tree.parent, hid, seg)
    err = max_rel_err(g, o)
    print(f"  hidden max-rel-err {err:.3e}", flush=True)
    assert err < TOL["bf16"]
    # logits of the last segment's rows
    n = min(seg, cfg.tree_size)
    rows = synth.storage(cfg, o[:n].astype(np.float32))
    lo, _ = pair.orc.logits(rows.astype(np.float64))
    lg, am = pair.gpu.tree_logits(to_dev(rows, torch.bfloat16))
    err = max_rel_err(lg.float().cpu().numpy(), lo)
    print(f"  logits max-rel-err {err:.3e}", flush=True)
    assert err < TOL["bf16"]


def test_w4_64_row_segment_head_dim_64():
    from tests.gpu_util import TOL, Pair, max_rel_err
    cfg = synth.StageConfig("w4-hd64", "bf16", 1, 384, 6, 3, 64, 896, 0, 70, 64, 64, 6, 4)
    print("case w4 hd64 seg=64", flush=True)
    pair = Pair(cfg, seed=5, w4=True)
    tree = synth.config_tree(cfg, seed=5)
    hid = synth.hidden(cfg, cfg.tree_size, 0, 5)
    o, g = pair.verify_tree(tree.parent, hid, 64)
    err = max_rel_err(g, o)
    print(f"  hidden max-rel-err {err:.3e}", flush=True)
    assert err < TOL["bf16"]


def test_w4_13b_shape_two_layers():
    """LLaMA2-13B layer shape (d 5120, 40 heads, FFN 13824, segment 24), two layers, with the head."""
    import torch
    from tests.gpu_util import TOL, Pair, max_rel_err, to_dev
    cfg = synth.CONFIGS["C3"].with_(n_layers=2)
    print("case w4 C3 shape, 2 layers", flush=True)
    pair = Pair(cfg, seed=2, head=True, w4=True)
    tree = synth.config_tree(cfg, seed=2)
    hid = synth.hidden(cfg, cfg.tree_size, 0, 2)
    o, g = pair.verify_tree(tree.parent, hid, cfg.seg_len)
    err = max_rel_err(g, o)
    print(f"  hidden max-rel-err {err:.3e}", flush=True)
    assert err < TOL["bf16"]
    rows = synth.storage(cfg, o[:cfg.seg_len].astype(np.float32))
    lo, _ = pair.orc.logits(rows.astype(np.float64))
    lg, am = pair.gpu.tree_logits(to_dev(rows, torch.bfloat16))
    lg = lg.float().cpu().numpy()
    err = max_rel_err(lg, lo)
    print(f"  logits max-rel-err {err:.3e}", flush=True)
    assert err < TOL["bf16"]
    # argmax: equal wherever the oracle's top two are further apart than the bf16-level error of a logit
    top2 = np.sort(lo, axis=1)[:, -2:]
    clear = (top2[:, 1] - top2[:, 0]) > 4 * TOL["bf16"] * np.abs(lo).max()
    assert np.array_equal(am.cpu().numpy()[clear], lo.argmax(axis=1)[clear])


def test_w4_many_row_chain():
    """A 200-row chain in one segment with 4-bit weights (row blocks of the few-row kernel)."""
    from tests.gpu_util import TOL, Pair, max_rel_err
    cfg = synth.StageConfig("w4-chain", "bf16", 2, 512, 4, 4, 128, 1408, 0, 60, 200, 200, 200, 1)
    print("case w4 chain 200 rows", flush=True)
    pair = Pair(cfg, seed=8, w4=True)
    hid = synth.hidden(cfg, 200, 0, 8)
    o, g = pair.verify_tree(np.arange(-1, 199, dtype=np.int32), hid, 200)
    err = max_rel_err(g, o)
    print(f"  hidden max-rel-err {err:.3e}", flush=True)
    assert err < TOL["bf16"]


def test_w4_rejects_f32_and_bad_shapes():
    from paper_2507_02620_amd import flowspec as fs
    with pytest.raises(fs.FlowSpecError):
        fs.Stage(n_layers=1, d_model=256, n_q_heads=4, n_kv_heads=4, head_dim=64, d_ffn=512, vocab=0, dtype=fs.FS_F32, rms_eps=1e-5,
                 rope_theta=1e4, kv_capacity=64, max_tree=16, max_seg=16, layers=[], weight_format=fs.FS_WFMT_INT4_G128)


def _random_w4(i):
    r = np.random.default_rng(8200 + i)
    hd = int(r.choice([64, 128]))
    n_kv = int(r.choice([1, 2, 4]))
    n_q = n_kv * int(r.choice([1, 2, 4]))
    while (n_q * hd) % 128:   # one scale per 128 input columns of the attention output projection
        n_q += n_kv
    return synth.StageConfig(f"w4-rnd{i}", "bf16", int(r.integers(1, 3)), int(r.integers(2, 8)) * 128, n_q, n_kv, hd, int(r.integers(3, 12)) * 128,
                             int(r.choice([0, 777, 2000])), int(r.choice([0, 5, int(r.integers(6, 1200))])), int(r.integers(2, 120)),
                             int(r.integers(1, 66)), int(r.integers(2, 20)), int(r.choice([0, 2, 4])), qkv_bias=bool(i % 2))


@pytest.mark.parametrize("i", range(8))
def test_w4_random_shapes(i):
    """Seeded random 4-bit stages (widths in multiples of the 128-column scale group, ragged trees and segments, with and
    without head): hidden states, appended K/V and logits against the oracle."""
    import torch
    from tests.gpu_util import TOL, Pair, max_rel_err, to_dev
    cfg = _random_w4(i)
    print(f"[case] {cfg}", flush=True)
    pair = Pair(cfg, seed=60 + i, head=cfg.vocab > 0, w4=True)
    tree = synth.config_tree(cfg, seed=60 + i)
    hid = synth.hidden(cfg, tree.size, 0, 60 + i)
    o, g = pair.verify_tree(tree.parent, hid, cfg.seg_len)
    err = max_rel_err(g, o)
    L = cfg.l_glo + tree.size
    kerr = max_rel_err(pair.kv[:, :, :, cfg.l_glo:L].float().cpu().numpy(), pair.orc.kv[:, :, :, cfg.l_glo:L])
    print(f"  hidden max-rel-err {err:.3e}, appended K/V {kerr:.3e}", flush=True)
    assert err < TOL["bf16"] and kerr < TOL["bf16"]
    if cfg.vocab:
        n = min(cfg.seg_len, tree.size)
        rows = synth.storage(cfg, o[:n].astype(np.float32))
        lo, _ = pair.orc.logits(rows.astype(np.float64))
        lg, _ = pair.gpu.tree_logits(to_dev(rows, torch.bfloat16))
        lerr = max_rel_err(lg.float().cpu().numpy(), lo)
        print(f"  logits max-rel-err {lerr:.3e}", flush=True)
        assert lerr < TOL["bf16"]


@pytest.mark.parametrize("name,cfg,rows", [
    # QKV and gate/up in 128-row blocks, the residual projections (short K: test_w4_residual_projections_of_a_short_k) in the few-row kernel
    ("all", synth.StageConfig("w4b-all", "bf16", 2, 1024, 16, 16, 128, 3328, 0, 40, 577, 577, 577, 1, qkv_bias=True), 577),
    # residual projections and LM head in 64-row blocks, the attention output with one K slice; the others in the few-row kernel
    ("resid", synth.StageConfig("w4b-resid", "bf16", 2, 4992, 2, 2, 64, 1152, 34000, 30, 33, 33, 5, 3), 33),
    ("resid", synth.StageConfig("w4b-resid", "bf16", 1, 4992, 2, 2, 64, 1152, 34000, 30, 64, 64, 5, 3), 64),
    # gate/up only: 64-row blocks, and 128-row blocks (161 rows: 6 and 5 row tiles, the last one with a single row)
    ("gateup", synth.StageConfig("w4b-gu", "bf16", 2, 128, 2, 1, 64, 17024, 0, 30, 64, 64, 5, 3), 64),
    ("gateup", synth.StageConfig("w4b-gu", "bf16", 2, 128, 2, 1, 64, 9728, 0, 30, 161, 161, 161, 1), 161),
    # one row tile, gate/up of 1376 tiles (half groups: the next test)
    ("half", synth.StageConfig("w4b-half", "bf16", 1, 128, 2, 1, 64, 11008, 0, 30, 16, 16, 5, 3), 16),
])
def test_w4_row_blocks(name, cfg, rows):
    """The many-row 4-bit kernel where it takes over from the few-row one, alone and mixed with it in one layer."""
    import torch
    from tests.gpu_util import TOL, Pair, max_rel_err, to_dev
    print(f"[case] {name} rows={rows}", flush=True)
    pair = Pair(cfg, seed=rows, head=cfg.vocab > 0, w4=True)
    parent = np.arange(-1, rows - 1, dtype=np.int32) if cfg.max_branch == 1 else synth.config_tree(cfg, seed=rows).parent
    hid = synth.hidden(cfg, rows, 0, rows)
    o, g = pair.verify_tree(parent, hid, rows)
    L = cfg.l_glo + rows
    err = max_rel_err(g, o)
    kerr = max_rel_err(pair.kv[:, :, :, cfg.l_glo:L].float().cpu().numpy(), pair.orc.kv[:, :, :, cfg.l_glo:L])
    print(f"  hidden {err:.2e}, K/V {kerr:.2e}", flush=True)
    assert err < TOL["bf16"] and kerr < TOL["bf16"]
    if cfg.vocab:
        x = synth.storage(cfg, o.astype(np.float32))
        lo, _ = pair.orc.logits(x.astype(np.float64))
        lg, _ = pair.gpu.tree_logits(to_dev(x, torch.bfloat16))
        assert max_rel_err(lg.cpu().numpy(), lo) < TOL["bf16"]


@pytest.mark.parametrize("rows", [1, 16])
def test_w4_half_groups(rows):
    """One row tile, gate/up of 592 groups of four tiles: half a group per workgroup."""
    from tests.gpu_util import TOL, Pair, kernel_names, max_rel_err
    cfg = synth.StageConfig(f"w4-half-{rows}", "bf16", 1, 256, 2, 2, 128, 18944, 0, 30, rows, rows, 5, 3)
    print(f"[case] {cfg.name}", flush=True)
    pair = Pair(cfg, seed=rows, w4=True)
    got = []
    names = kernel_names(lambda: got.extend(pair.verify_tree(synth.config_tree(cfg, seed=rows).parent, synth.hidden(cfg, rows, 0, rows), rows)))
    assert max_rel_err(got[1], got[0]) < TOL["bf16"]
    assert any("skinny_gemm_w4_kernel<1, 2, 2, 2>" in n for n in names), names   # two of a group's four tiles


@pytest.mark.parametrize("rows,ffn,wn", [(33, 5504, 2), (64, 5504, 2), (33, 11008, 4), (64, 11008, 4)])
def test_w4_streaming_kernel_behind_a_few_row_producer(rows, ffn, wn):
    """4096 columns: the output projection leaves 256 partial sums of squares, more than a thread of gate/up loads ahead of the ring."""
    from tests.gpu_util import TOL, Pair, kernel_names, max_rel_err
    cfg = synth.StageConfig(f"w4-ssp-{rows}-{ffn}", "bf16", 1, 4096, 1, 1, 128, ffn, 0, 20, rows, rows, 5, 3)
    print(f"[case] {cfg.name}", flush=True)
    pair = Pair(cfg, seed=rows, w4=True)
    got = []
    names = kernel_names(lambda: got.extend(pair.verify_tree(synth.config_tree(cfg, seed=rows).parent, synth.hidden(cfg, rows, 0, rows), rows)))
    assert max_rel_err(got[1], got[0]) < TOL["bf16"]
    assert any(f"stream_gemm_w4_kernel<2, {wn}, 2, 4" in n for n in names), names
    assert any("skinny_gemm_w4_kernel" in n and ", 1, " in n for n in names), names   # the output projection


@pytest.mark.parametrize("rows", [500, 641])
def test_w4_residual_projections_of_a_short_k(rows):
    """1536 input columns: few-row kernel in row blocks up to about 570 rows, beyond in 128-row blocks (6 or 5 row
    tiles, the last one with a single row) in K slices."""
    from tests.gpu_util import TOL, Pair, max_rel_err
    cfg = synth.StageConfig(f"w4-short-k-{rows}", "bf16", 2, 1536, 12, 2, 128, 1536, 0, 20, rows, rows, rows, 1)
    print(f"[case] {cfg.name}", flush=True)
    pair = Pair(cfg, seed=6, w4=True)
    o, g = pair.verify_tree(np.arange(-1, rows - 1, dtype=np.int32), synth.hidden(cfg, rows, 0, 6), rows)
    assert max_rel_err(g, o) < TOL["bf16"]


@pytest.mark.parametrize("rows,ffn", [(1, 8320), (16, 8320), (17, 5248), (32, 5248), (33, 10368), (64, 10368)])
def test_w4_streaming_kernel(rows, ffn):
    """Up to 64 rows through the LDS-fed 4-bit kernel: QKV and gate/up in blocks of four and eight tiles, the down projection in
    K slices of an odd number of chunks, a head whose last block is ragged; both ends of each row-tile count."""
    import torch
    from tests.gpu_util import TOL, Pair, kernel_names, max_rel_err, to_dev
    cfg = synth.StageConfig(f"w4s-{rows}", "bf16", 2, 256, 36, 18, 128, ffn, 11300, 20, rows, rows, 5, 3, qkv_bias=True)
    print(f"[case] {cfg.name}", flush=True)
    pair = Pair(cfg, seed=rows, head=True, w4=True)
    got = []
    names = kernel_names(lambda: got.extend(pair.verify_tree(synth.config_tree(cfg, seed=rows).parent, synth.hidden(cfg, rows, 0, rows), rows)))
    o, g = got[:2]   # (more where the profile had to be taken again)
    assert [sum(f"stream_gemm_w4_kernel<{kind}," in n for n in names) for kind in (0, 2)] == [2, 2], names
    assert any("stream_gemm_w4_kernel<1," in n for n in names), names
    L = cfg.l_glo + rows
    kerr = max_rel_err(pair.kv[:, :, :, cfg.l_glo:L].float().cpu().numpy(), pair.orc.kv[:, :, :, cfg.l_glo:L])
    x = synth.storage(cfg, o.astype(np.float32))
    lo, _ = pair.orc.logits(x.astype(np.float64))
    names = kernel_names(lambda: got.extend(pair.gpu.tree_logits(to_dev(x, torch.bfloat16))))
    lg = got[-2]
    assert any("stream_gemm_w4_kernel<3," in n for n in names), names
    assert max_rel_err(g, o) < TOL["bf16"] and kerr < TOL["bf16"] and max_rel_err(lg.cpu().numpy(), lo) < TOL["bf16"]


@pytest.mark.parametrize("rows", [140, 177, 225])
@pytest.mark.parametrize("d,ffn", [(4864, 3072), (128, 9728)])
def test_w4_row_blocks_of_equal_height(rows, d, ffn):
    """128-row blocks that share the row tiles evenly (5, 6 and 8 tiles; waves of 3 + 2, 3 + 3 and 4 + 4): the down projection of 19 feature
    blocks in K slices (4864 columns), gate/up (128 columns)."""
    from tests.gpu_util import TOL, Pair, max_rel_err
    cfg = synth.StageConfig(f"w4e-{rows}", "bf16", 1 if d > 128 else 2, d, 2, 1, 64, ffn, 0, 20, rows, rows, rows, 1)
    print(f"[case] {cfg.name} {d}", flush=True)
    pair = Pair(cfg, seed=rows, w4=True)
    o, g = pair.verify_tree(np.arange(-1, rows - 1, dtype=np.int32), synth.hidden(cfg, rows, 0, rows), rows)
    assert max_rel_err(g, o) < TOL["bf16"]


@pytest.mark.parametrize("rows,d,heads,slices", [(257, 4096, 8, 2), (300, 4096, 8, 2), (300, 5120, 10, 2)])
def test_w4_residual_projections_of_a_short_k_are_cut(rows, d, heads, slices):
    """1024 and 1280 input columns, a few row blocks: one slice leaves most of the chip idle (31 against 22 us)."""
    from tests.gpu_util import TOL, Pair, kernel_names, max_rel_err
    cfg = synth.StageConfig(f"w4c-{rows}-{d}", "bf16", 1, d, heads, 1, 128, 128, 0, 20, rows, rows, rows, 1)
    print(f"[case] {cfg.name}", flush=True)
    pair = Pair(cfg, seed=rows, w4=True)
    hid, par = synth.hidden(cfg, rows, 0, rows), np.arange(-1, rows - 1, dtype=np.int32)
    got = []
    names = kernel_names(lambda: got.extend(pair.verify_tree(par, hid, rows)))
    assert max_rel_err(got[1], got[0]) < TOL["bf16"]
    assert sum(f"wide_fixup_kernel<{slices}, 4>" in n for n in names) == 1, names   # the output projection (the down projection has one chunk)


@pytest.mark.parametrize("rows", [257, 320, 321])
def test_w4_row_blocks_of_full_height(rows):
    """Three row blocks of 88 feature blocks: 33 an XCD.  Up to 320 rows two blocks of eight row tiles and one of 1 to 4, whose second
    row of waves has no rows; from 321 rows on equal heights."""
    from tests.gpu_util import TOL, Pair, max_rel_err
    cfg = synth.StageConfig(f"w4h-{rows}", "bf16", 1, 256, 2, 1, 64, 11136, 0, 20, rows, rows, rows, 1)
    print(f"[case] {cfg.name}", flush=True)
    pair = Pair(cfg, seed=rows, w4=True)
    o, g = pair.verify_tree(np.arange(-1, rows - 1, dtype=np.int32), synth.hidden(cfg, rows, 0, rows), rows)
    assert max_rel_err(g, o) < TOL["bf16"]


@pytest.mark.parametrize("rows,ffn", [
    (300, 22528),   # 66 blocks an XCD in three row blocks, two rounds and two: full heights
    (321, 22528),   # the last row block of full height would have five tiles: equal
    (530, 6656),    # 35 blocks in five row blocks: full
    (530, 8192),    # 40: equal
    (385, 8448),    # four row blocks of seven tiles, the last of four: its second row of waves has no rows
    (389, 1024),    # the same in the residual projections' slices and in gate/up
])
def test_w4_row_blocks_of_either_height(rows, ffn):
    from tests.gpu_util import TOL, Pair, max_rel_err
    d = 128 if ffn > 1024 else 2176
    cfg = synth.StageConfig(f"w4r-{rows}-{ffn}", "bf16", 1, d, 17 if ffn == 1024 else 2, 1, 128 if ffn == 1024 else 64, ffn, 0, 20, rows, rows, rows, 1)
    print(f"[case] {cfg.name}", flush=True)
    pair = Pair(cfg, seed=rows, w4=True)
    o, g = pair.verify_tree(np.arange(-1, rows - 1, dtype=np.int32), synth.hidden(cfg, rows, 0, rows), rows)
    assert max_rel_err(g, o) < TOL["bf16"]


@pytest.mark.parametrize("rows,ffn,block", [(128, 5632, False), (100, 5632, False), (80, 9216, True), (65, 11008, True)])
def test_w4_residual_projections_between_the_two_lines(rows, ffn, block):
    """4096 features, 65 to 128 rows: two full rounds of few-row workgroups, which a K of 5632 does not make longer than the row blocks."""
    from tests.gpu_util import TOL, Pair, kernel_names, max_rel_err
    cfg = synth.StageConfig(f"w4l-{rows}-{ffn}", "bf16", 1, 4096, 1, 1, 128, ffn, 0, 20, rows, rows, rows, 1)
    print(f"[case] {cfg.name}", flush=True)
    pair = Pair(cfg, seed=rows, w4=True)
    hid, par = synth.hidden(cfg, rows, 0, rows), np.arange(-1, rows - 1, dtype=np.int32)
    got = []
    names = kernel_names(lambda: got.extend(pair.verify_tree(par, hid, rows)))
    assert max_rel_err(got[1], got[0]) < TOL["bf16"]
    assert any("block_gemm_w4_kernel<1," in n for n in names) == block, names


# the kernels of QKV, gate/up and the down projection
_FEW, _STREAM = "skinny_gemm_w4_kernel<", "stream_gemm_w4_kernel<"


@pytest.mark.parametrize("d,heads,kv,ffn,rows,qkv,gateup,down", [
    # one full round of few-row workgroups: 256 groups of two tiles (QKV), 128 groups and two row blocks (gate/up)
    (4096, 32, 16, 2048, 16, _FEW, _FEW, _FEW),
    (4096, 32, 16, 2048, 32, _FEW, _FEW, _FEW),
    (2560, 20, 20, 2048, 33, _FEW, _FEW, _FEW),
    (2560, 20, 20, 2048, 64, _FEW, _FEW, _FEW),
    # more than a round: 320 groups of two tiles (QKV), gate/up of 1312 and 1920 tiles; the down projection of 5248 and 7680 columns
    (1024, 40, 20, 7680, 24, _STREAM, _STREAM, _STREAM),
    # close to each other: QKV of 960 tiles, 15.3 against 17.3 us
    (5120, 40, 40, 2048, 24, _STREAM, _FEW, _FEW),
    (5120, 4, 4, 5248, 24, _FEW, _STREAM, _STREAM),
    (5120, 4, 4, 5248, 33, _FEW, _STREAM, _STREAM),
    (5120, 4, 4, 5248, 64, _FEW, _STREAM, _STREAM),
])
def test_w4_streaming_kernel_where_it_is_the_faster_one(d, heads, kv, ffn, rows, qkv, gateup, down):
    from tests.gpu_util import TOL, Pair, kernel_names, max_rel_err
    cfg = synth.StageConfig(f"w4r-{d}-{ffn}-{rows}", "bf16", 1, d, heads, kv, 128, ffn, 0, 20, rows, rows, 5, 3)
    print(f"[case] {cfg.name}", flush=True)
    pair = Pair(cfg, seed=rows, w4=True)
    hid, par = synth.hidden(cfg, rows, 0, rows), synth.config_tree(cfg, seed=rows).parent
    got = []
    names = kernel_names(lambda: got.extend(pair.verify_tree(par, hid, rows)))
    assert max_rel_err(got[1], got[0]) < TOL["bf16"]
    # template arguments: projection kind first (streaming kernel) or third (few-row kernel)
    kinds = [(_STREAM, n.split(_STREAM)[1].split(",")[0]) if _STREAM in n else (_FEW, n.split(_FEW)[1].split(",")[2].strip())
             for n in names if _STREAM in n or _FEW in n]
    print("  ", kinds, flush=True)
    assert [k for k, _ in kinds if _ == "0"] == [qkv] and [k for k, _ in kinds if _ == "2"] == [gateup]
    assert [k for k, _ in kinds if _ == "1"][-1] == down
