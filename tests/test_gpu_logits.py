"""LM head + row argmax of the HIP path vs the oracle."""
import numpy as np
import pytest

from paper_2507_02620_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg,rows", [
    (synth.CONFIGS["C1"], 16),
    (synth.StageConfig("lg-bf16", "bf16", 1, 512, 4, 4, 128, 1376, 32000, 8, 16, 24, 4, 3), 24),
    (synth.StageConfig("lg-bf16-odd-vocab", "bf16", 1, 1024, 8, 2, 128, 1376, 50257, 8, 16, 64, 4, 3), 64),
    (synth.StageConfig("lg-f32", "f32", 1, 256, 4, 4, 64, 688, 1000, 8, 16, 5, 4, 3), 5),
    # 40 rows: the kernel that streams weights and activations through LDS; 100 rows: one partly filled 128-row block of the many-row kernel, padding tiles
    (synth.StageConfig("lg-bf16-40", "bf16", 1, 512, 4, 4, 128, 1376, 32000, 8, 16, 40, 4, 3), 40),
    (synth.StageConfig("lg-bf16-100-odd-vocab", "bf16", 1, 1024, 8, 2, 128, 1376, 50257, 8, 16, 100, 4, 3), 100),
])
def test_logits_and_argmax(cfg, rows):
    import torch
    from tests.gpu_util import TOL, Pair, max_rel_err, to_dev
    print(f"[case] {cfg.name} rows={rows} vocab={cfg.vocab}", flush=True)
    p = Pair(cfg, 3, head=True)
    hid = synth.hidden(cfg, rows, 7, 3)
    o_lg, o_am = p.orc.logits(hid.astype(np.float64))
    g_lg, g_am = p.gpu.tree_logits(to_dev(hid, p.tdtype))
    torch.cuda.synchronize()
    g_lg, g_am = g_lg.cpu().numpy(), g_am.cpu().numpy()
    err = max_rel_err(g_lg, o_lg)
    print(f"  logits max-rel-err {err:.3e}", flush=True)
    assert err < TOL[cfg.dtype]
    # the device argmax is exact for the device's own fp32 logits (lowest index on ties) ...
    assert np.array_equal(g_am, np.argmax(g_lg, axis=1))
    # ... and agrees with the oracle wherever the oracle's top-2 gap exceeds the numerical error bound
    top2 = np.sort(o_lg, axis=1)[:, -2:]
    clear = (top2[:, 1] - top2[:, 0]) > 2 * TOL[cfg.dtype] * np.abs(o_lg).max()
    assert np.array_equal(g_am[clear], o_am[clear])
    # elsewhere the chosen entry must be within the bound of the oracle's maximum
    for r in np.nonzero(~clear)[0]:
        assert o_lg[r, g_am[r]] >= top2[r, 1] - 2 * TOL[cfg.dtype] * np.abs(o_lg).max()


@pytest.mark.parametrize("vocab,rows", [(32768, 33), (32769, 40), (32769, 41), (49152, 17), (49153, 32), (49153, 33), (65408, 24), (65409, 17)])
def test_head_of_17_to_48_rows_at_the_edges_of_its_routes(vocab, rows):
    """256, 257, 384, 385, 511 and 512 blocks of 128 features, rows on both sides of the line between two kernels."""
    import torch
    from tests.gpu_util import TOL, Pair, max_rel_err, to_dev
    cfg = synth.StageConfig(f"lg-{vocab}", "bf16", 1, 256, 2, 2, 128, 256, vocab, 8, 16, rows, 4, 3)
    print(f"[case] {cfg.name} rows={rows}", flush=True)
    p = Pair(cfg, 3, head=True)
    hid = synth.hidden(cfg, rows, 7, 3)
    o_lg, _ = p.orc.logits(hid.astype(np.float64))
    g_lg, g_am = p.gpu.tree_logits(to_dev(hid, torch.bfloat16))
    g_lg, g_am = g_lg.cpu().numpy(), g_am.cpu().numpy()
    assert max_rel_err(g_lg, o_lg) < TOL["bf16"]
    assert np.array_equal(g_am, np.argmax(g_lg, axis=1))


@pytest.mark.parametrize("dtype,w4,rows,vocab,shift", [
    ("bf16", False, 16, 1004, 0), ("bf16", False, 5, 1004, 1), ("bf16", False, 40, 996, 0), ("bf16", False, 128, 2004, 0), ("bf16", False, 128, 2004, 2),
    ("bf16", False, 300, 1000, 0), ("bf16", False, 17, 1003, 0), ("bf16", True, 24, 1004, 0), ("bf16", True, 100, 1004, 3), ("f32", False, 16, 1004, 0),
    ("f32", False, 7, 1002, 0), ("f32", False, 3, 4, 0),
])
def test_logits_in_rows_on_16_bytes_and_not(dtype, w4, rows, vocab, shift):
    """Vocabularies that are and are not a multiple of four, inside the last tile, and a buffer off 16 bytes; nothing beyond the rows is written."""
    import torch
    from tests.gpu_util import TOL, Pair, max_rel_err, to_dev
    cfg = synth.StageConfig(f"lg-vec-{vocab}", dtype, 1, 256, 2, 2, 128, 256, vocab, 8, 16, rows, 4, 3)
    print(f"[case] {cfg.name} {dtype} w4={w4} rows={rows} shift={shift}", flush=True)
    p = Pair(cfg, 3, head=True, w4=w4)
    hid = synth.hidden(cfg, rows, 7, 3)
    o_lg, _ = p.orc.logits(hid.astype(np.float64))
    buf = torch.full((rows * vocab + 64,), -7.0, device="cuda")
    view = buf[shift:shift + rows * vocab].view(rows, vocab)
    _, am = p.gpu.tree_logits(to_dev(hid, p.tdtype), view, torch.empty(rows, dtype=torch.int32, device="cuda"))
    got = view.cpu().numpy()
    assert max_rel_err(got, o_lg) < TOL[dtype]
    assert np.array_equal(am.cpu().numpy(), np.argmax(got, axis=1))
    assert bool((buf[:shift] == -7.0).all()) and bool((buf[shift + rows * vocab:] == -7.0).all())
