"""Host rules that choose a launch's shape, at the lines where first one side and then the other was measured the faster one.  CPU only."""
import ctypes as C
import heapq

import numpy as np
import pytest

from paper_2507_02620_amd import flowspec as fs


@pytest.mark.parametrize("vocab,rows,chunks", [
    (152064, 40, 13), (152064, 80, 12), (100000, 200, 5), (32001, 256, 4),      # about 512 to 1024 workgroups
    (152064, 257, 7), (152065, 400, 5), (100000, 512, 4), (32000, 600, 3),      # many rows: about 2048
    (4096, 16, 1), (16385, 1, 5), (1, 1, 1), (152064, 1024, 2),
])
def test_chunks_of_a_sampled_row(vocab, rows, chunks):
    assert fs.lib().sample_chunks(C.c_int(vocab), C.c_int(rows)) == chunks


def _longest_first(tiles, wgs, slots):
    a = (C.c_int * len(tiles))(*tiles)
    b = (C.c_int * len(wgs))(*wgs)
    return bool(fs.lib().attn_longest_first(a, b, len(tiles), slots))


def _end(jobs, slots):
    """Workgroup by workgroup: each starts where a place falls free first."""
    free = [0] * slots
    for t in jobs:
        heapq.heapreplace(free, free[0] + t + 6)
    return max(free)


def test_longest_contexts_first_only_where_that_is_shorter():
    rng, chosen = np.random.default_rng(4), 0
    for _ in range(300):
        n, slots = int(rng.integers(1, 33)), int(rng.choice([256, 512]))
        tiles = [int(t) for t in rng.integers(1, int(rng.choice([4, 20, 70])) + 1, n)]
        wgs = [int(rng.choice([4, 32, 40])) * int(rng.integers(1, 4)) for _ in range(n)]
        order = sorted(range(n), key=lambda i: -tiles[i])
        ends = [_end([tiles[i] for i in o for _ in range(wgs[i])], slots) for o in (range(n), order)]
        chosen += ends[1] * 100 < ends[0] * 97
        assert _longest_first(tiles, wgs, slots) == (ends[1] * 100 < ends[0] * 97), (tiles, wgs, slots, ends)
    assert 50 < chosen < 250


def test_a_few_workgroups_beyond_two_rounds_keep_their_order():
    """26 requests of 40 heads, contexts of 9 to 18 tiles (550 .. 1100 slots): 1040 workgroups on 512 places; sorted, the last 16 are a round of their own."""
    tiles = [9 + (7 * i) % 10 for i in range(26)]
    assert not _longest_first(tiles, [40] * 26, 512)
    assert _longest_first([9 + (7 * i) % 10 for i in range(32)], [32] * 32, 512)


def _plan(M, G, kv, slots, hd=128, elem=2):
    """The attention plan of one request of M rows, G query heads to each of kv KV heads."""
    out = [C.c_int() for _ in range(8)]
    req = C.create_string_buffer(64)   # not looked at: one request's tiles in pairs are balanced
    fs.lib().attn_plan(elem, hd, M, G, kv, slots, req, 1, 64, 0, 0, 0, 0, 0, *(C.byref(o) for o in out))
    return dict(zip(("waves", "row_tiles", "row_blocks", "splits", "tiles_per_split", "ring", "dma", "pair"), (o.value for o in out)))


@pytest.mark.parametrize("M,G,kv,hd,slots,splits", [
    (16, 2, 4, 128, 28 * 64, 28), (16, 2, 4, 128, 28 * 64 + 1, 15), (16, 2, 4, 128, 33 * 64 - 1, 17), (16, 2, 4, 128, 64 * 64, 32),
    (16, 2, 4, 128, 65 * 64, 22), (16, 2, 4, 128, 112 * 64, 38), (16, 2, 4, 128, 113 * 64, 29), (16, 3, 4, 128, 96 * 64, 32), (16, 3, 4, 128, 97 * 64, 25),
    (16, 2, 4, 128, 128 * 64, 32), (16, 2, 4, 128, 128 * 64 + 1, 43), (5, 1, 4, 64, 29 * 64, 15), (5, 1, 4, 64, 81 * 64, 27),
    (16, 1, 12, 128, 80 * 64, 27), (16, 1, 12, 128, 100 * 64, 34), (1, 1, 5, 128, 128 * 64, 43),   # one row tile (12 heads: 43 wanted)
    (45, 8, 4, 128, 36 * 64, 18), (45, 8, 4, 128, 66 * 64, 17), (45, 8, 4, 128, 76 * 64, 19), (45, 8, 4, 128, 80 * 64, 27),   # 12 workgroups of 8 waves
    (7, 3, 2, 128, 29 * 64, 29),                                             # two KV heads: a tile to a split
])
def test_splits_of_few_kv_heads(M, G, kv, hd, slots, splits):
    p = _plan(M, G, kv, slots, hd)
    assert p["splits"] == splits and not p["pair"], p
    assert p["splits"] * p["tiles_per_split"] * 64 >= slots


@pytest.mark.parametrize("M,G,kv,slots,dma", [
    (16, 4, 4, 28 * 64, False), (16, 4, 4, 28 * 64 + 1, True), (13, 4, 8, 128 * 64, True), (16, 4, 8, 128 * 64 + 1, False),
    (12, 4, 4, 64 * 64, False), (17, 4, 4, 64 * 64, False), (16, 4, 3, 64 * 64, False), (16, 4, 9, 64 * 64, False),
])
def test_four_row_tiles_on_few_kv_heads(M, G, kv, slots, dma):
    p = _plan(M, G, kv, slots)
    assert (p["dma"] == 2 and p["row_tiles"] == 1 and p["waves"] == 4) == dma, p
