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
