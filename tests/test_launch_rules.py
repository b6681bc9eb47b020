"""Host rules that choose a launch's shape, at the lines where first one side and then the other was measured the faster one.  CPU only."""
import ctypes as C

import pytest

from paper_2507_02620_amd import flowspec as fs


@pytest.mark.parametrize("vocab,rows,chunks", [
    (152064, 40, 13), (152064, 80, 12), (100000, 200, 5), (32001, 256, 4),      # about 512 to 1024 workgroups
    (152064, 257, 7), (152065, 400, 5), (100000, 512, 4), (32000, 600, 3),      # many rows: about 2048
    (4096, 16, 1), (16385, 1, 5), (1, 1, 1), (152064, 1024, 2),
])
def test_chunks_of_a_sampled_row(vocab, rows, chunks):
    assert fs.lib().sample_chunks(C.c_int(vocab), C.c_int(rows)) == chunks
