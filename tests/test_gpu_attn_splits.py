"""Tree attention of few KV heads at the ends of the rule on how many KV splits a context goes into, against the oracle."""
import pytest

from paper_2507_02620_amd import synth
from tests.test_gpu_parity import _check_stage

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,kv,hd,rows", [(8, 4, 128, 16), (4, 4, 64, 5), (6, 2, 128, 7), (16, 4, 128, 16), (32, 8, 128, 13), (16, 4, 128, 12)])
@pytest.mark.parametrize("slots", [28 * 64, 28 * 64 + 1, 33 * 64 - 1, 65 * 64, 128 * 64, 128 * 64 + 1])
def test_splits_of_few_kv_heads(heads, kv, hd, rows, slots):
    """28 and 29 tiles, an odd number of them, more than 64 (32 splits of several), 128 and 129; (2 KV heads: the rule does not apply;
    four row tiles of 4 and 8 KV heads: the direct-to-LDS kernel in that range, three: not)."""
    cfg = synth.StageConfig(f"splits-{hd}-{slots}", "bf16", 1, 128, heads, kv, hd, 256, 0, slots - rows, rows, rows, 6, 3)
    _check_stage(cfg, slots, rows)
