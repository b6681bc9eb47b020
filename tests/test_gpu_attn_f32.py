"""f32 tree attention of one row tile per KV head (its slots divided over the waves) against the oracle: contexts that end in every wave's
share of a tile, waves that see no slot, draft slots in some shares only, one split and several, one tile in flight and two."""
import pytest

from paper_2507_02620_amd import synth
from tests.test_gpu_parity import _check_stage

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,kv,hd,rows", [(4, 4, 64, 16), (4, 4, 64, 1), (6, 3, 64, 8), (4, 4, 128, 16), (4, 2, 128, 5), (4, 4, 64, 17)])
@pytest.mark.parametrize("l_glo", [0, 1, 15, 16, 33, 47, 49, 64, 111, 113, 176, 177, 1000])
def test_slots_divided_over_the_waves(heads, kv, hd, rows, l_glo):
    """(17 rows: two row tiles, the form with a row tile per wave.)"""
    cfg = synth.StageConfig(f"f32-{hd}-{l_glo}-{rows}", "f32", 1, 128, heads, kv, hd, 256, 0, l_glo, 2 * rows, rows, 6, 3)
    _check_stage(cfg, l_glo + rows, rows)   # two segments: the second one's tree reaches back into the cache


@pytest.mark.parametrize("l_glo,wgs", [(700, 4), (705, 8), (4000, 16)])
def test_long_splits_with_two_tiles_in_flight(l_glo, wgs, monkeypatch):
    monkeypatch.setenv("FLOWSPEC_ATTN_WGS", str(wgs))
    cfg = synth.StageConfig(f"f32-ring-{l_glo}", "f32", 1, 128, 2, 2, 64, 256, 0, l_glo, 30, 16, 6, 3)
    _check_stage(cfg, l_glo, 16)


@pytest.mark.parametrize("hd,slots,one", [(64, 192, True), (64, 193, False), (128, 64, True), (128, 65, False)])
def test_short_contexts_in_one_split(hd, slots, one):
    from tests.gpu_util import kernel_names
    cfg = synth.StageConfig(f"f32-ends-{hd}-{slots}", "f32", 1, 128, 4, 4, hd, 256, 0, slots - 16, 16, 16, 6, 4)
    _check_stage(cfg, slots, 16)
    names = kernel_names(lambda: _check_stage(cfg, slots, 16))
    assert any("tree_attn" in n for n in names) and any("attn_merge_kernel" in n for n in names) != one, names
