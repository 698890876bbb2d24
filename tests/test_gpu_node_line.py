"""Which calls of gw_lnl_batch sum over frequency nodes, by detector count and
precision: seen from the plans' size classes, which the two kinds of calls do not share.
The rows on both sides of the line round to the same power of two.
"""
import pytest

pytestmark = pytest.mark.gpu

# (detectors, precision, bins, most rows that are summed bin by bin): the next row starts a group of 256
LINES = ([(d, "fp64", 16_384, 1280) for d in (1, 2, 3, 5, 8)]
         + [(d, "mixed", 16_384, 2304) for d in (1, 2)] + [(d, "mixed", 16_384, 1792) for d in (3, 4, 8)]
         + [(d, "mixed", 65_536, 256) for d in (1, 3, 8)])


@pytest.mark.parametrize("n_det,precision,n_bins,rows", LINES)
def test_line(n_det, precision, n_bins, rows):
    import torch
    import paper_1904_02863_amd as gw
    assert torch.cuda.is_available(), "these tests need the GPU"
    ws = gw.Workspace(0)
    above = ws.lnl_plan(n_bins, n_det, rows + 1, precision)
    tile = above["tile_bins"] // 2
    ws.set_plan(n_bins, n_det, rows, tile, 0, precision)
    assert ws.lnl_plan(n_bins, n_det, rows, precision)["tile_bins"] == tile
    assert ws.lnl_plan(n_bins, n_det, rows + 1, precision) == above
