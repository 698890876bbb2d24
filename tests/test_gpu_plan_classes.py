"""Plans of gw_lnl_batch are kept per size class, and a call that sums over frequency
nodes is of another class than one that sums every bin, also where their
sizes round to the same powers of two: a plan of one is not used for the other.
"""
import pytest

pytestmark = pytest.mark.gpu

# (bins that are summed one by one, bins on nodes, rows): the same floor(log2) in each
SHAPES = [(16_384, 32_767, 1024), (33_000, 65_000, 500), (8_192, 16_383, 2300)]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("on_bins,on_nodes,rows", SHAPES)
def test_nodes_have_their_own_plans(on_bins, on_nodes, rows, precision):
    import torch
    import paper_1904_02863_amd as gw
    assert torch.cuda.is_available(), "these tests need the GPU"
    for first, second in ((on_bins, on_nodes), (on_nodes, on_bins)):
        ws = gw.Workspace(0)
        default = {n: ws.lnl_plan(n, 3, rows, precision) for n in (first, second)}
        tile = default[first]["tile_bins"] // 2
        ws.set_plan(first, 3, rows, tile, 0, precision)
        assert ws.lnl_plan(first, 3, rows, precision)["tile_bins"] == tile
        assert ws.lnl_plan(second, 3, rows, precision) == default[second]
        # sizes of the same class share the plan, as without nodes
        assert ws.lnl_plan(first - 1 if first == on_nodes else first + 1, 3, rows, precision)["tile_bins"] == tile
        ws.set_plan(first, 3, rows, 0, 0, precision)
        assert ws.lnl_plan(first, 3, rows, precision) == default[first]
    # with the template end there are no nodes: one class
    ws = gw.Workspace(0)
    tile = ws.lnl_plan(on_nodes, 3, rows, precision, gw.FLAG_TERM_ISCO)["tile_bins"] // 2
    ws.set_plan(on_nodes, 3, rows, tile, 0, precision, gw.FLAG_TERM_ISCO)
    assert ws.lnl_plan(on_bins, 3, rows, precision, gw.FLAG_TERM_ISCO)["tile_bins"] == tile
