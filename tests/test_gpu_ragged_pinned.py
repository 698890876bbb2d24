"""gw_lnl_ragged on a workspace that a graph was captured from.  The graph's
replays write the captured call's sections over the arena without a call into the
library, so a ragged call between them must not take its events, its maps or its
bin tables as still standing there: it repeats its first result bit for bit,
and that one is within 1e-10 relative (the repository's FP64 bar) of the oracle.

The captured call writes either the first event's tables alone or more than
the whole ragged plan; the ragged call sums every bin or frequency nodes.
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

# (1/delta_f, bins, rows) of the ragged call's events
EVENTS = {"bins": [(8.0, 3001, 70), (4.0, 1500, 257), (8.0, 2000, 1)],
          "nodes": [(64.0, 60_001, 300), (32.0, 40_000, 256), (4.0, 37, 20)]}
CAPTURED_BINS = {"tables": 300, "everything": 500_000}


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("captured", list(CAPTURED_BINS))
@pytest.mark.parametrize("route", list(EVENTS))
def test_replays_between_ragged_calls(route, captured):
    import torch
    import paper_1904_02863_amd as gw
    ws = gw.Workspace(0)
    ws.set_tuning(False)
    ws.reserve(1_000_000, 3, 600)
    one = synth.small_event(60, 3, CAPTURED_BINS[captured], 300, 9, delta_f=1.0 / 64.0)
    args = (one.grid, one.tensors, one.vertices, _dev(oracle.workload_data(one)), _dev(one.psd), _dev(one.theta))
    eager = gw.lnl_batch(*args, workspace=ws).clone()
    replayed = torch.empty_like(eager)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        gw.lnl_batch(*args, workspace=ws, out=replayed)
    torch.cuda.synchronize()

    evs = [synth.small_event(61 + i, 3, m, n, 9, delta_f=1.0 / t) for i, (t, m, n) in enumerate(EVENTS[route])]
    data = [oracle.workload_data(w) for w in evs]
    events, _, rows = gw.make_events([w.grid for w in evs], [w.tensors for w in evs], [w.vertices for w in evs],
                                     [len(w.theta) for w in evs])
    packed = (_dev(np.concatenate([d.ravel() for d in data])), _dev(np.concatenate([w.psd.ravel() for w in evs])),
              _dev(np.concatenate([w.theta for w in evs])))
    out = torch.empty(rows, dtype=torch.float64, device="cuda:0")
    first = None
    for rep in range(4):
        out.fill_(float("nan"))
        print(f"{route} {captured} ragged {rep}", flush=True)
        gw.lnl_ragged(events, len(evs), *packed, out=out, workspace=ws)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        if first is None:
            first = got
            at = 0
            for w, d in zip(evs, data):
                pick = np.unique(np.linspace(0, len(w.theta) - 1, 6).astype(int))
                g = w.grid
                ref = oracle.lnl(g.f_low, g.delta_f, g.n_bins, w.tensors, w.vertices, d, w.psd, w.theta[pick])
                assert (np.abs(got[at + pick] - ref) <= 1e-10 * np.abs(ref)).all(), g.n_bins
                at += len(w.theta)
        np.testing.assert_array_equal(got, first, err_msg=f"ragged call {rep}")
        replayed.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(replayed.cpu().numpy(), eager.cpu().numpy(), err_msg=f"replay {rep}")
