"""Likelihood calls on a workspace that cannot grow any more (a call on it was
captured) and has room for the sections of a sum over every bin, but not for those
of the frequency nodes that the call would otherwise take: they run, and their rows
are within 1e-10 relative (the repository's FP64 bar) of the oracle.
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def _pinned(gw, n_bins):
    """A workspace whose capacity a waveform call of n_bins set, and that a capture of it pinned."""
    import torch
    ws = gw.Workspace(0)
    ws.set_tuning(False)
    one = synth.small_event(70, 1, 8, 1, 9)
    args = ((20.0, 1.0 / 64.0, n_bins), one.tensors, one.vertices, _dev(one.theta))
    out = gw.waveform_batch(*args, workspace=ws)
    torch.cuda.synchronize()
    with torch.cuda.graph(torch.cuda.CUDAGraph()):
        gw.waveform_batch(*args, workspace=ws, out=out)
    torch.cuda.synchronize()
    return ws


def _check(w, data, rows, got):
    g = w.grid
    ref = oracle.lnl(g.f_low, g.delta_f, g.n_bins, w.tensors, w.vertices, data, w.psd, w.theta[rows])
    assert (np.abs(got[rows] - ref) <= 1e-10 * np.abs(ref)).all()


def test_batch():
    import paper_1904_02863_amd as gw
    w = synth.small_event(71, 3, 40_001, 4000, 9, delta_f=1.0 / 64.0)
    need = gw.lnl_batch_static_bytes(w.grid, 3, 4000)
    # the waveform's two tables take 48 bytes a bin, the workspace an eighth more; the
    # nodes' own sections take about 18 KB here
    ws = _pinned(gw, int((need - 4000) / 54.0) - 30)
    assert need - 9000 < ws.nbytes < need
    data = oracle.workload_data(w)
    got = gw.lnl_batch(w.grid, w.tensors, w.vertices, _dev(data), _dev(w.psd), _dev(w.theta), workspace=ws)
    _check(w, data, np.array([0, 1, 2047, 3999]), got.cpu().numpy())
    assert ws.nbytes < need


def test_ragged():
    import paper_1904_02863_amd as gw
    w = synth.small_event(72, 3, 100_003, 256, 9, delta_f=1.0 / 64.0)
    # tables and D take 9.6 MB, the partial sums 0.05 MB on bins and 3.2 MB on nodes
    ws = _pinned(gw, 200_000)
    assert 10.5e6 < ws.nbytes < 11.0e6
    data = oracle.workload_data(w)
    events, _, rows = gw.make_events([w.grid], [w.tensors], [w.vertices], [256])
    args = (events, 1, _dev(data.ravel()), _dev(w.psd.ravel()), _dev(w.theta))
    got = gw.lnl_ragged(*args, workspace=ws).cpu().numpy()
    _check(w, data, np.array([0, 100, 255]), got)
    np.testing.assert_array_equal(gw.lnl_ragged(*args, workspace=ws).cpu().numpy(), got)
