"""gw_lnl_ragged on frequency nodes against the CPU oracle, where the events'
split into items can go wrong: detector counts side by side, events of a few
bins among long ones (no nodes at all), one row and rows past a block, more
rows than one plan reads ranges for, arrival times that leave an event on
single bins, and the mixed path's two passes (one of them empty for some events).

Bars: the repository's, 1e-10 of lnL for FP64 (the nodes recover a bin's phasor to
4e-16, so the sums differ from direct ones by rounding) and 1e-3 in lnL for the
mixed path; a replay of the captured pass is bitwise equal to the first.
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

# per event: (detectors, 1/delta_f, bins, rows, kind of rows)
CALLS = {
    "lengths": [(3, 64, 60_001, 300, "prior"), (3, 8, 16_225, 1, "prior"), (3, 4, 37, 257, "prior"),
                (3, 4, 1, 5, "prior"), (3, 128, 100_003, 256, "late")],
    "detectors": [(1, 64, 60_001, 70, "prior"), (8, 32, 9_001, 20, "prior"), (2, 32, 30_000, 64, "prior"),
                  (4, 64, 40_003, 65, "prior"), (3, 64, 50_000, 33, "prior"), (5, 16, 8_192, 3, "prior")],
    "rows": [(2, 16, 16_225, 16_500, "prior"), (2, 64, 40_000, 1, "prior"), (1, 16, 20_000, 511, "prior")],
    "spread": [(3, 64, 60_000, 40, "scattered"), (3, 64, 60_000, 40, "prior"), (2, 4, 2_000, 40, "prior")],
}


def _call(gw, name, precision, flags=0):
    import torch
    evs, datas, thetas = [], [], []
    for i, (n_det, duration, n_bins, n_rows, kind) in enumerate(CALLS[name]):
        w = synth.small_event(80 + i, n_det, n_bins, n_rows, 9, delta_f=1.0 / duration)
        th = np.array(w.theta)
        if kind == "late":
            th[:, 4] += 0.9 * duration
        elif kind == "scattered":
            th[:, 4] = np.random.default_rng(i).uniform(0.0, duration, n_rows)
        evs.append(w)
        datas.append(oracle.workload_data(w))
        thetas.append(th)
    events, _, rows = gw.make_events([w.grid for w in evs], [w.tensors for w in evs], [w.vertices for w in evs],
                                     [len(t) for t in thetas])
    dev = torch.device("cuda", 0)
    pack = lambda a: torch.from_numpy(np.concatenate([x.ravel() for x in a])).to(dev)  # noqa: E731
    data, psd = pack(datas), pack([np.array(w.psd) for w in evs])
    theta = torch.from_numpy(np.concatenate(thetas)).to(dev)
    ws, out = gw.Workspace(0), torch.zeros(rows, dtype=torch.float64, device=dev)
    got = []
    for _ in range(2):
        out.fill_(7.0)
        gw.lnl_ragged(events, len(evs), data, psd, theta, precision=precision, flags=flags, out=out, workspace=ws)
        torch.cuda.synchronize()
        got.append(out.cpu().numpy())
    np.testing.assert_array_equal(got[0], got[1])
    return evs, datas, thetas, got[0]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("name", list(CALLS))
def test_ragged_nodes_match_oracle(name, precision):
    import paper_1904_02863_amd as gw
    print(f"{name} {precision}", flush=True)
    evs, datas, thetas, got = _call(gw, name, precision)
    row = 0
    for w, data, th in zip(evs, datas, thetas):
        pick = np.unique(np.linspace(0, len(th) - 1, min(len(th), 20)).astype(int))
        g = w.grid
        ref = oracle.lnl(g.f_low, g.delta_f, g.n_bins, w.tensors, w.vertices, data, w.psd, th[pick])
        err = np.abs(got[row + pick] - ref)
        if precision == "fp64":
            assert (err <= 1e-10 * np.abs(ref)).all(), (g.n_bins, err.max())
        else:
            assert err.max() <= 1e-3, (g.n_bins, err.max())
        row += len(th)
    assert row == len(got)


def test_ragged_nodes_norm_flag():
    import paper_1904_02863_amd as gw
    evs, _, thetas, plain = _call(gw, "spread", "fp64")
    normed = _call(gw, "spread", "fp64", flags=gw.FLAG_ADD_NORM)[3]
    norm = np.repeat([float(np.sum(np.log(2.0 * np.pi * w.psd))) for w in evs], [len(t) for t in thetas])
    assert (np.abs(normed - (plain - norm)) <= 1e-12 * np.abs(norm)).all()
