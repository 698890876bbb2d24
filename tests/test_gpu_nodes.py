"""The split-form likelihood on frequency nodes (csrc/gw_nodes.h) against the
CPU oracle, where its geometry and its plan can go wrong: the smallest bands
that take nodes and one bin either side, every detector count (each packs
the matrix instruction's columns its own way), bands that leave single bins below
the levels or end inside a cell, batches of one row, of rows without spread, of more
rows than the plan reads ranges for, batches whose arrival times lie late in the segment
(a reference carrier) or are spread so far that no level applies, rows outside the
domain among valid ones, and one far-off row.

Bar: the repository's FP64 bar, 1e-10 of lnL for every row, and for noise-free
data (where lnL is not dominated by <d,d>) 1e-10 of <d,d>; the nodes recover a
bin's phasor to 4e-16, so the sums differ from direct ones by FP64 rounding.
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

RTOL = 1e-10


@pytest.fixture(scope="module")
def gw():
    import torch
    import paper_1904_02863_amd as gw
    assert torch.cuda.is_available(), "these tests need the GPU"
    gw.load_library()
    return gw


def _lnl(gw, grid, w, data, theta, precision="fp64", flags=0):
    import torch
    dev = torch.device("cuda", 0)
    ws = gw.Workspace(0)
    ws.set_tuning(False)
    out = gw.lnl_batch(grid, w.tensors, w.vertices, torch.from_numpy(np.ascontiguousarray(data)).to(dev),
                       torch.from_numpy(np.array(w.psd)).to(dev),
                       torch.from_numpy(np.ascontiguousarray(theta)).to(dev), precision=precision, flags=flags,
                       workspace=ws)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def _ref(w, data, theta):
    g = w.grid
    return oracle.lnl(g.f_low, g.delta_f, g.n_bins, w.tensors, w.vertices, data, w.psd, theta)


def _rows(kind, w, rng):
    th = np.array(w.theta)
    if kind == "same":
        th[:] = th[0]
    elif kind == "narrow":
        th = synth.near_fiducial(th[0], len(th), rng)
    elif kind == "late":                       # merger late in the segment
        th[:, 4] += 0.9 / w.grid.delta_f
    elif kind == "scattered":                  # arrival times all over the segment: single bins only
        th[:, 4] = rng.uniform(0.0, 1.0 / w.grid.delta_f, len(th))
    elif kind == "outlier":                    # one light binary among heavy ones
        th[len(th) // 2, 0] = 0.9
    elif kind == "invalid":
        th[0, 0], th[1, 1], th[2, 2], th[3, 4] = -1.0, 1.5, np.nan, np.inf
        th[4] = th[5]
    return th


# (kind of rows, detectors, 1/delta_f, f_low, bins, rows, parameters)
CASES = [
    ("prior", 3, 8, 20.0, 8191, 70, 9),
    ("prior", 3, 8, 20.0, 8192, 70, 9),
    ("prior", 3, 8, 20.0, 8193, 1, 9),
    ("prior", 1, 64, 20.0, 60_001, 130, 5),
    ("prior", 2, 64, 20.0, 50_000, 64, 9),
    ("prior", 4, 64, 20.0, 40_003, 65, 9),
    ("prior", 5, 32, 20.0, 20_011, 33, 9),
    ("prior", 6, 32, 15.0, 20_000, 33, 9),
    ("prior", 7, 32, 20.0, 20_001, 20, 9),
    ("prior", 8, 128, 20.0, 30_007, 20, 9),
    ("same", 3, 128, 10.0, 100_003, 9, 9),
    ("narrow", 3, 256, 20.0, 90_001, 40, 9),
    ("late", 3, 64, 20.0, 64_001, 50, 9),
    ("scattered", 2, 64, 20.0, 20_000, 40, 9),
    ("outlier", 3, 64, 20.0, 60_000, 60, 9),
    ("invalid", 3, 64, 20.0, 40_001, 66, 9),
    ("prior", 3, 16, 20.0, 16_225, 16_449, 9),
]


@pytest.mark.parametrize("kind,n_det,duration,f_low,n_bins,n_rows,n_param", CASES)
def test_nodes_match_oracle(gw, kind, n_det, duration, f_low, n_bins, n_rows, n_param):
    print(f"{kind} det {n_det} 1/df {duration} bins {n_bins} rows {n_rows}", flush=True)
    w = synth.small_event(60 + n_det, n_det, n_bins, n_rows, n_param, f_low=f_low, delta_f=1.0 / duration)
    rng = np.random.default_rng(n_bins)
    th = _rows(kind, w, rng)
    # the oracle on a spread of rows (all of them in the small batches)
    pick = np.unique(np.linspace(0, n_rows - 1, min(n_rows, 66)).astype(int))
    data = oracle.workload_data(w)
    got, ref = _lnl(gw, w.grid, w, data, th)[pick], _ref(w, data, th[pick])
    np.testing.assert_array_equal(np.isnan(got), np.isnan(ref))
    np.testing.assert_array_equal(np.isinf(got), np.isinf(ref))
    ok = np.isfinite(ref)
    err = np.abs(got[ok] - ref[ok])
    print(f"  noise: worst {np.max(err / np.abs(ref[ok])):.2e} of lnL", flush=True)
    assert (err <= RTOL * np.abs(ref[ok])).all()
    # the signal alone
    h = oracle.waveform(w.grid.f_low, w.grid.delta_f, n_bins, w.tensors, w.vertices, w.theta_inj[None])[0]
    far = np.array(w.theta_inj)[None].copy()
    far[0, 2] = 1e30
    dd = -2.0 * _ref(w, h, far)[0]
    got, ref = _lnl(gw, w.grid, w, h, th)[pick], _ref(w, h, th[pick])
    scale = np.maximum(dd, np.abs(ref[ok]))
    err = np.abs(got[ok] - ref[ok])
    print(f"  signal: worst {np.max(err / scale):.2e} of <d,d> = {dd:.3g}", flush=True)
    assert (err <= RTOL * scale).all()


def test_mixed_precision_and_norm_on_nodes(gw):
    """The mixed path keeps its bar of 1e-3 in lnL against the oracle; GW_FLAG_ADD_NORM
    subtracts the same constant from every row."""
    w = synth.small_event(71, 3, 60_000, 300, 9, delta_f=1.0 / 64.0)
    data = oracle.workload_data(w)
    mixed = _lnl(gw, w.grid, w, data, w.theta, precision="mixed")
    assert np.abs(mixed[:40] - _ref(w, data, w.theta[:40])).max() <= 1e-3
    norm = float(np.sum(np.log(2.0 * np.pi * w.psd)))
    a = _lnl(gw, w.grid, w, data, w.theta)
    b = _lnl(gw, w.grid, w, data, w.theta, flags=gw.FLAG_ADD_NORM)
    assert np.all(np.abs(b - (a - norm)) <= 1e-12 * abs(norm))


def test_bad_psd_makes_every_row_nan_on_nodes(gw):
    w = synth.small_event(72, 2, 30_000, 20, 9, delta_f=1.0 / 64.0)
    data = oracle.workload_data(w)
    w.psd = np.array(w.psd)
    w.psd[1, 29_999] = 0.0
    assert np.isnan(_lnl(gw, w.grid, w, data, w.theta)).all()
