"""Interpolation error of the frequency nodes for chirps, on the CPU.

The weights recover a phasor of constant rate, up to 0.2 turns per node, to 4e-16
(test_node_host.py).  A template's rate falls with the frequency, and over the 32 nodes
of a bin it may change by a lot: the lowest cells of a level, whose lowest nodes
have the largest rate that a plan allows, are off by 1e-12 to 2e-10, the more the fewer
spacings there are below them; five cells up the error is 1e-13 and less.  Here every
term of the phase in turn has the largest rate, at the lowest node of a level of the
fewest cells a level may have.

Bar: what the error adds to a sum over the level's bins is at most its mean size over
them, times the sum of the terms' sizes.  That mean is held to 1e-11, a tenth of the
1e-10 that the likelihood is held to.
"""
import os
import sys

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_1904_02863_amd", "csrc")
SPACINGS = (8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512, 768, 1024)
POWERS = {"tau": 3, "c7": 2, "c6": 1, "c4": -1, "c3": -2, "c2": -3, "c0": -5}     # of u = f^(1/3)
L = np.longdouble


@pytest.fixture(scope="module")
def gen():
    sys.path.insert(0, CSRC)
    try:
        import gen_resample
    finally:
        sys.path.remove(CSRC)
    return gen_resample


def _errors(gen, coef, f_low, df, term, q):
    """|phasor - its interpolation| over the cells of a level, [cells, points]."""
    p = L(POWERS[term]) / 3
    two_pi = 2 * L("3.14159265358979323846264338327950288")
    f0 = max(0.5 * f_low, f_low - 16 * q * df)                  # the level's lowest node
    amp = L(0.2) / (L(q) * df) / (abs(p) * L(f0) ** (p - 1))
    phasor = lambda f: np.exp(1j * np.asarray(two_pi * amp * f ** p))  # noqa: E731
    n = min(q, 32)
    x = np.arange(n) * (q // n) / q
    w = gen.evaluate(coef, x).astype(L)
    cells = np.arange(40)                                       # kNodeLowCells
    at_nodes = phasor(L(f0) + np.arange(40 + gen.TAPS).astype(L) * L(q) * L(df))
    got = np.stack([w @ at_nodes[c:c + gen.TAPS] for c in cells])
    bins = L(f0) + (cells[:, None] + gen.P - 1 + x[None].astype(L)) * L(q) * L(df)
    return np.abs(got - phasor(bins)).astype(np.float64)


@pytest.mark.parametrize("f_low", [3.0, 5.0, 10.0, 20.0, 40.0])
def test_chirps(gen, f_low):
    coef = gen.polynomials()
    mean, bin_ = dict.fromkeys(POWERS, 0.0), dict.fromkeys(POWERS, 0.0)
    for term in POWERS:
        for df in (1.0 / 4.0, 1.0 / 64.0, 1.0 / 512.0):
            for q in SPACINGS:
                e = _errors(gen, coef, f_low, df, term, q)
                mean[term], bin_[term] = max(mean[term], e.mean()), max(bin_[term], e.max())
    print(f"mean over a level {max(mean.values()):.1e}, one bin {max(bin_.values()):.1e}")
    assert max(mean.values()) <= 1e-11
    assert bin_["tau"] <= 1e-15            # a constant rate (4e-16, and the sums' rounding)
    assert bin_["c0"] >= 1e-13             # the falling rate costs the lowest cells digits
