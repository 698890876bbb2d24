"""gw_pop_lnl where its weights take another form or its launch another shape:
mass-ratio indices on both sides of those whose samples share a division, samples
just above the smallest mass (where the mass ratio's normalisation is a small
difference), spin magnitudes of exactly 0 and 1, sample counts at the edges of
a block's share, and few enough blocks that the points are shared out.

Bar: the oracle's and the kernel's weights are products of a few exponentials
whose exponents (below 100) are sums of at most 8 rounded terms, so ln of a mean of
positive weights agrees to 8 * 100 * 2^-53 = 1e-13; a sample whose q_min is 1 - x
carries in addition the rounding of ln m_min - ln m1 (about 1e-15) over x.
"""
import numpy as np
import pytest

import synth
from oracle import population as pop

pytestmark = pytest.mark.gpu

BETAS = (-3.0, -1.0 - 1e-6, -1.0, -1.0 + 0.9e-3, -1.0 + 1.1e-3, 0.0, 1.7, 12.0)


def _run(samples, hyper, prepared=False):
    import torch
    import paper_1904_02863_amd as gw
    dev = torch.device("cuda", 0)
    s = torch.from_numpy(np.ascontiguousarray(samples)).to(dev)
    out = gw.pop_lnl(gw.pop_prepare(s) if prepared else s, torch.from_numpy(np.ascontiguousarray(hyper)).to(dev))
    return out.cpu().numpy()


def _hyper(betas):
    h = np.tile([2.1, 0.0, 5.0, 80.0, 0.1, 35.0, 4.0, 1.6, 2.4, 0.6, 0.9, 1.3], (len(betas), 1))
    h[:, 1] = betas
    return h


def _samples(rng, n_events, n_per):
    s = np.empty((7, n_events, n_per))
    s[0] = rng.uniform(6.0, 70.0, (n_events, n_per))
    s[1] = rng.uniform(0.05, 1.0, (n_events, n_per))
    s[2:4] = rng.uniform(0.0, 1.0, (2, n_events, n_per))
    s[4:6] = rng.uniform(-1.0, 1.0, (2, n_events, n_per))
    s[6] = -5.0
    return s


@pytest.mark.parametrize("n_events,n_per", [(1, 1), (1, 255), (2, 256), (3, 257), (1, 1023), (1, 1025), (40, 70)])
def test_every_form_of_the_mass_ratio(n_events, n_per):
    rng = np.random.default_rng(n_per)
    s = _samples(rng, n_events, n_per)
    s[1, :, 0], s[0, :, 0] = 0.9, 20.0            # every event keeps a sample inside the support
    h = _hyper(BETAS)
    ref = pop.lnl(s, h)
    for prepared in (False, True):
        got = _run(s, h, prepared)
        assert np.isfinite(ref).all()
        # the oracle's normalisation near beta = -1 is (1 - q_min^(1 + beta)) / (1 + beta): its 1 - q_min^(1 + beta)
        # keeps an absolute error of about 1e-16 (q_min below 5/6 here)
        own = np.array([0.0 if b == -1.0 else 1e-15 / (abs(1.0 + b) * 0.18) for b in BETAS])
        assert (np.abs(got - ref) <= n_events * (1e-13 * np.maximum(1.0, np.abs(ref)) + own)).all()


@pytest.mark.parametrize("x", [1e-5, 1e-3, 2.5e-3, 3e-2])
def test_samples_just_above_the_smallest_mass(x):
    s = _samples(np.random.default_rng(3), 1, 1)
    s[0], s[1] = 5.0 / (1.0 - x), 1.0 - 0.25 * x
    h = _hyper((-2.5, -1.0, 0.0, 3.0))
    ref = pop.lnl(s, h)
    got = _run(s, h)
    assert (np.abs(got - ref) <= 1e-13 * np.maximum(1.0, np.abs(ref)) + 1e-15 / x).all(), np.abs(got - ref).max()


def test_spin_magnitudes_at_their_ends():
    """A Beta density above 1 vanishes at the ends: those samples weigh nothing."""
    s = _samples(np.random.default_rng(4), 1, 300)
    s[1], s[0] = 0.9, 20.0
    h = _hyper((1.0, -2.0))
    keep = np.ones(300, bool)
    s[2, 0, 10], s[3, 0, 11], s[2, 0, 12] = 0.0, 1.0, 1.0
    keep[10:13] = False
    got, ref = _run(s, h), pop.lnl(s[:, :, keep], h) + np.log(297.0 / 300.0)
    assert (np.abs(got - ref) <= 1e-13 * np.maximum(1.0, np.abs(ref))).all()
