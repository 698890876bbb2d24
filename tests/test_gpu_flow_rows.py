"""The one-kernel couplings where a block's rows, waves and stores have edges: row
counts around the 16 of a block, the smallest and largest dimension, both widths they
serve, chains longer than one launch, and rows read and written in place.

Bars: the inverse of the forward map returns z to 1e-9 (both see the same MLP
outputs; the FP64 couplings lose at most e^3 of the digits in each of the layers,
log-scales being tanh-bounded), every row is bitwise the one a larger batch gives,
and in place is bitwise out of place.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _flow(dim, hidden, layers):
    import paper_1904_02863_amd as gw
    from paper_1904_02863_amd import sampler
    flow = gw.Flow(dim, sampler.default_masks(dim, layers, 0), hidden=hidden, device=0)
    rng = np.random.default_rng(dim + hidden + layers)
    flow.set_params(sampler.init_flow_params(dim, hidden, layers, 5, scale_last=0.3), rng.normal(size=dim),
                    0.2 * rng.normal(size=dim))
    return flow


@pytest.mark.parametrize("dim,hidden,layers", [(2, 128, 4), (11, 256, 8), (16, 256, 3), (5, 128, 18), (16, 128, 17)])
def test_rows_at_the_edges_of_a_block(dim, hidden, layers):
    import torch
    flow = _flow(dim, hidden, layers)
    z = torch.randn((300, dim), dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(3))
    x_all, q_all = (t.clone() for t in flow.forward(z))
    for n in (1, 15, 16, 17, 33, 256, 300):
        part = z[:n].contiguous()
        x, q = flow.forward(part)
        assert torch.equal(x, x_all[:n]) and torch.equal(q, q_all[:n])
        back, q_back = flow.inverse(x)
        assert (back - part).abs().max() <= 1e-9 and (q_back - q).abs().max() <= 1e-9
        keep = x.clone()
        in_place, q_in = flow.inverse(keep, z_out=keep)
        assert torch.equal(in_place, back) and torch.equal(q_in, q_back)


@pytest.mark.parametrize("hidden,layers", [(256, 4), (128, 18)])
def test_gradients_add_over_rows(hidden, layers):
    """A mean over n rows is the mean of the halves' means: the same products in another
    grouping (FP32 sums of BF16 products, so 1e-4 of the gradient's size)."""
    import torch
    flow = _flow(11, hidden, layers)
    x = torch.randn((2 * 272, 11), dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(4))
    g, loss = (t.clone() for t in flow.gradients(x))
    a, la = (t.clone() for t in flow.gradients(x[:272].contiguous()))
    b, lb = (t.clone() for t in flow.gradients(x[272:].contiguous()))
    # the gradient of a row enters its BF16 products divided by n: halving it is exact
    assert (g - 0.5 * (a + b)).abs().max() <= 1e-4 * g.abs().max()
    assert abs(float(loss) - 0.5 * float(la + lb)) <= 1e-12 * abs(float(loss))
