"""GPU: henry_sample_stats at the largest number of columns a launch of one
256-thread block per column can have (2^24 - 1; the launch's threads are
counted in 32 bits), and at column counts that do not divide by the eight
XCDs its blocks are dealt to, against torch in FP64 (two samples: the mean is
half their sum, the variance half their difference squared, the median the
mean; each to a few units of roundoff, 1e-15 of numbers below 2)."""
import pytest

import henry_inputs as hi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nvals", [1, 2, 7, 8, 9, 15, 17, 1001, 2 ** 24 - 1])
def test_every_column_once(nvals):
    import torch

    import paper_2302_07804_amd as hm
    ctx = hm.Context(hi.PHYS, 0)
    g = torch.Generator(device="cuda:0").manual_seed(nvals)
    x = 1.0 + torch.rand((2, nvals), dtype=torch.float64, device="cuda:0", generator=g)
    mean, var, _ = hm.henry_sample_stats(ctx, x)
    m = 0.5 * (x[0] + x[1])
    assert (mean - m).abs().max() <= 1e-15
    assert (var - 0.5 * (x[0] - x[1]) ** 2).abs().max() <= 1e-15
    mean2, var2, q = hm.henry_sample_stats(ctx, x, probs=(0.5,))
    assert torch.equal(mean2, mean) and torch.equal(var2, var)
    assert (q[0] - m).abs().max() <= 1e-15
    ctx.close()
