"""GPU: henry_residual_batch either side of the width from which it forms the
face coefficients from K and phi and loads four rows ahead (128 columns), and
at the largest, where a thread's band has more rows than a wavefront has
lanes, with the caller's own rough fields, against the oracle.  Both sides
are FP64 and add the same face terms, possibly in another order: the bar is
the smaller grids', 1e-13 of the largest |R| of each solve and equation."""
import numpy as np
import pytest

import henry_inputs as hi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", [64, 128, 512, 1024])
def test_residual_of_rough_fields(nx):
    import torch

    import oracle
    import paper_2302_07804_amd as hm
    ny, steps, n = nx // 2, 100, 2
    rng = np.random.default_rng(nx)
    phi = 0.35 * (1 + 0.2 * rng.uniform(-1, 1, (n, ny, nx)))
    logk = np.log(hi.PHYS["k0"]) + 0.6 * rng.uniform(-1, 1, (n, ny, nx))
    q = hi.PHYS["q_in"] * (1 + 0.2 * rng.uniform(-1, 1, n))
    y = -1.0 + (np.arange(ny)[:, None] + 0.5) / ny
    c, cn = rng.uniform(0, 1, (n, ny, nx)), rng.uniform(0, 1, (n, ny, nx))
    p = -1010.0 * 9.81 * y + 50.0 * rng.uniform(-1, 1, (n, ny, nx))
    ctx = hm.Context(hi.PHYS, 0)
    dev = lambda a: torch.tensor(np.ascontiguousarray(a).ravel(), device="cuda:0")
    got = hm.residual(ctx, [(nx, ny, steps)] * n, dev(p), dev(c), dev(cn), phi=dev(phi), logk=dev(logk), qin=dev(q))
    got = [g.cpu().numpy().reshape(n, ny, nx) for g in got]
    ctx.close()
    for k in range(n):
        want = oracle.residual(hi.PHYS, steps, phi[k], np.exp(logk[k]), q[k], p[k], c[k], cn[k])
        for g, w in zip(got, want):
            assert np.abs(g[k] - w).max() <= 1e-13 * np.abs(w).max()
