"""GPU: the levels that one wavefront runs alone (henry_wave.hpp).  Every
width that can be the first of them (2 to 32 columns), below them nothing,
above them a level of the whole workgroup (64x32), in both precisions,
forward and transposed, against the oracle."""
import numpy as np
import pytest

import henry_inputs as hi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("nx,nsteps", [(2, 6), (4, 6), (8, 6), (16, 6), (32, 4), (64, 2)])
def test_solve_matches_oracle(nx, nsteps, prec):
    """A step stops at a scaled residual of 1e-10, of which c keeps about as
    much; 1e-8 is the parity bar of the FP64 and mixed solves."""
    import torch

    import oracle
    import paper_2302_07804_amd as hm
    ph = dict(hi.PHYS, T=360.0 * nsteps / max(1, nx // 16))
    xi = hm.henry_sample_xi(3, 0, 0, 5, 3)
    ctx = hm.Context(ph, 0)
    out = hm.solve(ctx, [(nx, nx // 2, nsteps)] * 5, xi=torch.tensor(xi, device="cuda:0"),
                   opts=hm.make_opts(prec=prec, max_outer=60))
    assert (out["status"].cpu().numpy() == 0).all()
    c = out["c"].cpu().numpy().reshape(5, nx // 2, nx)
    for k in range(5):
        ref = oracle.solve_xi(ph, nx, nx // 2, nsteps, xi[k])
        assert np.abs(c[k] - ref["c"]).max() <= 1e-8 * np.abs(ref["c"]).max()
    ctx.close()


@pytest.mark.parametrize("nx,nsteps", [(2, 3), (4, 4), (8, 4), (16, 4), (32, 3)])
def test_adjoint_matches_oracle(nx, nsteps):
    """The transposed cycles; the transposed systems are solved to 1e-10."""
    import torch

    import oracle
    import paper_2302_07804_amd as hm
    ph = dict(hi.PHYS, T=360.0 * nsteps / max(1, nx // 16))
    xi = hm.henry_sample_xi(4, 0, 0, 2, 3)
    ctx = hm.Context(ph, 0)
    a = hm.adjoint(ctx, [(nx, nx // 2, nsteps)] * 2, xi=torch.tensor(xi, device="cuda:0"),
                   opts=hm.make_opts(max_outer=60), ckpt_every=2)
    assert (a["status"].cpu().numpy() == 0).all()
    for k in range(2):
        _, dxi, _ = oracle.adjoint_xi(ph, nx, nx // 2, nsteps, xi[k])
        assert np.abs(a["dq_dxi"][k].cpu().numpy() - dxi).max() <= 1e-6 * np.abs(dxi).max()
    ctx.close()
