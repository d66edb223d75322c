"""GPU: the ways a multigrid level is smoothed and transferred -- passes over
global memory, cells held in registers (one, two or four per thread and
colour), x-lines of 16, 32 or 64 lanes in one or several passes, strips with
a halo in LDS (four or eight cells per thread), a level handed to the leader's
LDS -- are chosen from the grid, the workgroup and the cluster.  The general
path, which one wavefront per solve takes on every level of more than 512
cells, is the reference: every choice gives its bits."""
import pytest

import henry_inputs as hi

pytestmark = pytest.mark.gpu

PREC_FP64, PREC_MIXED = 0, 1
KEYS = ("c", "qoi", "iters", "status")


def run(nx, nsteps, prec, threads, cluster, nsolves=2, **opts):
    import torch

    import paper_2302_07804_amd as hm
    ctx = hm.Context(dict(hi.PHYS, T=360.0 * nsteps / (nx // 16)), 0)
    xi = torch.tensor(hm.henry_sample_xi(5, 0, 0, nsolves, 3), device="cuda:0")
    out = hm.solve(ctx, [(nx, nx // 2, nsteps)] * nsolves, xi=xi,
                   opts=hm.make_opts(prec=prec, threads=threads, cluster=cluster, max_outer=60, **opts))
    out = {k: out[k].cpu() for k in KEYS}
    ctx.close()
    return out


def same(a, b):
    import torch
    return [k for k in KEYS if not torch.equal(a[k], b[k])]


@pytest.mark.parametrize("prec", [PREC_FP64, PREC_MIXED])
@pytest.mark.parametrize("nx,nsteps", [(64, 4), (128, 3), (256, 2), (512, 1)])
def test_every_path_gives_the_general_paths_bits(nx, nsteps, prec):
    ref = run(nx, nsteps, prec, 64, 1)
    assert (ref["status"] == 0).all()
    for threads in (64, 128, 256, 512) + ((1024,) if prec == PREC_MIXED else ()):
        for cluster in (1, 2, 4, 8):
            assert not same(run(nx, nsteps, prec, threads, cluster), ref), (threads, cluster)


@pytest.mark.parametrize("nx,nsolves", [(16, 513), (32, 513), (64, 513), (64, 1), (128, 33), (128, 65)])
def test_built_in_choice_gives_the_general_paths_bits(nx, nsolves):
    """Either side of the batch sizes at which the built-in workgroup and
    cluster sizes change; the launches of a chunked solve start from the
    stored state."""
    ref = run(nx, 2, PREC_MIXED, 64, 1, nsolves)
    assert not same(run(nx, 2, PREC_MIXED, 0, 0, nsolves), ref)
    assert not same(run(nx, 2, PREC_MIXED, 0, 0, nsolves, steps_per_launch=1), ref)


@pytest.mark.parametrize("nx,nsteps", [(64, 3), (128, 2), (256, 2)])
def test_adjoint_paths_agree(nx, nsteps):
    """The transposed cycles, whose levels take registers and lines but no
    strips: the gradient of every workgroup and cluster size.  The sums over
    cells are taken by thread, so they agree to rounding, not to the bit: sums
    of at most 32768 FP64 terms, whose order changes them by less than 32768
    times the unit roundoff (4e-12) of the sum of their magnitudes, a hundred
    times the largest entry at most."""
    import torch

    import paper_2302_07804_amd as hm
    ctx = hm.Context(dict(hi.PHYS, T=360.0 * nsteps / (nx // 16)), 0)
    xi = torch.tensor(hm.henry_sample_xi(6, 0, 0, 2, 3), device="cuda:0")

    def grad(threads, cluster):
        a = hm.adjoint(ctx, [(nx, nx // 2, nsteps)] * 2, xi=xi,
                       opts=hm.make_opts(threads=threads, cluster=cluster, max_outer=60), ckpt_every=2)
        assert (a["status"].cpu() == 0).all()
        return a["dq_dxi"].cpu()

    ref = grad(64, 1)
    for threads in (128, 256, 512):
        for cluster in (1, 2, 4):
            g = grad(threads, cluster)
            assert (g - ref).abs().max() <= 4e-10 * ref.abs().max(), (threads, cluster)
    ctx.close()
