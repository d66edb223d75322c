"""GPU: calls that leave the number of workgroups per solve to the library
and shared no solve on 128x64 cells before the built-in choice took clusters
there do not report HENRY_STATUS_SYNC: a bound on the members' waits that is
below the time they need (1 us) changes neither the status nor a bit."""
import pytest

import henry_inputs as hi

pytestmark = pytest.mark.gpu

PTS = [(1.0, -0.5), (1.6, -0.9)]


def _ctx(hm, nsteps):
    return hm.Context(dict(hi.PHYS, T=45.0 * nsteps), 0)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("beside,spl", [(0, 0), (0, 1), (3, 0), (3, 2)])
def test_solves_with_a_short_wait(prec, beside, spl):
    import torch

    import paper_2302_07804_amd as hm
    ctx = _ctx(hm, 4)
    solves = [(128, 64, 4)] * 5 + [(16, 8, 4)] * beside
    xi = torch.tensor(hm.henry_sample_xi(8, 0, 0, len(solves), 3), device="cuda:0")

    def run(**kw):
        out = hm.solve(ctx, solves, xi=xi, want_p=True, trace=(2, PTS),
                       opts=hm.make_opts(prec=prec, max_outer=60, steps_per_launch=spl, **kw))
        return {k: out[k].cpu() for k in ("c", "p", "qoi", "status", "iters", "trace")}

    ref, got = run(cluster=1), run(cluster_wait_us=1)
    ctx.close()
    assert (ref["status"] == 0).all()
    for k in ref:
        assert torch.equal(got[k], ref[k]), k


@pytest.mark.parametrize("prec", [0, 1])
def test_adjoints_with_a_short_wait(prec):
    import torch

    import paper_2302_07804_amd as hm
    ctx = _ctx(hm, 2)
    xi = torch.tensor(hm.henry_sample_xi(8, 0, 0, 3, 3), device="cuda:0")

    def run(**kw):
        a = hm.adjoint(ctx, [(128, 64, 2)] * 3, xi=xi, opts=hm.make_opts(prec=prec, max_outer=60, **kw), ckpt_every=1)
        return {k: a[k].cpu() for k in ("qoi", "dq_dxi", "dq_dq", "dq_dlogk", "dq_dphi", "status", "iters")}

    ref, got = run(cluster=1), run(cluster_wait_us=1)
    ctx.close()
    assert (ref["status"] == 0).all()
    for k in ref:
        assert torch.equal(got[k], ref[k]), k


@pytest.mark.parametrize("prec", [0, 1])
def test_initial_state_overwritten_by_the_result(prec):
    """A resumed solve whose c_out is its c0: the second attempt starts from
    c0 too."""
    import torch

    import paper_2302_07804_amd as hm
    ctx = _ctx(hm, 3)
    solves = [(128, 64, 3)] * 2
    n = 2 * 128 * 64
    f64 = dict(dtype=torch.float64, device="cuda:0")
    xi = torch.tensor(hm.henry_sample_xi(9, 0, 0, 2, 3), device="cuda:0")
    c0 = 0.5 * torch.rand(n, generator=torch.Generator(device="cuda:0").manual_seed(1), **f64)

    def run(**kw):
        o = hm.make_opts(prec=prec, max_outer=60, **kw)
        c, q, st = c0.clone(), torch.empty(2, **f64), torch.empty(2, dtype=torch.int32, device="cuda:0")
        ws = hm.aligned_workspace(hm.henry_workspace_bytes(solves, o), torch.device("cuda:0"))
        hm.henry_solve_batch(ctx, solves, hm.FIELD_CLOSED3, xi=xi, c0=c, opts=o, c_out=c, qoi_out=q, status=st, workspace=ws)
        return c.cpu(), q.cpu(), st.cpu()

    ref, got = run(cluster=1), run(cluster_wait_us=1)
    ctx.close()
    assert (ref[2] == 0).all()
    for a, b in zip(ref, got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("prec", [0, 1])
def test_gradient_over_the_coefficients(prec):
    """The two-layer gradient reads xi again at the end, where dq_dxi may
    overwrite it."""
    import torch

    import paper_2302_07804_amd as hm
    ctx = _ctx(hm, 2)
    solves = [(128, 64, 2)] * 2
    f64 = dict(dtype=torch.float64, device="cuda:0")
    x0 = torch.tensor(hm.henry_sample_xi(9, 0, 0, 2, 3), device="cuda:0")

    def run(**kw):
        o = hm.make_opts(prec=prec, max_outer=60, **kw)
        xi, q, st = x0.clone(), torch.empty(2, **f64), torch.empty(2, dtype=torch.int32, device="cuda:0")
        ws = hm.aligned_workspace(hm.henry_adjoint_workspace_bytes(solves, o, 1), torch.device("cuda:0"))
        hm.henry_adjoint_batch(ctx, solves, hm.FIELD_TWOLAYER3, xi=xi, opts=o, ckpt_every=1, qoi_out=q, dq_dxi=xi,
                               status=st, workspace=ws)
        return xi.cpu(), q.cpu(), st.cpu()

    ref, got = run(cluster=1), run(cluster_wait_us=1)
    ctx.close()
    assert (ref[2] == 0).all()
    for a, b in zip(ref, got):
        assert torch.equal(a, b)
