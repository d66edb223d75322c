"""GPU: a sample's gradient does not depend on how many others are in its
batch, also past the number of solves above which the built-in workgroup is
half as large (the sums over cells are taken by thread)."""
import pytest

import henry_inputs as hi

pytestmark = pytest.mark.gpu

KEYS = ("qoi", "dq_dxi", "dq_dq", "dq_dlogk", "dq_dphi", "iters", "status")


@pytest.mark.parametrize("nx,model,prec", [(4, None, 1), (16, None, 1), (16, "kl", 1), (32, None, 0), (32, "two_layer", 1),
                                           (32, "kl", 0), (64, None, 1), (64, "two_layer", 0), (64, "kl", 1)])
def test_gradient_does_not_depend_on_the_batch(nx, model, prec):
    import torch

    import paper_2302_07804_amd as hm
    ctx = hm.Context(dict(hi.PHYS, T=360.0 * 2 / max(1, nx // 16)), 0)
    if model == "kl":
        ctx.set_kl(nx, nx // 2)
        xi = hm.henry_sample_xi_kl(7, 0, 0, 257)
    else:
        xi = hm.henry_sample_xi(7, 0, 0, 257, 3)
    xi = torch.tensor(xi, device="cuda:0")

    def first(n):
        a = hm.adjoint(ctx, [(nx, nx // 2, 2)] * n, xi=xi[:n].contiguous(), opts=hm.make_opts(prec=prec, max_outer=60),
                       ckpt_every=2, model="two_layer" if model == "two_layer" else None)
        return {k: a[k].view(n, -1)[:2].cpu() for k in KEYS}

    few, most, more = first(2), first(256), first(257)
    ctx.close()
    assert (few["status"] == 0).all()
    for k in KEYS:
        assert torch.equal(most[k], few[k]), k
        assert torch.equal(more[k], few[k]), k
