"""GPU: one multigrid cycle of each kind, as the solves run it, against the
oracle's operators and relaxations.  A solve of one step and one outer
iteration adds one pressure cycle's result to p and one transport cycle's to
c; an adjoint of one step and one transposed iteration forms its gradient
from one transposed transport cycle and one pressure cycle.  The reference
below is the cycle in FP64 on sparse matrices, so a wrong coarse coefficient,
transfer weight or line is off by its size and not only by iterations.

Bars: a cycle is about a hundred dependent phases of some ten roundings, of
which each may cost a unit of roundoff of the largest value: 1e3 * 1.1e-16,
and a hundred times that for the residual the cycle starts from, a difference
of terms larger than it: 1e-11 in FP64; 1e3 * 6e-8 in FP32.  The gradient's
reference is a central difference of the oracle's residual (step 1e-5: 1e-10
of truncation, 1e-11 of the residual's terms by rounding): 1e-7."""
import numpy as np
import pytest

import henry_inputs as hi
import oracle

pytestmark = pytest.mark.gpu

BAR = {0: 1e-11, 1: 6e-5}


def prolongation(nx, ny):
    """Bilinear, constant past the boundary: fine cells from coarse ones."""
    def one(n):
        P = np.zeros((n, n // 2))
        for i in range(n):
            I = i // 2
            P[i, I] += 0.75
            P[i, min(max(I + (1 if i & 1 else -1), 0), n // 2 - 1)] += 0.25
        return P
    return one(nx), one(ny)


def half_x(a):
    return a[:, 0::2] + a[:, 1::2]


def half_y(a):
    return a[0::2] + a[1::2]


def pressure_cycle(te, tn, b):
    """V(2,2), red-black Gauss-Seidel; exact on 2 x 1 cells."""
    ny, nx = te.shape
    A = oracle.pressure_operator(te, tn)
    if ny == 1:
        return np.linalg.solve(A.toarray(), b.ravel()).reshape(ny, nx)
    x = oracle.gauss_seidel_rb(A, b, np.zeros((ny, nx)), nx, ny, 2)
    r = b - (A @ x.ravel()).reshape(ny, nx)
    Px, Py = prolongation(nx, ny)
    tec = 0.5 * half_y(te)[:, 1::2]
    tnc = 0.5 * half_x(tn)[1::2]
    x = x + Py @ pressure_cycle(tec, tnc, Py.T @ r @ Px) @ Px.T
    return oracle.gauss_seidel_rb(A, b, x, nx, ny, 2)


def transport_cycle(parts, b, trans):
    """Even, then odd x-lines; the coarser cycle; the same again, with y-lines
    on levels of at most 512 cells."""
    acc, mx, my, dx, dy, mr, dr, dl, ml = parts
    ny, nx = acc.shape
    A = oracle.transport_operator(*parts)
    if trans:
        A = A.T.tocsr()
    x = oracle.zebra_lines(A, b, np.zeros((ny, nx)), nx, ny, 1)
    if ny == 1:
        return x
    r = b - (A @ x.ravel()).reshape(ny, nx)
    Px, Py = prolongation(nx, ny)
    coarse = (half_x(half_y(acc)), half_y(mx)[:, 1::2], half_x(my)[1::2], 0.5 * half_y(dx)[:, 1::2],
              0.5 * half_x(dy)[1::2], half_y(mr), 0.5 * half_y(dr), 0.5 * half_y(dl), half_y(ml))
    x = x + Py @ transport_cycle(coarse, Py.T @ r @ Px, trans) @ Px.T
    return oracle.zebra_lines(A, b, x, nx, ny, 1, ylines=nx * ny <= 512)


def coefficients(ph, nsteps, phi, K, q, p, c, cn):
    """The two systems' level 0 coefficients at a state (Sec. 2.3)."""
    ny, nx = phi.shape
    h = 1.0 / ny
    rho = lambda v: ph["rho0"] + (ph["rho1"] - ph["rho0"]) * v
    r = rho(c)
    harm = lambda a, b: 2.0 * a * b / (a + b)
    te, tn, mx, my, dx, dy = (np.zeros((ny, nx)) for _ in range(6))
    rf = 0.5 * (r[:, :-1] + r[:, 1:])
    te[:, :-1] = rf * harm(K[:, :-1], K[:, 1:]) / ph["mu"]
    mx[:, :-1] = -te[:, :-1] * (p[:, 1:] - p[:, :-1])
    dx[:, :-1] = rf * harm(phi[:, :-1], phi[:, 1:]) * ph["D"]
    rf = 0.5 * (r[:-1] + r[1:])
    tn[:-1] = rf * harm(K[:-1], K[1:]) / ph["mu"]
    my[:-1] = -tn[:-1] * (p[1:] - p[:-1] + rf * ph["g"] * h)
    dy[:-1] = rf * harm(phi[:-1], phi[1:]) * ph["D"]
    rs = 0.5 * (r[:, -1] + ph["rho1"])  # the seawater face, half a cell away
    te[:, -1] = rs * 2.0 * K[:, -1] / ph["mu"]
    y = -1.0 + (np.arange(ny) + 0.5) * h
    mr = -te[:, -1] * (-ph["rho1"] * ph["g"] * y - p[:, -1])
    dr = rs * 2.0 * phi[:, -1] * ph["D"]
    dl = (r[:, 0] + ph["rho0"]) * phi[:, 0] * ph["D"]
    ml = np.full(ny, ph["rho0"] * q * h)
    acc = h * h / (ph["T"] / nsteps) * phi * rho(cn)
    return (te, tn), (acc, mx, my, dx, dy, mr, dr, dl, ml)


def phys(nx):
    return dict(hi.PHYS, T=5760.0 / nx)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("nx,threads,cluster", [(2, 0, 0), (4, 0, 0), (8, 0, 0), (16, 0, 0), (32, 0, 0), (64, 0, 0),
                                                (64, 64, 1), (128, 0, 1), (128, 0, 2), (128, 256, 4)])
def test_one_pressure_and_one_transport_cycle(nx, threads, cluster, prec):
    import torch

    import paper_2302_07804_amd as hm
    ny, ph = nx // 2, phys(nx)
    xi = hm.henry_sample_xi(11, 0, 0, 1, 3)
    phi, K, q = oracle.fields_closed(ph, nx, ny, xi[0])
    X, Y = np.meshgrid((np.arange(nx) + 0.5) / ny, -1.0 + (np.arange(ny) + 0.5) / ny)
    c0 = 0.5 + 0.3 * np.sin(2.0 * X + 3.0 * Y) + 0.1 * np.random.default_rng(nx).uniform(-1, 1, (ny, nx))
    ctx = hm.Context(ph, 0)
    out = hm.solve(ctx, [(nx, ny, 1)], xi=torch.tensor(xi, device="cuda:0"), c0=torch.tensor(c0.ravel(), device="cuda:0"),
                   want_p=True, opts=hm.make_opts(prec=prec, max_outer=1, threads=threads, cluster=cluster))
    p, c = (out[k].cpu().numpy().reshape(ny, nx) for k in ("p", "c"))
    assert out["status"].item() == hm.STATUS_NOCONV
    ctx.close()
    p0 = -(ph["rho0"] + (ph["rho1"] - ph["rho0"]) * c0) * ph["g"] * Y
    (te, tn), _ = coefficients(ph, 1, phi, K, q, p0, c0, c0)
    Rp, _ = oracle.residual(ph, 1, phi, K, q, p0, c0, c0)
    dp = pressure_cycle(te, tn, -Rp)
    assert np.abs(p - p0 - dp).max() <= BAR[prec] * np.abs(dp).max()
    _, parts = coefficients(ph, 1, phi, K, q, p, c0, c0)  # at the pressure the solve has
    Rp, Rc = oracle.residual(ph, 1, phi, K, q, p, c0, c0)
    dc = transport_cycle(parts, -(Rc - c0 * Rp), False)
    assert np.abs(c - c0 - dc).max() <= BAR[prec] * np.abs(dc).max()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("nx", [2, 4, 8, 16, 32])
def test_one_transposed_cycle(nx, prec):
    import torch

    import paper_2302_07804_amd as hm
    ny, ph = nx // 2, phys(nx)
    n, h = nx * ny, 1.0 / ny
    xi = hm.henry_sample_xi(12, 0, 0, 1, 3)
    xt = torch.tensor(xi, device="cuda:0")
    phi, K, q = oracle.fields_closed(ph, nx, ny, xi[0])
    ctx = hm.Context(ph, 0)
    out = hm.solve(ctx, [(nx, ny, 1)], xi=xt, want_p=True, opts=hm.make_opts(prec=prec, max_outer=60))
    a = hm.adjoint(ctx, [(nx, ny, 1)], xi=xt, opts=hm.make_opts(prec=prec, max_outer=60), ckpt_every=1, adj_max_it=1)
    ctx.close()
    p, c = (out[k].cpu().numpy().reshape(ny, nx) for k in ("p", "c"))
    cn = np.zeros((ny, nx))
    (te, tn), parts = coefficients(ph, 1, phi, K, q, p, c, cn)
    bc = h * h * phi * (ph["rho0"] + 2.0 * (ph["rho1"] - ph["rho0"]) * c)
    bc[:, nx // 2:] = 0.0
    mu_c = transport_cycle(parts, bc, True)
    J = oracle.jacobian_dense(ph, 1, phi, K, q, p, c, cn)  # cells with y fastest, p and c interleaved
    lam = np.stack([(-c * mu_c).T.ravel(), mu_c.T.ravel()], 1).ravel()
    mu_p = pressure_cycle(te, tn, -(J.T @ lam)[0::2].reshape(nx, ny).T)
    lam_p, lam_c = mu_p - c * mu_c, mu_c

    def gradient(which):
        """-lam^T dR / d(phi or log K), per cell."""
        g, e = np.empty(n), 1e-5
        for k in range(n):
            R, d = [], []
            for s in (e, -e):
                f = [phi.copy().ravel(), K.copy().ravel()]
                f[which][k] *= np.exp(s)
                d.append(f[0][k] if which == 0 else s)
                rp, rc = oracle.residual(ph, 1, f[0].reshape(ny, nx), f[1].reshape(ny, nx), q, p, c, cn)
                R.append((lam_p * rp + lam_c * rc).sum())
            g[k] = -(R[0] - R[1]) / (d[0] - d[1])
        return g

    explicit = h * h * (ph["rho0"] + (ph["rho1"] - ph["rho0"]) * c) * c
    explicit[:, nx // 2:] = 0.0
    wants = {"dq_dphi": explicit.ravel() + gradient(0)}
    if nx > 4:  # with one or two rows the flow hardly depends on K
        wants["dq_dlogk"] = gradient(1)
    for name, want in wants.items():
        assert np.abs(a[name].cpu().numpy() - want).max() <= max(BAR[prec], 1e-7) * np.abs(want).max(), name
