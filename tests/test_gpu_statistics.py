"""GPU: the level and ensemble statistics at the edges of their kernels'
tiles: samples per thread and threads per cell (mlmc_level_estimate), sort
widths (henry_sample_stats), against numpy in FP64."""
import numpy as np
import pytest

import henry_inputs as hi

pytestmark = pytest.mark.gpu


def _estimate(hm, torch, ctx, grids, m, rng):
    dev = "cuda:0"
    cells = [g[0] * g[1] for g in grids]
    cf = [rng.uniform(0, 1, (ml, n)) for ml, n in zip(m, cells)]
    cc = [None] + [rng.uniform(0, 1, (ml, n // 4)) for ml, n in zip(m[1:], cells[1:])]
    qf = [rng.uniform(1, 2, ml) for ml in m]
    qc = [None] + [rng.uniform(1, 2, ml) for ml in m[1:]]
    up = lambda a: None if a is None else torch.tensor(a, device=dev)
    out = [torch.full((n,), float("nan"), dtype=torch.float64, device=dev) for n in cells * 2]
    L1 = len(grids)
    qs, ec, est = (torch.full((n,), float("nan"), dtype=torch.float64, device=dev) for n in (2 * L1, cells[-1], 2))
    for _ in range(2):  # a second call finds the first one's outputs
        hm.mlmc_level_estimate(ctx, grids, m, [up(a) for a in cf], [up(a) for a in cc], [up(a) for a in qf],
                               [up(a) for a in qc], out[:L1], out[L1:], qs, ec, est)
    e = v = np.zeros(1)
    for l, (g, n) in enumerate(zip(grids, cells)):
        fine = cf[l].reshape(m[l], g[1], g[0])
        if l > 0:
            fine = fine - np.repeat(np.repeat(cc[l].reshape(m[l], g[1] // 2, g[0] // 2), 2, 1), 2, 2)
            e, v = (np.repeat(np.repeat(a.reshape(g[1] // 2, g[0] // 2), 2, 0), 2, 1) for a in (e, v))
        q = qf[l] - (qc[l] if l > 0 else 0.0)
        yield out[l], fine.mean(0), out[L1 + l], fine.var(0, ddof=1)
        yield qs[2 * l:2 * l + 1], q.mean(), qs[2 * l + 1:2 * l + 2], q.var(ddof=1)
        e, v = e + fine.mean(0), v + fine.var(0, ddof=1) / m[l]
    vq = sum(qs[2 * l + 1].item() / m[l] for l in range(L1))
    yield ec, e, est, np.array([vq, v.max()])


# 2 .. 2049 samples: one per thread, the last register, and past it; 2x1
# cells: a tile that is mostly past the end; 512x256: 8 threads per cell
@pytest.mark.parametrize("grids,m", [([(2, 1, 1)], [2]), ([(2, 1, 1)], [2049]), ([(16, 8, 1)], [63]),
                                     ([(16, 8, 1), (32, 16, 1)], [2500, 65]),
                                     ([(64, 32, 1), (128, 64, 1), (256, 128, 1)], [513, 257, 3]),
                                     ([(512, 256, 1)], [31]), ([(512, 256, 1)], [257])])
def test_level_estimate(grids, m):
    """Sums of m terms of size one in a tree of 64 classes: relative rounding
    below (m / 64 + 8) 2^-53 of the terms' size, so 1e-13 bounds means of
    [0, 1) values and their variances (of size 1/12) with room."""
    import torch

    import paper_2302_07804_amd as hm
    ctx = hm.Context(hi.PHYS, 0)
    for a, ra, b, rb in _estimate(hm, torch, ctx, grids, m, np.random.default_rng(m[0])):
        assert np.abs(a.cpu().numpy() - np.ravel(ra)).max() <= 1e-13
        assert np.abs(b.cpu().numpy() - np.ravel(rb)).max() <= 1e-13
    ctx.close()


@pytest.mark.parametrize("n", [1, 2, 63, 255, 256, 257, 512, 513, 1025, 2049, 4097, 8191, 8192])
@pytest.mark.parametrize("sub", [False, True])
def test_sample_stats(n, sub):
    """Order statistics are exact (a sort moves values); their interpolation
    rounds twice.  Ties, infinities and NaN (after every number) included."""
    import torch

    import paper_2302_07804_amd as hm
    rng = np.random.default_rng(n)
    x = rng.integers(-50, 50, (n, 5)) / 8.0
    x[:, 1] = rng.uniform(-1, 1, n)
    x[rng.integers(0, n), 2] = np.inf
    x[rng.integers(0, n), 3] = np.nan
    x[:, 4] = np.sort(x[:, 4])[::-1]
    xs = rng.integers(-4, 4, (n, 5)) / 8.0 if sub else np.zeros((n, 5))
    probs = (0.0, 0.025, 0.25, 0.5, 0.8, 1.0)
    ctx = hm.Context(hi.PHYS, 0)
    up = lambda a: torch.tensor(a, device="cuda:0")
    mean, var, q = (t.cpu().numpy() for t in hm.henry_sample_stats(ctx, up(x), probs, x_sub=up(xs) if sub else None))
    y = x - xs
    srt = np.sort(y, axis=0)  # numpy sorts NaN last
    with np.errstate(invalid="ignore"):
        for k, p in enumerate(probs):
            h = (n - 1) * p
            lo = int(np.floor(h))
            hi_ = min(lo + 1, n - 1)
            ref = srt[lo] + (h - lo) * (srt[hi_] - srt[lo])
            assert np.array_equal(np.isnan(q[k]), np.isnan(ref))
            ok = np.isfinite(ref)
            assert np.array_equal(q[k][~ok & ~np.isnan(ref)], ref[~ok & ~np.isnan(ref)])
            assert np.abs(q[k][ok] - ref[ok]).max(initial=0.0) <= 1e-14 * 10
    for v in (0, 1, 4):
        assert abs(mean[v] - y[:, v].mean()) <= 1e-13
        assert abs(var[v] - (y[:, v].var(ddof=1) if n > 1 else 0.0)) <= 1e-11
    assert np.isnan(mean[3]) and not np.isfinite(mean[2])
    ctx.close()
