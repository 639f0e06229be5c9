"""Transposed extraction inside the adjoint passes with several points on one
theta row of a tile: up to the number the passes take at a grid point (3) and
beyond it (the unfused route), points sharing a column, rows at the poles and
at tile edges, many points along a row.  A gradient that is not finite reaches
no more of the cotangents than the stencils carry it to.  Cotangents against the oracle's reverse pass, and by one and two steps per
pass bit for bit."""
import math

import numpy as np
import pytest

from paper_1010_3816_amd import inputs

TOL = 1e-11  # cotangents against the oracle, normwise (the reverse pass's bar)


@pytest.mark.gpu
@pytest.mark.parametrize("npts,cols,row,rows,n", [
    (1, [60.0], 5.3, 5, 4),
    (2, [59.5, 60.25], 4.0, 5, 5),
    (3, [59.5, 60.25, 61.0], 9.6, 5, 6),
    (3, [2.5, 2.5, 63.75], -0.3, 1, 3),       # below the first row centre: the pole's ghost
    (4, [59.5, 60.25, 61.0, 90.0], 5.3, 16, 4),
    (4, [59.5, 60.25, 60.5, 61.0], 5.3, 16, 4),  # more than the passes take: unfused
    (16, [8.0 * k + 0.5 for k in range(16)], 8.4, 16, 5),
    (5, [10.5, 20.0, 30.0, 40.0, 50.0], 18.2, 7, 5),
])
def test_points_on_one_row(gpu, npts, cols, row, rows, n):
    import torch

    import oracle

    a, s, m, nr, nth = 0.6, -2, 1, 130, 20
    rmin, rmax = -40.0, 60.0
    dr, dth = (rmax - rmin) / (nr - 1), math.pi / nth
    er = [rmin + c * dr for c in cols]
    et = [max((row + 0.5) * dth, 0.0)] * npts
    dt = inputs.stable_dt(dr, nth, m, s, 1000)
    rng = np.random.default_rng(npts * 100 + n)
    gs = rng.standard_normal((n, npts)) + 1j * rng.standard_normal((n, npts))
    lam = inputs.random_state(nr, nth, seed=3)
    out = []
    for spp in (1, 2):
        g = gpu.TeukGrid(a, s, m, nr, nth, rmin, rmax, dt, extract_rstar=er, extract_theta=et)
        g.enable_adjoint()
        g.set_adjoint_tile(rows, 4)
        g.set_steps_per_pass(spp)
        lp, lq = (torch.from_numpy(x.copy()).cuda() for x in lam)
        g.adjoint(n, lp, lq, torch.from_numpy(gs).cuda(), None, project_initial=True, spin=False)
        out.append((lp.cpu().numpy(), lq.cpu().numpy()))
        g.close()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    o = oracle.OracleGrid(a, s, m, nr, nth, rmin, rmax, dt)
    p, q = lam[0].copy(), lam[1].copy()
    for k in range(n - 1, -1, -1):
        for e in range(npts):
            p = o.extract_adjoint(p, er[e], et[e], gs[k, e])
        p, q = o.adjoint_step(p, q)
    p, q = o.project(p, q)
    for got, ref in zip(out[0], (p, q)):
        assert np.abs(got - ref).max() <= TOL * np.abs(ref).max()


@pytest.mark.gpu
@pytest.mark.parametrize("spp,n", [(1, 1), (2, 2)])
def test_non_finite_gradient_stays_local(gpu, spp, n):
    """The transposed step reaches two columns; the rest keeps its values."""
    import torch

    a, s, m, nr, nth = 0.6, -2, 1, 130, 20
    rmin, rmax = -40.0, 60.0
    dr = (rmax - rmin) / (nr - 1)
    out = []
    for value in (0.0, math.nan):
        g = gpu.TeukGrid(a, s, m, nr, nth, rmin, rmax, inputs.stable_dt(dr, nth, m, s, 1000),
                         extract_rstar=[rmin + 40.5 * dr], extract_theta=[math.pi / 2])
        g.enable_adjoint()
        g.set_adjoint_tile(5, 4)
        g.set_steps_per_pass(spp)
        lp, lq = (torch.from_numpy(x.copy()).cuda() for x in inputs.random_state(nr, nth, seed=4))
        gs = torch.full((n, 1), value, dtype=torch.complex128, device="cuda")
        g.adjoint(n, lp, lq, gs, None, spin=False)
        out.append(np.stack([lp.cpu().numpy(), lq.cpu().numpy()]))
        g.close()
    bad = np.isnan(out[1]).any(axis=(0, 1))
    assert bad[40:42].all() and not bad[:40 - 2 * n].any() and not bad[42 + 2 * n:].any()
    ok = ~np.isnan(out[1])
    assert np.array_equal(out[0][ok], out[1][ok])
