"""The adjoint tile pass (cotangents only), which grids take by default where
it is estimated fastest: equal, bit for bit, to the adjoint sweeps (one step
per pass), and to the oracle's transposed steps within the reverse pass's bar:
shapes of one to three rows a lane, whole grids and theta tiles, both pole
signs, points at poles, at the radial ends, sharing a row or a column, step
counts that do and do not divide the steps of a launch, no sample gradients."""
import math

import numpy as np
import pytest

from paper_1010_3816_amd import inputs

TOL = 1e-11  # cotangents against the oracle, normwise (the reverse pass's bar)


@pytest.mark.gpu
@pytest.mark.parametrize("a,s,m,nr,nth,n,npts", [
    (0.0, -2, 2, 3, 2, 4, 1),
    (0.5, -2, 1, 200, 16, 31, 2),
    (0.9, 0, -3, 401, 31, 17, 3),
    (0.7, -2, 2, 63, 65, 9, 4),
    (0.3, -1, 1, 1200, 100, 12, 1),
    (0.99, -2, 2, 130, 301, 7, 8),
    (0.6, 2, -2, 3201, 96, 6, 0),
])
def test_adjoint_tile_pass(gpu, a, s, m, nr, nth, n, npts):
    import torch

    import oracle

    rmin, rmax = -40.0, 60.0
    dr, dth = (rmax - rmin) / (nr - 1), math.pi / nth
    cols = [0.5, nr - 1.5, 0.4 * nr, 0.4 * nr, 0.4 * nr + 1.0, 0.4 * nr - 1.25, 0.1 * nr, 0.4 * nr][:npts]
    thetas = [0.1 * dth, math.pi - 0.2 * dth, 1.5, 1.5 + 0.4 * dth, 1.5, 1.5 - dth, 1.5, 1.5 + dth][:npts]
    er = [rmin + min(max(c, 0.0), nr - 1.0) * dr for c in cols]
    dt = inputs.stable_dt(dr, nth, m, s, 1000)
    rng = np.random.default_rng(nr + nth)
    gs = rng.standard_normal((n, npts)) + 1j * rng.standard_normal((n, npts))
    lam = inputs.random_state(nr, nth, seed=3)
    out = []
    for spp in (2, 1):
        g = gpu.TeukGrid(a, s, m, nr, nth, rmin, rmax, dt, extract_rstar=er, extract_theta=thetas)
        g.enable_adjoint()
        g.set_steps_per_pass(spp)
        lp, lq = (torch.from_numpy(x.copy()).cuda() for x in lam)
        g.adjoint(n, lp, lq, torch.from_numpy(gs).cuda() if npts else None, None, project_initial=True, spin=False)
        out.append((lp.cpu().numpy(), lq.cpu().numpy()))
        g.close()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    o = oracle.OracleGrid(a, s, m, nr, nth, rmin, rmax, dt)
    p, q = lam[0].copy(), lam[1].copy()
    for k in range(n - 1, -1, -1):
        for e in range(npts):
            p = o.extract_adjoint(p, er[e], thetas[e], gs[k, e])
        p, q = o.adjoint_step(p, q)
    p, q = o.project(p, q)
    for got, ref in zip(out[0], (p, q)):
        assert np.abs(got - ref).max() <= TOL * np.abs(ref).max()
