"""The tile pass (several steps per launch on register tiles), which a grid
takes by default where it is estimated fastest: equal, bit for bit, to the
sweeps, and to the oracle within the forward path's bar.  Grids are chosen so
that each of its shapes runs (rows per lane, columns a group, one theta tile or
several, ragged last tiles, a tile that runs past the last row), with step
counts that do and do not divide the steps of a launch, both pole signs and
extraction points at poles, at both radial ends and next to each other."""
import math

import numpy as np
import pytest

from paper_1010_3816_amd import inputs

TOL = 1e-11  # of the forward path (normwise, against the oracle)


def _run(gpu, w, n, u, sweeps):
    import torch

    g = gpu.TeukGrid(w["a"], w["s"], w["m"], w["nr"], w["nth"], -60.0, 140.0, w["dt"], extract_rstar=w["er"],
                     extract_theta=w["et"])
    if sweeps:
        g.set_block_steps(0)
    g.set_initial_data(*(torch.from_numpy(x).cuda() for x in u))
    series = [g.step(n - n // 3), g.step(n // 3)]
    out = [t.cpu().numpy() for t in g.state()] + [np.concatenate([s.cpu().numpy() for s in series])]
    assert g.steps == n
    g.close()
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("a,s,m,nr,nth,n", [
    (0.0, -2, 2, 3, 2, 5),          # all of the smallest grid in one wavefront
    (0.5, -2, 2, 200, 16, 40),
    (0.0, 0, 1, 400, 32, 25),       # theta split or whole, odd m
    (0.9, -2, -3, 401, 31, 26),     # a row past the last in the tile
    (0.7, 2, 2, 63, 65, 17),
    (0.99, -2, 2, 1600, 64, 13),
    (0.3, -1, 1, 700, 101, 20),
    (0.6, -2, 2, 130, 500, 11),     # many theta tiles
    (0.8, 0, -1, 1601, 129, 9),
    (0.5, -2, 2, 6400, 17, 21),
    (0.5, -2, 2, 3201, 128, 10),    # more workgroups than the device holds at once
])
def test_tile_pass(gpu, a, s, m, nr, nth, n):
    import oracle

    dr, dth = 200.0 / (nr - 1), math.pi / nth
    cols = [0.5, nr - 1.5, 0.37 * nr, 0.37 * nr + 0.5]
    thetas = [0.1 * dth, math.pi - 0.2 * dth, 0.5 * math.pi, 0.5 * math.pi + 0.3 * dth]
    w = dict(a=a, s=s, m=m, nr=nr, nth=nth, dt=inputs.stable_dt(dr, nth, m, s, 1000),
             er=[-60.0 + min(max(c, 0.0), nr - 1.0) * dr for c in cols], et=thetas)
    u = inputs.random_state(nr, nth, seed=nr + nth)
    tile, ref = _run(gpu, w, n, u, False), _run(gpu, w, n, u, True)
    for k in range(3):
        assert np.array_equal(tile[k], ref[k]), k
    o = oracle.OracleGrid(a, s, m, nr, nth, -60.0, 140.0, w["dt"])
    p, q = o.project(*u)
    exp = o.evolve(p, q, n, w["er"], w["et"])
    for k in range(3):
        assert np.abs(tile[k] - exp[k]).max() <= TOL * np.abs(exp[k]).max(), k


@pytest.mark.gpu
def test_launch_settings_choose_the_pass(gpu):
    """The tile and block settings: turning the block pass off leaves the
    sweeps, the default tile brings the grid's own choice back, another tile
    applies to the sweeps; the results do not depend on any of it."""
    import torch

    w = dict(a=0.6, s=-2, m=2, nr=900, nth=96, dt=0.01, er=[10.0], et=[1.0])
    u = inputs.random_state(w["nr"], w["nth"], seed=1)
    ref = _run(gpu, w, 12, u, False)
    g = gpu.TeukGrid(w["a"], w["s"], w["m"], w["nr"], w["nth"], -60.0, 140.0, w["dt"], extract_rstar=w["er"],
                     extract_theta=w["et"])
    tile = g.tile()
    for setting in (lambda: g.set_block_steps(0), lambda: g.set_tile(*tile), lambda: g.set_tile(7, 2),
                    lambda: g.set_tile(*tile), lambda: g.set_steps_per_pass(1), lambda: g.set_finite_check(5)):
        setting()
        g.set_initial_data(*(torch.from_numpy(x).cuda() for x in u))
        series = g.step(12)
        for got, want in zip([*g.state(), series], ref):
            assert np.array_equal(got.cpu().numpy(), want)
    g.close()
