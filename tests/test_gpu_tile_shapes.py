"""Each shape of the tile passes, forward and adjoint, by the pass the grid
reports: equal to the sweeps bit for bit, with extraction points at a pole, a
boundary column and next to each other; and the block pass, which grids take
only by a launch of their own or with an in-loop check, against the oracle."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_1010_3816_amd import inputs
from parity import rel_err, run_oracle

pytestmark = pytest.mark.gpu
TOL = 1e-11  # of the forward path (normwise, against the oracle)


def _points(nr, nth):
    dr, dth = 200.0 / (nr - 1), math.pi / nth
    cols = [0.5, nr - 1.5, 0.45 * nr, 0.45 * nr, 0.45 * nr + 1.0]
    th = [0.2 * dth, math.pi - 0.3 * dth, 1.5, 1.5 + 0.4 * dth, 1.5 + dth]
    return [-60.0 + min(max(c, 0.0), nr - 1.0) * dr for c in cols], [min(t, math.pi) for t in th]


def _grid(gpu, nr, nth, m):
    er, et = _points(nr, nth)
    dt = inputs.stable_dt(200.0 / (nr - 1), nth, m, -2, 1000)
    return gpu.TeukGrid(0.7, -2, m, nr, nth, -60.0, 140.0, dt, extract_rstar=er, extract_theta=et)


def _expect(g, run, shape):
    """The pass the cost model chooses on the device it was fitted to."""
    p = g.get_pass(run)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert (p["kind"], p["cols"], p["rows"]) == ("tile", *shape), p
    return p


def _cuda(x):
    return [torch.from_numpy(np.array(a)).cuda() for a in x]


# (nr, ntheta): shape; one theta tile, one that runs past the last row, several
FORWARD = [((12, 47), (16, 1)), ((56, 32), (16, 1)), ((700, 26), (32, 1)), ((200, 17), (32, 1)), ((64, 9), (32, 1)),
           ((1601, 52), (32, 1)), ((700, 28), (32, 2)), ((700, 101), (32, 2)), ((700, 11), (64, 1)),
           ((700, 12), (64, 2)), ((3201, 18), (64, 3)), ((700, 200), (64, 3))]


@pytest.mark.parametrize("grid,shape", FORWARD)
def test_forward_shapes(gpu, grid, shape):
    nr, nth = grid
    g = _grid(gpu, nr, nth, 1 + nr % 2)
    p = _expect(g, "series", shape)
    n = 2 * p["steps"] + 3
    u = inputs.random_state(nr, nth, seed=nr)
    out = []
    for k in range(2):
        g.set_initial_data(*_cuda(u))
        s = g.step(n)
        out.append([t.cpu().numpy() for t in (*g.state(), s)])
        if k == 0:
            g.set_block_launch(0)
            assert g.get_pass("series")["kind"] == "sweep"
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    g.close()


ADJOINT = [((121, 26), (16, 1)), ((90, 32), (16, 1)), ((700, 22), (32, 1)), ((700, 21), (32, 1)), ((700, 28), (32, 2)),
           ((700, 101), (32, 2)), ((700, 9), (64, 1)), ((700, 10), (64, 2)), ((3201, 18), (64, 3)),
           ((700, 200), (64, 3))]


@pytest.mark.parametrize("grid,shape", ADJOINT)
def test_adjoint_shapes(gpu, grid, shape):
    nr, nth = grid
    g = _grid(gpu, nr, nth, 1 + nr % 2)
    g.enable_adjoint()
    n = 2 * _expect(g, "cotangents", shape)["steps"] + 3
    lam = inputs.random_state(nr, nth, seed=nth)
    rng = np.random.default_rng(nr)
    gs = _cuda([rng.standard_normal((n, 5)) + 1j * rng.standard_normal((n, 5))])[0]
    out = []
    for spp in (2, 1):  # single steps: the sweep
        g.set_steps_per_pass(spp)
        lp, lq = _cuda(lam)
        g.adjoint(n, lp, lq, gs, None, project_initial=True, spin=False)
        out.append((lp.cpu().numpy(), lq.cpu().numpy()))
    assert g.get_pass("cotangents")["kind"] == "sweep"
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    g.close()


def test_block_pass_of_its_own(gpu):
    """400 x 32 over 300 steps by a block launch other than the default, and by
    the default one with an in-loop check that never falls due: the block pass,
    against the oracle and equal to the tile pass bit for bit."""
    w = dict(inputs.workload("schwarzschild_400x32"))
    n = 300
    w["extract_rstar"] = w["extract_rstar"] + [w["center"] + 0.3 * n * w["dt"]]
    w["extract_theta"] = w["extract_theta"] + [math.pi / 2]
    u = inputs.initial_data(w)
    exp = run_oracle(w, *u, n)
    out = []
    for launch, check in ((None, 0), ((5, 16), 0), (None, 10 * n)):
        g = gpu.TeukGrid(w["a"], w["s"], w["m"], w["nr"], w["ntheta"], w["rstar_min"], w["rstar_max"], w["dt"],
                         extract_rstar=w["extract_rstar"], extract_theta=w["extract_theta"])
        if launch:
            g.set_block_launch(*launch)
        g.set_finite_check(check)
        if torch.cuda.get_device_properties(0).multi_processor_count == 256:
            assert g.get_pass("series")["kind"] == ("block" if launch or check else "tile")
        g.set_initial_data(*_cuda(u))
        s = g.step(n)
        out.append([t.cpu().numpy() for t in (*g.state(), s)])
        g.close()
    for k, e in enumerate(exp):
        assert rel_err(out[1][k], e) <= TOL
        assert np.array_equal(out[1][k], out[0][k]) and np.array_equal(out[2][k], out[0][k])
