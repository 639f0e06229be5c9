"""Sweeps over tiles of a few rows, whose last rows go one by one: heights of
every remainder of the row loops' groups, from one row to all of them, equal
to the tallest tile's results, and those to the oracle's within the paths'
bars.  Rows whose number a height does not divide, both pole signs, strips on
both sides of a boundary column."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_1010_3816_amd import inputs
from parity import rel_err

pytestmark = pytest.mark.gpu
TOL = 1e-11  # of the forward and reverse paths (normwise, against the oracle)
NR, NTH = 122, 13
HEIGHTS = [1, 2, 3, 4, 5, 6, 7, NTH]


def _grid(gpu, m, coef=False):
    dr, dth = 200.0 / (NR - 1), math.pi / NTH
    # a pole row, the last row of a tile of four and a boundary column's cell
    er, et = [-60.0 + 61.5 * dr, 140.0 - 0.5 * dr], [0.2 * dth, 3.9 * dth]
    dt = inputs.stable_dt(dr, NTH, m, -2, 1000)
    g = gpu.TeukGrid(0.7, -2, m, NR, NTH, -60.0, 140.0, dt, extract_rstar=er, extract_theta=et,
                     coef_mode=gpu.TEUK_COEF_USER if coef else gpu.TEUK_COEF_KERR)
    if g.block_steps():
        g.set_block_steps(0)
    return g, oracle.OracleGrid(0.7, -2, m, NR, NTH, -60.0, 140.0, dt, kerr=not coef), er, et


def _cuda(x):
    return [torch.from_numpy(np.array(a)).cuda() for a in x]


@pytest.mark.parametrize("m", [1, 2])
@pytest.mark.parametrize("kind", ["one", "two", "store", "source", "user"])
def test_forward(gpu, kind, m):
    n = 6
    g, o, er, et = _grid(gpu, m, kind == "user")
    u = inputs.random_state(NR, NTH, seed=m)
    rng = np.random.default_rng(m)
    if kind == "user":
        c = [0.1 * rng.standard_normal((gpu.TEUK_NCOEF, NTH, w)) for w in (NR, NR - 1)]
        g.set_coefficients(*_cuda(c))
        o.set_coefficients(*c)
    if kind == "source":
        prof = [rng.standard_normal((NTH, w)) + 1j * rng.standard_normal((NTH, w)) for w in (NR, NR - 1)]
        f = rng.standard_normal((n, 2)) + 1j * rng.standard_normal((n, 2))
        g.set_source(*_cuda(prof))
        o.set_source(*prof)
    if kind == "two":
        g.set_finite_check(1000)  # no check within the run: its steps go in pairs
    if kind == "one":
        g.set_steps_per_pass(1)
    ref = None
    for rows in reversed(HEIGHTS):
        g.set_tile(rows, 2)
        g.set_initial_data(*_cuda(u))
        out = []
        if kind == "store":
            win = g.new_window(n)
            out.append(g.step_store(n, win))
            out += [t for k in range(n) for t in g.window_slot(win, k)]
        elif kind == "source":
            out.append(g.step_source(f))
        else:
            out.append(g.step(n))
        out = [t.cpu().numpy() for t in (*g.state(), *out)]
        if ref is None:
            ref = out
        for k, (a, b) in enumerate(zip(out, ref)):
            assert np.array_equal(a, b), (rows, k)
    p, q = o.project(*u)
    exp = o.evolve_source(p, q, f, er, et) if kind == "source" else o.evolve(p, q, n, er, et)
    for a, b in zip(ref[:3], exp):
        assert rel_err(a, b) <= TOL
    g.close()


DLDA_TOL = 1e-10  # of the spin gradient, relative (a sum over all points and steps)


@pytest.mark.parametrize("m", [1, 2])
@pytest.mark.parametrize("spp", [1, 2])
@pytest.mark.parametrize("kind", ["cotangents", "tangents", "states"])
def test_adjoint(gpu, kind, spp, m):
    n = 5
    g, o, er, et = _grid(gpu, m)
    u = inputs.random_state(NR, NTH, seed=10 + m)
    rng = np.random.default_rng(10 + m)
    gser = rng.standard_normal((n, 2)) + 1j * rng.standard_normal((n, 2))
    g.enable_adjoint()
    g.set_steps_per_pass(spp)
    g.set_initial_data(*_cuda(u))
    win = g.new_window(n)
    if kind == "tangents":
        g.step_tangent(n, win)
    else:
        g.step_store(n, win, series=False)
    zero = np.zeros((NTH, NR), dtype=np.complex128)
    exp = o.adjoint_evolve(*o.project(*u), n, er, et, gser)
    ref = None
    for rows in reversed(HEIGHTS):
        g.set_adjoint_tile(rows, 4 if rows > 1 and rows % 2 else 2)
        lam = _cuda((zero, zero))
        dlda = g.adjoint(n, *lam, _cuda([gser])[0], win, project_initial=True, spin=kind != "cotangents",
                         tangent=kind == "tangents")
        torch.cuda.synchronize()
        out = [t.cpu().numpy() for t in lam]
        if ref is None:
            ref = out
        assert np.array_equal(out[0], ref[0]) and np.array_equal(out[1], ref[1]), rows
        if kind != "cotangents":
            assert abs(dlda - exp[2]) <= DLDA_TOL * abs(exp[2]), (rows, dlda, exp[2])
    p, q = o.project(exp[0], exp[1])
    assert rel_err(ref[0], p) <= TOL and rel_err(ref[1], q) <= TOL
    g.close()


@pytest.mark.parametrize("m", [1, 2])
def test_tangents(gpu, m):
    """The step with its spin derivative and the step that stores its tangent."""
    n = 4
    g, o, er, et = _grid(gpu, m)
    u, v = inputs.random_state(NR, NTH, seed=20 + m), inputs.random_state(NR, NTH, seed=30 + m)
    g.enable_spin_tangent()
    win = g.new_window(n)
    ref = None
    for rows in reversed(HEIGHTS):
        g.set_adjoint_tile(rows, 4 if rows > 1 and rows % 2 else 2)
        g.set_initial_data(*_cuda(u))
        g.set_spin_tangent(*_cuda(v))
        out = [*g.step_spin_tangent(n)]
        out = [*g.state(), *g.spin_tangent(), *out]
        g.set_initial_data(*_cuda(u))
        g.step_tangent(n, win)
        out = [t.cpu().numpy() for t in (*out, *g.state(), *(f for k in range(n) for f in g.window_slot(win, k)))]
        if ref is None:
            ref = out
        for k, (a, b) in enumerate(zip(out, ref)):
            assert np.array_equal(a, b), (rows, k)
    p, q = o.project(*u)
    exp = o.evolve_spin_tangent(p, q, *o.project(*v), n, er, et)
    for a, b in zip(ref[:6], exp):
        assert rel_err(a, b) <= TOL
    for k in range(n):
        for a, b in zip(ref[8 + 2 * k:10 + 2 * k], o.tangent_a(p, q)):
            assert rel_err(a, b) <= TOL
        p, q = o.step(p, q)
    g.close()
