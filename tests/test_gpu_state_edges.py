"""Edges of what a state takes: copied out into one array for both fields, or
overlapping ones (Phi, then Pi over it, as two copies in turn leave it), and
advanced by a step of next to nothing."""
import numpy as np
import pytest
import torch

from paper_1010_3816_amd import inputs

pytestmark = pytest.mark.gpu


def test_one_array_for_both_fields(gpu):
    nr, nth = 300, 40
    g = gpu.TeukGrid(0.5, -2, 2, nr, nth, -50.0, 150.0, 0.001)
    g.set_initial_data(*(torch.from_numpy(x).cuda() for x in inputs.random_state(nr, nth, seed=1)))
    g.step(3)
    phi, pi = (t.cpu().numpy() for t in g.state())
    buf = torch.zeros((nth, nr), dtype=torch.complex128, device="cuda")
    gpu.teuk_get_state(g.handle, buf, buf)
    assert np.array_equal(buf.cpu().numpy(), pi)
    flat = torch.zeros(nr * nth + 100, dtype=torch.complex128, device="cuda")
    gpu.teuk_get_state(g.handle, flat, flat[100:])
    exp = np.concatenate([phi.ravel()[:100], pi.ravel()])
    assert np.array_equal(flat.cpu().numpy(), exp)
    gpu.teuk_get_state(g.handle, flat[100:], flat)
    exp = np.concatenate([pi.ravel(), phi.ravel()[-100:]])
    assert np.array_equal(flat.cpu().numpy(), exp)
    g.close()


def test_step_of_next_to_nothing(gpu):
    """A step so short that its inverse is no finite number leaves the state."""
    nr, nth = 300, 40
    g = gpu.TeukGrid(0.5, -2, 2, nr, nth, -50.0, 150.0, 1e-310)
    u = inputs.random_state(nr, nth, seed=2)
    g.set_initial_data(*(torch.from_numpy(x).cuda() for x in u))
    before = [t.cpu().numpy() for t in g.state()]
    for spp in (1, 2):
        g.set_steps_per_pass(spp)
        g.step(5)
        for a, b in zip(g.state(), before):
            assert np.array_equal(a.cpu().numpy(), b)
    lam = [torch.from_numpy(x).cuda() for x in before]
    g.enable_adjoint()
    g.adjoint(3, *lam, None, None, project_initial=True, spin=False)
    for a, b in zip(lam, before):
        assert np.array_equal(a.cpu().numpy(), b)
    g.close()
