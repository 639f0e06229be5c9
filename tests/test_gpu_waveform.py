"""All azimuthal modes of one problem as one batch, and the field summed from
them at observers (C ABI teuk_batch_extract, teuk_assemble_modes; module
waveform): batched samples equal single-grid samples bit for bit, mode
samples match the oracle within the forward tolerance, and the assembled
field matches the oracle's mode sum (oracle.mode_sum) of the oracle's
samples."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_1010_3816_amd import binding, inputs
from parity import rel_err

pytestmark = pytest.mark.gpu
TOL = 1e-11


def test_batch_extract_equals_single_grids(gpu):
    base = [(0.3, -2, 2, 130, 20, ((20.0, 1.5), (-5.0, 0.2))),
            (0.8, 0, -3, 187, 33, ((40.0, 2.9),)),
            (0.0, -2, 1, 64, 9, ((1.0, 0.0), (2.0, math.pi), (3.0, 1.0)))]
    members = []
    for a, s, m, nr, nth, ext in base:
        members.append(dict(a=a, s=s, m=m, nr=nr, ntheta=nth, rstar_min=-30.0, rstar_max=60.0,
                            dt=inputs.stable_dt(90.0 / (nr - 1), nth, m, s, 100),
                            extract_rstar=[e[0] for e in ext], extract_theta=[e[1] for e in ext]))
    data = [inputs.random_state(mb["nr"], mb["ntheta"], seed=500 + k) for k, mb in enumerate(members)]
    b = gpu.TeukBatch(members)
    assert b.n_extract() == 6
    for k, (p, q) in enumerate(data):
        b.set_initial_data(k, torch.from_numpy(p).cuda(), torch.from_numpy(q).cuda())
    b.step(5)
    got = b.extract().cpu().numpy()
    ref = []
    for k, mb in enumerate(members):
        g = gpu.TeukGrid(mb["a"], mb["s"], mb["m"], mb["nr"], mb["ntheta"], mb["rstar_min"], mb["rstar_max"], mb["dt"])
        g.set_initial_data(torch.from_numpy(data[k][0]).cuda(), torch.from_numpy(data[k][1]).cuda())
        g.step(5)
        ref.append(g.extract(mb["extract_rstar"], mb["extract_theta"]).cpu().numpy())
        g.close()
    assert np.array_equal(got, np.concatenate(ref))
    b.close()


def test_mode_sum_against_oracle(gpu):
    from paper_1010_3816_amd.waveform import ModeSet

    a, s, nr, nth, rmin, rmax = 0.6, -2, 150, 24, -30.0, 60.0
    modes = [-2, -1, 0, 1, 2]
    dt = min(inputs.stable_dt((rmax - rmin) / (nr - 1), nth, m, s, 60) for m in modes)
    observers = [(15.0, math.pi / 2, 0.0), (25.0, 1.0, 0.7), (8.0, 2.5, -2.1)]
    ms = ModeSet(a, s, modes, nr, nth, rmin, rmax, dt, observers)
    init = {}
    for j, m in enumerate(modes):
        phi0, pi0 = inputs.gaussian_pulse(nr, nth, rmin, rmax, 5.0 + j, 3.0, "regular", m, s)
        rnd = inputs.random_state(nr, nth, seed=600 + j)
        phi0 = phi0 + 0.01 * rnd[0]
        init[m] = (phi0, pi0)
        ms.set_initial_data(m, torch.from_numpy(phi0).cuda(), torch.from_numpy(pi0).cuda())
    n_samples, every = 20, 3
    samples = ms.evolve(n_samples, every)
    psi = ms.assemble(samples).cpu().numpy()
    samples = samples.cpu().numpy()

    ref = np.zeros((n_samples, len(modes), len(observers)), dtype=np.complex128)
    obs_r = [o[0] for o in observers]
    obs_t = [o[1] for o in observers]
    for j, m in enumerate(modes):
        o = oracle.OracleGrid(a, s, m, nr, nth, rmin, rmax, dt)
        p, q = o.project(*init[m])
        _, _, ser = o.evolve(p, q, n_samples * every, obs_r, obs_t)
        ref[:, j, :] = ser[every - 1::every]
    assert rel_err(samples, ref) <= TOL
    psi_ref = oracle.mode_sum(a, modes, obs_r, [ob[2] for ob in observers], ref)
    assert rel_err(psi, psi_ref) <= TOL
    ms.close()


@pytest.mark.parametrize("n_modes,n_obs,n_samples", [(1, 1, 1), (9, 4, 37), (64, 64, 3), (17, 5, 300)])
def test_assemble_modes_against_oracle(gpu, n_modes, n_obs, n_samples):
    """teuk_assemble_modes on random mode samples, the observers' radii from
    teuk_radius, against the oracle's mode sum (its own tortoise inversion),
    up to the library's limits of 64 modes and 64 observers."""
    rng = np.random.default_rng(n_modes * 1000 + n_obs)
    a = 0.83
    modes = list(rng.choice(np.arange(-40, 41), size=n_modes, replace=False))
    rstar = rng.uniform(-20.0, 300.0, n_obs)
    phi = rng.uniform(-math.pi, math.pi, n_obs)
    smp = rng.standard_normal((n_samples, n_modes, n_obs)) + 1j * rng.standard_normal((n_samples, n_modes, n_obs))
    r = [binding.teuk_radius(a, x) for x in rstar]
    stream = torch.cuda.current_stream()
    d_smp = torch.from_numpy(smp).cuda()
    psi = torch.empty((n_samples, n_obs), dtype=torch.complex128, device="cuda")
    binding.teuk_assemble_modes(d_smp, modes, phi, r, psi, stream)
    torch.cuda.synchronize()
    ref = oracle.mode_sum(a, modes, rstar, phi, smp)
    assert rel_err(psi.cpu().numpy(), ref) <= TOL


@pytest.mark.gpu
@pytest.mark.parametrize("every,n_samples,share", [(1, 7, False), (2, 5, False), (3, 4, True), (5, 3, False),
                                                   (2, 4, True), (17, 2, False)])
def test_samples_inside_the_passes(gpu, every, n_samples, share):
    """Samples taken inside the batch's passes equal, bit for bit, those of
    stepping and sampling in turn, for intervals on both sides of a pass's
    steps, observers that differ in azimuth alone, uneven members, and points
    that share a tile (share: sampled by launches of their own)."""
    import torch

    pts = [(20.0, 1.2), (20.0, 1.2), (-30.0, 0.01), (55.0, 3.1)] + ([(20.5, 1.21)] if share else [])
    members = [dict(a=0.3 * k, s=-2, m=k - 1, nr=130 + 61 * k, ntheta=24 + 7 * k, rstar_min=-40.0, rstar_max=60.0,
                    dt=0.01, extract_rstar=[p[0] for p in pts], extract_theta=[p[1] for p in pts]) for k in range(3)]
    out = []
    for route in range(2):
        b = gpu.TeukBatch(members)
        for k in range(3):
            b.set_initial_data(k, *(torch.from_numpy(x).cuda() for x in inputs.random_state(130 + 61 * k, 24 + 7 * k, 5 + k)))
        if route:
            got = b.step_samples(n_samples, every)
        else:
            rows = []
            for _ in range(n_samples):
                b.step(every)
                rows.append(b.extract())
            got = torch.stack(rows)
        out.append((got.cpu(), [[t.cpu() for t in b.state(k)] for k in range(3)]))
        b.close()
    assert torch.equal(out[0][0], out[1][0])
    for x, y in zip(out[0][1], out[1][1]):
        assert torch.equal(x[0], y[0]) and torch.equal(x[1], y[1])
