"""The work users of this library have it do, as timed cases.

listed() gives the cases, draw(rng) more of the same ranges, prepare() what a
program holds before the call (fields and handles on the GPU), run() one pass
through the public entry points, work() the bytes and operations a pass cannot
do without, and exact() the same outputs by plain torch in 64 bits.

Kinds of work:
  evolve    initial data in, n steps with the waveform series, state out
  source    the same with a source term f(t) g(r*, theta)
  batch     several uneven grids advanced together
  modes     all m-modes of one problem, sampled, summed at observers, states out
  gradient  series of an evolution and the gradients of its misfit with
            respect to the initial data, and to the spin by either route
"""
import math

import numpy as np
import torch

from paper_1010_3816_amd import autograd, binding, inputs
from paper_1010_3816_amd.waveform import ModeSet

R0, R1 = -100.0, 600.0  # the radial range of the repository's Kerr workloads


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------


def _case(kind, nr, ntheta, steps, a=0.9, s=-2, m=2, rmin=R0, rmax=R1, points=1, horizon=10000, **more):
    """horizon: the run length the time step is chosen for (its part of `steps` steps is timed)."""
    dr = (rmax - rmin) / (nr - 1)
    dt = inputs.stable_dt(dr, ntheta, m, s, max(horizon, steps))
    return dict(kind=kind, nr=nr, ntheta=ntheta, steps=steps, a=a, s=s, m=m, rmin=rmin, rmax=rmax, dt=dt,
                points=points, **more)


def _modes(nr, ntheta, a, m_max, samples, every, name=None):
    # the modes share one time step: that of the largest |m|
    c = _case("modes", nr, ntheta, samples * every, a=a, m=m_max, points=4, m_max=m_max, samples=samples, every=every)
    return dict(c, name=name) if name else c


def listed():
    def named(name, *args, **kw):
        return dict(_case(*args, **kw), name=name)

    return [
        # a live monitor that asks for a few steps at a time on a small grid: launches and latency
        named("monitor_200x16", "evolve", 200, 16, 16, a=0.0, rmin=-50.0, rmax=150.0),
        # the standard small run, all of its steps
        named("run_400x32", "evolve", 400, 32, 1000, a=0.0, rmin=-50.0, rmax=150.0, points=1),
        # parameter scans at medium resolution: a grid too tall for one workgroup, too small to fill the chip
        named("scan_1600x128", "evolve", 1600, 128, 500, a=0.5, s=0, m=1, points=2),
        # nothing a multiple of anything, odd m (anti-symmetric poles), an odd number of steps
        named("ragged_5003x197", "evolve", 5003, 197, 151, a=0.37, m=-3, points=3),
        # the production waveform run (part of its 20000 steps)
        named("waveform_6400x256", "evolve", 6400, 256, 400, a=0.9, horizon=20000),
        # the headline resolution, no extraction
        named("large_25600x512", "evolve", 25600, 512, 100, a=0.99, rmin=-200.0, rmax=1200.0, points=0),
        # a particle-driven run
        named("source_6400x256", "source", 6400, 256, 200, a=0.9, points=1),
        # a parameter study: uneven members advanced together
        named("batch_24", "batch", 12800, 256, 40, members=24, points=0),
        # the field at observers from nine azimuthal modes
        _modes(6400, 128, 0.7, 4, 60, 2, name="modes9_6400x128"),
        # gradient of a waveform misfit with respect to the initial data and the spin (default route)
        named("gradient_6400x256", "gradient", 6400, 256, 300, a=0.7, wrt="all", spin="forward", horizon=8000),
        # source inversion: only the initial data need gradients
        named("gradient_data_3200x128", "gradient", 3200, 128, 400, a=0.7, wrt="data", spin="forward"),
        # the checkpointed route
        named("gradient_ckpt_3200x128", "gradient", 3200, 128, 200, a=0.5, m=-1, wrt="all", spin="reverse"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["evolve"] * 5 + ["source", "batch", "modes"] + ["gradient"] * 3)
    a, m, s = rng.uniform(0.0, 0.99), rng.randint(-4, 4), rng.choice([0, -2, -2])
    points = rng.randint(0, 4)
    if kind == "batch":
        return _case("batch", _log_int(rng, 1600, 12800), rng.choice([64, 100, 128, 200, 256]), rng.randint(11, 40),
                     a=a, members=rng.randint(4, 24), points=0)
    if kind == "modes":
        return _modes(_log_int(rng, 500, 6400), _log_int(rng, 32, 128), a, rng.randint(1, 4), rng.randint(10, 60),
                      rng.randint(1, 4))
    if kind == "evolve":
        nr, ntheta = _log_int(rng, 200, 25600), _log_int(rng, 16, 512)
        most = 1.3e9
    else:
        nr, ntheta = _log_int(rng, 800, 6400), _log_int(rng, 48, 256)
        most = 2.5e8
    steps = max(16, min(_log_int(rng, 16, 1000), int(most / (nr * ntheta))))
    if kind == "gradient":
        return _case(kind, nr, ntheta, min(steps, 400), a=a, s=s, m=m, points=max(points, 1),
                     wrt=rng.choice(["all", "all", "data"]), spin=rng.choice(["forward", "reverse"]))
    return _case(kind, nr, ntheta, steps, a=a, s=s, m=m, points=points)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

CHECKPOINT_EVERY = 100
SOURCE_OMEGA, SOURCE_AMPLITUDE = 0.4, 50.0


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _rng(seed, salt=0):
    return np.random.default_rng([int(seed), int(salt), 1010])


def _pulses(nr, ntheta, rmin, rmax, m, s, rng):
    """Phi and Pi: three Gaussian pulses each with complex amplitudes and the
    angular profile that vanishes at the poles as the equation requires."""
    dev = _device()
    x = torch.linspace(0.0, 1.0, nr, dtype=torch.float64, device=dev) * (rmax - rmin) + rmin
    th = (torch.arange(ntheta, dtype=torch.float64, device=dev) + 0.5) * (math.pi / ntheta)
    ang = torch.sin(th / 2) ** abs(m + s) * torch.cos(th / 2) ** abs(m - s)
    out = []
    for scale in (1.0, 0.1):
        f = torch.zeros((ntheta, nr), dtype=torch.complex128, device=dev)
        for _ in range(3):
            centre, width = rng.uniform(5.0, 40.0), rng.uniform(2.0, 6.0)
            amp = scale * complex(rng.normal(), rng.normal())
            tilt = 1.0 + 0.3 * rng.uniform(-1.0, 1.0) * torch.cos(th)
            f += amp * (ang * tilt)[:, None] * torch.exp(-((x - centre) ** 2) / (2.0 * width * width))[None, :]
        out.append(f)
    return out


def _points(case, rng):
    """Extraction points where the pulses are (and one further out)."""
    n = case["points"]
    r = [rng.uniform(10.0, 60.0) for _ in range(n)]
    t = [rng.uniform(0.2, math.pi - 0.2) for _ in range(n)]
    if n:
        t[0] = math.pi / 2
    if n > 2:
        r[2] = 0.8 * case["rmax"]
    return r, t


def _source(case, rng):
    gi, gh = (torch.from_numpy(g).to(_device()) for g in inputs.localised_source(
        case["nr"], case["ntheta"], case["rmin"], case["rmax"], rng.uniform(8.0, 20.0), width=2.0))
    f = inputs.oscillating_factors(case["steps"], case["dt"], SOURCE_OMEGA, SOURCE_AMPLITUDE)
    return gi, gh, f


def _members(case):
    """Uneven members around the case's largest size; fixed by the case."""
    rng = _rng(case["members"], case["nr"] * 4096 + case["ntheta"])
    out = []
    for _ in range(case["members"]):
        nr = int(rng.integers(max(case["nr"] // 8, 3), case["nr"] + 1))
        ntheta = max(int(case["ntheta"] * rng.choice([0.25, 0.5, 1.0])), 2)
        m, s = int(rng.integers(-4, 5)), int(rng.choice([0, -2]))
        dr = (case["rmax"] - case["rmin"]) / (nr - 1)
        out.append(dict(a=float(rng.uniform(0.0, 0.99)), s=s, m=m, nr=nr, ntheta=ntheta, rstar_min=case["rmin"],
                        rstar_max=case["rmax"], dt=inputs.stable_dt(dr, ntheta, m, s, 5000)))
    return out


def _mode_values(case):
    return list(range(-case["m_max"], case["m_max"] + 1))


OBSERVERS = [(30.0, math.pi / 2, 0.0), (30.0, math.pi / 2, math.pi / 3), (20.0, math.pi / 4, 0.0), (45.0, 2.0, 1.0)]


def _fields(case, seed):
    """The seeded inputs of a case that both run() and exact() start from."""
    rng = _rng(seed)
    kind = case["kind"]
    if kind == "batch":
        mbs = _members(case)
        return dict(members=mbs, data=[_pulses(q["nr"], q["ntheta"], q["rstar_min"], q["rstar_max"], q["m"], q["s"],
                                               rng) for q in mbs])
    if kind == "modes":
        return dict(data=[_pulses(case["nr"], case["ntheta"], case["rmin"], case["rmax"], m, case["s"], rng)
                          for m in _mode_values(case)])
    out = dict(data=_pulses(case["nr"], case["ntheta"], case["rmin"], case["rmax"], case["m"], case["s"], rng),
               points=_points(case, rng))
    if kind == "source":
        out["source"] = _source(case, rng)
    if kind == "gradient":
        # the observed series the misfit is taken against: a ringing signal
        t = np.arange(case["steps"]) * case["dt"]
        amp = rng.normal(size=case["points"]) + 1j * rng.normal(size=case["points"])
        obs = 0.3 * amp[None, :] * np.exp(1j * 0.5 * t)[:, None]
        out["target"] = torch.from_numpy(obs).to(_device())
    return out


def prepare(case, seed):
    f = _fields(case, seed)
    kind = case["kind"]
    st = dict(f, case=case)
    if kind == "batch":
        st["batch"] = binding.TeukBatch(f["members"])
    elif kind == "modes":
        st["modes"] = ModeSet(case["a"], case["s"], _mode_values(case), case["nr"], case["ntheta"], case["rmin"],
                              case["rmax"], case["dt"], OBSERVERS)
    elif kind == "gradient":
        r, t = f["points"]
        st["cfg"] = dict(s=case["s"], m=case["m"], nr=case["nr"], ntheta=case["ntheta"], rstar_min=case["rmin"],
                         rstar_max=case["rmax"], dt=case["dt"], extract_rstar=r, extract_theta=t)
        st["spin"] = torch.tensor(case["a"], dtype=torch.float64, device=_device())
    else:
        r, t = f["points"]
        g = binding.TeukGrid(case["a"], case["s"], case["m"], case["nr"], case["ntheta"], case["rmin"], case["rmax"],
                             case["dt"], extract_rstar=r, extract_theta=t)
        if kind == "source":
            gi, gh, _ = f["source"]
            g.set_source(gi, gh)
        st["grid"] = g
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------


def _named(series, phi, pi):
    out = {"phi": phi, "pi": pi}
    if series is not None:
        out["series"] = series
    return out


def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "evolve":
        g = state["grid"]
        g.set_initial_data(*state["data"])
        series = g.step(case["steps"])
        return _named(series, *g.state())
    if kind == "source":
        g = state["grid"]
        g.set_initial_data(*state["data"])
        series = g.step_source(state["source"][2])
        return _named(series, *g.state())
    if kind == "batch":
        b = state["batch"]
        for k, (phi, pi) in enumerate(state["data"]):
            b.set_initial_data(k, phi, pi)
        b.step(case["steps"])
        return [b.state(k) for k in range(len(b))]
    if kind == "modes":
        ms = state["modes"]
        for m, (phi, pi) in zip(ms.m_values, state["data"]):
            ms.set_initial_data(m, phi, pi)
        samples = ms.evolve(case["samples"], case["every"])
        return {"samples": samples, "psi": ms.assemble(samples),
                "state": [ms.batch.state(k) for k in range(len(ms.m_values))]}
    phi, pi = (x.detach().requires_grad_() for x in state["data"])
    a = state["spin"].detach()
    if case["wrt"] == "all":
        a.requires_grad_()
    series = autograd.evolve(phi, pi, a, state["cfg"], case["steps"], CHECKPOINT_EVERY, spin=case["spin"])
    loss = 0.5 * (series - state["target"]).abs().square().sum()
    loss.backward()
    out = {"series": series.detach(), "phi": phi.grad, "pi": pi.grad}
    if a.grad is not None:
        out["a"] = a.grad
    return out


# ---------------------------------------------------------------------------
# the work a pass cannot do without
# ---------------------------------------------------------------------------

# One step at one point, its coefficients at hand: two stages, each the sums
# and differences of two complex values of Phi and Pi (8), the Phi row (8) and
# the Pi row with three complex and three real coefficients (34), in flops.
STEP_FLOPS = 100


def work(case):
    kind, pts, n = case["kind"], case["nr"] * case["ntheta"], case["steps"]
    if kind == "batch":
        pts = sum(q["nr"] * q["ntheta"] for q in _members(case))
        return {"bytes": 64 * pts, "flops": STEP_FLOPS * pts * n}
    if kind == "modes":
        k = 2 * case["m_max"] + 1
        return {"bytes": 64 * pts * k + 16 * case["samples"] * (k + 1) * len(OBSERVERS),
                "flops": STEP_FLOPS * pts * n * k}
    series = 16 * n * case["points"]
    if kind == "source":
        return {"bytes": 64 * pts + 32 * pts + series, "flops": (STEP_FLOPS + 16) * pts * n}
    if kind == "gradient":
        # the step, its transpose, and the step's derivative in the spin (the tangent and the coefficients')
        per = STEP_FLOPS * (4 if case["wrt"] == "all" else 2)
        return {"bytes": 64 * pts + 2 * series, "flops": per * pts * n}
    return {"bytes": 64 * pts + series, "flops": STEP_FLOPS * pts * n}


# ---------------------------------------------------------------------------
# the same in plain torch, 64 bits
# ---------------------------------------------------------------------------


def _tortoise(a, x):
    """r* of x = r - r_+ (M = 1)."""
    q = np.sqrt(1 - a * a)
    return 1 + q + x + ((1 + q) / q) * np.log(x / 2) - ((1 - q) / q) * np.log(x / 2 + q)


def _invert(a, rstar):
    """x = r - r_+ at r*, and dx/da at fixed r*, in extended precision."""
    L = np.longdouble
    a, rs = L(a), np.asarray(rstar, dtype=L)
    q = np.sqrt(1 - a * a)
    near = np.log(L(2)) + (rs - 1 - q) * q / (1 + q)
    u = np.where(rs > 4, np.log(np.maximum(rs, L(1))), near)
    for _ in range(100):
        x = np.exp(u)
        r = 1 + q + x
        du = (_tortoise(a, x) - rs) * (x + 2 * q) / (r * r + a * a)
        u = u - np.clip(du, -2, 2)
    x = np.exp(u)
    r = 1 + q + x
    h = L(1e-40)
    dr_da = np.imag(_tortoise(np.clongdouble(a + 1j * h), x.astype(np.clongdouble))) / h
    return x.astype(np.float64), (-dr_da * x * (x + 2 * q) / (r * r + a * a)).astype(np.float64)


class _Plain:
    """The two-step Lax-Wendroff scheme on one grid (arXiv:1010.3816, Sec. 3)."""

    def __init__(self, case, need_da=False):
        self.nr, self.nth, self.dt = case["nr"], case["ntheta"], case["dt"]
        self.s, self.m = case["s"], case["m"]
        self.dr = (case["rmax"] - case["rmin"]) / (self.nr - 1)
        self.rmin = case["rmin"]
        self.dth = math.pi / self.nth
        self.sigma = 1.0 if self.m % 2 == 0 else -1.0
        dev = _device()
        th = (torch.arange(self.nth, dtype=torch.float64, device=dev) + 0.5) * self.dth
        self.sn, self.cs = torch.sin(th)[:, None], torch.cos(th)[:, None]
        self.ci, self.ch = self._coefs(case["a"], self.nr, 0.0), self._coefs(case["a"], self.nr - 1, 0.5)
        if need_da:
            self.dci = self._coefs(case["a"], self.nr, 0.0, True)
            self.dch = self._coefs(case["a"], self.nr - 1, 0.5, True)

    def _coefs(self, a, n, shift, derivative=False):
        x, dx = _invert(a, self.rmin + (np.arange(n, dtype=np.longdouble) + shift) * np.longdouble(self.dr))
        x, dx = (torch.from_numpy(v).to(self.sn.device)[None, :] for v in (x, dx))
        h = 1e-30
        if derivative:  # complex step along da at fixed r*
            a, x = torch.complex(torch.full_like(x, a), torch.full_like(x, h)), torch.complex(x, h * dx)
            q = torch.sqrt(1 - a * a)
        else:
            q = math.sqrt(1.0 - a * a)
        s, m, sn2, cs = self.s, self.m, self.sn**2, self.cs
        r = 1 + q + x
        D = x * (x + 2 * q)
        rho = r * r + a * a
        S2 = rho * rho - a * a * D * sn2
        S = torch.sqrt(S2)
        b = rho / S
        bp = (2 * r - (rho / S2) * (2 * r * rho - a * a * (r - 1) * sn2)) * D / (rho * S)
        ctr = 2 * s * (r * D - (r * r - a * a)) / S2
        cti = (4 * a * m * r + 2 * s * a * D * cs) / S2
        b1 = (rho * (6 * D / r + 2 * s * (r - 1)) + 2 * r * D) / S2
        a2 = D / S2
        a1 = a2 * cs / self.sn
        v0r = (D * ((m + s * cs) ** 2 / sn2 - s) - m * m * a * a
               - 6 * D * ((s + 2) * r * r - (s + 3) * r + a * a) / (r * r)) / S2
        v0i = -2 * s * m * a * (r - 1) / S2
        real = dict(b=b, cr=b * (bp - ctr) - b1, cim=-b * cti, ctr=ctr, cti=cti, a2=a2 / self.dth**2,
                    a1=a1 / (2 * self.dth), v0r=v0r, v0i=v0i)
        if derivative:
            real = {k: v.imag / h for k, v in real.items()}
        pair = lambda re, im: torch.complex(re, im.expand_as(re).contiguous())  # noqa: E731
        return dict(b=real["b"], c=pair(real["cr"], real["cim"]), ct=pair(real["ctr"], real["cti"]), a2=real["a2"],
                    a1=real["a1"], v0=pair(real["v0r"], real["v0i"]))

    def _rhs(self, k, dp, dq, fp, fq):
        """Rates of (Phi, Pi) for r* derivatives (dp, dq) and values (fp, fq), coefficients k."""
        up = torch.cat([fp[1:], self.sigma * fp[-1:]])
        dn = torch.cat([self.sigma * fp[:1], fp[:-1]])
        sq = -k["ct"] * fq + k["a2"] * (up - 2 * fp + dn) + k["a1"] * (up - dn) - k["v0"] * fp
        return -k["b"] * dp, -(k["c"] * dp - k["b"] * dq) + sq

    def _half(self, p, q):
        """Averages and r* differences of neighbouring columns."""
        up, uq = (p[:, 1:] + p[:, :-1]) / 2, (q[:, 1:] + q[:, :-1]) / 2
        dp, dq = (p[:, 1:] - p[:, :-1]) / self.dr, (q[:, 1:] - q[:, :-1]) / self.dr
        return up, uq, dp, dq

    def _bound(self, p, q):
        for f in (p, q):
            f[:, 0] = 0
            f[:, -1] = 0
        return p, q

    def _wrap(self, inner, like):
        out = torch.zeros_like(like)
        out[:, 1:-1] = inner
        return out

    def step(self, p, q, source=None, f=None):
        up, uq, dp, dq = self._half(p, q)
        rp, rq = self._rhs(self.ch, dp, dq, up, uq)
        if source is not None:
            rq = rq + f[0] * source[1]
        hp, hq = up + self.dt / 2 * (rp + uq), uq + self.dt / 2 * rq
        ap, aq, ep, eq = self._half(hp, hq)
        mid = {n: c[:, 1:-1] for n, c in self.ci.items()}
        rp, rq = self._rhs(mid, ep, eq, ap, aq)
        if source is not None:
            rq = rq + f[1] * source[0][:, 1:-1]
        return (self._wrap(p[:, 1:-1] + self.dt * (rp + aq), p), self._wrap(q[:, 1:-1] + self.dt * rq, q))

    def step_with_tangent(self, p, q, v, w):
        """One step of (p, q) and of its derivative in the spin (v, w)."""
        up, uq, dp, dq = self._half(p, q)
        vp, vq, ep, eq = self._half(v, w)
        rp, rq = self._rhs(self.ch, dp, dq, up, uq)
        sp, sq = self._rhs(self.ch, ep, eq, vp, vq)
        tp, tq = self._rhs(self.dch, dp, dq, up, uq)
        k = self.dt / 2
        hp, hq = up + k * (rp + uq), uq + k * rq
        gp, gq = vp + k * (sp + tp + vq), vq + k * (sq + tq)
        ap, aq, dp, dq = self._half(hp, hq)
        bp, bq, ep, eq = self._half(gp, gq)
        mid = {n: c[:, 1:-1] for n, c in self.ci.items()}
        dmid = {n: c[:, 1:-1] for n, c in self.dci.items()}
        rp, rq = self._rhs(mid, dp, dq, ap, aq)
        sp, sq = self._rhs(mid, ep, eq, bp, bq)
        tp, tq = self._rhs(dmid, dp, dq, ap, aq)
        new = (p[:, 1:-1] + self.dt * (rp + aq), q[:, 1:-1] + self.dt * rq)
        tan = (v[:, 1:-1] + self.dt * (sp + tp + bq), w[:, 1:-1] + self.dt * (sq + tq))
        return tuple(self._wrap(n, p) for n in new + tan)

    def sampler(self, rstar, theta):
        """Phi -> bilinear samples at the points (as a differentiable function)."""
        rows, cols, wts = [], [], []
        for r, t in zip(rstar, theta):
            x = (r - self.rmin) / self.dr
            i = min(max(int(math.floor(x)), 0), self.nr - 2)
            y = t / self.dth - 0.5
            j = min(max(int(math.floor(y)), -1), self.nth - 1)
            for row, wt in ((j, 1 - (y - j)), (j + 1, y - j)):
                if row < 0 or row >= self.nth:  # the pole's ghost row
                    row, wt = min(max(row, 0), self.nth - 1), wt * self.sigma
                for col, wr in ((i, 1 - (x - i)), (i + 1, x - i)):
                    rows.append(row)
                    cols.append(col)
                    wts.append(wt * wr)
        dev = self.sn.device
        n = len(rows) // 4
        rows, cols = torch.tensor(rows, device=dev), torch.tensor(cols, device=dev)
        wts = torch.tensor(wts, dtype=torch.float64, device=dev)
        return lambda p: (p[rows, cols] * wts).view(n, 4).sum(1)


def _evolve_plain(case, fields, every=1, source=None, f=None):
    w = _Plain(case)
    take = w.sampler(*fields["points"]) if fields["points"][0] else None
    p, q = w._bound(*(x.clone() for x in fields["data"]))
    series = []
    for k in range(case["steps"]):
        p, q = w.step(p, q, source, None if f is None else (complex(f[k][0]), complex(f[k][1])))
        if take is not None and (k + 1) % every == 0:
            series.append(take(p))
    return (torch.stack(series) if series else None), p, q


def _gradient_plain(case, fields):
    everything = case["wrt"] == "all"
    w = _Plain(case, need_da=everything)
    take = w.sampler(*fields["points"])
    p, q = w._bound(*(x.clone() for x in fields["data"]))
    v, t = torch.zeros_like(p), torch.zeros_like(p)
    series, tangents = [], []
    for _ in range(case["steps"]):
        if everything:
            p, q, v, t = w.step_with_tangent(p, q, v, t)
            tangents.append(take(v))
        else:
            p, q = w.step(p, q)
        series.append(take(p))
    series = torch.stack(series)
    g = series - fields["target"]
    lp, lq = torch.zeros_like(p), torch.zeros_like(p)
    zero = torch.zeros_like(p)
    for k in range(case["steps"] - 1, -1, -1):
        x = [zero.clone().requires_grad_(), zero.clone().requires_grad_()]
        y = w.step(*x)  # linear: the point of expansion does not matter
        lp, lq = torch.autograd.grad([*y, take(y[0])], x, [lp, lq, g[k]])
    lp, lq = w._bound(lp.clone(), lq.clone())
    out = {"series": series, "phi": lp, "pi": lq}
    if everything:
        out["a"] = (g.conj() * torch.stack(tangents)).real.sum()
    return out


def exact(case, seed):
    kind = case["kind"]
    fields = _fields(case, seed)
    if kind == "gradient":
        return _gradient_plain(case, fields)
    if kind == "batch":
        out = []
        for q, data in zip(fields["members"], fields["data"]):
            c = dict(q, rmin=q["rstar_min"], rmax=q["rstar_max"], steps=case["steps"])
            out.append(_evolve_plain(c, dict(data=data, points=([], [])))[1:])
        return out
    if kind == "modes":
        obs = np.asarray(OBSERVERS)
        pts = (obs[:, 0].tolist(), obs[:, 1].tolist())
        per_mode = [_evolve_plain(dict(case, m=m), dict(data=d, points=pts), every=case["every"])
                    for m, d in zip(_mode_values(case), fields["data"])]
        samples = torch.stack([e[0] for e in per_mode], dim=1)
        x, _ = _invert(case["a"], obs[:, 0])
        r3 = torch.from_numpy((1 + math.sqrt(1 - case["a"] ** 2) + x) ** 3).to(samples.device)
        ph = torch.from_numpy(np.outer(_mode_values(case), obs[:, 2])).to(samples.device)
        psi = r3 * (torch.polar(torch.ones_like(ph), ph) * samples).sum(1)
        return {"samples": samples, "psi": psi, "state": [e[1:] for e in per_mode]}
    source = f = None
    if kind == "source":
        gi, gh, f = fields["source"]
        source = (gi, gh)
    series, p, q = _evolve_plain(case, fields, source=source, f=f)
    return _named(series, p, q)
