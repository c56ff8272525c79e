"""Cases for timing the framework, each a call a user's program makes.

A program that uses the integrator holds initial conditions in host arrays (the
``Simulation`` and many-system calls take and return numpy arrays) or in
device tensors (the derivative and no-allocation calls), keeps one simulation
object, and asks for one stretch of time steps: one output interval of a long
run, one set of initial conditions of a scan, one gradient of a fit.  A pass
is that whole call: states in, integration, states and removal records out.

Sizes come from the package's own workloads and tests: 64 particles up to the
200,000 of the resonant workload, 1 to 8 planets, 100 to 10,000 steps, odd and
ragged counts among them.  Strongly chaotic orbits (the belt between Uranus
and Neptune, a particle next to a giant planet) are kept to stretches short
enough that their states still mean something digit by digit; the distant
resonant belt runs for more than one of the library's chunks.

``exact`` is an independent 64-bit evaluation of the same map in numpy and
torch: planets by the Wisdom-Holman map in Jacobi coordinates, particles by
kick - Kepler drift - kick about the central mass, removal at step boundaries.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2011_03484_amd as tpm
from paper_2011_03484_amd import autograd as tpm_autograd
from paper_2011_03484_amd import workloads as W

# Longest stretch per kind (see above) and the most particle-steps of a case.
MAX_STEPS = {"giants": 2000, "single": 500, "resonant": 10_000, "high_e": 250, "handoff": 800,
             "batch": 800, "static": 1500, "adjoint": 500, "tangent": 500, "diagnostics": 4000}
MAX_PARTICLE_STEPS = 2_000_000_000


def listed():
    return [
        # A handful of test particles followed for a few orbits: one wavefront,
        # so the call's latency is all that counts.
        {"name": "giants_64", "kind": "giants", "n": 64, "steps": 256},
        # The single-planet workload at its own size, one planet.
        {"name": "single_planet_1024", "kind": "single", "n": 1024, "steps": 500},
        # The length of the paper's own benchmark, with one particle more than
        # the 13,312 at which its card filled up: two chunks, the chip part full.
        {"name": "resonant_13313", "kind": "resonant", "n": 13_313, "steps": 10_000},
        # The benchmark's workload at full size, one output interval.
        {"name": "giants_100k", "kind": "giants", "n": 100_000, "steps": 2000},
        # The resonant belt at full size over several chunks: the largest call.
        {"name": "resonant_200k", "kind": "resonant", "n": 200_000, "steps": 10_000},
        # High eccentricities and unbound orbits with the universal drift,
        # working set ordered by eccentricity.
        {"name": "high_e_4096", "kind": "high_e", "n": 4096, "steps": 250, "sort": True},
        # Close encounters handed off and followed with 16 substeps.
        {"name": "handoff_20k", "kind": "handoff", "n": 20_000, "steps": 800, "substeps": 16},
        # A hundred-odd independent systems of 1 to 8 planets in one call.
        {"name": "batch_96", "kind": "batch", "nsys": 96, "nmax": 4096, "steps": 800},
        # A run on device buffers that allocates nothing (a serving loop).
        {"name": "static_16k", "kind": "static", "n": 16_384, "steps": 1000},
        # Forward and gradient of a loss on the final states, checkpointed.
        {"name": "adjoint_16k", "kind": "adjoint", "n": 16_384, "steps": 500, "ckpt": 125},
        # Forward and a directional derivative, ragged particle count.
        {"name": "tangent_2047", "kind": "tangent", "n": 2047, "steps": 500, "ckpt": 200},
        # The applications' sampled diagnostics: e_max and the 3:1 angle with
        # Neptune every 100 steps.
        {"name": "diagnostics_25k", "kind": "diagnostics", "n": 25_001, "steps": 2000,
         "every": 100},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["giants", "giants", "single", "resonant", "resonant", "high_e", "handoff",
                       "batch", "static", "adjoint", "tangent", "diagnostics"])
    top = {"giants": 150_000, "single": 2048, "resonant": 200_000, "high_e": 16_384,
           "handoff": 40_000, "static": 262_144, "adjoint": 20_000, "tangent": 16_384,
           "diagnostics": 100_000}
    c = {"kind": kind}
    if kind == "batch":
        c["nsys"] = _log_int(rng, 2, 200)
        c["nmax"] = _log_int(rng, 128, 4096)
        c["steps"] = _log_int(rng, 200, MAX_STEPS[kind])
        return c
    c["n"] = _log_int(rng, 1 if kind in ("giants", "static") else 64, top[kind])
    c["steps"] = min(_log_int(rng, 100, MAX_STEPS[kind]), MAX_PARTICLE_STEPS // c["n"])
    if kind == "high_e":
        c["sort"] = rng.random() < 0.5
    if kind == "handoff":
        c["substeps"] = rng.choice([4, 8, 16])
    if kind in ("adjoint", "tangent"):
        c["ckpt"] = rng.choice([50, 125, 333, 1000])
    if kind == "diagnostics":
        c["every"] = rng.choice([50, 100, 250, 1000])
    return c


# ------------------------------------------------------------------- inputs
def _workload(case, seed):
    """The package's own seeded initial conditions (planets and particles)."""
    kind, s = case["kind"], 77_000_000 + int(seed)
    if kind == "single":
        return W.single_planet(n=case["n"], seed=s)
    if kind in ("resonant", "diagnostics"):
        return W.resonant_200k(n=case["n"], seed=s)
    if kind == "high_e":
        return W.high_e(n=case["n"], seed=s)
    if kind in ("adjoint", "tangent"):
        return W.adjoint_16k(n=case["n"], seed=s)
    return W.giants_100k(n=case["n"], seed=s)


def _systems(case, seed):
    """Systems of 64 to nmax particles (their counts spread evenly in the
    logarithm, the same for every seed), in the workload's random order of
    planet counts."""
    nsys, nmax = case["nsys"], case["nmax"]
    full = W.make_batched(nsys=nsys, nmin=nmax, nmax=nmax, nsteps=case["steps"],
                          seed=77_000_000 + int(seed))
    return [w.subset(n=k) for w, k in zip(full, _system_sizes(nsys, nmax))]


def _system_sizes(nsys, nmax):
    golden = 0.5 * (math.sqrt(5.0) - 1.0)
    return [int(round(64.0 * (nmax / 64.0) ** (golden * (s + 1) % 1.0))) for s in range(nsys)]


REMOVAL_RADIUS = 0.05          # au, of the hand-off cases (as in the benchmark)


def _vectors(case, seed):
    """Two seeded vectors per particle: a gradient or a direction."""
    rng = np.random.Generator(np.random.PCG64(78_000_000 + int(seed)))
    return rng.normal(size=(case["n"], 3)), rng.normal(size=(case["n"], 3))


def _tensor(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def prepare(case, seed):
    kind = case["kind"]
    state = {"case": case}
    if kind == "batch":
        state["systems"] = _systems(case, seed)
        return state
    w = state["w"] = _workload(case, seed)
    if kind == "static":
        n = w.n
        state["r"], state["v"] = _tensor(w.r), _tensor(w.v)
        state["out"] = {"r": torch.empty_like(state["r"]), "v": torch.empty_like(state["v"]),
                        "deact_step": torch.empty(n, dtype=torch.int64, device="cuda"),
                        "reason": torch.empty(n, dtype=torch.int32, device="cuda"),
                        "planet": torch.empty(n, dtype=torch.int32, device="cuda"),
                        "info": torch.empty(2, dtype=torch.int64, device="cuda")}
        return state
    sim = state["sim"] = tpm.Simulation(r_escape=w.rmax, universal_drift=kind in ("high_e", "handoff"),
                                        sort_by_e=bool(case.get("sort", False)),
                                        handoff_substeps=case.get("substeps", 0))
    sim.set_central(w.mu0)
    if kind in ("adjoint", "tangent"):
        sim.set_planets(w.mu, w.rp, w.vp, w.rcrit)
        state["r"], state["v"] = _tensor(w.r), _tensor(w.v)
        a, b = _vectors(case, seed)
        state["a"], state["b"] = _tensor(a), _tensor(b)
    return state


# --------------------------------------------------------------- one call each
def run(state):
    case = state["case"]
    kind, T = case["kind"], case["steps"]
    if kind == "batch":
        res, stats = tpm.batch_integrate(state["systems"], nsteps=T, strict=False)
        keys = ("r", "v", "deact_step", "reason", "planet")
        out = {k: np.concatenate([x[k] for x in res]) for k in keys}
        out["planet_flag"] = stats["planet_flag"]
        return out
    w = state["w"]
    if kind == "static":
        o = state["out"]
        tpm.integrate_static(w.mu0, w.mu, w.rp, w.vp, w.rcrit, state["r"].data_ptr(),
                             state["v"].data_ptr(), T, w.dt, o["r"].data_ptr(), o["v"].data_ptr(),
                             o["deact_step"].data_ptr(), o["reason"].data_ptr(),
                             o["planet"].data_ptr(), d_info=o["info"].data_ptr(),
                             stream=torch.cuda.current_stream().cuda_stream, r_escape=w.rmax, n=w.n)
        return o
    sim = state["sim"]
    if kind == "adjoint":
        r0 = state["r"].detach().requires_grad_(True)
        v0 = state["v"].detach().requires_grad_(True)
        rT, vT, step, reason = tpm_autograd.integrate(sim, r0, v0, T, w.dt, case["ckpt"])
        gr, gv = torch.autograd.grad([rT, vT], [r0, v0], [state["a"], state["b"]])
        return {"r": rT.detach(), "v": vT.detach(), "grad_r": gr, "grad_v": gv, "deact_step": step,
                "reason": reason}
    if kind == "tangent":
        rT, vT, step, reason = tpm_autograd.integrate(sim, state["r"], state["v"], T, w.dt,
                                                      case["ckpt"])
        dr, dv = tpm_autograd.tangent(sim, state["a"], state["b"])
        return {"r": rT, "v": vT, "dr": dr, "dv": dv, "deact_step": step, "reason": reason}
    sim.set_planets(w.mu, w.rp, w.vp, w.rcrit)
    if kind == "handoff":
        sim.set_removal_radii(np.full(w.np_, REMOVAL_RADIUS))
    sim.set_particles(w.r, w.v)
    if kind == "diagnostics":
        sim.set_diagnostics(case["every"], ref_planet=3, resonances=[(3, 1)])
    sim.integrate(T, w.dt)
    out = sim.particles()
    out["planet_r"], out["planet_v"] = sim.planets()
    if kind == "diagnostics":
        out.update(sim.diagnostics())
    return out


# ------------------------------------------------------------------------ work
def _flops(planets):
    """FP64 operations of one particle step with one Newton step of Kepler's
    equation: the drift and kicks (about 190) and one planet term (39) each."""
    return 190.0 + 39.0 * planets


def work(case):
    kind, T = case["kind"], case["steps"]
    if kind == "batch":
        n = sum(_system_sizes(case["nsys"], case["nmax"]))
        return {"bytes": 112.0 * n, "flops": n * T * _flops(4.5)}
    n, planets = case["n"], 1 if kind == "single" else 4
    bytes_, flops = 112.0 * n, n * T * _flops(planets)
    if kind == "adjoint":       # the gradient in and out; a reverse step is about two forward
        bytes_, flops = bytes_ + 96.0 * n, 3.0 * flops
    if kind == "tangent":
        bytes_, flops = bytes_ + 96.0 * n, 2.0 * flops + flops
    if kind == "diagnostics":
        bytes_ += 36.0 * n
    return {"bytes": bytes_, "flops": flops}


# ----------------------------------------------------- the map in plain 64 bits
def _kepler_x(ec, es, dM, where, fabs, sin, iters):
    """Root x of x - ec sin x + es (1 - cos x) = dM, Newton kept in a bracket."""
    w = 2.0 * (fabs(ec) + fabs(es))
    lo, hi = dM - w, dM + w
    x = dM / (1.0 - ec)
    x = where((x < lo) | (x > hi) | (ec > 0.9), dM, x)
    for _ in range(iters):
        s, h = sin(x), sin(0.5 * x)
        om = 2.0 * h * h                                      # 1 - cos x
        F = x - ec * s + es * om - dM
        lo, hi = where(F < 0.0, x, lo), where(F > 0.0, x, hi)
        xn = x - F / (1.0 - ec + ec * om + es * s)
        x = where((xn >= lo) & (xn <= hi), xn, 0.5 * (lo + hi))
    return x


def _planet_table(systems, T):
    """Planet positions [T+1][S][P][3], indirect term [T+1][S][3] and final
    heliocentric planet states of S systems (padded to P planets of no mass),
    planets in order of semi-major axis; also that order."""
    S, P = len(systems), max(1, max(w.np_ for w in systems))
    mu0 = np.array([w.mu0 for w in systems])
    dt = np.array([w.dt for w in systems])[:, None]
    mu = np.zeros((S, P + 1))
    r, v = np.zeros((S, P + 1, 3)), np.zeros((S, P + 1, 3))
    order = np.zeros((S, P), int)
    for s, w in enumerate(systems):
        k = w.np_
        rr = np.linalg.norm(w.rp, axis=1)
        a = 1.0 / (2.0 / rr - np.sum(w.vp * w.vp, axis=1) / (w.mu0 + w.mu))
        o = np.argsort(a, kind="stable")
        order[s] = np.concatenate([o, np.arange(k, P)])
        mu[s, 1:k + 1], r[s, 1:k + 1], v[s, 1:k + 1] = w.mu[o], w.rp[o], w.vp[o]
        for b in range(k + 1, P + 1):                         # idle bodies, far out
            r[s, b] = [1000.0 + b, 0.0, 0.0]
            v[s, b] = [0.0, math.sqrt(w.mu0 / (1000.0 + b)), 0.0]
    mu[:, 0] = mu0
    eta = np.cumsum(mu, axis=1)
    mup = mu0[:, None] * eta[:, 1:] / eta[:, :-1]             # Jacobi Kepler constants
    wj = (mu[:, 1:] / eta[:, 1:])[:, :, None]

    def jacobi(h):
        c = np.cumsum(mu[:, :, None] * h, axis=1) / eta[:, :, None]
        return h[:, 1:] - c[:, :-1]

    def helio(j):
        R = np.cumsum(wj * j, axis=1)
        h = np.zeros((S, P + 1, 3))
        h[:, 1:] = j
        h[:, 2:] += R[:, :-1]
        return h

    off = np.eye(P + 1)[None]

    def accel(j):
        h = helio(j)
        d = h[:, :, None, :] - h[:, None, :, :]
        d3 = (np.sum(d * d, axis=3) + off) ** 1.5
        a = -np.sum((mu[:, None, :] / d3)[..., None] * d, axis=2)
        c = np.cumsum(mu[:, :, None] * a, axis=1) / eta[:, :, None]
        j3 = np.sum(j * j, axis=2) ** 1.5
        return h, -a[:, 0], a[:, 1:] - c[:, :-1] + (mup / j3)[..., None] * j

    def drift(j, w):
        r0 = np.sqrt(np.sum(j * j, axis=2))
        u = np.sum(j * w, axis=2)
        al = 2.0 / r0 - np.sum(w * w, axis=2) / mup
        n = np.sqrt(mup * al) * al
        ec, es = 1.0 - r0 * al, u * np.sqrt(al / mup)
        x = _kepler_x(ec, es, n * dt, np.where, np.abs, np.sin, 6)
        s, hs = np.sin(x), np.sin(0.5 * x)
        om = 2.0 * hs * hs
        r1 = (1.0 - ec + ec * om + es * s) / al
        f, g = 1.0 - om / (al * r0), dt + (s - x) / n
        fd, gd = -n * s / (al * al * r1 * r0), 1.0 - om / (al * r1)
        return (f[..., None] * j + g[..., None] * w, fd[..., None] * j + gd[..., None] * w)

    J, Wj = jacobi(r), jacobi(v)
    pos, h0 = np.zeros((T + 1, S, P, 3)), np.zeros((T + 1, S, 3))
    h, z, a = accel(J)
    pos[0], h0[0] = h[:, 1:], z
    hh = 0.5 * dt[..., None]
    for t in range(1, T + 1):
        J, Wj = drift(J, Wj + hh * a)
        h, z, a = accel(J)
        Wj = Wj + hh * a
        pos[t], h0[t] = h[:, 1:], z
    return mu[:, 1:], order, pos, h0, helio(J)[:, 1:], helio(Wj)[:, 1:]


def _drift(mu0, dt, r, v, iters, differentiable, unbound):
    """Kepler drift of particles [n][3] about mu0 by dt (numbers or [n])."""
    r0 = torch.sqrt((r * r).sum(1))
    u = (r * v).sum(1)
    al = 2.0 / r0 - (v * v).sum(1) / mu0
    ab = al.abs() if unbound else al
    n = torch.sqrt(mu0 * ab) * ab
    ec, es = 1.0 - r0 * al, u * torch.sqrt(ab / mu0)
    dM = n * dt
    if differentiable:
        with torch.no_grad():
            x = _kepler_x(ec, es, dM, torch.where, torch.abs, torch.sin, iters)
            hs = torch.sin(0.5 * x)
            slope = 1.0 - ec + ec * 2.0 * hs * hs + es * torch.sin(x)
        hs = torch.sin(0.5 * x)
        x = x - (x - ec * torch.sin(x) + es * 2.0 * hs * hs - dM) / slope
    else:
        turns = 2.0 * math.pi * torch.round(dM / (2.0 * math.pi)) if unbound else 0.0
        x = _kepler_x(ec, es, dM - turns, torch.where, torch.abs, torch.sin, iters)
    s, hs = torch.sin(x), torch.sin(0.5 * x)
    om = 2.0 * hs * hs
    xm = x - s
    r1 = (1.0 - ec + ec * om + es * s) / al
    g = dt - xm / n
    if unbound:
        # whole turns leave g alone (it holds sin x - x of the reduced anomaly)
        g = torch.where(turns == 0.0, g, (dM - turns - xm) / n)
        # hyperbolic: es (cosh x - 1) + ec sinh x - x = dM, x between 0 and dM/(e - 1)
        hyp = al < 0.0
        e = torch.sqrt(torch.clamp(ec * ec - es * es, min=1.0 + 1e-12))
        lo, hi = torch.zeros_like(dM), torch.where(hyp, dM / (e - 1.0), 0.0)
        hi = torch.clamp(hi, max=60.0)
        y = torch.minimum(hi, torch.asinh(dM / e) + 1.0)
        for _ in range(40):
            sh, c1 = torch.sinh(y), 2.0 * torch.sinh(0.5 * y) ** 2
            F = es * c1 + ec * sh - y - dM
            lo, hi = torch.where(F < 0.0, y, lo), torch.where(F > 0.0, y, hi)
            yn = y - F / (es * sh + ec * (1.0 + c1) - 1.0)
            y = torch.where((yn >= lo) & (yn <= hi), yn, 0.5 * (lo + hi))
        sh, c1 = torch.sinh(y), 2.0 * torch.sinh(0.5 * y) ** 2
        r1h = (es * sh + ec * (1.0 + c1) - 1.0) / ab
        s, r1 = torch.where(hyp, sh, s), torch.where(hyp, r1h, r1)
        om = torch.where(hyp, c1, om)                         # |1 - cos| resp. cosh - 1
        g = torch.where(hyp, dt - (sh - y) / n, g)
    f = 1.0 - om / (ab * r0)
    fd, gd = -n * s / (ab * ab * r1 * r0), 1.0 - om / (ab * r1)
    return (f[:, None] * r + g[:, None] * v, fd[:, None] * r + gd[:, None] * v)


def _particles(systems, T, iters=6, differentiable=False, unbound=False, r=None, v=None):
    """Particle states after T steps, by the map in 64 bits (removed particles
    keep the state of their removal), and the planets' final states."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    mu, order, pos, h0, hr, hv = _planet_table(systems, T)
    pos, h0, mu = (torch.tensor(a, device=dev) for a in (pos, h0, mu))
    P = mu.shape[1]
    one = len(systems) == 1
    sys_of = torch.tensor(np.repeat(np.arange(len(systems)), [w.n for w in systems]), device=dev)

    def col(values):
        return values[0] if one else torch.tensor(values, dtype=torch.float64, device=dev)[sys_of]

    mu0, dt, rmax = (col([getattr(w, k) for w in systems]) for k in ("mu0", "dt", "rmax"))
    rcrit = np.zeros((len(systems), P))
    for s, w in enumerate(systems):
        rcrit[s, :w.np_] = w.rcrit[order[s, :w.np_]]
    rcrit = torch.tensor(rcrit, device=dev)
    m, rc = (mu, rcrit) if one else (mu[sys_of], rcrit[sys_of])
    if r is None:
        r = torch.tensor(np.concatenate([w.r for w in systems]), device=dev)
        v = torch.tensor(np.concatenate([w.v for w in systems]), device=dev)
    h = 0.5 * dt if one else 0.5 * dt[:, None]
    live = torch.ones(r.shape[0], dtype=torch.bool, device=dev)

    def accel(t, r):
        p, z = (pos[t], h0[t]) if one else (pos[t][sys_of], h0[t][sys_of])
        d = r[:, None, :] - p
        d2 = (d * d).sum(2)
        return z - ((m / (d2 * torch.sqrt(d2)))[..., None] * d).sum(1), (d2 < rc * rc).any(1)

    a, near = accel(0, r)
    live = live & ~near & ((r * r).sum(1) <= rmax * rmax)
    for t in range(1, T + 1):
        nr, nv = _drift(mu0, dt, r, v + h * a, iters, differentiable, unbound)
        b, near = accel(t, nr)
        nv = nv + h * b
        on = live[:, None]
        r, v, a = torch.where(on, nr, r), torch.where(on, nv, v), torch.where(on, b, a)
        live = live & ~near & ((r * r).sum(1) <= rmax * rmax)
    return r, v, order, hr, hv


def exact(case, seed):
    kind, T = case["kind"], case["steps"]
    if kind == "handoff":
        return None     # substeps of a few particles at nearly every step: minutes in torch
    none = dict.fromkeys(("deact_step", "reason", "planet"))
    if kind == "batch":
        systems = _systems(case, seed)
        r, v, *_ = _particles(systems, T)
        return {"r": r, "v": v, **none, "planet_flag": None}
    w = _workload(case, seed)
    if kind == "adjoint":
        dev = "cuda" if torch.cuda.is_available() else "cpu"
        if case["n"] * T > 20_000_000:
            return None                                       # the graph would not fit
        r0 = torch.tensor(w.r, device=dev).requires_grad_(True)
        v0 = torch.tensor(w.v, device=dev).requires_grad_(True)
        rT, vT, *_ = _particles([w], T, differentiable=True, r=r0, v=v0)
        ga, gb = (torch.tensor(x, device=dev) for x in _vectors(case, seed))
        gr, gv = torch.autograd.grad([rT, vT], [r0, v0], [ga, gb])
        return {"r": rT.detach(), "v": vT.detach(), "grad_r": gr, "grad_v": gv,
                "deact_step": None, "reason": None}
    if kind == "tangent":
        import torch.autograd.forward_ad as fwd
        dev = "cuda" if torch.cuda.is_available() else "cpu"
        a, b = (torch.tensor(x, device=dev) for x in _vectors(case, seed))
        with torch.no_grad(), fwd.dual_level():
            rT, vT, *_ = _particles([w], T, differentiable=True,
                                    r=fwd.make_dual(torch.tensor(w.r, device=dev), a),
                                    v=fwd.make_dual(torch.tensor(w.v, device=dev), b))
            (r, dr), (v, dv) = (tuple(x.clone() for x in fwd.unpack_dual(q)) for q in (rT, vT))
        return {"r": r, "v": v, "dr": dr, "dv": dv, "deact_step": None, "reason": None}
    high = kind == "high_e"
    r, v, order, hr, hv = _particles([w], T, iters=25 if high else 6, unbound=high)
    out = {"r": r, "v": v, **none}
    if kind == "static":
        return {**out, "info": None}
    back = np.empty_like(order[0])
    back[order[0]] = np.arange(len(back))
    out["planet_r"], out["planet_v"] = hr[0][back], hv[0][back]
    if kind == "diagnostics":
        out.update(dict.fromkeys(("emax", "emax_step", "flags", "lo", "hi")))
    return out
