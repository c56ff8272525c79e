"""The drift of long arcs and large eccentricities, t^2 <= q max(1, 4 q) with
t = dM/(1 - e cos E) and q = 1 - e^2, within and around that range: against the
oracle's converged drift to the bar of tests/test_gpu_short_drift.py, or, where the
fixed-count solve itself (a threshold below 1e-14 keeps a call on it) is further
off than that, to twice its error; that solve's bits outside the range, and its
refusals; the same bits whoever shares the wavefront; the gradients of such steps
against those through the fixed-count solve; and the time of a step, which with a
first attempt in vain and the fixed-count solve was longer than with that solve
alone."""
import math

import numpy as np
import pytest

from paper_2011_03484_amd import workloads as W

pytestmark = pytest.mark.gpu

MU, A = W.MU_SUN, 7.0
FIXED = 9e-15               # threshold that leaves every drift to the fixed-count solve


@pytest.fixture(scope="module")
def tpm():
    import paper_2011_03484_amd as P
    P.load()
    return P


def _states(e, E, seed):
    """Orbits of semi-major axis A at eccentric anomalies E, in random planes."""
    rng = np.random.default_rng(seed)
    n = len(E)
    ang = [rng.uniform(0, 2 * math.pi, n) for _ in range(3)]
    return W.elements_to_cartesian(MU, np.full(n, A), e, ang[0], ang[1], ang[2], E - e * np.sin(E))


def _edge(e):
    q = 1.0 - e * e
    return np.sqrt(q * np.maximum(1.0, 4.0 * q))


@pytest.mark.parametrize("e", [0.0, 0.1, 0.4, 0.53, 0.7, 0.8, 0.9, 0.99])
@pytest.mark.parametrize("part", [0.3, 0.9, 0.999, 1.001, 1.3, -0.5, -0.999])
def test_against_converged_drift(tpm, orc, e, part):
    """Each particle with the step that brings its t to `part` of the edge (beyond
    it, |t| > 0.14, only the fixed-count solve serves)."""
    n = 67
    E = np.concatenate([[0.0, math.pi, 0.5 * math.pi], np.random.default_rng(3).uniform(-math.pi, math.pi, n - 3)])
    e = np.full(n, e)
    r, v = _states(e, E, 11)
    arcs = part * _edge(e) * (1.0 - e * np.cos(E))
    worst = fixed = 0.0
    for i in range(n):
        dt = arcs[i] / math.sqrt(MU / A ** 3)
        gr, gv, ok = tpm.debug_drift(MU, r[i:i + 1], v[i:i + 1], dt)
        hr, hv, okf = tpm.debug_drift(MU, r[i:i + 1], v[i:i + 1], dt, kepler_ftol=FIXED)
        okc, rr, vv, _ = orc.drift(MU, r[i], v[i], dt, kfix=5)
        assert ok[0] == okc
        if abs(part) < 1.0:
            assert okc
        if not (okc and okf[0]):
            continue
        if abs(part) > 1.0:
            assert np.array_equal(gr, hr) and np.array_equal(gv, hv)
            continue
        _, r2, v2, _ = orc.drift(MU, r[i] * (1 + 2.0 ** -52), v[i], dt, kfix=5)
        rel = lambda x, y: np.linalg.norm(x - y) / np.linalg.norm(y)
        bound = 8 * max(rel(r2, rr), rel(v2, vv)) + 2e-15 + 8 * 2.0 ** -52 * abs(arcs[i]) / (1 - e[i])
        worst = max(worst, rel(gr[0], rr) / bound, rel(gv[0], vv) / bound)
        fixed = max(fixed, rel(hr[0], rr) / bound, rel(hv[0], vv) / bound)
    assert worst <= max(1.0, 2 * fixed), (worst, fixed)


@pytest.mark.parametrize("mode", ["fixed", "universal"])
def test_lanes_do_not_depend_on_their_wavefront(tpm, mode):
    """Lanes of every kind mixed (short, second step, wide, out of all, unbound)
    give the bits each gives alone."""
    rng = np.random.default_rng(5)
    n = 256
    e = np.concatenate([np.linspace(0.0, 0.99, n // 2), rng.uniform(0.0, 0.2, n // 2)])
    E = rng.uniform(-math.pi, math.pi, n)
    r, v = _states(e, E, 12)
    v[7::32] *= 2.5                                            # unbound
    r[: n // 4] *= 8.0                                         # short arcs
    v[: n // 4] /= math.sqrt(8.0)
    k = rng.permutation(n)
    r, v = r[k], v[k]
    for arc in (0.2, 0.6, 1.2, 2.5):
        dt = arc / math.sqrt(MU / A ** 3)
        run = ((lambda a, b: tpm.debug_drift(MU, a, b, dt)) if mode == "fixed"
               else (lambda a, b: tpm.debug_drift_universal(MU, a, b, dt, mode=1)))
        mixed = run(r, v)
        for i in range(0, n, 5):
            for x, y in zip(mixed, run(r[i:i + 1], v[i:i + 1])):
                assert np.array_equal(x[i:i + 1], y), (arc, i)


def test_gradients_of_long_steps(tpm):
    """How far the two sweeps are from each other's transpose, at most twice what it
    is through the fixed-count solve (the same sweeps about the same orbits, their
    rounding alone different)."""
    import torch
    from paper_2011_03484_amd import autograd as AG
    n, T = 130, 20
    rng = np.random.default_rng(8)
    e, E = rng.uniform(0.0, 0.6, n), rng.uniform(-math.pi, math.pi, n)
    r, v = _states(e, E, 13)
    w = W.giants_100k(n=1, seed=14)
    t = lambda x: torch.tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")
    dr, dv, gr, gv = (t(rng.normal(size=(n, 3))) for _ in range(4))
    dt = 0.8 / math.sqrt(MU / A ** 3)
    norm = lambda *x: torch.sqrt(sum((y * y).sum(1) for y in x))

    def mismatch(**opts):
        s = tpm.Simulation(**opts)
        s.set_central(w.mu0)
        s.set_planets(w.mu, w.rp * 10.0, w.vp / math.sqrt(10.0), np.full(4, 1e-3))
        r0, v0 = t(r).requires_grad_(True), t(v).requires_grad_(True)
        rT, vT, step, _ = AG.integrate(s, r0, v0, T, dt, 7)
        jr, jv = AG.tangent(s, dr, dv)
        ar, av = torch.autograd.grad([rT, vT], [r0, v0], [gr, gv])
        off = ((jr * gr).sum(1) + (jv * gv).sum(1) - (dr * ar).sum(1) - (dv * av).sum(1)).abs()
        off = off / (norm(jr, jv) * norm(gr, gv) + norm(dr, dv) * norm(ar, av))
        return off[step < 0], step

    (wide, step), (fixed, fstep) = mismatch(), mismatch(kepler_ftol=FIXED)
    assert torch.equal(step, fstep) and len(wide) > n // 2    # (fast ones are refused a drift)
    assert float(wide.max()) <= 2 * float(fixed.max())


@pytest.mark.parametrize("steps,universal,bound", [(15, False, 2.15), (15, True, 2.75), (6, True, 4.1)])
def test_step_time(tpm, steps, universal, bound):
    """Milliseconds for 2,000 steps of a wavefront on a supplied table; 2.46, 3.30 and
    5.70 with the short drift's attempt before the fixed-count solve (universal:
    the universal one), 1.77, 2.07 and 2.73 now, the bound between."""
    w = W.giants_100k(n=1, seed=3)
    rng = np.random.default_rng(4)
    w.r, w.v = W._particles(rng, 64, 2.0, 2.1, 0.0, 0.1, 3.0)
    dt = 2 * math.pi * math.sqrt(2.0 ** 3 / MU) / steps
    s = tpm.Simulation(r_escape=1e4, universal_drift=universal)
    s.set_central(w.mu0)
    s.set_planets(w.mu, w.rp, w.vp, np.full(4, 1e-4))
    table = s.planet_table(2000, dt)
    best = np.inf
    for _ in range(5):
        s.set_planets(w.mu, w.rp, w.vp, np.full(4, 1e-4))
        s.set_particles(w.r, w.v)
        s.set_planet_table(table)
        s.integrate(2000, dt)
        best = min(best, s.stats()["particle_ms"])
    assert best < bound, best
