"""Workspaces kept from call to call: a simulation given other particles and
planets (more, fewer, none, with and without the hand-off and the diagnostics),
and many-system calls of other sizes, give the bits of a fresh one; also from
two threads at once."""
import threading

import numpy as np
import pytest

from paper_2011_03484_amd import workloads as W

pytestmark = pytest.mark.gpu

KEYS = ("r", "v", "deact_step", "reason", "planet")


@pytest.fixture(scope="module")
def tpm():
    import paper_2011_03484_amd as P
    P.load()
    return P


def _run(tpm, s, w, T, ho):
    s.set_central(w.mu0)
    s.set_planets(w.mu, w.rp, w.vp, w.rcrit)
    if ho:
        s.set_removal_radii(0.1 * w.rcrit)
    s.set_particles(w.r, w.v)
    s.integrate(T, w.dt)
    out = s.particles()
    out["planets"] = np.concatenate(s.planets(), axis=1)
    st = s.stats()
    out["steps"] = np.array([st["active_particle_steps"], st["n_active"], st["handoffs"]])
    return out


def _cases():
    yield W.giants_100k(n=3000, seed=1), 150
    yield W.single_planet(n=70, seed=2), 300
    yield W.giants_100k(n=1, seed=3).subset(n=0), 20
    yield W.giants_100k(n=20_000, seed=4), 40
    eight = [w for w in W.make_batched(nsys=60, nmin=90, nmax=90, seed=3) if w.np_ == 8][0]
    yield eight, 100
    yield W.giants_100k(n=3000, seed=1), 150


@pytest.mark.parametrize("ho", [0, 4])
def test_one_simulation_for_many_sets(tpm, ho):
    opts = dict(r_escape=900.0, handoff_substeps=ho, chunk_steps=64)
    kept = tpm.Simulation(**opts)
    for w, T in _cases():
        fresh = tpm.Simulation(**opts)
        a, b = _run(tpm, kept, w, T, ho), _run(tpm, fresh, w, T, ho)
        for k in a:
            assert np.array_equal(a[k], b[k]), (w.name, w.n, k)
        blob = kept.get_state()
        other = tpm.Simulation(**opts)
        other.set_state(blob)
        assert other.get_state() == blob
        if not ho:
            kept.set_diagnostics(10)
            kept.integrate(30, w.dt)
            fresh.set_diagnostics(10)
            fresh.integrate(30, w.dt)
            assert np.array_equal(kept.diagnostics()["emax"], fresh.diagnostics()["emax"])


def test_many_system_calls_of_other_sizes(tpm):
    sizes = [(3, 200, 90), (9, 64, 700), (2, 900, 30), (9, 64, 700)]
    for nsys, nmax, T in sizes:
        systems = W.make_batched(nsys=nsys, nmin=40, nmax=nmax, seed=nsys)
        res, st = tpm.batch_integrate(systems, nsteps=T, strict=False)
        steps = 0
        for w, g in zip(systems, res):
            s = tpm.Simulation(r_escape=systems[0].rmax)
            s.set_central(w.mu0)
            s.set_planets(w.mu, w.rp, w.vp, w.rcrit)
            s.set_particles(w.r, w.v)
            try:
                s.integrate(T, w.dt)
            except tpm.PlanetEncounterError:
                pass
            ref = s.particles()
            for k in KEYS:
                assert np.array_equal(g[k], ref[k]), (nsys, k)
            steps += s.stats()["active_particle_steps"]
        assert st["active_particle_steps"] == steps


def test_refused_options_stay_refused(tpm):
    w = W.make_batched(nsys=1, nmin=40, nmax=40, seed=5)
    for bad in (dict(kepler_iters=65), dict(block_threads=96), dict(waves_per_simd=9),
                dict(chunk_steps=-1), dict(resync_chunks=-1), dict(r_escape=np.inf)):
        with pytest.raises(tpm.TpmError):
            tpm.batch_integrate(w, nsteps=5, **bad)


def test_two_threads(tpm):
    a, b = W.giants_100k(n=2000, seed=7), W.make_batched(nsys=5, nmin=40, nmax=300, seed=8)
    ref_a = tpm.run_workload(a, nsteps=80)
    ref_b = tpm.batch_integrate(b, nsteps=120, strict=False)[0]
    bad = []

    def one():
        for _ in range(5):
            g = tpm.run_workload(a, nsteps=80)
            bad.extend(k for k in KEYS if not np.array_equal(g[k], ref_a[k]))

    def two():
        for _ in range(5):
            g = tpm.batch_integrate(b, nsteps=120, strict=False)[0]
            bad.extend(k for x, y in zip(g, ref_b) for k in KEYS if not np.array_equal(x[k], y[k]))

    t = [threading.Thread(target=f) for f in (one, two)]
    for x in t:
        x.start()
    for x in t:
        x.join()
    assert not bad
