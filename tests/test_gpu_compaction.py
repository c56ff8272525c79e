"""The compaction at the edges of its tiles of 1,024 entries, over more than 64
tiles (a look-back of more than one round), and where none, all or a pattern of
the particles goes: a run compacted after every step equals the run compacted
only at its end, bit for bit, and counts its survivors.
"""
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


def _run(tpm, w, v, steps, resync, **opts):
    s = tpm.Simulation(r_escape=w.rmax, chunk_steps=1, resync_chunks=resync, **opts)
    s.set_central(w.mu0)
    s.set_planets(w.mu, w.rp, w.vp, w.rcrit)
    s.set_particles(w.r, v)
    s.integrate(steps, w.dt)
    mid = s.stats()["n_active"]
    s.integrate(2, w.dt)
    return s.particles(), mid, s.stats()["n_active"]


@pytest.mark.parametrize("n", [1, 63, 1023, 1024, 1025, 2049, 66_001])
@pytest.mark.parametrize("goes", ["none", "all", "odd", "first", "random"])
def test_every_step_equals_end_only(tpm, n, goes):
    """Particles that go are sent outwards fast enough to leave within 4 steps,
    at different ones."""
    w = W.giants_100k(n=n, seed=17)
    rng = np.random.default_rng(n)
    k = np.arange(n)
    out = {"none": k < 0, "all": k >= 0, "odd": k % 2 == 1, "first": k < (n + 1) // 2,
           "random": rng.random(n) < 0.3}[goes]
    u = w.r / np.linalg.norm(w.r, axis=1)[:, None]
    speed = w.rmax / abs(w.dt) * rng.choice([1.2, 0.6, 0.3], n)
    v = np.where(out[:, None], u * speed[:, None], w.v)
    got, mid, end = _run(tpm, w, v, 5, 1, universal_drift=True)
    want, mid1, end1 = _run(tpm, w, v, 5, 1000, universal_drift=True)
    for key in KEYS:
        assert np.array_equal(got[key], want[key]), (key, n, goes)
    assert np.all(got["reason"][out] != tpm.ACTIVE)
    assert mid == mid1 and end == end1 == np.sum(got["reason"] == tpm.ACTIVE)
