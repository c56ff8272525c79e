"""Diagnostics sampled from states that the particle launches store on their way,
against the same run with a launch ending at every sample (a snapshot callback
asks for that): the same accumulators and states, bit for bit, with samples at,
before and after chunk, item and call boundaries, and with every kind of removal
between them."""
import numpy as np
import pytest

from paper_2011_03484_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tpm():
    import paper_2011_03484_amd as P
    P.load()
    return P


def _run(tpm, w, pieces, every, snapshot, res, **opts):
    s = tpm.Simulation(r_escape=w.rmax, **opts)
    s.set_central(w.mu0)
    s.set_planets(w.mu, w.rp, w.vp, w.rcrit)
    s.set_particles(w.r, w.v)
    k = {"ref_planet": w.np_ - 1, "resonances": res} if res else {}
    s.set_diagnostics(every, snapshot=(lambda step, d: None) if snapshot else None, **k)
    for T in pieces:
        s.integrate(T, w.dt)
    return s.diagnostics(), s.particles(), s.stats()["n_active"]


def _equal(a, b):
    if isinstance(a, dict):
        return all(_equal(a[k], b[k]) for k in a)
    if isinstance(a, (tuple, list)):
        return all(_equal(x, y) for x, y in zip(a, b))
    return np.array_equal(a, b)


@pytest.mark.parametrize("every,pieces,opts", [
    (1, [40], {}), (7, [100, 6, 1], {}), (16, [16, 16, 31], {}), (100, [250, 49, 1], {"chunk_steps": 64}),
    (10, [95], {"chunk_steps": 10}), (25, [130], {"chunk_steps": 100, "sub_chunks": 100}),
    (64, [200], {"chunk_steps": 64, "resync_chunks": 2}), (1000, [130], {}), (1 << 40, [50], {}),
])
@pytest.mark.parametrize("res", [(), [(3, 1)]])
def test_stored_equals_cut(tpm, every, pieces, opts, res):
    w = W.giants_100k(n=700, seed=401)
    rng = np.random.default_rng(1)
    # removals on the way: hand-picked particles beside planets, and outward ones
    k = rng.choice(w.n, 90, replace=False)
    w.r[k[:60]] = w.rp[rng.integers(0, 4, 60)] + rng.normal(size=(60, 3)) * 0.8
    w.v[k[60:]] *= 1.5
    w.rmax = 40.0
    a = _run(tpm, w, pieces, every, False, res, **opts)
    b = _run(tpm, w, pieces, every, True, res, **opts)
    assert _equal(a, b)
    if sum(pieces) >= 100:
        assert np.sum(a[1]["reason"] != tpm.ACTIVE) > 0


def test_refused_drifts_and_many_tiles(tpm):
    """Near-parabolic particles without the universal fallback: refused drifts."""
    w = W.high_e(n=9000, seed=402)
    a = _run(tpm, w, [60, 30], 9, False, [])
    b = _run(tpm, w, [60, 30], 9, True, [])
    assert _equal(a, b)
    assert np.sum(a[1]["reason"] == tpm.KEPLER) > 0


@pytest.mark.parametrize("k", [1, 2, 6])
def test_planet_counts(tpm, k):
    w = [w for w in W.make_batched(nsys=40, nmin=300, nmax=300, seed=12) if w.np_ == k][0]
    a = _run(tpm, w, [75], 10, False, [(2, 1), (3, 2)], universal_drift=True)
    b = _run(tpm, w, [75], 10, True, [(2, 1), (3, 2)], universal_drift=True)
    assert _equal(a, b)
