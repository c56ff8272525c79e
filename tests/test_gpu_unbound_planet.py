"""A planet whose orbit becomes unbound in a drift, with no close pair before: the
event is reported as that, the body is left where the drift found it, and the
run goes on; rows and end states are the oracle's, for the matrix form of the
planet map (two to four planets), the form of a body per lane, and the
many-system map."""
import ctypes as C
import math

import numpy as np
import pytest

from paper_2011_03484_amd import workloads as W

pytestmark = pytest.mark.gpu

T = 200


@pytest.fixture(scope="module")
def tpm():
    import paper_2011_03484_amd as P
    P.load()
    return P


def _starts(orc, k):
    """Two starts of k planets in order of semi-major axis: light ones on circular
    orbits, a heavy one, and a light one on an eccentric orbit across that one's,
    whose kicks (at long steps) free it; drawn until the oracle reports an unbound
    orbit as the first event."""
    rng = np.random.default_rng(1000 + k)
    found = []
    while len(found) < 2:
        a = np.concatenate([3.0 * 1.6 ** np.arange(k - 2), [rng.uniform(30, 60)], [rng.uniform(70, 200)]])
        e = np.concatenate([np.full(k - 1, 0.01), [rng.uniform(0.85, 0.97)]])
        mu = W.MU_SUN * np.concatenate([np.full(k - 2, 1e-9), [10 ** rng.uniform(-2, -0.5)], [1e-9]])
        ang = [rng.uniform(0, 2 * math.pi, k) for _ in range(3)]
        rp, vp = W.elements_to_cartesian(W.MU_SUN + mu, a, e, np.full(k, 0.01), *ang)
        dt = rng.uniform(0.05, 0.6) * 2 * math.pi * math.sqrt(3.0 ** 3 / W.MU_SUN)
        eph = orc.ephemeris(W.MU_SUN, mu, rp, vp, T, dt)
        if eph.flag == -2:
            found.append((mu, rp, vp, dt, eph))
    return found


def _bar(orc, mu, rp, vp, dt, ref):
    """Largest relative distance of a table from ref, and what is allowed: 1e-11 or
    a hundred times the oracle's response to an ulp and to its rounding sequence."""
    k = len(mu)

    def off(t):
        d = np.linalg.norm((t - ref).reshape(T + 1, k + 1, 3), axis=2)
        return np.max(d / np.linalg.norm(ref.reshape(T + 1, k + 1, 3), axis=2))

    other = orc.ephemeris(W.MU_SUN, mu, np.nextafter(rp, np.inf), vp, T, dt).table
    with orc.rounding_probe():
        probe = orc.ephemeris(W.MU_SUN, mu, rp, vp, T, dt).table
    return off, max(1e-11, 100 * off(other), 100 * off(probe))


@pytest.mark.parametrize("k", [2, 3, 4, 5, 8])
def test_flagged_and_stays(tpm, orc, k):
    for mu, rp, vp, dt, eph in _starts(orc, k):
        off, bar = _bar(orc, mu, rp, vp, dt, eph.table)
        assert bar < 1e-3                     # the start says something
        s = tpm.Simulation(chunk_steps=64)
        s.set_central(W.MU_SUN)
        s.set_planets(mu, rp, vp, np.zeros(k))
        rows = np.full((T + 1, 3 * k + 3), np.nan)
        rc = tpm.load().tpm_planet_table(s._h, T, dt, rows.ctypes.data_as(C.c_void_p))
        assert rc == tpm.TPM_EPLANET and b"unbound" in tpm.load().tpm_last_error()
        assert np.all(np.isfinite(rows)) and off(rows) <= bar
        # the run of a simulation, its end state the last row's
        s.set_particles(np.array([[900.0, 0.0, 0.0]]), np.array([[0.0, 0.02, 0.0]]))
        with pytest.raises(tpm.PlanetEncounterError, match="unbound"):
            s.integrate(T, dt)
        r, v = s.planets()
        assert np.all(np.isfinite(r)) and np.all(np.isfinite(v))
        ends = np.concatenate([rows[:-1], np.concatenate([r.ravel(), rows[-1, 3 * k:]])[None]])
        assert off(ends) <= bar
        # the particle passes the same planets one by one and in many systems
        w = W.Workload("unbound", W.MU_SUN, mu, rp, vp, np.zeros(k), 1e6,
                       np.array([[900.0, 0.0, 0.0]]), np.array([[0.0, 0.02, 0.0]]), dt, T)
        res, st = tpm.batch_integrate([w, w], nsteps=T, strict=False)
        assert list(st["planet_flag"]) == [-2, -2]
        for g in res:
            assert np.array_equal(g["r"], s.particles()["r"])
