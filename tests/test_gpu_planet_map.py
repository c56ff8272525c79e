"""The planet map on matrix instructions (one to four planets) where it leaves
its fast form: eccentric orbits, on which the short sine range or two Newton
steps do not suffice for some or all of the steps, and long steps.  Against the
oracle's table, to the 1e-11 of the parity bar or a hundred times the oracle's
own response to a one-ulp change of a planet's start and to its rounding
sequence, whichever is larger."""
import math

import numpy as np
import pytest

from paper_2011_03484_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tpm():
    import paper_2011_03484_amd as P
    P.load()
    return P


def _planets(k, e, seed):
    rng = np.random.default_rng(seed)
    a = 3.0 * 2.2 ** np.arange(k)
    mu = W.MU_SUN * 10 ** rng.uniform(-6, -4, k)
    ang = [rng.uniform(0, 2 * math.pi, k) for _ in range(3)]
    rp, vp = W.elements_to_cartesian(W.MU_SUN + mu, a, np.full(k, e), rng.uniform(0, 0.1, k), *ang)
    return mu, rp, vp, 2 * math.pi * math.sqrt(a[0] ** 3 / W.MU_SUN)


@pytest.mark.parametrize("k", [1, 2, 3, 4])
@pytest.mark.parametrize("e,steps_per_orbit,T", [(0.02, 40, 333), (0.08, 25, 300), (0.12, 40, 300),
                                                 (0.4, 60, 200), (0.05, 9, 100)])
def test_rows_match_oracle(tpm, orc, k, e, steps_per_orbit, T):
    mu, rp, vp, period = _planets(k, e, 40 + k)
    dt = period / steps_per_orbit
    s = tpm.Simulation()
    s.set_central(W.MU_SUN)
    s.set_planets(mu, rp, vp, np.zeros(k))
    got = s.planet_table(T, dt)
    ref = orc.ephemeris(W.MU_SUN, mu, rp, vp, T, dt).table
    other = orc.ephemeris(W.MU_SUN, mu, np.nextafter(rp, np.inf), vp, T, dt).table
    with orc.rounding_probe():
        probe = orc.ephemeris(W.MU_SUN, mu, rp, vp, T, dt).table

    def off(t):
        d = np.linalg.norm((t - ref).reshape(T + 1, k + 1, 3), axis=2)
        return np.max(d / np.linalg.norm(ref.reshape(T + 1, k + 1, 3), axis=2))

    assert off(got) <= max(1e-11, 100 * off(other), 100 * off(probe))
    # the same rows when the run is cut at every step or two
    cut = tpm.Simulation(chunk_steps=7)
    cut.set_central(W.MU_SUN)
    cut.set_planets(mu, rp, vp, np.zeros(k))
    assert np.array_equal(cut.planet_table(T, dt), got)
    # and the state a run arrives at is the last row's
    cut.set_particles(np.array([[500.0, 0, 0]]), np.array([[0, 0.2, 0]]))
    cut.integrate(T, dt)
    last = got[-1, :3 * k].reshape(k, 3)
    assert np.allclose(cut.planets()[0], last, rtol=0, atol=4e-16 * np.abs(rp).max() * 8)


def test_unbound_planet_is_flagged_and_stays(tpm):
    """A planet kicked past escape by a close companion: the event is reported,
    and the run goes on with finite rows."""
    mu = np.array([W.MU_SUN * 1e-3, W.MU_SUN * 0.2])
    rp = np.array([[5.0, 0, 0], [5.2, 0.02, 0]])
    vc = math.sqrt(W.MU_SUN / 5.0)
    vp = np.array([[0, vc, 0], [0, vc * 1.05, 0]])
    s = tpm.Simulation()
    s.set_central(W.MU_SUN)
    s.set_planets(mu, rp, vp, np.zeros(2))
    with pytest.raises(tpm.PlanetEncounterError):
        s.planet_table(400, 0.05)
