"""The planet map's one-step Kepler solve at the edges of what it serves (arcs of
three quarters of a radian from the mean motion's, eccentricities about 0.4,
forwards and backwards, and orbits of which some steps are served and some not):
rows against the oracle to the bar of tests/test_gpu_planet_map.py, and the same
rows, bit for bit, however a run is cut (the choice is each body's own)."""
import math

import numpy as np
import pytest

from paper_2011_03484_amd import workloads as W
from test_gpu_planet_map import _planets, tpm  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 2, 4])
@pytest.mark.parametrize("e,steps_per_orbit,T", [(0.0, 8.5, 120), (0.2, 10, 120), (0.25, 25, 200),
                                                 (0.38, 50, 200), (0.41, 50, 200), (0.7, 120, 240),
                                                 (0.05, -30, 200), (0.3, 3.7, 40)])
def test_rows(tpm, orc, k, e, steps_per_orbit, T):  # noqa: F811
    mu, rp, vp, period = _planets(k, e, 70 + k)
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
    # live maps of one call, of steps one by one, and of short chunks
    ends = []
    for chunk, pieces in ((0, [T]), (0, [1] * T), (5, [T]), (17, [T - 3, 3])):
        c = tpm.Simulation(chunk_steps=chunk)
        c.set_central(W.MU_SUN)
        c.set_planets(mu, rp, vp, np.zeros(k))
        c.set_particles(np.array([[500.0, 0, 0]]), np.array([[0, 0.2, 0]]))
        for p in pieces:
            c.integrate(p, dt)
        ends.append(np.concatenate(c.planets()))
    for q in ends[1:]:
        assert np.array_equal(q, ends[0])
