"""The planet map of five to eight planets, a body per lane, whose drift is the
one-step solve where that serves and the general form elsewhere: the checks of
tests/test_gpu_planet_step.py (rows against the oracle, the same rows however a
run is cut), and the same particle from the many-system call."""
import numpy as np
import pytest

from paper_2011_03484_amd import workloads as W
from test_gpu_planet_map import _planets, tpm  # noqa: F401
from test_gpu_planet_step import test_rows as _check_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [5, 6, 7, 8])
@pytest.mark.parametrize("e,steps_per_orbit,T", [(0.0, 8.5, 120), (0.2, 10, 120), (0.38, 50, 200),
                                                 (0.41, 50, 200), (0.7, 120, 240),
                                                 (0.05, -30, 200), (0.3, 3.7, 40)])
def test_rows(tpm, orc, k, e, steps_per_orbit, T):  # noqa: F811
    _check_rows(tpm, orc, k, e, steps_per_orbit, T)


@pytest.mark.parametrize("k", [5, 8])
@pytest.mark.parametrize("e", [0.03, 0.39, 0.7])
def test_many_systems(tpm, k, e):  # noqa: F811
    mu, rp, vp, period = _planets(k, e, 90 + k)
    r, v = np.array([[0.0, 9e3, 0.0], [0.7, 0.0, 0.1]]), np.array([[0.02, 0.0, 0.0], [0.0, 7.0, 0.0]])
    w = W.Workload("many", W.MU_SUN, mu, rp, vp, np.zeros(k), 1e5, r, v, period / 40.0, 300)
    s = tpm.Simulation(r_escape=w.rmax)
    s.set_central(w.mu0)
    s.set_planets(mu, rp, vp, w.rcrit)
    s.set_particles(r, v)
    s.integrate(300, w.dt)
    got, _ = tpm.batch_integrate([w, w], nsteps=300)
    for g in got:
        assert np.array_equal(g["r"], s.particles()["r"])


def test_eight_planets_in_registers(tpm):  # noqa: F811
    """A step of the map takes 1.26 us; 1.83 where its state spills to memory in the
    loop.  The bound lies between."""
    mu, rp, vp, period = _planets(8, 0.02, 98)
    s = tpm.Simulation()
    s.set_central(W.MU_SUN)
    s.set_planets(mu, rp, vp, np.zeros(8))
    s.set_particles(np.array([[9e3, 0.0, 0.0]]), np.array([[0.0, 0.02, 0.0]]))
    best = np.inf
    for _ in range(4):
        s.integrate(20_000, period / 40.0)
        best = min(best, s.stats()["ephemeris_ms"] * 1e3 / 20_000)
    assert best < 1.55, best
