"""What a simulation costs before it holds anything: a few kilobytes of host
memory, not a staging block of its own; and results that go through the shared
staging come back right from many simulations in turn."""
import numpy as np
import pytest

from paper_2011_03484_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tpm():
    import paper_2011_03484_amd as P
    P.load()
    return P


def _address_space():
    for line in open("/proc/self/status"):
        if line.startswith("VmSize"):
            return int(line.split()[1]) * 1024


def test_many_simulations_are_small(tpm):
    w = W.giants_100k(n=500, seed=91)
    tpm.run_workload(w, nsteps=3)            # streams, staging and code objects are there
    before = _address_space()
    sims = [tpm.Simulation(r_escape=w.rmax) for _ in range(64)]
    grown = _address_space() - before
    # 256 KiB are seen; with a block of 1 MiB each it is 64 MiB
    assert grown < (16 << 20), grown
    parts = [w.subset(n=1 + 7 * k) for k in range(64)]
    for s, p in zip(sims, parts):
        s.set_central(p.mu0)
        s.set_planets(p.mu, p.rp, p.vp, p.rcrit)
        s.set_particles(p.r, p.v)
    for s, p in zip(sims, parts):
        got = s.particles()
        assert np.array_equal(got["r"], p.r) and np.array_equal(got["v"], p.v)
        assert np.all(got["deact_step"] == -1) and np.all(got["planet"] == -1)
