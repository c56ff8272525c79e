"""Diagnostics where the planet table fits the device but the memory for stored
samples does not (chunks of some hundred million steps): the run ends a launch
at each sample and gives the bits of the run that stores them."""
import numpy as np
import pytest

from paper_2011_03484_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tpm():
    import paper_2011_03484_amd as P
    P.load()
    return P


def test_samples_without_room(tpm):
    import torch
    torch.cuda.empty_cache()
    w = W.giants_100k(n=300, seed=81)
    got = []
    # eight slots of rows of 15 doubles: three fifths of what is free; with rows of
    # 12 velocities beside them, more than there is
    free = torch.cuda.mem_get_info()[0]
    for chunk in (0, int(0.6 * free / (8 * 15 * 8))):
        with tpm.Simulation(r_escape=w.rmax, chunk_steps=chunk) as s:
            s.set_central(w.mu0)
            s.set_planets(w.mu, w.rp, w.vp, w.rcrit)
            s.set_particles(w.r, w.v)
            s.set_diagnostics(10, ref_planet=3, resonances=[(3, 1)])
            s.integrate(125, w.dt)
            s.integrate(30, w.dt)
            got.append({**s.particles(), **s.diagnostics()})
    for k in got[0]:
        assert np.array_equal(got[0][k], got[1][k]), k
