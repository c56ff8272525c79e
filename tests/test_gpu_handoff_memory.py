"""The planet rows that a hand-off call keeps stay within the memory it may take
for them, also in chunks of a step or two, whose ring slots are padded to whole
groups of rows; the pieces a long call is run in change no result."""
import numpy as np
import pytest

from paper_2011_03484_amd import workloads as W

pytestmark = pytest.mark.gpu

MiB = 1 << 20
KEYS = ("r", "v", "deact_step", "reason", "planet")


@pytest.fixture(scope="module")
def tpm():
    import paper_2011_03484_amd as P
    P.load()
    return P


def _sim(tpm, w, **opts):
    s = tpm.Simulation(r_escape=w.rmax, handoff_substeps=4, **opts)
    s.set_central(w.mu0)
    s.set_planets(w.mu, w.rp, w.vp, w.rcrit)
    s.set_removal_radii(0.1 * w.rcrit)
    s.set_particles(w.r, w.v)
    return s


@pytest.mark.parametrize("chunk", [1, 2, 20])
def test_rows_within_their_memory(tpm, monkeypatch, chunk):
    import torch
    w = W.giants_100k(n=64, seed=71)
    T = 8000
    want = _sim(tpm, w)
    want.integrate(T, w.dt)
    want = want.particles()
    # the rows of the whole call would take 8,000 (chunk + 1)/chunk * 216 bytes or
    # more: 2 to 13 times the bound
    monkeypatch.setenv("TPM_HANDOFF_RING_BYTES", str(MiB))
    s = _sim(tpm, w, chunk_steps=chunk)
    s.integrate(1, w.dt)
    s.set_particles(w.r, w.v)
    s.set_planets(w.mu, w.rp, w.vp, w.rcrit)
    s.set_removal_radii(0.1 * w.rcrit)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    s.integrate(T, w.dt)
    taken = free - torch.cuda.mem_get_info()[0]
    # two allocations, each up to 2 MiB more than asked for, and the list lengths
    assert taken <= MiB + 5 * MiB, taken / MiB
    got = s.particles()
    for k in KEYS:
        assert np.array_equal(got[k], want[k]), k
