"""A simulation whose integrate call failed on the device (the work queue's error
flag) gives the bits of a fresh one once planets and particles are set again:
nothing of the failed call's bookkeeping (planet rows published, step sums,
counts, the encounter list) is taken for the new one's."""
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


def _set(s, w, ho):
    s.set_central(w.mu0)
    s.set_planets(w.mu, w.rp, w.vp, w.rcrit)
    if ho:
        s.set_removal_radii(0.1 * w.rcrit)
    s.set_particles(w.r, w.v)


def _run(s, w, T):
    s.integrate(T, w.dt)
    out = s.particles()
    out["planets"] = np.concatenate(s.planets(), axis=1)
    st = s.stats()
    out["stats"] = np.array([st[k] for k in ("active_particle_steps", "n_active", "handoffs", "step")])
    return out


@pytest.mark.parametrize("ho", [0, 4])
@pytest.mark.parametrize("T", [40, 300])
def test_new_start_after_failure(tpm, T, ho):
    opts = dict(r_escape=900.0, handoff_substeps=ho, chunk_steps=64)
    first, second = W.giants_100k(n=2000, seed=51), W.giants_100k(n=1500, seed=52)
    s = tpm.Simulation(**opts)
    _set(s, first, ho)
    s.integrate(70, first.dt)
    assert tpm.load().tpm_debug_queue_error(s._h) == tpm.TPM_OK
    with pytest.raises(tpm.TpmError) as e:
        s.integrate(300, first.dt)
    assert e.value.code == tpm.TPM_EDEVICE
    _set(s, second, ho)
    got = _run(s, second, T)
    fresh = tpm.Simulation(**opts)
    _set(fresh, second, ho)
    want = _run(fresh, second, T)
    for k in want:
        assert np.array_equal(got[k], want[k]), k
    assert 0 < got["stats"][0]
