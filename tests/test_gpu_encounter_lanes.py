"""The encounter integrator with one particle on four lanes, at the planet
counts where its lanes fill differently (one planet: three idle lanes; four:
full; five and eight: two planets per lane) and list lengths that leave a
wavefront's sixteen entries partly empty.  Every particle starts beside a
planet, so every one is handed off.

  * with one substep the run is the plain map's bit for bit: the sums over the
    planets are the same chain of FMAs;
  * with several it agrees with the oracle to the bar of tests/test_gpu_handoff.py.
"""
import numpy as np
import pytest

from paper_2011_03484_amd import workloads as W
from test_gpu_handoff import KEYS, _handoff_reference, _sim
from test_gpu_parity import _compare

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tpm():
    import paper_2011_03484_amd as P
    P.load()
    return P


def _beside_planets(np_, n, seed):
    """Planets: the first np_ giants, or the four and lighter bodies farther out
    on their outermost one's orbit scaled up; particles beside each in turn."""
    w = W.giants_100k(n=n, seed=seed)
    f = np.array([1.0, 1.0, 1.0, 1.0, 1.5, 1.9, 2.4, 3.0])[:np_]
    k = np.minimum(np.arange(np_), 3)
    w.mu = w.mu[k] * np.where(f > 1, 0.1, 1.0)
    w.rp, w.vp = w.rp[k] * f[:, None], w.vp[k] / np.sqrt(f)[:, None]
    w.rcrit = w.rcrit[k]
    rng = np.random.default_rng(seed)
    at = np.arange(n) % np_
    u = rng.normal(size=(n, 3))
    u /= np.linalg.norm(u, axis=1)[:, None]
    w.r = w.rp[at] + u * (w.rcrit[at] * rng.uniform(0.3, 0.95, n))[:, None]
    w.v = w.vp[at] * (1 + 0.03 * rng.normal(size=(n, 1)))
    return w


@pytest.mark.parametrize("np_,n", [(1, 17), (3, 64), (4, 1), (5, 47), (8, 97)])
def test_one_substep_equals_plain_map(tpm, np_, n):
    w = _beside_planets(np_, n, 90 + np_)
    rrem = np.full(np_, 0.02)
    s = _sim(tpm, w, w.rcrit, rrem, handoff_substeps=1, chunk_steps=64, universal_drift=True)
    ref = _sim(tpm, w, rrem, chunk_steps=64, universal_drift=True)
    for T in (150, 1, 49):                       # a second call resumes at a step boundary
        s.integrate(T, w.dt)
        ref.integrate(T, w.dt)
    got, want = s.particles(), ref.particles()
    assert s.stats()["handoffs"] <= n
    for k in KEYS:
        assert np.array_equal(got[k], want[k]), k


@pytest.mark.parametrize("np_,n,M", [(1, 33, 7), (4, 65, 16), (6, 48, 4), (8, 31, 3)])
def test_substeps_match_oracle(tpm, orc, np_, n, M):
    """Chunks of 16 steps: the budget of one launch stops entries inside a step."""
    w = _beside_planets(np_, n, 190 + np_)
    T = 60
    rrem = np.full(np_, 0.02)
    s = _sim(tpm, w, w.rcrit, rrem, handoff_substeps=M, chunk_steps=16, universal_drift=True)
    s.integrate(T, w.dt)
    res, near, spread, _ = _handoff_reference(orc, w, T, rrem, M, True)
    assert s.stats()["handoffs"] == n
    _compare(s.particles(), res, near, spread, f"encounter lanes np={np_} M={M}")
