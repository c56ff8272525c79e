"""The short drift at the edges of its ranges (arc 1/4, |ec| + |es| = 3/4, one
or two Newton steps, whole periods), against the oracle's converged drift
within eight times the oracle's response to a one-ulp change of the position
plus 2e-15 plus the rounding of the mean-anomaly step (8 eps |n dt|/(1 - e)),
and the refusals of the fixed-count rule where it does not serve."""
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


def _states(e, n, seed):
    rng = np.random.default_rng(seed)
    a = np.full(n, 7.0)
    ang = [rng.uniform(0, 2 * math.pi, n) for _ in range(4)]
    return W.elements_to_cartesian(W.MU_SUN, a, np.full(n, e), *ang)


@pytest.mark.parametrize("e", [0.0, 0.05, 0.3, 0.52, 0.74, 0.75, 0.76])
@pytest.mark.parametrize("arc", [1e-6, 0.01, 0.05, 0.1, 0.2499, 0.2501, 0.5, -0.1, -0.25, 6.4, -13.0])
def test_against_converged_drift(tpm, orc, e, arc):
    n = 67                       # a full wavefront and a ragged one
    mu = W.MU_SUN
    r, v = _states(e, n, 7)
    dt = arc / math.sqrt(mu / 7.0 ** 3)          # mean anomaly step
    gr, gv, ok = tpm.debug_drift(mu, r, v, dt)
    worst = 0.0
    for i in range(n):
        okc, rr, vv, _ = orc.drift(mu, r[i], v[i], dt, kfix=5)
        assert ok[i] == okc
        if not okc:
            continue
        _, r2, v2, _ = orc.drift(mu, r[i] * (1 + 2.0 ** -52), v[i], dt, kfix=5)
        rel = lambda x, y: np.linalg.norm(x - y) / np.linalg.norm(y)
        bound = 8 * max(rel(r2, rr), rel(v2, vv)) + 2e-15 + 8 * 2.0 ** -52 * abs(arc) / (1 - e)
        worst = max(worst, rel(gr[i], rr) / bound, rel(gv[i], vv) / bound)
    assert worst <= 1.0, worst


def test_lanes_do_not_depend_on_their_wavefront(tpm):
    """Short-arc, second-step, out-of-range and unbound lanes mixed in one
    wavefront give the bits each kind gives alone."""
    mu = W.MU_SUN
    parts = [_states(e, 16, 30 + k) for k, e in enumerate((0.02, 0.5, 0.74, 0.9))]
    r = np.concatenate([p[0] for p in parts])
    v = np.concatenate([p[1] for p in parts])
    v[5] *= 3.0
    dt = 0.15 / math.sqrt(mu / 7.0 ** 3)
    mixed = tpm.debug_drift(mu, r, v, dt)
    order = np.arange(64).reshape(4, 16).T.ravel()
    for part in (order[:20], order[20:]):
        alone = tpm.debug_drift(mu, r[part], v[part], dt)
        for x, y in zip(mixed, alone):
            assert np.array_equal(x[part], y)
    assert not mixed[2][5]


@pytest.mark.parametrize("ftol", [1e-13, 1e-14, 1e-15, 1e-30])
def test_thresholds_below_its_own(tpm, orc, ftol):
    """A failure threshold below rounding refuses drifts, as the rule says."""
    mu = W.MU_SUN
    r, v = _states(0.3, 64, 9)
    dt = 0.1 / math.sqrt(mu / 7.0 ** 3)
    _, _, ok = tpm.debug_drift(mu, r, v, dt, kepler_ftol=ftol)
    assert ok.all() if ftol >= 1e-15 else not ok.all()
