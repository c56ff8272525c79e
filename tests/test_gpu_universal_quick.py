"""The universal drift's short form at the edges of its range (|alpha| chi^2 = 1,
parabolic energy, pericentre passages its steps do not settle), against the
oracle's universal drift within eight times the oracle's response to a one-ulp
change of the state plus 4e-15, and independence of the wavefront's make-up."""
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


def _states(energy, n, seed):
    """States at r ~ 5 with v^2 = energy * mu / r and any direction."""
    rng = np.random.default_rng(seed)
    d, t = rng.normal(size=(n, 3)), rng.normal(size=(n, 3))
    r = rng.uniform(2, 8, n)[:, None] * d / np.linalg.norm(d, axis=1)[:, None]
    sp = np.sqrt(energy * W.MU_SUN / np.linalg.norm(r, axis=1))
    return r, sp[:, None] * t / np.linalg.norm(t, axis=1)[:, None]


@pytest.mark.parametrize("energy", [0.3, 1.0, 1.9, 1.999999, 2.0, 2.000001, 2.4, 6.0])
@pytest.mark.parametrize("dt", [1e-6, 0.05, 0.33, -0.33, 1.3, 1.9, -4.0])
def test_against_oracle(tpm, orc, energy, dt):
    n = 67
    r, v = _states(energy, n, 5)
    gr, gv, ok = tpm.debug_drift_universal(W.MU_SUN, r, v, dt, mode=2)
    assert ok.all()
    worst = 0.0
    for i in range(n):
        okc, rr, vv = orc.drift_universal(W.MU_SUN, r[i], v[i], dt)
        assert okc
        rel = lambda x, y: np.linalg.norm(x - y) / np.linalg.norm(y)
        bound = 4e-15
        for fr, fv in ((1 + 2.0 ** -52, 1.0), (1.0, 1 + 2.0 ** -52)):
            _, r2, v2 = orc.drift_universal(W.MU_SUN, r[i] * fr, v[i] * fv, dt)
            bound = max(bound, 4e-15 + 8 * max(rel(r2, rr), rel(v2, vv)))
        worst = max(worst, rel(gr[i], rr) / bound, rel(gv[i], vv) / bound)
    assert worst <= 1.0, worst


def test_lanes_do_not_depend_on_their_wavefront(tpm):
    parts = [_states(e, 16, 60 + k) for k, e in enumerate((0.9, 1.98, 2.0, 3.0))]
    r = np.concatenate([p[0] for p in parts])
    v = np.concatenate([p[1] for p in parts])
    order = np.arange(64).reshape(4, 16).T.ravel()
    for mode in (1, 2):
        mixed = tpm.debug_drift_universal(W.MU_SUN, r, v, 1.1, mode=mode)
        for part in (order[:20], order[20:], order[::7]):
            alone = tpm.debug_drift_universal(W.MU_SUN, r[part], v[part], 1.1, mode=mode)
            for x, y in zip(mixed, alone):
                assert np.array_equal(x[part], y)
