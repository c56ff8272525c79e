"""Tangent and adjoint at the edges of their segments: every checkpoint
interval gives the gradient of one segment, and the two sweeps are transposes
of each other for 0 to 8 planets, ragged counts, one to a few steps and
particles removed inside a segment, at its ends and at the start."""
import numpy as np
import pytest

from paper_2011_03484_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2011_03484_amd as P
    from paper_2011_03484_amd import autograd as AG
    P.load()
    return torch, P, AG


def _sweeps(env, w, T, ckpt):
    torch, P, AG = env
    s = P.Simulation(r_escape=w.rmax)
    s.set_central(w.mu0)
    s.set_planets(w.mu, w.rp, w.vp, w.rcrit)
    rng = np.random.default_rng(5)
    t = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    dr, dv, gr, gv = (t(rng.normal(size=(w.n, 3))) for _ in range(4))
    r0, v0 = t(w.r).requires_grad_(True), t(w.v).requires_grad_(True)
    rT, vT, step, _ = AG.integrate(s, r0, v0, T, w.dt, ckpt)
    jr, jv = AG.tangent(s, dr, dv)
    ar, av = torch.autograd.grad([rT, vT], [r0, v0], [gr, gv])
    num = [x.cpu().numpy() for x in (jr, jv, ar, av, dr, dv, gr, gv)]
    return num, step.cpu().numpy()


def _identity(num, T):
    """<J d, g> = <d, J^T g> per particle, relative to |J d||g| + |d||J^T g|, which
    bounds its rounding: 300 operations a step, each 2^-53."""
    jr, jv, ar, av, dr, dv, gr, gv = num
    J, A = np.concatenate([jr, jv], 1), np.concatenate([ar, av], 1)
    d, g = np.concatenate([dr, dv], 1), np.concatenate([gr, gv], 1)
    norm = lambda x: np.linalg.norm(x, axis=1)
    off = np.abs(np.sum(J * g, 1) - np.sum(d * A, 1)) / (norm(J) * norm(g) + norm(d) * norm(A))
    assert off.max() <= 300 * max(T, 1) * 2.0 ** -53, off.max()


@pytest.mark.parametrize("k", [0, 1, 3, 4, 5, 8])
@pytest.mark.parametrize("n,T,ckpt", [(1, 1, 1), (65, 2, 1), (63, 33, 32), (130, 40, 7)])
def test_transposes(env, k, n, T, ckpt):
    w = [x for x in W.make_batched(nsys=60, nmin=n, nmax=n, seed=21) if x.np_ == max(k, 1)][0]
    if k == 0:
        w.mu, w.rp, w.vp, w.rcrit = w.mu[:0], w.rp[:0], w.vp[:0], w.rcrit[:0]
    num, _ = _sweeps(env, w, T, ckpt)
    _identity(num, T)


def test_checkpoint_interval_does_not_matter(env):
    """With removals: particles near Jupiter's orbit, a tenth of them inside its
    radius at the start."""
    w = W.adjoint_16k(n=300, seed=31)
    T = 96
    base, step = _sweeps(env, w, T, T)
    assert np.sum(step == 0) > 0 and np.sum(step > 0) > 0 and np.sum(step < 0) > 0
    _identity(base, T)
    for ckpt in (1, 5, 32, 48, 95, 1000):
        num, st = _sweeps(env, w, T, ckpt)
        assert np.array_equal(st, step)
        _identity(num, T)
        for x, y in zip(num[:4], base[:4]):
            size = np.linalg.norm(y, axis=1, keepdims=True) + 1e-300
            assert np.max(np.abs(x - y) / size) <= 300 * T * 2.0 ** -53 * 100
