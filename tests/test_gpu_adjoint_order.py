"""Derivative calls of one simulation that follow each other without a host
synchronisation, on one stream or two, with the planets moved in between or
another time step: each gives the bits of a synchronised run."""
import numpy as np
import pytest

from paper_2011_03484_amd import workloads as W

pytestmark = pytest.mark.gpu

N, T, CKPT = 3000, 1500, 125


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2011_03484_amd as P
    from paper_2011_03484_amd import autograd as AG
    P.load()
    return torch, P, AG


def _setup(env):
    torch, P, _ = env
    w = W.adjoint_16k(n=N, seed=41)
    s = P.Simulation(r_escape=w.rmax)
    s.set_central(w.mu0)
    s.set_planets(w.mu, w.rp, w.vp, w.rcrit)
    s.set_particles(w.r[:1], w.v[:1])
    rng = np.random.default_rng(6)
    t = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    a, b = t(rng.normal(size=(N, 3))), t(rng.normal(size=(N, 3)))
    # what a first pass allocates, so that no later one has a reason to wait
    r, v = t(w.r).requires_grad_(True), t(w.v).requires_grad_(True)
    _gradient(env, s, r, v, a, b, w.dt)
    torch.cuda.synchronize()
    return w, s, r, v, a, b


def _gradient(env, s, r, v, a, b, dt, sweep="adjoint"):
    torch, _, AG = env
    rT, vT, _, _ = AG.integrate(s, r, v, T, dt, CKPT)
    if sweep == "adjoint":
        return torch.autograd.grad([rT, vT], [r, v], [a, b])
    return AG.tangent(s, a, b)


@pytest.mark.parametrize("second", ["same stream", "other stream"])
@pytest.mark.parametrize("change", ["planets move", "other step"])
@pytest.mark.parametrize("sweep", ["adjoint", "tangent"])
def test_next_forward_waits(env, sweep, change, second):
    torch, P, _ = env
    got = {}
    for wait in (True, False):
        w, s, r, v, a, b = _setup(env)
        one, two = torch.cuda.Stream(), torch.cuda.Stream()
        with torch.cuda.stream(one):
            first = _gradient(env, s, r, v, a, b, w.dt, sweep)
        if wait:
            torch.cuda.synchronize()
        if change == "planets move":
            s.integrate(1, w.dt)
        with torch.cuda.stream(one if second == "same stream" else two):
            other = _gradient(env, s, r, v, a, b, w.dt if change == "planets move" else 0.5 * w.dt,
                              sweep)
        torch.cuda.synchronize()
        got[wait] = [x.detach().cpu().numpy() for x in (*first, *other)]
    for x, y in zip(got[True], got[False]):
        assert np.array_equal(x, y)
    assert not np.array_equal(got[True][0], got[True][2])
