"""Compactions whose launch has blocks to spare: most entries are gone, but the
grid is still that of all of them, as in every no-allocation and many-system
run.  Their results equal those of a run that compacts only at its end, or of
the systems one by one, bit for bit."""
import numpy as np
import pytest

from paper_2011_03484_amd import workloads as W

pytestmark = pytest.mark.gpu

KEYS = ("r", "v", "deact_step", "reason", "planet")
STEPS = 24


@pytest.fixture(scope="module")
def tpm():
    import paper_2011_03484_amd as P
    P.load()
    return P


def _outwards(w, stay, steps, seed):
    """Velocities that take all but the particles of `stay` beyond rmax, at
    steps from 1 on."""
    rng = np.random.default_rng(seed)
    u = w.r / np.linalg.norm(w.r, axis=1)[:, None]
    speed = w.rmax / abs(w.dt) * rng.choice([1.2, 0.6, 0.3], w.n)
    return np.where(stay[:, None], w.v, u * speed[:, None])


@pytest.mark.parametrize("keep", [0, 1, 1024, 1025, 5000])
@pytest.mark.parametrize("n", [1025, 5000, 66_001])
def test_static(tpm, n, keep):
    import torch
    w = W.giants_100k(n=n, seed=23)
    stay = np.zeros(n, bool)
    stay[np.random.default_rng(n).permutation(n)[:keep]] = True
    w.v = _outwards(w, stay, STEPS, 3)
    t = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    r, v = t(w.r), t(w.v)
    got = []
    for resync in (1, 1000):
        out = {"r": torch.empty_like(r), "v": torch.empty_like(v),
               "deact_step": torch.empty(n, dtype=torch.int64, device="cuda"),
               "reason": torch.empty(n, dtype=torch.int32, device="cuda"),
               "planet": torch.empty(n, dtype=torch.int32, device="cuda")}
        info = torch.empty(2, dtype=torch.int64, device="cuda")
        tpm.integrate_static(w.mu0, w.mu, w.rp, w.vp, w.rcrit, r.data_ptr(), v.data_ptr(), STEPS, w.dt,
                             *(out[k].data_ptr() for k in KEYS), d_info=info.data_ptr(),
                             stream=torch.cuda.current_stream().cuda_stream, r_escape=w.rmax, n=n,
                             chunk_steps=1, resync_chunks=resync)
        torch.cuda.synchronize()
        assert int(info[1]) == 0
        got.append({k: x.cpu().numpy() for k, x in out.items()})
    for k in KEYS:
        assert np.array_equal(got[0][k], got[1][k]), k
    assert np.sum(got[0]["reason"] == tpm.ACTIVE) <= keep


def test_many_systems(tpm):
    systems = W.make_batched(nsys=6, nmin=700, nmax=3000, seed=29)
    for k, w in enumerate(systems):
        stay = np.arange(w.n) % 50 == 0
        w.rmax = systems[0].rmax
        w.v = _outwards(w, stay, STEPS, k)
    res, st = tpm.batch_integrate(systems, nsteps=STEPS, chunk_steps=2, resync_chunks=1, strict=False)
    assert st["compactions"] > 5
    for w, g in zip(systems, res):
        ref = tpm.batch_integrate([w], nsteps=STEPS, chunk_steps=STEPS, strict=False)[0][0]
        for k in KEYS:
            assert np.array_equal(g[k], ref[k]), k
