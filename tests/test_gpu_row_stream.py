"""Planet rows written by the particle launch that uses them, against the same
run on a supplied table (tpm_planet_table's rows, all there before the launch):
bit-identical particles and planets at the edges of the row blocks (8 to 32
steps), of the tiles, of the one-wavefront-per-SIMD launches and of the chunks
the map may run ahead into."""
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


def _sim(tpm, w, **opts):
    s = tpm.Simulation(r_escape=w.rmax, kepler_iters=w.kepler_iters, **opts)
    s.set_central(w.mu0)
    s.set_planets(w.mu, w.rp, w.vp, w.rcrit)
    s.set_particles(w.r, w.v)
    return s


def _both(tpm, w, pieces, **opts):
    """Results of the live map over the given calls, and through a table."""
    a, b = _sim(tpm, w, **opts), _sim(tpm, w, **opts)
    b.set_planet_table(b.planet_table(sum(pieces), w.dt))
    for T in pieces:
        a.integrate(T, w.dt)
        b.integrate(T, w.dt)
    return a, a.particles(), b.particles()


@pytest.mark.parametrize("n,pieces,opts", [
    (1, [1], {}), (64, [7], {}), (65, [8], {}), (63, [9], {}), (64, [31, 1], {}),
    (130, [32, 33], {}), (64, [129], {}), (191, [300, 17], {}),
    (70, [100], {"chunk_steps": 5}), (70, [257], {"chunk_steps": 32, "resync_chunks": 3}),
    (700, [90], {"chunk_steps": 64, "block_threads": 256}),
    (700, [90], {"sub_chunks": 64}), (700, [333], {"waves_per_simd": 2, "sub_chunks": 7}),
    (65_472, [70], {}), (65_536, [70], {}), (140_001, [40], {}),
    (64, [8192 + 40], {}), (64, [3000, 6000], {"chunk_steps": 1000}),
])
def test_live_map_equals_supplied_table(tpm, n, pieces, opts):
    w = W.giants_100k(n=n, seed=301)
    s, a, b = _both(tpm, w, pieces, **opts)
    for k in KEYS:
        assert np.array_equal(a[k], b[k]), (n, pieces, opts, k)
    t = _sim(tpm, w, **opts)
    row = t.planet_table(sum(pieces), w.dt)[-1]
    assert np.array_equal(s.planets()[0].ravel(), row[:12])


@pytest.mark.parametrize("k", [0, 1, 3, 8])
def test_planet_counts(tpm, k):
    systems = [w for w in W.make_batched(nsys=40, nmin=100, nmax=100, seed=12) if w.np_ == max(k, 1)]
    w = systems[0]
    if k == 0:
        w.mu, w.rp, w.vp, w.rcrit = w.mu[:0], w.rp[:0], w.vp[:0], w.rcrit[:0]
    s, a, b = _both(tpm, w, [77, 50], universal_drift=True)
    for key in KEYS:
        assert np.array_equal(a[key], b[key]), (k, key)


def test_planets_go_on_without_particles(tpm):
    """All particles inside a planet's radius at the start: the launches after
    the first have no tiles, and the planets still reach the end."""
    w = W.giants_100k(n=100, seed=302)
    w.rcrit = np.full(4, 1e3)
    s = _sim(tpm, w, chunk_steps=40)
    s.integrate(500, w.dt)
    assert np.all(s.particles()["deact_step"] == 0)
    row = _sim(tpm, w).planet_table(500, w.dt)[-1]
    assert np.array_equal(s.planets()[0].ravel(), row[:12])


def test_static_run_over_several_chunks(tpm):
    """The one-slot ring of the no-allocation run: its map may not run ahead."""
    import torch
    w = W.giants_100k(n=1000, seed=303)
    T = 217
    r, v = (torch.tensor(x, device="cuda") for x in (w.r, w.v))
    ro, vo = torch.empty_like(r), torch.empty_like(v)
    st = torch.empty(w.n, dtype=torch.int64, device="cuda")
    rs, pl = (torch.empty(w.n, dtype=torch.int32, device="cuda") for _ in range(2))
    for chunk in (0, 50, 8):
        tpm.integrate_static(w.mu0, w.mu, w.rp, w.vp, w.rcrit, r.data_ptr(), v.data_ptr(), T, w.dt,
                             ro.data_ptr(), vo.data_ptr(), st.data_ptr(), rs.data_ptr(),
                             pl.data_ptr(), stream=torch.cuda.current_stream().cuda_stream,
                             r_escape=w.rmax, chunk_steps=chunk, n=w.n)
        torch.cuda.synchronize()
        s = _sim(tpm, w)
        s.integrate(T, w.dt)
        g = s.particles()
        assert np.array_equal(ro.cpu().numpy(), g["r"]) and np.array_equal(vo.cpu().numpy(), g["v"])
        assert np.array_equal(st.cpu().numpy(), g["deact_step"])
