"""Rows read without an acquire, and tiles handed between wavefronts on different
dies through memory: bit-identical to a run on a supplied table with one item per
tile, at the ends of the row groups (16 rows), in ring slots used again and again,
for every row length, and with items of a few steps on every compute unit."""
import numpy as np
import pytest

from paper_2011_03484_amd import workloads as W
from test_gpu_row_stream import KEYS, _sim, tpm  # noqa: F401

pytestmark = pytest.mark.gpu


def _equal(tpm, w, pieces, ref_opts, **opts):
    a, b = _sim(tpm, w, **opts), _sim(tpm, w, **ref_opts)
    b.set_planet_table(b.planet_table(sum(pieces), w.dt))
    for T in pieces:
        a.integrate(T, w.dt)
        b.integrate(T, w.dt)
    a, b = a.particles(), b.particles()
    for k in KEYS:
        assert np.array_equal(a[k], b[k]), (k, pieces, opts)


@pytest.mark.parametrize("pieces", [[1], [14, 1], [15, 16], [16, 15], [17], [46, 1, 1], [47, 33],
                                    [48, 16], [79]])
@pytest.mark.parametrize("chunk", [0, 15, 16, 17, 33])
def test_row_groups(tpm, pieces, chunk):  # noqa: F811
    _equal(tpm, W.giants_100k(n=3000, seed=311), pieces, {"sub_chunks": 1}, chunk_steps=chunk)


@pytest.mark.parametrize("k", [0, 1, 2, 3, 5, 8])
def test_row_lengths(tpm, k):  # noqa: F811
    w = [w for w in W.make_batched(nsys=40, nmin=400, nmax=400, seed=12) if w.np_ == max(k, 1)][0]
    if k == 0:
        w.mu, w.rp, w.vp, w.rcrit = w.mu[:0], w.rp[:0], w.vp[:0], w.rcrit[:0]
    _equal(tpm, w, [75, 300], {"sub_chunks": 1, "universal_drift": True}, universal_drift=True,
           chunk_steps=40)


@pytest.mark.parametrize("n,steps,opts", [
    (30_000, 400, {"chunk_steps": 128, "sub_chunks": 64}),
    (100_000, 300, {"chunk_steps": 300, "sub_chunks": 100}),
    (140_001, 130, {"chunk_steps": 65, "sub_chunks": 65, "waves_per_simd": 2}),
    (66_000, 200, {"chunk_steps": 100, "sub_chunks": 25, "block_threads": 256}),
])
def test_short_items(tpm, n, steps, opts):  # noqa: F811
    """Removals on the way: a tile's removed particles stay removed for whoever
    takes its next item."""
    w = W.giants_100k(n=n, seed=312)
    w.rcrit = w.rcrit * 4
    _equal(tpm, w, [steps, 60], {"sub_chunks": 1}, **opts)
