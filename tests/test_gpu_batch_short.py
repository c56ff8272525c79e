"""Many-system runs of a few hundred steps: the bits of the run in one chunk,
however the library cuts them, and cut only where the chunks can overlap."""
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


@pytest.mark.parametrize("T", [1, 127, 128, 129, 255, 384, 511, 512, 513, 700])
def test_same_bits_as_one_chunk(tpm, T):
    systems = W.make_batched(nsys=7, nmin=40, nmax=300, seed=61)
    got, _ = tpm.batch_integrate(systems, nsteps=T, strict=False)
    want, _ = tpm.batch_integrate(systems, nsteps=T, chunk_steps=1024, strict=False)
    for g, x in zip(got, want):
        for k in KEYS:
            assert np.array_equal(g[k], x[k]), (T, k)


@pytest.mark.parametrize("T,chunks", [(1, 1), (129, 1), (512, 1), (513, 4), (700, 4)])
def test_cut_only_where_chunks_overlap(tpm, T, chunks):
    """A run that fits the shortest chunk of the tuner has one ring slot: cut, its
    chunks would go one after the other (512 steps of 200 systems 2.2 ms for 1.8)."""
    systems = W.make_batched(nsys=7, nmin=40, nmax=300, seed=62)
    _, st = tpm.batch_integrate(systems, nsteps=T, strict=False)
    assert st["chunks"] == chunks


@pytest.mark.parametrize("T", [300, 800, 1900])
@pytest.mark.parametrize("resync", [1, 2])
def test_given_options_stay(tpm, T, resync):
    """An interval of compactions that is given is not rescaled in a cut run."""
    systems = W.make_batched(nsys=7, nmin=40, nmax=300, seed=63)
    _, st = tpm.batch_integrate(systems, nsteps=T, strict=False, resync_chunks=resync, sub_chunks=4)
    assert st["resync_chunks"] == resync and st["sub_chunks"] == 4
    cut = 512 < T < 4 * st["chunk_steps"]
    assert st["chunks"] == (4 if cut else -(-T // st["chunk_steps"]))
    assert st["compactions"] == (st["chunks"] - 1) // resync
