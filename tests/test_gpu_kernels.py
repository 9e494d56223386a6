"""Edges of single kernels on the GPU: tile and batch remainders, the smallest
and largest sizes a launch rule takes, against the CPU oracle."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fl():
    from paper_2606_22180_amd import build, felog
    import os
    if not os.path.exists(build.LIB):
        build.build()
    felog.load()
    return felog


@pytest.fixture(scope="module")
def ctx(fl):
    return fl.Context(0)


def _mixed_degrees():
    """Node v of 0 .. 67 has v neighbours among the 68 to the right plus a few
    shared hubs, so that every degree from 0 to beyond 64 occurs."""
    e = [(v, 70 + u) for v in range(69) for u in range(v)]
    return synth.csr_from_edges(140, np.array(e, np.int64))


# k_s below, at and beyond the rows scored at a time (4) and the lanes of a wave
@pytest.mark.parametrize("k_s", [1, 3, 4, 5, 7, 8, 63, 64])
@pytest.mark.parametrize("dim", [64, 128, 256])
def test_psi_batches(fl, ctx, orc, dim, k_s):
    g = _mixed_degrees()
    G = fl.Graph.from_csr(ctx, g.indptr, g.indices)
    M = fl.Model.create(G, dim=dim, seed=1)
    tin = np.random.default_rng(k_s).normal(0, 1, (g.n, dim)).astype(np.float32)
    tin[71] = 0.0
    M.write(fl.TABLE_IN, tin)
    _, psi = M.feedback(mu=0.0, k_s=k_s, seed=5, round=2, want_psi=True)
    ref = orc.psi(tin, g, np.arange(g.n), k_s, 5, 2)
    assert np.array_equal(np.isnan(psi), np.isnan(ref))
    ok = ~np.isnan(ref)
    # FP64 sums of at most 256 terms and 64 cosines on both sides
    assert np.abs(psi[ok] - ref[ok]).max() <= 1e-12


# walks and steps around the 64 x 64 tile, reads below and above the size that
# is turned on the device
@pytest.mark.parametrize("L", [1, 2, 63, 64, 65, 129])
@pytest.mark.parametrize("n", [5, 63, 64, 65, 4100])
def test_read_walk_rows(fl, ctx, orc, n, L):
    e = np.array([(i, i + 1) for i in range(n - 2)] + [(0, n - 2)] * (n > 4), np.int64)
    g = synth.csr_from_edges(n, np.unique(e, axis=0))        # the last node is isolated
    G = fl.Graph.from_csr(ctx, g.indptr, g.indices)
    W = fl.Walks.generate(G, r=1, L=L, seed=3)
    ref = orc.walks_uniform(g, np.arange(n), 1, L, 3)
    assert np.array_equal(W.read(), ref)
    for first, count in ((0, 1), (1, n - 1), (n // 2, n - n // 2), (n, 0)):
        assert np.array_equal(W.read_range(first, count), ref[first:first + count])


def test_read_walks_within_a_budget(fl, orc):
    """A context whose budget leaves no room for the block still reads."""
    n, L = 3000, 40
    g = synth.csr_from_edges(n, np.array([(i, i + 1) for i in range(n - 1)], np.int64))
    for spare in (0, 8, 200 * L * 4, 1100 * L * 4):
        probe = fl.Context(0)
        G = fl.Graph.from_csr(probe, g.indptr, g.indices)
        W = fl.Walks.generate(G, r=1, L=L, seed=3)
        held = probe.bytes_in_use()
        c = fl.Context(0, hbm_budget=held + 64 + spare)      # the upload's check word fits too
        G2 = fl.Graph.from_csr(c, g.indptr, g.indices)
        W2 = fl.Walks.generate(G2, r=1, L=L, seed=3)
        assert np.array_equal(W2.read(), orc.walks_uniform(g, np.arange(n), 1, L, 3))
        assert c.bytes_in_use() == held
