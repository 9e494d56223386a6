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


def _two_paths(fl, g, *, dim, K, P, first, count, r=2, L=12, window=3):
    """Tables and counts of the same minibatches on both update paths."""
    out = []
    for path in (0, 1):
        c = fl.Context(0)
        c.set_sgns_path(path)
        G = fl.Graph.from_csr(c, g.indptr, g.indices)
        W = fl.Walks.generate(G, r=r, L=L, seed=4)
        M = fl.Model.create(G, dim=dim, seed=6)
        rng = np.random.default_rng(7)
        for which in (fl.TABLE_IN, fl.TABLE_OUT):
            M.write(which, rng.normal(0, 0.2, (g.n, dim)).astype(np.float32))
        st = M.train_steps(W, fl.train_params(window=window, negatives=K, minibatch_pairs=P,
                                              seed=9), first, count)
        assert st.path == (1 - path if P * (K + 2) <= 8192 else 0)
        out.append((M.read(fl.TABLE_IN), M.read(fl.TABLE_OUT), st.loss, st.pairs, st.rows_in,
                    st.rows_out, st.rows_out_single))
    return out


# touches around a round of the plan's sort (1,024) and at the largest of its
# two sizes (8,192 and 16,384, the second of planned launches only); node
# counts around a power of two, the largest row keys of a digit and below
@pytest.mark.parametrize("P,K,n", [(1, 1, 3), (341, 1, 255), (342, 1, 256), (146, 5, 257),
                                   (147, 5, 1000), (1024, 6, 1023), (1170, 5, 1024),
                                   (2730, 1, 65535), (372, 20, 65536), (1024, 6, 65537),
                                   (1171, 5, 1200), (2340, 5, 3000), (5461, 1, 4097),
                                   (744, 20, 800)])
def test_plan_sizes(fl, orc, P, K, n):
    rng = np.random.default_rng(n)
    e = np.stack([rng.integers(0, n, 4 * n), rng.integers(0, n, 4 * n)], 1)
    e = np.concatenate([np.sort(e[e[:, 0] != e[:, 1]], 1), [[0, n - 1]]])
    g = synth.csr_from_edges(n, np.unique(e, axis=0))
    first = 3 if n > 100 else 0
    a, b = _two_paths(fl, g, dim=128, K=K, P=P, first=first, count=3)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    assert a[3:] == b[3:] and abs(a[2] - b[2]) <= 1e-12 * abs(b[2])
    # the oracle's minibatches one after another: each stored entry within the
    # per-row bar of the deltas plus one FP32 spacing per minibatch
    rng = np.random.default_rng(7)
    tab = [rng.normal(0, 0.2, (n, 128)).astype(np.float32) for _ in range(2)]
    walks = orc.walks_uniform(g, np.arange(n), 2, 12, 4)
    cdf = orc.neg_cdf(g.degrees().astype(np.uint64))
    prm = fl.train_params(window=3, negatives=K, minibatch_pairs=P, seed=9)
    slices = sum(1 for j in range(12) for o in range(-3, 4) if o and 0 <= j + o < 12)
    B = -(-2 * int((g.degrees() > 0).sum()) * slices // P)
    moved = [np.zeros(n), np.zeros(n)]
    for i in range(first, min(first + 3, B)):
        mb = orc.minibatch_pairs(walks, 3, P, i)
        d = orc.sgns_step(tab[0], tab[1], mb.ctx, mb.ctr, orc.draw_negatives(mb, 0, K, 9, cdf),
                          orc.lr_at(i, B, prm.lr_start, prm.lr_end))
        moved[0][d.rows_in] += np.linalg.norm(d.d_in, axis=1)
        moved[1][d.rows_out] += np.linalg.norm(d.d_out, axis=1)
    for got, ref, mv in zip(a[:2], tab, moved):
        assert (np.abs(got.astype(np.float64) - ref) <=
                1e-5 * mv[:, None] + 3 * np.spacing(np.abs(ref)) + 1e-12).all()


def test_plan_one_hub(fl):
    """Every context or centre is one node: segments of hundreds of touches,
    and negatives that are skipped as often as drawn."""
    n = 64
    g = synth.csr_from_edges(n, np.array([(0, i) for i in range(1, n)], np.int64))
    a, b = _two_paths(fl, g, dim=64, K=5, P=1024, first=0, count=2, r=20)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]) and a[3:] == b[3:]


# odd pair counts at d = 64, where a wave holds two pairs side by side and the
# last of an odd number stands alone; many negatives equal their centre
@pytest.mark.parametrize("P", [1, 3, 255, 257])
@pytest.mark.parametrize("K", [1, 9, 15, 20])
def test_forward_odd_pairs_d64(fl, orc, K, P):
    n = 40
    e = np.array([(i, j) for i in range(n) for j in range(i + 1, min(n, i + 6))], np.int64)
    g = synth.csr_from_edges(n, e)
    c = fl.Context(0)
    c.set_sgns_path(1)
    G = fl.Graph.from_csr(c, g.indptr, g.indices)
    W = fl.Walks.generate(G, r=8, L=12, seed=4)
    M = fl.Model.create(G, dim=64, seed=6)
    rng = np.random.default_rng(K)
    tab = [rng.normal(0, 0.2, (n, 64)).astype(np.float32) for _ in range(2)]
    for which in (0, 1):
        M.write(which, tab[which])
    walks = orc.walks_uniform(g, np.arange(n), 8, 12, 4)
    cdf = orc.neg_cdf(g.degrees().astype(np.uint64))
    prm = fl.train_params(window=3, negatives=K, minibatch_pairs=P, seed=9, lr_start=0.02,
                          lr_end=0.02)
    for b in (2, 3, 4):
        mb = orc.minibatch_pairs(walks, 3, P, b)
        ref = orc.sgns_step(tab[0], tab[1], mb.ctx, mb.ctr, orc.draw_negatives(mb, 0, K, 9, cdf),
                            float(np.float32(0.02)), apply=False)
        ri, di, ro, do, _ = M.train_delta(W, prm, b)
        for rows, d, rrows, rd in ((ri, di, ref.rows_in, ref.d_in), (ro, do, ref.rows_out, ref.d_out)):
            assert np.array_equal(np.sort(rows), np.sort(rrows))
            d, rd = d[np.argsort(rows)], rd[np.argsort(rrows)]
            err = np.linalg.norm(d.astype(np.float64) - rd, axis=1)
            assert (err <= 1e-5 * np.linalg.norm(rd, axis=1) + 1e-12).all()


@pytest.mark.parametrize("P,K", [(200, 5), (2000, 5)])
def test_launches_within_a_budget(fl, P, K):
    """Per-minibatch launches under shrinking budgets: fewer plans per launch,
    then none (the ids of each minibatch instead), then ENOMEM; every call that
    succeeds gives the same tables."""
    n = 300
    rng = np.random.default_rng(1)
    e = np.sort(np.stack([rng.integers(0, n, 2000), rng.integers(0, n, 2000)], 1), 1)
    g = synth.csr_from_edges(n, np.unique(e[e[:, 0] != e[:, 1]], axis=0))
    prm = fl.train_params(window=3, negatives=K, minibatch_pairs=P, seed=9)

    def train(budget):
        c = fl.Context(0, hbm_budget=budget)
        c.set_sgns_path(1)
        c.set_single_stream(True)
        G = fl.Graph.from_csr(c, g.indptr, g.indices)
        W = fl.Walks.generate(G, r=4, L=12, seed=4)
        M = fl.Model.create(G, dim=64, seed=6)
        held = c.bytes_in_use()
        M.train_steps(W, prm, 0, 30)
        return M.read(fl.TABLE_IN), M.read(fl.TABLE_OUT), held

    ref = train(0)
    done = 0
    for spare in (64 << 20, 4 << 20, 1500000, 900000, 500000, 250000, 100000, 20000):
        try:
            got = train(ref[2] + spare)
        except fl.FelogError as err:
            assert err.status == fl.FELOG_ENOMEM
            continue
        done += 1
        assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1])
    assert done >= 2


def _one_edge(n):
    return np.minimum(np.arange(n + 1, dtype=np.int64), 2), np.array([1, 0], np.int32)


# Host reads of rows * 256 bytes: below and at the staged size (4 MiB), chunk
# edges (2 MiB), the threaded size (16 MiB) and past one turn of the ring
@pytest.mark.parametrize("rows", [16383, 16384, 24575, 24577, 65535, 65536, 65537, 163841])
def test_large_reads(fl, ctx, rows):
    G = fl.Graph.from_csr(ctx, *_one_edge(rows))
    M = fl.Model.create(G, dim=64, seed=1)
    want = np.arange(rows * 64, dtype=np.uint32).view(np.float32).reshape(rows, 64)
    M.write(fl.TABLE_IN, want)
    for _ in range(2):   # a new ring, one that waited
        assert (M.read(fl.TABLE_IN).view(np.uint32) == want.view(np.uint32)).all()


def test_large_reads_from_threads(fl):
    """More readers than rings are kept, each with a context of its own."""
    from concurrent.futures import ThreadPoolExecutor

    def job(i):
        c = fl.Context(0)
        G = fl.Graph.from_csr(c, *_one_edge(90000 + i))
        M = fl.Model.create(G, dim=64, seed=1)
        want = np.full((90000 + i, 64), i + 1, np.float32)
        want[:, 0] = np.arange(90000 + i)
        M.write(fl.TABLE_IN, want)
        return all((M.read(fl.TABLE_IN) == want).all() for _ in range(3))

    with ThreadPoolExecutor(4) as ex:
        assert all(ex.map(job, range(4)))


# Counted in LDS: one range of nodes filled exactly, one node more (two
# ranges), fewer than eight parts, a remainder of 1 to 3 positions in a part;
# by atomics: too few positions, too many nodes, no room for the parts' counts
@pytest.mark.parametrize("n,r,L,spare", [
    (40960, 1, 103, None), (40961, 1, 103, None), (100001, 1, 13, None), (300, 700, 5, None),
    (1203, 875, 1, None), (65536, 1, 15, None), (1400000, 1, 2, None), (40961, 1, 103, 400000)])
def test_corpus_counts(fl, orc, n, r, L, spare):
    """The unigram counts and the codec's profile against a host count; a
    quarter of the nodes are isolated (padded walks), node 0 is a hub."""
    m = n - n // 4
    v = np.arange(1, m, dtype=np.int64)
    e = np.unique(np.sort(np.concatenate([np.stack([0 * v, v], 1), np.stack([v[:-1], v[1:]], 1)]),
                          axis=1), axis=0)
    g = synth.csr_from_edges(n, e)

    def run(budget):
        c = fl.Context(0, hbm_budget=budget)
        G = fl.Graph.from_csr(c, g.indptr, g.indices)
        M = fl.Model.create(G, dim=64, seed=1)
        W = fl.Walks.generate(G, r=r, L=L, seed=5)
        held = c.bytes_in_use()
        M.set_unigram(W)
        return M.read_cdf(), W, held

    cdf, W, held = run(0)
    if spare is not None:
        # room for the counts, the weights and the table, not for parts of them
        cdf, W, _ = run(held + 20 * n + spare)
    x = W.read().ravel()
    counts = np.bincount(x[x >= 0], minlength=n)
    assert np.array_equal(cdf, orc.neg_cdf(counts.astype(np.uint32)))
    if spare is None:
        _, sym, cnt, total = W.fabc_profile()
        assert total == x.size
        all_counts = np.concatenate([[np.count_nonzero(x < 0)], counts]).astype(np.uint64)
        order = np.lexsort((np.arange(-1, n), -all_counts.astype(np.int64)))[:len(sym)]
        assert np.array_equal(sym, order - 1) and np.array_equal(cnt, all_counts[order])


# Every lane at its own transition: one step and none, few lanes of a wave,
# walks that end at once beside long ones, and transitions that only end at the
# cap (leaving a leaf needs the return to prev, accepted once in 10^6 attempts)
@pytest.mark.parametrize("n,r,L,p,q,weighted", [
    (5, 1, 1, 0.5, 2.0, False), (63, 1, 2, 0.5, 2.0, True), (65, 3, 33, 8.0, 0.125, True),
    (200, 2, 50, 0.05, 20.0, False), (67, 1, 4, 1e6, 1.0, True)])
def test_node2vec_lanes(fl, ctx, orc, n, r, L, p, q, weighted):
    rng = np.random.default_rng(n)
    m = n - n // 5                       # the last fifth is isolated
    v = np.arange(1, m, dtype=np.int64)
    e = np.concatenate([np.stack([0 * v, v], 1), rng.integers(0, max(m // 2, 2), (2 * n, 2))])
    e = np.sort(e[e[:, 0] != e[:, 1]], axis=1)
    e = np.unique(e, axis=0)
    g = synth.csr_from_edges(n, e, *([synth.edge_weights(e.shape[0], 3)] if weighted else []))
    G = fl.Graph.from_csr(ctx, g.indptr, g.indices, *([g.weights] if weighted else []))
    W = fl.Walks.generate(G, r=r, L=L, seed=11, id_base=3, kind=fl.WALK_NODE2VEC, p=p, q=q)
    want, capped = orc.walks_node2vec(g, np.arange(n), r, L, p, q, 11, 3)
    assert np.array_equal(W.read(), want)
    assert W.capped() == capped and (capped > 0) == (p == 1e6)


# Id batches of the BF16 form: just past the narrow batch, at and past the wide
# one, and cut by the chunks' ends; a context with a budget keeps the narrow one
@pytest.mark.parametrize("n_mb,chunk", [(65, 0), (256, 0), (257, 0), (600, 90)])
def test_bf16_id_batches(fl, n_mb, chunk):
    n = 400
    rng = np.random.default_rng(2)
    e = np.sort(rng.integers(0, n, (2500, 2)), 1)
    g = synth.csr_from_edges(n, np.unique(e[e[:, 0] != e[:, 1]], axis=0))

    def train(budget):
        c = fl.Context(0, hbm_budget=budget)
        G = fl.Graph.from_csr(c, g.indptr, g.indices)
        W = fl.Walks.generate(G, r=4, L=20, seed=4)
        M = fl.Model.create(G, dim=64, seed=6, precision=fl.PREC_BF16)
        prm = fl.train_params(window=3, negatives=5, minibatch_pairs=64, seed=9,
                              shared_negatives=64, chunk_walks=chunk)
        st = M.train_steps(W, prm, 0, n_mb)
        assert st.minibatches == n_mb
        return M.read(fl.TABLE_IN), M.read(fl.TABLE_OUT), st.loss

    wide, narrow = train(0), train(1 << 30)
    assert np.array_equal(wide[0], narrow[0]) and np.array_equal(wide[1], narrow[1])
    assert wide[2] == narrow[2]


def test_empty_noise_table_is_refused(fl, ctx):
    """Counts of a corpus without walks are refused, and the model goes on with
    the table that it has."""
    n = 200
    rng = np.random.default_rng(5)
    e = np.sort(rng.integers(0, n, (900, 2)), 1)
    g = synth.csr_from_edges(n, np.unique(e[e[:, 0] != e[:, 1]], axis=0))
    G = fl.Graph.from_csr(ctx, g.indptr, g.indices)
    W = fl.Walks.generate(G, r=4, L=12, seed=4)
    none = fl.Walks.generate(G, r=1, L=12, seed=4, starts=fl.Active.from_host(G, np.zeros(0, np.int32)))
    M, R = (fl.Model.create(G, dim=64, seed=6) for _ in range(2))
    with pytest.raises(fl.FelogError) as err:
        M.set_unigram(none)
    assert err.value.status == fl.FELOG_EINVAL
    assert np.array_equal(M.read_cdf(), R.read_cdf())
    prm = fl.train_params(window=3, negatives=5, minibatch_pairs=256, seed=9)
    for m in (M, R):
        m.train_steps(W, prm, 0, 4)
    for which in (0, 1):
        assert np.array_equal(M.read(which), R.read(which))


# q = 1 (no searches): one, two and four attempts in flight, by weights, p and
# whether the entries pass 16 MB; walks that end at once, leaves whose only
# neighbour is the previous node, transitions that end at the cap
@pytest.mark.parametrize("n,m,p,weighted", [
    (65, 200, 0.25, False), (65, 200, 0.25, True), (500, 3000, 1.0, False),
    (500, 3000, 2.0, True), (64, 80, 1e6, False), (200000, 4300000, 0.5, False),
    (200000, 4300000, 1.0, True), (100000, 2200000, 0.25, True)])
def test_node2vec_without_searches(fl, ctx, orc, n, m, p, weighted):
    rng = np.random.default_rng(n)
    e = rng.integers(0, n - n // 8, (m, 2))                  # the last eighth is isolated
    e = np.unique(np.sort(e[e[:, 0] != e[:, 1]], axis=1), axis=0)
    g = synth.csr_from_edges(n, e, *([synth.edge_weights(e.shape[0], 3)] if weighted else []))
    G = fl.Graph.from_csr(ctx, g.indptr, g.indices, *([g.weights] if weighted else []))
    starts = np.arange(0, n, max(1, n // 700), dtype=np.int32)
    W = fl.Walks.generate(G, r=3, L=17, seed=11, id_base=5, kind=fl.WALK_NODE2VEC, p=p, q=1.0,
                          starts=fl.Active.from_host(G, starts))
    want, capped = orc.walks_node2vec(g, starts, 3, 17, p, 1.0, 11, 5)
    assert np.array_equal(W.read(), want)
    assert W.capped() == capped and (capped > 0) == (p == 1e6)


# q other than 1 beyond 24 MB of indices: rows of like length walked in step (above
# 48 MB, or without weights and p >= 1), a hub or p < 1 that keep lanes at their own
# transitions; leaves, where a transition ends at the cap
@pytest.mark.parametrize("n,m,p,q,weighted,hub", [
    (200000, 3300000, 1.0, 2.0, False, False), (200000, 3300000, 2.0, 1.5, False, True),
    (200000, 3300000, 0.5, 4.0, False, False), (200000, 3300000, 1.0, 0.5, False, False),
    (400000, 6600000, 0.5, 4.0, True, False), (400000, 6600000, 1e6, 2.0, False, False)])
def test_node2vec_beyond_the_caches(fl, ctx, orc, n, m, p, q, weighted, hub):
    rng = np.random.default_rng(m)
    k = n - n // 8                       # the last eighth: leaves, every other one isolated
    e = np.sort(rng.integers(0, k, (m, 2)), axis=1)
    e = e[e[:, 0] != e[:, 1]]
    if hub:
        e = np.concatenate([e, np.stack([np.zeros(400, np.int64), np.arange(1, 401)], 1)])
    leaf = np.arange(k, n, 2, dtype=np.int64)
    e = np.concatenate([e, np.stack([leaf - k, leaf], 1)])
    key = np.unique(e[:, 0] * n + e[:, 1])
    e = np.stack([key // n, key % n], 1)
    g = synth.csr_from_edges(n, e, *([synth.edge_weights(e.shape[0], 3)] if weighted else []))
    assert g.indices.shape[0] * 4 > (24 if n == 200000 else 48) << 20
    G = fl.Graph.from_csr(ctx, g.indptr, g.indices, *([g.weights] if weighted else []))
    starts = np.arange(0, n, n // 700, dtype=np.int32)
    W = fl.Walks.generate(G, r=2, L=21, seed=11, id_base=5, kind=fl.WALK_NODE2VEC, p=p, q=q,
                          starts=fl.Active.from_host(G, starts))
    want, capped = orc.walks_node2vec(g, starts, 2, 21, p, q, 11, 5)
    assert np.array_equal(W.read(), want)
    assert W.capped() == capped and (capped > 0) == (p == 1e6)


# the fewest parts that counts are split over: four for the noise table, two for
# the codec's profile, and one less of each
@pytest.mark.parametrize("n,r,L", [(70000, 1, 17), (70000, 1, 15), (140000, 1, 9), (140000, 1, 7),
                                   (262144, 1, 7)])
def test_corpus_counts_of_few_parts(fl, orc, n, r, L):
    test_corpus_counts(fl, orc, n, r, L, None)


# around the sizes above which walks of one, two and three steps are turned on
# the device (62k, 34k and 5k ints), and a single walk of four
@pytest.mark.parametrize("n,L", [(61439, 1), (65536, 1), (16383, 2), (18432, 2), (1365, 3),
                                 (1366, 3), (2731, 3), (5, 4)])
def test_read_short_walks(fl, ctx, orc, n, L):
    test_read_walk_rows(fl, ctx, orc, n, L)
