"""The three routes of the FP32 update against each other and the oracle: the
persistent update, planned launches, and launches with ids, scans and two
applies (the only one that shares no plan and no apply with the others).

Minibatches of up to 16,384 touches take the third route when a budget has no
room for a plan; the tests make room for everything else and fill the rest."""
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


def _random_graph(n, seed=1):
    rng = np.random.default_rng(seed)
    e = np.stack([rng.integers(0, n, 4 * n), rng.integers(0, n, 4 * n)], 1)
    e = np.concatenate([np.sort(e[e[:, 0] != e[:, 1]], 1), [[0, n - 1]]])
    return synth.csr_from_edges(n, np.unique(e, axis=0))


def _star(n):
    return synth.csr_from_edges(n, np.array([(0, i) for i in range(1, n)], np.int64))


def _tables(n, dim, seed=7):
    rng = np.random.default_rng(seed)
    return [rng.normal(0, 0.2, (n, dim)).astype(np.float32) for _ in range(2)]


def _build(fl, c, g, *, dim, r, L):
    G = fl.Graph.from_csr(c, g.indptr, g.indices)
    W = fl.Walks.generate(G, r=r, L=L, seed=4)
    M = fl.Model.create(G, dim=dim, seed=6)
    for which, t in enumerate(_tables(g.n, dim)):
        M.write(which, t)
    return G, W, M


def _train(fl, g, prm, first, count, *, route, dim, r=2, L=12):
    """Tables and row counts of minibatches [first, first + count)."""
    P, T = prm.minibatch_pairs, prm.minibatch_pairs * (prm.negatives + 2)
    if route == "ids":
        # the id buffers (a capture of minibatch 0 takes them) and the call's
        # own; the capture's rows are the largest need
        def prepare(budget):
            c = fl.Context(0, hbm_budget=budget)
            c.set_sgns_path(1)
            G, W, M = _build(fl, c, g, dim=dim, r=r, L=L)
            A = fl.Active.from_host(G, np.zeros(1, np.int32))
            M.train_delta(W, prm, 0)
            return c, G, W, M, A
        own = 8 * (P + 8) + 8 * prm.window * L + 64      # loss slots, slices
        objs = prepare(0)
        need = objs[0].bytes_in_use()
        c, G, W, M, A = prepare(need + 4 * T * dim + own)
        room = need + 4 * T * dim + own - c.bytes_in_use() - own
        F = fl.Walks.generate(G, r=room // 4, L=1, seed=1, starts=A)
        held = c.bytes_in_use()
        assert held <= need + 4 * T * dim <= held + 16
    else:
        c = fl.Context(0)
        c.set_sgns_path(0 if route == "persistent" else 1)
        G, W, M = _build(fl, c, g, dim=dim, r=r, L=L)
        held = c.bytes_in_use()
    c.set_timing(1)
    st = M.train_steps(W, prm, first, count)
    assert st.path == (1 if route == "persistent" else 0)
    if route == "ids":          # two applies, and nothing allocated for plans
        assert 0 < st.ms_apply_first < st.ms_apply and c.bytes_in_use() == held
    else:                       # plans; their launches apply in one
        assert c.bytes_in_use() > held and st.ms_apply_first == st.ms_apply
    return (M.read(fl.TABLE_IN), M.read(fl.TABLE_OUT), st.loss,
            (st.pairs, st.rows_in, st.rows_out, st.rows_out_single))


# all dimensions; few nodes (long segments, skipped negatives) and many; one
# pair; the largest K; the edges of the persistent update (8,192 touches) and
# of planned launches (16,384); two launch groups of 64 plans; more than 2,048
# pairs, whose ids run on a second stream with counters zeroed whole
@pytest.mark.parametrize("n,dim,K,P,first,count", [
    (300, 64, 5, 256, 0, 140), (5000, 128, 5, 1024, 2, 20), (64, 256, 3, 333, 1, 30),
    (40, 128, 1, 1, 3, 5), (700, 128, 20, 372, 0, 12), (700, 64, 14, 511, 0, 12),
    (700, 64, 20, 744, 0, 8), (3000, 64, 5, 2340, 0, 12), (1500, 256, 1, 5461, 0, 6),
    (20000, 128, 5, 1170, 0, 70)])
def test_routes_agree(fl, n, dim, K, P, first, count):
    g = _random_graph(n)
    prm = fl.train_params(window=3, negatives=K, minibatch_pairs=P, seed=9)
    ids = _train(fl, g, prm, first, count, route="ids", dim=dim, r=20 if n < 1000 else 2)
    small = P * (K + 2) <= 8192 and not (dim == 64 and K > 14)
    for route in ["planned"] + ["persistent"] * small:
        got = _train(fl, g, prm, first, count, route=route, dim=dim, r=20 if n < 1000 else 2)
        assert np.array_equal(got[0].view(np.uint32), ids[0].view(np.uint32)), route
        assert np.array_equal(got[1].view(np.uint32), ids[1].view(np.uint32)), route
        assert got[3] == ids[3] and abs(got[2] - ids[2]) <= 1e-12 * abs(ids[2]), route


@pytest.mark.parametrize("dim", [64, 128, 256])
def test_one_hub(fl, orc, dim):
    """A star: every context or centre is node 0, so segments have hundreds of
    touches and negatives are skipped as often as drawn.  The three routes agree
    and one minibatch after another is the oracle's, within the per-row bar of
    its deltas plus the table's rounding."""
    n, P, K, r, L = 64, 1024, 5, 20, 12
    g = _star(n)
    prm = fl.train_params(window=3, negatives=K, minibatch_pairs=P, seed=9)
    res = [_train(fl, g, prm, 0, 6, route=x, dim=dim, r=r) for x in ("ids", "planned", "persistent")]
    for x in res[1:]:
        assert np.array_equal(x[0], res[0][0]) and np.array_equal(x[1], res[0][1])
        assert x[3] == res[0][3]
    walks = orc.walks_uniform(g, np.arange(n), r, L, 4)
    cdf = orc.neg_cdf(g.degrees().astype(np.uint64))
    B, _ = orc.count_minibatches(walks, 3, P)
    for path in (0, 1):
        c = fl.Context(0)
        c.set_sgns_path(path)
        _, W, M = _build(fl, c, g, dim=dim, r=r, L=L)
        for b in (0, 1, B - 1):
            tab = _tables(n, dim, seed=b)
            for which in (0, 1):
                M.write(which, tab[which])
            M.train_steps(W, prm, b, 1)
            mb = orc.minibatch_pairs(walks, 3, P, b)
            before = [t.copy() for t in tab]
            d = orc.sgns_step(tab[0], tab[1], mb.ctx, mb.ctr, orc.draw_negatives(mb, 0, K, 9, cdf),
                              orc.lr_at(b, B, prm.lr_start, prm.lr_end))
            for which, rows, delta in ((0, d.rows_in, d.d_in), (1, d.rows_out, d.d_out)):
                moved = np.zeros(n)
                moved[rows] = np.linalg.norm(delta, axis=1)
                err = np.abs(M.read(which).astype(np.float64) - tab[which])
                assert (err <= 1e-5 * moved[:, None] + np.spacing(np.abs(tab[which])) + 1e-12).all()
                assert (moved > 0).any() and not np.array_equal(tab[which], before[which])


# groups of eight and of four minibatches' ids; chunks whose last minibatch is
# ragged; both rings used again; row counters zeroed whole, and reset row by row
# (n above eight times a minibatch's touches)
@pytest.mark.parametrize("n,dim,K,P,chunk,count", [
    (3000, 64, 5, 3000, 1100, 41), (4000, 128, 20, 2200, 0, 37), (2000, 64, 1, 70000, 0, 11),
    (300000, 64, 5, 2500, 0, 25), (3000, 256, 7, 5000, 777, 20)])
def test_id_groups(fl, orc, n, dim, K, P, chunk, count):
    """Minibatches whose ids are drawn in groups against the same minibatches
    trained one call at a time, and (the smaller tables) against the oracle."""
    g = _random_graph(n)
    r = max(2, -(-count * P // (48 * min(n, 3000))) + 1)
    starts = np.arange(min(n, 3000), dtype=np.int32)
    prm = fl.train_params(window=3, negatives=K, minibatch_pairs=P, seed=9, chunk_walks=chunk)
    res = []
    for step in (count, 1):
        c = fl.Context(0)
        G = fl.Graph.from_csr(c, g.indptr, g.indices)
        W = fl.Walks.generate(G, r=r, L=12, seed=4, starts=fl.Active.from_host(G, starts))
        M = fl.Model.create(G, dim=dim, seed=6)
        for which, t in enumerate(_tables(n, dim)):
            M.write(which, t)
        pairs = rows = 0
        for b in range(0, count, step):
            st = M.train_steps(W, prm, b, step)
            assert st.path == 0 and st.minibatches == step
            pairs += st.pairs
            rows += st.rows_in + st.rows_out + st.rows_out_single
        res.append((M.read(fl.TABLE_IN), M.read(fl.TABLE_OUT), pairs, rows))
    assert np.array_equal(res[0][0], res[1][0]) and np.array_equal(res[0][1], res[1][1])
    assert res[0][2:] == res[1][2:]
    if chunk:
        assert res[0][2] < count * P        # a ragged minibatch was among them
    if n > 4000 or K > 7 or P > 5000:
        return
    tab = _tables(n, dim)
    walks = orc.walks_uniform(g, starts, r, 12, 4)
    cdf = orc.neg_cdf(g.degrees().astype(np.uint64))
    B, _ = orc.count_minibatches(walks, 3, P, *([chunk] if chunk else []))
    moved = [np.zeros(n), np.zeros(n)]
    for b in range(count):
        mb = orc.minibatch_pairs(walks, 3, P, b, *([chunk] if chunk else []))
        d = orc.sgns_step(tab[0], tab[1], mb.ctx, mb.ctr, orc.draw_negatives(mb, 0, K, 9, cdf),
                          orc.lr_at(b, B, prm.lr_start, prm.lr_end))
        moved[0][d.rows_in] += np.linalg.norm(d.d_in, axis=1)
        moved[1][d.rows_out] += np.linalg.norm(d.d_out, axis=1)
    for got, ref, mv in zip(res[0], tab, moved):
        err = np.abs(got.astype(np.float64) - ref)
        assert (err <= 1e-5 * mv[:, None] + count * np.spacing(np.abs(ref)) + 1e-12).all()


# calls below, at and above the fewest minibatches that planned launches serve,
# by touches; a budget that has room for plans but not for the ids' buffers
@pytest.mark.parametrize("P,K,counts", [(292, 5, (1, 2)), (293, 5, (1, 2, 3, 4)),
                                        (1171, 5, (1, 3, 4, 5)), (2340, 5, (1, 3, 4, 5))])
def test_few_minibatches(fl, P, K, counts):
    n, dim = 900, 64
    g = _random_graph(n)
    prm = fl.train_params(window=3, negatives=K, minibatch_pairs=P, seed=9)
    fewest = 1 if P * (K + 2) <= 2048 else 3 if P * (K + 2) <= 8192 else 4
    for count in counts:
        res = []
        for budget in (0, 1, 2):
            if budget == 2:
                budget = tight
            c = fl.Context(0, hbm_budget=0 if budget == 1 else budget)
            c.set_sgns_path(1)
            c.set_timing(1)
            G, W, M = _build(fl, c, g, dim=dim, r=6, L=12)
            held = c.bytes_in_use()
            if budget == 1:                              # one call per minibatch: the ids
                for b in range(count):
                    st = M.train_steps(W, prm, b, 1)
            else:
                st = M.train_steps(W, prm, 0, count)
            res.append((M.read(fl.TABLE_IN), M.read(fl.TABLE_OUT)))
            if budget == 0:
                assert (st.ms_apply_first == st.ms_apply) == (count >= fewest)
                # half of what the ids' buffers of these minibatches take
                tight = held + (8 + 16 + 20) * P * (K + 2) + 12 * P * dim + 20000
            elif budget > 1:
                assert st.ms_apply_first == st.ms_apply  # plans
        for r in res[1:]:
            assert np.array_equal(r[0], res[0][0]) and np.array_equal(r[1], res[0][1])
