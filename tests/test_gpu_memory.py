"""Device memory that training takes beyond what it needs: bounded, and not in
the way of anything that fits without it.  Results do not depend on it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fl():
    from paper_2606_22180_amd import build, felog
    import os
    if not os.path.exists(build.LIB):
        build.build()
    felog.load()
    return felog


def _ring(n):
    """The cycle 0, 1, .., n - 1."""
    v = np.arange(n, dtype=np.int64)
    nbr = np.sort(np.stack([(v - 1) % n, (v + 1) % n], 1), 1)
    return np.arange(0, 2 * n + 1, 2, dtype=np.int64), nbr.ravel().astype(np.int32)


def _model(fl, ctx, n, *, dim=64, starts=3000, L=12, precision=0):
    G = fl.Graph.from_csr(ctx, *_ring(n))
    A = fl.Active.from_host(G, np.arange(min(starts, n), dtype=np.int32))
    W = fl.Walks.generate(G, r=2, L=L, seed=3, starts=A)
    M = fl.Model.create(G, dim=dim, seed=5, precision=precision)
    return G, A, W, M


def _prm(fl, P, K=5):
    return fl.train_params(window=4, negatives=K, minibatch_pairs=P, seed=9)


def test_id_sets_are_bounded(fl):
    """2,500 pairs on 2^22 nodes: id sets of 67 MB, of which sixteen would let
    eight minibatches' ids share a launch.  Beyond the three of a model, an
    eighth of its tables (268 MB), and the same tables as three sets give."""
    n, prm = 1 << 22, _prm(fl, 2500)
    c = fl.Context(0)
    objs = _model(fl, c, n)
    held = c.bytes_in_use()
    objs[3].train_steps(objs[2], prm, 0, 20)
    grown = c.bytes_in_use() - held
    print("[gpu] grown by", grown, flush=True)
    assert grown <= 2 * 4 * n * 64 // 8 + (32 << 20)
    rows = [objs[3].read(t)[:4096] for t in (0, 1)]
    for o in reversed(objs):
        o.close()
    c2 = fl.Context(0, hbm_budget=held + (60 << 20))   # three sets only
    objs = _model(fl, c2, n)
    objs[3].train_steps(objs[2], prm, 0, 20)
    assert all(np.array_equal(a, objs[3].read(t)[:4096]) for t, a in enumerate(rows))


def test_larger_minibatches_after_groups(fl):
    """A budget that one minibatch of 60,000 pairs fits still does after groups
    of smaller minibatches took id sets from it."""
    n = 1 << 16

    def steps(budget, small_first):
        c = fl.Context(0, hbm_budget=budget)
        objs = _model(fl, c, n)
        if small_first:
            objs[3].train_steps(objs[2], _prm(fl, 2500), 0, 20)
        else:
            objs[3].train_delta(objs[2], _prm(fl, 64), 0)    # (the corpus's column list)
        objs[3].train_steps(objs[2], _prm(fl, 60000), 0, 1)
        return c.bytes_in_use()

    need = steps(0, False)
    print("[gpu] needed", need, flush=True)
    steps(need + (2 << 20), False)
    steps(need + (2 << 20), True)


# what comes after the groups: a second corpus, or a minibatch's captured deltas
@pytest.mark.parametrize("then", ["corpus", "deltas"])
def test_id_sets_make_room(fl, then):
    """Groups of minibatches take id sets from a budget; an allocation that
    fits beside three sets gets their memory, and training goes on."""
    n, prm = 1 << 18, _prm(fl, 2500, K=20)

    def steps(budget, spare):
        c = fl.Context(0, hbm_budget=budget)
        objs = _model(fl, c, n)
        held = c.bytes_in_use()
        objs[3].train_steps(objs[2], prm, 0, 20)
        used = c.bytes_in_use()
        if spare and then == "corpus":
            W = fl.Walks.generate(objs[0], r=1, L=spare // (4 * n), seed=4)
            assert np.array_equal(W.read_range(0, 5)[:, 0], np.arange(5))
            W.close()
        elif spare:
            objs[3].train_delta(objs[2], prm, 3)
        objs[3].train_steps(objs[2], prm, 20, 20)
        return held, used, [objs[3].read(t) for t in (0, 1)]

    held, many, rows = steps(0, 0)
    _, few, rows3 = steps(held + (40 << 20), 0)
    print("[gpu] %d bytes held with many id sets, %d with three" % (many, few), flush=True)
    assert many - few > 60 << 20 and all(np.array_equal(a, b) for a, b in zip(rows, rows3))
    # room for the many sets, but not for them and what follows
    budget = many + (5 << 20)
    _, used, got = steps(budget, budget - few - (4 << 20))
    assert used == many and all(np.array_equal(a, b) for a, b in zip(rows, got))


def test_plans_make_room(fl):
    """The same of the plans of a group of minibatches (update path 1)."""
    n, prm = 1 << 12, _prm(fl, 1024)

    def steps(budget, spare):
        c = fl.Context(0, hbm_budget=budget)
        c.set_sgns_path(1)
        objs = _model(fl, c, n)
        objs[3].train_steps(objs[2], prm, 0, 130)
        used = c.bytes_in_use()
        if spare:
            fl.Walks.generate(objs[0], r=1, L=spare // (4 * n), seed=4).close()
        objs[3].train_steps(objs[2], prm, 130, 130)
        return used, [objs[3].read(t) for t in (0, 1)]

    used, rows = steps(0, 0)
    for extra in (1 << 16, 1 << 20):
        got = steps(used + extra, extra + (8 << 20))
        assert got[0] == used and all(np.array_equal(a, b) for a, b in zip(rows, got[1]))


@pytest.mark.parametrize("mode", [1, 2])
def test_serving_estimate_of_plans(fl, mode):
    """A persistent or shared job reserves its plans (14 bytes per touch of 128
    minibatches) beside what a job of launches does, and holds no more."""
    n, P, K, dim = 1500, 1024, 5, 64
    est, peak = {}, {}
    for m in (0, mode):
        S = fl.Server(0, 0, slots=1, minibatch_pairs=P, negatives=K, update_mode=m)
        jid = S.submit(*_ring(n), dim=dim, r=8, L=20, window=3, seed=2)
        st = S.wait(jid, 60.0)
        S.close()
        assert st.state == fl.JOB_DONE
        est[m], peak[m] = st.device_bytes, st.peak_bytes
    print("[gpu] estimates %s, peaks %s" % (est, peak), flush=True)
    plans = 128 * (14 * P * (K + 2) + 16)
    pairs = 8 * P * (K + 2) + 8 * P * dim
    # descriptors, slices, control words and loss slots: below 256 KiB here
    assert 0 < est[mode] - est[0] <= (plans + pairs + (256 << 10)) * 17 // 16
    assert peak[mode] <= est[mode] and peak[0] <= est[0]


@pytest.mark.parametrize("route,large,small", [("bf16", 512, 64), ("persistent", 1024, 64),
                                               ("planned", 2048, 64), ("ids", 60000, 2500)])
def test_after_a_refused_call(fl, route, large, small):
    """Minibatches that do not fit a budget are refused by every call; smaller
    ones after them are refused too (buffers of the refused size that did fit are
    kept) or train as they do alone."""
    def prm(P):
        return fl.train_params(window=4, negatives=5, minibatch_pairs=P, seed=9,
                               shared_negatives=P if route == "bf16" else 0)

    def steps(budget, sizes):
        c = fl.Context(0, hbm_budget=budget)
        c.set_sgns_path(int(route == "planned"))
        objs = _model(fl, c, 4096, precision=fl.PREC_BF16 if route == "bf16" else 0)
        held, status = c.bytes_in_use(), []
        for P in sizes:
            try:
                objs[3].train_steps(objs[2], prm(P), 0, 6)
                status.append(0)
            except fl.FelogError as err:
                assert err.status == fl.FELOG_ENOMEM
                status.append(err.status)
        return held, c.bytes_in_use(), status, [objs[3].read(t) for t in (0, 1)]

    held, _, _, rows = steps(0, [small])
    _, all_held, _, both = steps(0, [large, large, small])
    refused = trained = 0
    for k in range(1, 36):                       # every buffer is the one too many
        _, _, status, got = steps(held + (all_held - held + (2 << 20)) * k // 35,
                                  [large, large, small])
        assert status[0] == status[1] and (status[0] or not status[2])
        refused += status[0] != 0
        trained += status[0] != 0 and not status[2]
        if not status[2]:
            assert all(np.array_equal(a, b) for a, b in zip(rows if status[0] else both, got))
    print("[gpu] %s: %d of 35 budgets refused, %d of them trained the smaller" %
          (route, refused, trained), flush=True)
    assert 0 < trained <= refused < 35
