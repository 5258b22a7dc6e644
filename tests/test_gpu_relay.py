"""Several expansions per step on five wavefronts per query (small batches): rows of one to sixteen lanes, slots with lanes
of their own and lists, pools so small that a step's candidates fill them, batches on both sides of two queries to a
compute unit, and a visited cache that forgets.  Against the oracle, bit for bit; with a bit per node the number of
evaluations, too."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits,d", [(8, 48), (8, 100), (8, 200), (8, 400), (8, 900), (4, 60), (4, 200), (4, 300), (4, 900), (4, 1500)])
@pytest.mark.parametrize("p,degree", [(4, 3), (4, 32), (8, 32), (8, 17)])
def test_rows_steps_and_pools(bits, d, p, degree):
    import gpu_harness as H
    import paper_2503_17911_amd as ann
    rng = np.random.default_rng(d + p + degree)
    n, nq = 900, 20
    X = rng.standard_normal((n, d)).astype(np.float32)
    X[500:600] = X[:100]  # equal keys: the order is by id
    adj = np.stack([rng.choice(n, degree, replace=False) for _ in range(n)]).astype(np.uint32)
    adj[rng.random(adj.shape) > 0.85] = 0xFFFFFFFF
    lv = oracle.sq_fit(X, bits)
    ix = H.GpuIndex(X, adj, 3, [lv], oracle.L2)
    Q = rng.standard_normal((nq, d)).astype(np.float32)
    for ef in (1, 5, 30, 64, 128, 250, 512):
        oi, ok, od, oc = oracle.search_batch(lv, d, adj, 3, Q, ef, expansions_per_step=p)
        for visited in (dict(visited_slots=0), dict(visited_kind=ann.VISITED_CACHE), dict(visited_kind=ann.VISITED_CACHE, visited_slots=64)):
            got = ix.search(Q, ef, mode=1, expansions_per_step=p, **visited)
            assert (got[0] == oi).all() and (got[1].view(np.uint32) == ok.view(np.uint32)).all() and (got[2] == od).all()
            assert (got[3][:, 0] == oc[:, 0]).all() and (got[3][:, 2] == oc[:, 2]).all()
            if "visited_kind" not in visited:
                assert (got[3][:, 1] == oc[:, 1]).all()
    ix.close()


@pytest.mark.parametrize("degree,ef,p", [(33, 200, 4), (48, 256, 4), (64, 512, 8)])
def test_long_adjacency_rows(degree, ef, p):
    """Degrees above 32, which the folded kernels take from four pool registers per lane on: steps of up to 512 ids."""
    import gpu_harness as H
    rng = np.random.default_rng(degree)
    n, d, nq = 3000, 64, 300
    X = rng.standard_normal((n, d)).astype(np.float32)
    adj = np.stack([rng.choice(n, degree, replace=False) for _ in range(n)]).astype(np.uint32)
    for bits in (8, 4):
        lv = oracle.sq_fit(X, bits)
        ix = H.GpuIndex(X, adj, 3, [lv], oracle.L2)
        ix.build_row_norms()
        Q = rng.standard_normal((nq, d)).astype(np.float32)
        oi, ok, od, oc = oracle.search_batch(lv, d, adj, 3, Q, ef, expansions_per_step=p)
        for layout in (0, 2):
            got = ix.search(Q, ef, mode=1, expansions_per_step=p, visited_slots=0, layout=layout)
            assert (got[0] == oi).all() and (got[1].view(np.uint32) == ok.view(np.uint32)).all() and (got[3][:, :3] == oc[:, :3]).all()
        ix.close()


@pytest.mark.parametrize("bits,d", [(8, 40), (8, 200), (4, 300)])
@pytest.mark.parametrize("p", [4, 8])
@pytest.mark.parametrize("metric", [oracle.L2, oracle.IP])
def test_options(bits, d, p, metric):
    """Entry nodes (some twice, some none), an order, pool sizes of each query's own and folded queries of an earlier call, with
    bits and with the cache."""
    import gpu_harness as H
    import paper_2503_17911_amd as ann
    import torch
    rng = np.random.default_rng(d + p)
    n, nq, degree, ef = 1100, 24, 20, 200 if p == 8 else 70
    X = rng.standard_normal((n, d)).astype(np.float32)
    if metric == oracle.IP:
        X /= np.linalg.norm(X, axis=1, keepdims=True)
    adj = np.stack([rng.choice(n, degree, replace=False) for _ in range(n)]).astype(np.uint32)
    lv = oracle.sq_fit(X, bits)
    ix = H.GpuIndex(X, adj, 3, [lv], metric)
    Q = rng.standard_normal((nq, d)).astype(np.float32)
    ent = rng.integers(0, n, (nq, 6)).astype(np.uint32)
    ent[::2, 1] = 0xFFFFFFFF
    ent[:, 4] = ent[:, 0]
    order = torch.from_numpy(rng.permutation(nq).astype(np.int32)).to(H.DEV)
    efs = np.array([1, 2, 30, ef] * (nq // 4), np.uint32)
    kw = dict(mode=1, expansions_per_step=p)
    for visited in (dict(visited_slots=0), dict(visited_kind=ann.VISITED_CACHE)):
        plain = oracle.search_batch(lv, d, adj, 3, Q, ef, metric=metric, expansions_per_step=p)
        for more in (dict(), dict(same_queries_as_last_call=True, reuse_folded_queries=True), dict(query_order=order)):
            got = ix.search(Q, ef, **kw, **visited, **more)
            assert all((g == w).all() for g, w in zip(got[:3], plain)) and (got[3][:, 0] == plain[3][:, 0]).all()
        want = oracle.search_batch(lv, d, adj, 3, Q, ef, metric=metric, entries=ent, expansions_per_step=p)
        for more in (dict(), dict(query_order=order)):
            got = ix.search(Q, ef, entries=ent, **kw, **visited, **more)
            assert all((g == w).all() for g, w in zip(got[:3], want)) and (got[3][:, 0] == want[3][:, 0]).all()
        got = ix.search(Q, ef, ef_per_query=torch.from_numpy(efs.view(np.int32)).to(H.DEV), **kw, **visited)
        for e in np.unique(efs):
            want = oracle.search_batch(lv, d, adj, 3, Q[efs == e], int(e), metric=metric, expansions_per_step=p)
            assert (got[0][efs == e][:, :e] == want[0]).all() and (got[0][efs == e][:, e:] == 0xFFFFFFFF).all()
            assert (got[1][efs == e][:, :e] == want[1]).all() and (got[3][efs == e][:, 0] == want[3][:, 0]).all()
    ix.close()


@pytest.mark.parametrize("n,degree", [(20_000, 12), (700_000, 6), (1_400_000, 6)])
def test_batches_and_base_sets_on_both_sides_of_what_is_resident(n, degree):
    """(Bits for 512 queries, for 256, and for none.)"""
    import gpu_harness as H
    d, ef = 16, 60
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, d)).astype(np.float32)
    adj = (np.arange(n, dtype=np.int64)[:, None] + rng.integers(1, n // degree, (n, degree)) + np.arange(degree) * (n // degree)) % n
    adj = adj.astype(np.uint32)
    lv = oracle.sq_fit(X, 8)
    ix = H.GpuIndex(X, adj, 11, [lv], oracle.L2)
    Q = rng.standard_normal((64, d)).astype(np.float32)
    want = oracle.search_batch(lv, d, adj, 11, Q, ef, expansions_per_step=4)
    for nq in (1, 2, 256, 257, 512, 513):
        rep = -(-nq // 64)
        got = ix.search(np.tile(Q, (rep, 1))[:nq], ef, mode=1, visited_slots=0)
        assert all((g == np.tile(w, (rep, 1))[:nq]).all() for g, w in zip(got[:3], want))
        assert (got[3][:, 0] == np.tile(want[3], (rep, 1))[:nq, 0]).all()
    ix.close()


def test_longer_rows_on_both_sides_of_what_fits():
    """Rows of four lanes and few neighbours: the kernel lists them, and its LDS holds the lists beside a query's bits.  (Bits with
    lists in 160 KB: up to 1,261,952 nodes with four expansions and one pool register per lane, 1,215,872 with eight and four.)"""
    import gpu_harness as H
    d, degree, most = 130, 16, 1_270_000
    rng = np.random.default_rng(4)
    X = rng.standard_normal((most, d), dtype=np.float32)
    lv = oracle.sq_fit(X, 8)
    Q = rng.standard_normal((3, d)).astype(np.float32)
    for n in (1_210_000, 1_230_000, 1_255_000, most):
        adj = (np.arange(n, dtype=np.int64)[:, None] + rng.integers(1, n // degree, (n, degree)) + np.arange(degree) * (n // degree)) % n
        adj = adj.astype(np.uint32)
        part = oracle.SQLevel(8, lv.lo, lv.delta, lv.codes[:n], lv.norm_term[:n])
        ix = H.GpuIndex(X[:n], adj, 11, [part], oracle.L2)
        for ef, p in ((40, 4), (200, 8)):
            got = ix.search(Q, ef, mode=1, expansions_per_step=p, visited_slots=0)
            want = oracle.search_batch(part, d, adj, 11, Q, ef, expansions_per_step=p)
            assert all((g == w).all() for g, w in zip(got[:3], want)) and (got[3][:, 0] == want[3][:, 0]).all()
        ix.close()
