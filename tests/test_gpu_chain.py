"""One expansion per step with a bit per node (small batches, the library's own choice of the visited set):
rows of one to sixteen lanes, slots with lanes of their own and lists of unvisited neighbours (of which some do not
fit the rows requested ahead), pools of one to eight registers, labels and the cap, and batches and base sets on both
sides of what is resident.  Against the oracle, bit for bit, the counts of evaluations too: nothing is forgotten."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _index(H, n, d, bits, degree, metric=oracle.L2, labels=False, seed=0, fill=1.0):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((n, d)).astype(np.float32)
    X[n // 2:n // 2 + n // 8] = X[:n // 8]  # equal keys: the order is by id
    if metric == oracle.IP:
        X /= np.linalg.norm(X, axis=1, keepdims=True)
    adj = np.stack([rng.choice(n, degree, replace=False) for _ in range(n)]).astype(np.uint32)
    adj[rng.random(adj.shape) > fill] = 0xFFFFFFFF
    lab = rng.integers(10, 21, adj.shape).astype(np.float32) / np.float32(10) if labels else None
    lv = oracle.sq_fit(X, bits)
    return H.GpuIndex(X, adj, 3, [lv], metric, labels=lab), lv, adj, lab, rng


def _same(got, want, counts=True):
    assert (got[0] == want[0]).all() and (got[1].view(np.uint32) == want[1].view(np.uint32)).all() and (got[2] == want[2]).all()
    if counts:
        assert (got[3][:, :3] == want[3][:, :3]).all() and (got[3][:, 3] == 0).all()


@pytest.mark.parametrize("bits,d", [(8, 48), (8, 100), (8, 200), (8, 400), (8, 900), (4, 48), (4, 200), (4, 300), (4, 900), (4, 1500)])
@pytest.mark.parametrize("degree", [5, 32, 33, 64])
def test_rows_and_degrees(bits, d, degree):
    import gpu_harness as H
    ix, lv, adj, lab, rng = _index(H, 700, d, bits, degree, labels=True, seed=d + degree, fill=0.8)
    Q = rng.standard_normal((20, d)).astype(np.float32)
    for ef in (7, 100, 200, 400):
        _same(ix.search(Q, ef, visited_slots=0), oracle.search_batch(lv, d, adj, 3, Q, ef))
        for kw in (dict(alpha_s=1.6), dict(m_s=max(1, degree // 3)), dict(alpha_s=1.6, m_s=max(1, degree // 3))):
            _same(ix.search(Q, ef, visited_slots=0, **kw), oracle.search_batch(lv, d, adj, 3, Q, ef, labels=lab, **kw))
    ix.close()


@pytest.mark.parametrize("n", [1, 2, 31, 33, 127, 128, 129, 1300])
def test_few_nodes_and_options(n):
    import gpu_harness as H
    import torch
    d, degree = 40, min(n, 24)
    for metric in (oracle.L2, oracle.IP):
        rng = np.random.default_rng(n)
        X = rng.standard_normal((n, d)).astype(np.float32)
        X /= np.linalg.norm(X, axis=1, keepdims=True)
        adj = np.stack([rng.permutation(n)[:degree] for _ in range(n)]).astype(np.uint32)
        lv = oracle.sq_fit(X, 8)
        ix = H.GpuIndex(X, adj, n - 1, [lv], metric)
        if metric == oracle.L2:
            ix.build_row_norms()
        Q = rng.standard_normal((9, d)).astype(np.float32)
        ent = rng.integers(0, n, (9, 4)).astype(np.uint32)
        ent[::2, 1] = 0xFFFFFFFF
        order = torch.from_numpy(rng.permutation(9).astype(np.int32)).to(H.DEV)
        for layout in (0, 2) if metric == oracle.L2 else (0,):
            _same(ix.search(Q, 20, visited_slots=0, layout=layout), oracle.search_batch(lv, d, adj, n - 1, Q, 20, metric=metric))
            _same(ix.search(Q, 20, visited_slots=0, layout=layout, entries=ent, query_order=order),
                  oracle.search_batch(lv, d, adj, n - 1, Q, 20, metric=metric, entries=ent))
        efs = np.array([1, 2, 20] * 3, np.uint32)
        got = ix.search(Q, 20, visited_slots=0, ef_per_query=torch.from_numpy(efs.view(np.int32)).to(H.DEV))
        for e in (1, 2, 20):
            want = oracle.search_batch(lv, d, adj, n - 1, Q[efs == e], e, metric=metric)
            assert (got[0][efs == e][:, :e] == want[0]).all() and (got[0][efs == e][:, e:] == 0xFFFFFFFF).all()
            assert (got[3][efs == e][:, :3] == want[3][:, :3]).all()
        ix.close()


@pytest.mark.parametrize("mode,n,nq", [(0, 500_000, 300), (1, 100_000, 400)])
def test_batches_on_several_streams(mode, n, nq):
    """Bits for a batch that is resident at once; not while another stream's batches would not fit next to it (the cache then
    forgets nodes, which the counts show), and again when that stream has been quiet for a while."""
    import gpu_harness as H
    import torch
    d, ef, degree, p = 16, 400, 12, 8
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, d)).astype(np.float32)
    adj = (np.arange(n, dtype=np.int64)[:, None] + rng.integers(1, n // degree, (n, degree)) + np.arange(degree) * (n // degree)) % n
    adj = adj.astype(np.uint32)
    lv = oracle.sq_fit(X, 8)
    ix = H.GpuIndex(X, adj, 11, [lv], oracle.L2)
    Q = np.tile(rng.standard_normal((20, d)).astype(np.float32), (nq // 20, 1))
    kw = dict(mode=mode, expansions_per_step=p if mode else 0, visited_slots=0)
    want = oracle.search_batch(lv, d, adj, 11, Q[:20], ef, expansions_per_step=p if mode else 1)
    want = tuple(np.tile(w, (nq // 20, 1)) for w in want)

    def forgotten():
        got = ix.search(Q, ef, **kw)
        assert all((g == w).all() for g, w in zip(got[:3], want)) and (got[3][:, 0] == want[3][:, 0]).all()
        return int((got[3][:, 1].astype(np.int64) - want[3][:, 1]).sum())

    assert forgotten() == 0
    others = [torch.cuda.Stream() for _ in range(2)]
    for s in others:
        with torch.cuda.stream(s):
            forgotten()
    assert forgotten() > 0
    for _ in range(32):
        forgotten()
    assert forgotten() == 0
    ix.close()


@pytest.mark.parametrize("n,degree,cap", [(9_000, 12, 0), (150_000, 12, 0), (600_000, 8, 3), (1_200_000, 8, 0), (1_200_000, 8, 3), (1_320_000, 8, 3)])
def test_batches_and_base_sets_on_both_sides_of_what_is_resident(n, degree, cap):
    """(The largest base set's bits do not fit a compute unit's LDS.)"""
    import gpu_harness as H
    d, ef = 16, 40
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, d)).astype(np.float32)
    adj = (np.arange(n, dtype=np.int64)[:, None] + rng.integers(1, n // degree, (n, degree)) + np.arange(degree) * (n // degree)) % n
    adj = adj.astype(np.uint32)
    lv = oracle.sq_fit(X, 8)
    ix = H.GpuIndex(X, adj, 11, [lv], oracle.L2)
    Q = rng.standard_normal((64, d)).astype(np.float32)
    want = oracle.search_batch(lv, d, adj, 11, Q, ef, m_s=cap)
    for nq in (1, 255, 257, 513, 1025, 2049, 4097):
        rep = -(-nq // 64)
        got = ix.search(np.tile(Q, (rep, 1))[:nq], ef, visited_slots=0, m_s=cap)
        _same(got, tuple(np.tile(w, (rep, 1))[:nq] for w in want), counts=False)
        assert (got[3][:, 0] == np.tile(want[3], (rep, 1))[:nq, 0]).all()
    ix.close()
