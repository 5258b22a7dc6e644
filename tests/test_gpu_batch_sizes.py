"""Batch sizes on both sides of the lines where the search takes four, two or one
wavefronts per query, for rows of one to sixteen lanes, against the oracle."""
import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,bits,degree,ef,p", [(40, 8, 16, 33, 4), (128, 8, 32, 128, 4), (100, 8, 24, 64, 8), (250, 8, 32, 200, 8),
                                                (480, 4, 32, 64, 4), (960, 4, 48, 256, 4), (768, 4, 48, 300, 8), (1024, 8, 20, 100, 8)])
def test_wavefronts_per_query(d, bits, degree, ef, p):
    import gpu_harness as H
    import paper_2503_17911_amd as ann
    w = inputs.Workload("team", 1500, d, 12, 0.3, 2304, bits=(bits,), seed=d + ef)
    X, Q = inputs.base_vectors(w), inputs.queries(w)
    adj, entry = inputs.build_graph(X, degree, 64)
    lv = oracle.sq_fit(X, bits)
    ix = H.GpuIndex(X, adj, entry, [lv], oracle.L2)
    oi, ok, od, oc = oracle.search_batch(lv, d, adj, entry, Q, ef, expansions_per_step=p)
    for nq in (1, 3, 1023, 1024, 1025, 2049, 2304):
        gi, gk, gd, gc = ix.search(Q[:nq], ef, mode=1, expansions_per_step=p, visited_kind=ann.VISITED_AUTO)
        assert (gi == oi[:nq]).all() and (gd == od[:nq]).all() and (gk.view(np.uint32) == ok[:nq].view(np.uint32)).all()
        assert (gc[:, 0] == oc[:nq, 0]).all() and (gc[:, 2] == oc[:nq, 2]).all()
    ix.close()


@pytest.mark.parametrize("d,bits,degree,ef", [(40, 8, 16, 33), (128, 8, 32, 128), (250, 8, 64, 200), (960, 4, 48, 40), (1024, 8, 20, 300)])
def test_one_expansion_per_step(d, bits, degree, ef):
    """Batches on both sides of 16 queries per compute unit."""
    import gpu_harness as H
    import paper_2503_17911_amd as ann
    w = inputs.Workload("small", 1200, d, 12, 0.3, 4200, bits=(bits,), seed=d + ef)
    X, Q = inputs.base_vectors(w), inputs.queries(w)
    adj, entry = inputs.build_graph(X, degree, 64)
    lv = oracle.sq_fit(X, bits)
    ix = H.GpuIndex(X, adj, entry, [lv], oracle.L2)
    oi, ok, od, oc = oracle.search_batch(lv, d, adj, entry, Q, ef)
    for nq in (1, 4096, 4097, 4200):
        gi, gk, gd, gc = ix.search(Q[:nq], ef, visited_kind=ann.VISITED_AUTO)
        assert (gi == oi[:nq]).all() and (gd == od[:nq]).all() and (gk.view(np.uint32) == ok[:nq].view(np.uint32)).all()
        assert (gc[:, 0] == oc[:nq, 0]).all() and (gc[:, 2] == oc[:nq, 2]).all()
    ix.close()


@pytest.mark.parametrize("metric,bits,d,ef,p", [(oracle.L2, 8, 48, 100, 4), (oracle.IP, 8, 128, 64, 4), (oracle.L2, 4, 96, 130, 8), (oracle.IP, 4, 64, 300, 8),
                                                (oracle.L2, 8, 128, 64, 1), (oracle.IP, 8, 40, 130, 1), (oracle.L2, 4, 64, 40, 1)])
def test_options_at_both_ends_of_the_batch_sizes(metric, bits, d, ef, p):
    """Norm terms with the rows, inner-product keys (plain and of unit vectors), several entries and a pool size
    per query: on the kernels for small batches and on those for full ones."""
    import gpu_harness as H
    import torch
    import paper_2503_17911_amd as ann
    nq = 4200 if p == 1 else 2304
    rng = np.random.default_rng(d + ef)
    w = inputs.Workload("options", 1200, d, 12, 0.3, nq, bits=(bits,), seed=d + ef)
    X, Q = inputs.base_vectors(w), inputs.queries(w)
    if metric == oracle.IP:
        X /= np.linalg.norm(X, axis=1, keepdims=True)
    adj, entry = inputs.build_graph(X, 24, 64)
    lv = oracle.sq_fit(X, bits)
    ent = rng.integers(0, 1200, (nq, 5)).astype(np.uint32)
    ent[::3, 2], ent[1::3, 4] = 0xFFFFFFFF, ent[1::3, 0]
    efs = rng.choice(np.array([1, ef // 2, ef], np.uint32), nq)
    step = dict(mode=int(p > 1), expansions_per_step=p if p > 1 else 0, visited_kind=ann.VISITED_AUTO)

    def check(ix, key_metric, m, **kw):
        e, per_query = kw.get("entries"), kw.pop("efs", None)
        if per_query is not None:
            kw["ef_per_query"] = torch.from_numpy(per_query.view(np.int32)).to(H.DEV)
        gi, gk, gd, gc = ix.search(Q[:m], ef, **step, **kw)
        for pool in ([ef] if per_query is None else np.unique(per_query)):
            at = np.arange(m) if per_query is None else np.flatnonzero(per_query == pool)
            oi, ok, od, oc = oracle.search_batch(lv, d, adj, entry, Q[at], int(pool), metric=key_metric, entries=None if e is None else e[at],
                                                 expansions_per_step=p)
            assert (gi[at, :pool] == oi).all() and (gi[at, pool:] == 0xFFFFFFFF).all()
            assert (gk[at, :pool].view(np.uint32) == ok.view(np.uint32)).all() and (gd[at, :pool] == od).all()
            assert (gc[at, 0] == oc[:, 0]).all() and (gc[at, 2] == oc[:, 2]).all()

    ix = H.GpuIndex(X, adj, entry, [lv], metric)
    for m in (100, nq):
        check(ix, metric, m, entries=ent[:m])
        check(ix, metric, m, efs=efs[:m])
    if metric == oracle.IP:
        ix.close()
        ix = H.GpuIndex(X, adj, entry, [lv], metric, unit_norm_l2_keys=True)
    ix.build_row_norms()
    for m in (100, nq):
        check(ix, oracle.L2, m, layout=2)
        check(ix, oracle.L2, m, layout=2, entries=ent[:m], efs=efs[:m])
    ix.close()
