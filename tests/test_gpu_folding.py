"""The folded query's constant term where its terms cancel (the sum's order then
decides the rounding) and at lengths that do not fill a wavefront."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [2, 63, 64, 66, 130, 256, 960])
def test_cancelling_terms(d):
    import gpu_harness as H
    rng = np.random.default_rng(d)
    n, nq = 64, 75
    X = rng.standard_normal((n, d)).astype(np.float32) * 100
    adj = np.stack([rng.permutation(n)[:8] for _ in range(n)]).astype(np.uint32)
    lv = oracle.sq_fit(X, 8)
    Q = rng.standard_normal((nq, d)).astype(np.float32)
    # project out the codebook's minima: qlo is a small difference of large terms
    lo = lv.lo.astype(np.float64)
    Q = (Q - (Q @ lo)[:, None] * lo / (lo @ lo)).astype(np.float32)
    Q[5] = 0.0
    ix = H.GpuIndex(X, adj, 0, [lv], oracle.L2)
    t, s, qlo = ix.query_prep(Q)
    want = np.zeros(nq, np.float32)
    for i in range(nq):
        acc = 0.0
        for j in range(d):
            acc += float(Q[i, j]) * float(lv.lo[j])
        want[i] = np.float32(acc)
    assert (qlo.view(np.uint32) == want.view(np.uint32)).all()
    # the kernel that folds and scans pivots together leaves the same folding: the search after it returns the oracle's keys
    ix.entry_scan(Q, 16, 1)
    got = ix.search(Q, 20, reuse_folded_queries=True, same_queries_as_last_call=True)
    oi, ok, od, _ = oracle.search_batch(lv, d, adj, 0, Q, 20)
    assert (got[0] == oi).all() and (got[1].view(np.uint32) == ok.view(np.uint32)).all()
    ix.close()


def _check_launches(H, ix, Q):
    """The search kernel alone is launched (no folding ahead of it) for small batches."""
    import torch
    kw = dict(mode=0, visited_kind=H.ann.VISITED_CACHE)
    ix.search(Q, 20, **kw)
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        ix.search(Q, 20, **kw)
    names = [e.name for e in prof.events()]
    assert any("search_small_kernel" in s for s in names), names
    assert not any("query_prep_kernel" in s for s in names), names


@pytest.mark.parametrize("d,bits", [(2, 8), (30, 4), (63, 8), (66, 8), (130, 4), (256, 8), (258, 8), (960, 4), (1024, 8), (2046, 4)])
def test_folding_inside_the_search(d, bits):
    """The search kernels' own folding: rows of one to sixteen lanes, cancelling terms, a zero query, with one and
    several wavefronts per query, and what it leaves for a call that reuses it."""
    import gpu_harness as H
    import paper_2503_17911_amd as ann
    rng = np.random.default_rng(d)
    n, nq = 300, 20
    X = rng.standard_normal((n, d)).astype(np.float32) * 100
    adj = np.stack([rng.permutation(n)[:8] for _ in range(n)]).astype(np.uint32)
    lv = oracle.sq_fit(X, bits)
    Q = rng.standard_normal((nq, d)).astype(np.float32)
    lo = lv.lo.astype(np.float64)
    Q = (Q - (Q @ lo)[:, None] * lo / (lo @ lo)).astype(np.float32)
    Q[5] = 0.0
    ix = H.GpuIndex(X, adj, 0, [lv], oracle.L2)
    _check_launches(H, ix, Q)
    for p in (1, 4):
        kw = dict(mode=0 if p == 1 else 1, expansions_per_step=p)
        oi, ok, od, _ = oracle.search_batch(lv, d, adj, 0, Q, 20, expansions_per_step=p)
        for kind in (ann.VISITED_CACHE, ann.VISITED_TABLE):
            got = ix.search(Q, 20, visited_kind=kind, **kw)
            again = ix.search(Q, 20, visited_kind=kind, reuse_folded_queries=True, same_queries_as_last_call=True, **kw)
            for ids, keys, dots, _ in (got, again):
                assert (ids == oi).all() and (dots == od).all() and (keys.view(np.uint32) == ok.view(np.uint32)).all()
    ix.close()
