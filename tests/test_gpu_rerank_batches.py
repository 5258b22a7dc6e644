"""Rerank on both sides of the lines where a query's rows are shared by four
wavefronts: batch sizes, list lengths, padding anywhere in the list, odd rows."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n_cand,k,nq", [(128, 24, 10, 40), (128, 25, 25, 40), (960, 4, 3, 9), (960, 80, 10, 2048), (960, 80, 10, 2049),
                                           (33, 70, 70, 17), (300, 1024, 64, 5), (300, 1025, 64, 5), (7, 26, 1, 2100)])
@pytest.mark.parametrize("metric", [oracle.L2, oracle.IP])
def test_rerank(d, n_cand, k, nq, metric):
    import gpu_harness as H
    rng = np.random.default_rng(d + n_cand)
    n = 1200
    X, Q = rng.standard_normal((n, d), dtype=np.float32), rng.standard_normal((nq, d), dtype=np.float32)
    adj = np.stack([rng.permutation(n)[:8] for _ in range(n)]).astype(np.uint32)
    ix = H.GpuIndex(X, adj, 0, [oracle.sq_fit(X, 8)], metric)
    cand = np.stack([rng.permutation(n)[:n_cand] for _ in range(nq)]).astype(np.uint32)
    pad = rng.random(cand.shape) < 0.1
    pad[0] = True                                # a list of padding only
    pad[1] = False
    cand[pad] = 0xFFFFFFFF
    ids, dist = ix.rerank(Q, cand, n_cand, k)
    # plain fp64: distance, then (distance, id)
    for i in list(range(min(nq, 40))) + [nq - 1]:
        c = cand[i][cand[i] != 0xFFFFFFFF]
        rows, q = X[c].astype(np.float64), Q[i].astype(np.float64)
        full = -(rows @ q) if metric == oracle.IP else np.square(rows - q).sum(1)
        order = np.lexsort((c, full.astype(np.float32)))[:k]
        want_d = np.full(k, np.inf, np.float32)
        want_i = np.full(k, 0xFFFFFFFF, np.uint32)
        want_d[:order.size], want_i[:order.size] = full[order], c[order]
        H.check_rerank(ids[i:i + 1], dist[i:i + 1], want_i[None], want_d[None])
    ix.close()
