"""The merge of a step's candidates into the pool: pool sizes on both sides of a register
and of half a register per lane, steps of up to 64, 256 and 512 candidates (long batches,
half-full ones and single ones as the search converges), and a visited cache so small that
nodes come back while they are in the pool, or twice in one step.  Against the oracle, bit for bit."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ef", [1, 2, 31, 33, 64, 65, 127, 128, 129, 256, 257, 511, 512])
def test_pool_sizes_and_step_sizes(ef):
    import gpu_harness as H
    import paper_2503_17911_amd as ann
    rng = np.random.default_rng(ef)
    n, d, nq = 1500, 48, 40
    X = rng.standard_normal((n, d)).astype(np.float32)
    X[700:900] = X[:200]  # equal keys: the order is by id
    Q = rng.standard_normal((nq, d)).astype(np.float32)
    lv = oracle.sq_fit(X, 8)
    for degree in (32, 64):
        adj = np.stack([rng.permutation(n)[:degree] for _ in range(n)]).astype(np.uint32)
        ix = H.GpuIndex(X, adj, 3, [lv], oracle.L2)
        for p in (1, 4, 8):
            oi, ok, od, oc = oracle.search_batch(lv, d, adj, 3, Q, ef, expansions_per_step=p)
            for slots in (0, 64):
                got = ix.search(Q, ef, mode=0 if p == 1 else 1, expansions_per_step=p, visited_kind=ann.VISITED_CACHE, visited_slots=slots)
                assert (got[0] == oi).all() and (got[1].view(np.uint32) == ok.view(np.uint32)).all() and (got[2] == od).all()
                assert (got[3][:, 0] == oc[:, 0]).all() and (got[3][:, 2] == oc[:, 2]).all()
        ix.close()
