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


# kernels that merge with more and with less in flight: rows of one to sixteen lanes, one and several expansions, rows that
# the kernels without run-time switches take and longer ones, labels, a visited cache that forgets and the table
@pytest.mark.parametrize("bits,d", [(8, 48), (8, 100), (8, 200), (8, 700), (4, 100), (4, 200), (4, 300), (4, 900)])
@pytest.mark.parametrize("ef", [33, 128, 200, 500])
def test_every_kernel_merges_the_same(bits, d, ef):
    import gpu_harness as H
    import paper_2503_17911_amd as ann
    rng = np.random.default_rng(d + ef)
    n, nq = 1500, 24
    X = rng.standard_normal((n, d)).astype(np.float32)
    X[700:900] = X[:200]  # equal keys: the order is by id
    Q = rng.standard_normal((nq, d)).astype(np.float32)
    lv = oracle.sq_fit(X, bits)
    for degree in (32, 48):
        adj = np.stack([rng.permutation(n)[:degree] for _ in range(n)]).astype(np.uint32)
        labels = rng.integers(10, 21, adj.shape).astype(np.float32) / np.float32(10)
        ix = H.GpuIndex(X, adj, 3, [lv], oracle.L2, labels=labels)
        for p in (1, 4, 8):
            mode = dict(mode=0 if p == 1 else 1, expansions_per_step=p)
            for labelled in (False, True):
                more = dict(alpha_s=1.7) if labelled else {}
                oi, ok, od, _ = oracle.search_batch(lv, d, adj, 3, Q, ef, expansions_per_step=p, **(dict(labels=labels, alpha_s=1.7) if labelled else {}))
                for visited in (dict(visited_kind=ann.VISITED_CACHE), dict(visited_kind=ann.VISITED_CACHE, visited_slots=64), dict(visited_kind=ann.VISITED_TABLE)):
                    got = ix.search(Q, ef, **mode, **visited, **more)
                    assert (got[0] == oi).all() and (got[1].view(np.uint32) == ok.view(np.uint32)).all() and (got[2] == od).all()
                # (a batch that the kernels for small ones do not take)
                got = ix.search(np.tile(Q, (180, 1)), ef, **mode, visited_kind=ann.VISITED_CACHE, **more)
                assert (got[0] == np.tile(oi, (180, 1))).all() and (got[2] == np.tile(od, (180, 1))).all()
        ix.close()


@pytest.mark.parametrize("bits,d,ef,p,most", [(8, 700, 128, 4, 1.5), (8, 200, 128, 4, 1.5)])
def test_a_slot_more_costs_little(bits, d, ef, p, most):
    """Rows of 33 slots, the last one empty, take the kernels with run-time switches: the same work as with 32."""
    import torch
    import gpu_harness as H
    import paper_2503_17911_amd as ann
    rng = np.random.default_rng(1)
    n, nq = 20_000, 8000
    X = rng.standard_normal((n, d)).astype(np.float32)
    adj = np.full((n, 33), 0xFFFFFFFF, np.uint32)
    adj[:, :32] = np.stack([rng.choice(n, 32, replace=False) for _ in range(n)])
    lv = oracle.sq_fit(X, bits)
    Q = torch.from_numpy(rng.standard_normal((nq, d)).astype(np.float32)).to(H.DEV)
    out = torch.empty((nq, ef), dtype=torch.int32, device=H.DEV)
    took, found = [], []
    for degree in (32, 33):
        ix = H.GpuIndex(X, np.ascontiguousarray(adj[:, :degree]), 0, [lv], oracle.L2)
        best = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            ann.ann_search_batch(ix.handle, Q, nq, k=10, ef=ef, out_ids=out, mode=1, expansions_per_step=p, stream=H.stream_ptr())
            b.record()
            b.synchronize()
            best.append(a.elapsed_time(b))
        took.append(min(best))
        found.append(H.as_u32(out))
        ix.close()
    assert (found[0] == found[1]).all()
    assert took[1] < most * took[0], took
