"""Device memory that is kept between objects: indexes and temporaries of
changing sizes, one after the other and from several threads, never see each
other's blocks."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("threads", [1, 3])
def test_indexes_of_changing_sizes(threads):
    import gpu_harness as H
    import torch

    def work(t):
        with torch.cuda.stream(torch.cuda.Stream()):
            for r in range(6):
                rng = np.random.default_rng(100 * t + r)
                n, d = [(3000, 24), (9000, 64), (2500, 100)][(r + t) % 3]
                X, Q = rng.standard_normal((n, d), dtype=np.float32), rng.standard_normal((9, d), dtype=np.float32)
                adj = np.stack([rng.permutation(n)[:16] for _ in range(n)]).astype(np.uint32)
                lv = oracle.sq_fit(X, 8)
                ix = H.GpuIndex(X, adj, 3, [lv], oracle.L2)
                gid, gdist = H.gpu_bruteforce(X, Q, 5, oracle.L2)
                gi, gk, gd, _ = ix.search(Q, 40)
                ix.close()
                lo, delta, codes, norm = H.gpu_sq_fit(X, 8)
                oi, ok, od, _ = oracle.search_batch(lv, d, adj, 3, Q, 40)
                assert (gi == oi).all() and (gd == od).all() and (gk.view(np.uint32) == ok.view(np.uint32)).all()
                oid, odist = oracle.bruteforce_topk(X, Q, 5)
                H.check_rerank(gid, gdist, oid, odist.astype(np.float32), rel=1e-6)
                assert (codes == lv.codes).all() and (norm.view(np.uint32) == lv.norm_term.view(np.uint32)).all()
        return True

    with ThreadPoolExecutor(threads) as pool:
        assert all(pool.map(work, range(threads)))


def test_kept_memory_is_given_back():
    import gpu_harness as H
    import torch
    import paper_2503_17911_amd as ann
    n, d, degree = 400_000, 128, 16
    lv = [(8, torch.zeros(n, d, dtype=torch.uint8, device=H.DEV), torch.zeros(d, device=H.DEV), torch.ones(d, device=H.DEV),
           torch.zeros(n, device=H.DEV))]
    adj = torch.stack([(torch.arange(n, device=H.DEV) + 1 + j) % n for j in range(degree)], 1).to(torch.int32)
    ann.ann_trim_memory()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    ix = ann.ann_upload_index(n=n, d=d, degree=degree, metric=ann.L2, vectors=None, levels=lv, adjacency=adj, entry_point=0, stream=H.stream_ptr())
    held = before - torch.cuda.mem_get_info()[0]
    assert held >= n * (d + 4 * degree)
    ann.ann_free_index(ix)
    kept = before - torch.cuda.mem_get_info()[0]
    assert kept <= held
    ann.ann_trim_memory()
    assert before - torch.cuda.mem_get_info()[0] <= 0
    ann.ann_trim_memory()
