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
