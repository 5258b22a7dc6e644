"""Codebook and encoder kernels at the edges of their pieces and row groups,
bit for bit against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import gpu_harness
    return gpu_harness


def _values(n, d, seed):
    rng = np.random.default_rng(seed)
    return (rng.standard_normal((n, d)) * np.exp(rng.standard_normal(d))).astype(np.float32)


def _fit(H, X, bits, offset=0):
    """Train and encode with x and the codes `offset` elements behind a 256-byte boundary."""
    import torch
    import paper_2503_17911_amd as ann
    n, d = X.shape
    rb = d if bits == 8 else d // 2
    xd = torch.empty(n * d + offset, device=H.DEV)
    xd[offset:] = H.dev(X).reshape(-1)
    codes = torch.zeros(n * rb + offset, dtype=torch.uint8, device=H.DEV)
    lo, delta, norm = (torch.empty(m, device=H.DEV) for m in (d, d, n))
    ann.ann_sq_train(xd[offset:], n, d, bits, lo, delta, H.stream_ptr())
    ann.ann_sq_encode(xd[offset:], n, d, bits, lo, delta, codes[offset:], norm, H.stream_ptr())
    return lo.cpu().numpy(), delta.cpu().numpy(), codes[offset:].cpu().numpy().reshape(n, rb), norm.cpu().numpy()


def _same(got, want):
    return (np.ascontiguousarray(got).view(np.uint32) == np.ascontiguousarray(want).view(np.uint32)).all()


# one piece per row and several; 8 to 64 lanes a row; rows that do not fill a group; scalar pieces (d % 4, offset)
@pytest.mark.parametrize("n,d,bits,offset", [(1, 1, 8, 0), (9, 3, 8, 0), (33, 4, 8, 0), (257, 32, 8, 0), (65, 36, 4, 0), (1027, 64, 8, 1),
                                             (63, 65, 8, 0), (130, 66, 4, 0), (129, 256, 8, 0), (31, 260, 8, 0), (70, 1028, 4, 0),
                                             (17, 2048, 8, 0), (19, 2048, 4, 3), (40000, 24, 8, 0), (12345, 10, 4, 2)])
def test_edges(H, n, d, bits, offset):
    X = _values(n, d, n + d)
    lv = oracle.sq_fit(X, bits)
    lo, delta, codes, norm = _fit(H, X, bits, offset)
    assert _same(lo, lv.lo) and _same(delta, lv.delta)
    assert (codes == lv.codes).all()
    assert _same(norm, lv.norm_term)


@pytest.mark.parametrize("bits", [8, 4])
def test_values_outside_the_range(H, bits):
    """Values far outside the codebook's range and infinities clamp; a column of one value has step 1."""
    import torch
    import paper_2503_17911_amd as ann
    X = _values(300, 72, 3)
    X[:, 5] = 1.5
    lv = oracle.sq_fit(X, bits)
    Y = X.copy()
    Y[::7] *= 1e6
    Y[3, 4], Y[5, 6], Y[8, 9], Y[9, 9] = np.inf, -np.inf, 3e38, -3e38
    want = oracle.sq_encode(Y, bits, lv.lo, lv.delta)
    codes = torch.empty(want.codes.shape, dtype=torch.uint8, device=H.DEV)
    norm = torch.empty(300, device=H.DEV)
    ann.ann_sq_encode(H.dev(Y), 300, 72, bits, H.dev(lv.lo), H.dev(lv.delta), codes, norm, H.stream_ptr())
    assert (codes.cpu().numpy() == want.codes).all()
    assert _same(norm.cpu().numpy(), want.norm_term)


# columns that do not fill a workgroup's 32, rows that do not fill its 16, equal values, signed zeros
@pytest.mark.parametrize("n,d,bits,coverage", [(2, 1, 8, 0.99), (255, 31, 8, 0.9), (257, 33, 8, 0.99), (5000, 65, 8, 0.75), (70001, 3, 8, 0.99),
                                               (4097, 34, 4, 0.999)])
def test_truncated_edges(H, n, d, bits, coverage):
    X = _values(n, d, n * 3 + d)
    X[:, 0] = np.round(X[:, 0])
    X[::2, d - 1] = -0.0
    lo_o, delta_o = oracle.sq_train_truncated(X, bits, coverage)
    lo, delta, _, _ = H.gpu_sq_fit(X, bits, coverage=coverage)
    assert (lo == lo_o).all() and _same(delta, delta_o)


# ranges from one pass over brackets (from 32,768 rows on): its smallest size, columns and rows that do not fill a group,
# lists of several sizes, ranks among the first values, rows in an order, few distinct values, infinities and NaN,
# more equal values than a list holds
@pytest.mark.parametrize("n,d,coverage,kind", [
    (32768, 1, 0.99, "values"), (32769, 33, 0.99, "values"), (40003, 70, 0.9999, "values"), (50000, 5, 0.99997, "values"), (33000, 31, 0.97, "values"),
    (400001, 4, 0.95, "values"), (1200003, 2, 0.97, "values"), (60000, 40, 0.99, "sorted"), (60000, 40, 0.99, "whole"), (60000, 24, 0.99, "mostly zero"),
    (50000, 12, 0.98, "not finite"), (70000, 9, 0.995, "one value"), (60000, 7, 0.8, "values")])
def test_truncated_by_brackets(H, n, d, coverage, kind):
    X = _values(n, d, n + d)
    if kind == "sorted":
        X.sort(axis=0)
        X[:, ::2] = X[::-1, ::2]
    elif kind == "whole":
        X = np.round(X)
    elif kind == "mostly zero":
        X[np.random.default_rng(1).random(X.shape) < 0.97] = 0.0
    elif kind == "not finite":
        X[::37], X[::41], X[5::1009, :4] = np.inf, -np.inf, np.nan
    elif kind == "one value":
        X[:, ::2], X[:, 1] = -2.5, 0.0
        X[::3, 1] = -0.0
    lo, delta, _, _ = H.gpu_sq_fit(X, 8, coverage=coverage)
    # the definition: order statistics of the ordered bit patterns
    u = np.ascontiguousarray(X).view(np.uint32)
    key = np.sort(np.where(u >> 31, ~u, u | 0x80000000), axis=0)
    k = int(np.floor((1.0 - coverage) * (n - 1)))
    mn, mx = (np.where(v >> 31, v & 0x7FFFFFFF, ~v).astype(np.uint32).view(np.float32) for v in (key[k], key[n - 1 - k]))
    assert (lo.view(np.uint32) == mn.view(np.uint32)).all()
    with np.errstate(invalid="ignore"):
        assert _same(delta, np.where(mx > mn, (mx - mn) / np.float32(255), np.float32(1)).astype(np.float32))


@pytest.mark.parametrize("degree", [1, 2, 7, 8, 9, 16, 31, 33, 64])
def test_adjacency_checks(H, degree):
    """Every pair of slots of a row is compared, every id is checked, and rows in order are taken."""
    import paper_2503_17911_amd as ann
    n, d = 300, 8
    rng = np.random.default_rng(degree)
    X = _values(n, d, degree)
    lv = oracle.sq_fit(X, 8)
    good = np.stack([rng.permutation(n)[:degree] for _ in range(n)]).astype(np.uint32)
    good[rng.random(good.shape) < 0.2] = 0xFFFFFFFF
    H.GpuIndex(X, good, 0, [lv], oracle.L2).close()
    pairs = [(a, b) for a in range(degree) for b in range(a + 1, degree)]
    for a, b in [pairs[i] for i in rng.permutation(len(pairs))[:20]] + pairs[-1:]:
        adj = good.copy()
        adj[n - 1] = 0xFFFFFFFF
        adj[n - 1, a] = adj[n - 1, b] = 7
        with pytest.raises(ann.AnnError) as e:
            H.GpuIndex(X, adj, 0, [lv], oracle.L2)
        assert e.value.status == ann.EINVAL and "twice" in str(e.value)
    adj = good.copy()
    adj[n - 1, degree - 1] = n
    with pytest.raises(ann.AnnError) as e:
        H.GpuIndex(X, adj, 0, [lv], oracle.L2)
    assert e.value.status == ann.EINVAL and ">= n" in str(e.value)


@pytest.mark.parametrize("n", [1, 9, 31, 33, 255, 257, 8191, 8193, 70_001])
@pytest.mark.parametrize("d,bits", [(4, 8), (6, 4), (33, 8), (128, 8)])
def test_rows_at_the_edges_of_the_passes(n, d, bits):
    """Row counts around the groups of rows that a thread and a workgroup take."""
    import gpu_harness as H
    X = np.random.default_rng(n + d).standard_normal((n, d)).astype(np.float32)
    X[-1] *= 9.0  # the last row holds an end of most ranges
    lv = oracle.sq_fit(X, bits)
    lo, delta, codes, norm = H.gpu_sq_fit(X, bits)
    assert (lo == lv.lo).all() and (delta == lv.delta).all() and (codes == lv.codes).all()
    assert (norm.view(np.uint32) == lv.norm_term.view(np.uint32)).all()


@pytest.mark.parametrize("n,d", [(32_768, 1000), (33_000, 33), (40_000, 32), (210_000, 30), (98_305, 8)])
def test_truncated_range_of_one_and_several_turns_of_workgroups(H, n, d):
    X = _values(n, d, n)
    X[:, 0] = np.maximum(X[:, 0], 0.0)  # half of a column equal: more than the few keys its bracket is searched among
    lo, delta, _, _ = H.gpu_sq_fit(X, 8, coverage=0.99)
    k = int(np.floor((1.0 - 0.99) * (n - 1)))
    S = np.sort(X, axis=0)
    mn, mx = S[k], S[n - 1 - k]
    assert (lo == mn).all() and _same(delta, ((mx - mn) / np.float32(255)).astype(np.float32))
