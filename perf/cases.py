"""The work that a user of the library has it do, as cases that can be timed.

Four kinds of case, each a sequence of calls of the public binding:

  search  a batch of queries on an index that is already on the GPU: (pivot scan
          and batch order,) graph search, (rescore with the finer codes,) exact
          rerank.  What a serving program does for every batch.
  truth   exact k nearest neighbours by exhaustive search: the ground truth of a
          recall measurement, or a flat index.
  codes   codebook and codes of a base set (the 8- or 4-bit scalar quantizer).
  index   the whole way from vectors and a graph to a searchable index and back:
          codebook, codes, upload, norm terms with the rows, pivot table, release.

Base sets are Gaussian mixtures, like the repository's benchmark workloads
(cluster counts, spreads, dimension scales and normalisation are theirs); the
graph is made on the GPU in a fraction of a second: near neighbours inside the
cluster, a few random nodes of the cluster and some of the whole set, to the
mean out-degree of the benchmark's graphs (about 20 of 32, 25 of 48).
"""
import math

import numpy as np
import torch

import paper_2503_17911_amd as ann

DEV = "cuda"
PAD = -1  # ANN_PAD_ID as int32


# ------------------------------------------------------------------ the cases
def _search(name, n, d, nq, ef, k, rerank, **more):
    case = dict(name=name, kind="search", n=n, d=d, nq=nq, ef=ef, k=k, rerank=rerank, clusters=max(8, n // 1000), sigma=0.3,
                aniso=0.0, metric="l2", bits=8, fine_bits=0, coverage=1.0, degree=32, mode=1, layout=0, pivots=0, filtered=False)
    case.update(more)
    return case


def _truth(name, n, d, nq, k, metric="l2"):
    return dict(name=name, kind="truth", n=n, d=d, nq=nq, k=k, metric=metric, clusters=max(8, n // 1000), sigma=0.3, aniso=0.0)


def _build(name, kind, n, d, bits, coverage, **more):
    case = dict(name=name, kind=kind, n=n, d=d, bits=bits, coverage=coverage, clusters=max(8, n // 1000), sigma=0.3, aniso=0.0,
                metric="l2", degree=32)
    case.update(more)
    return case


def listed():
    return [
        # one query at a time, host-synchronised or in a stream of requests: latency and launches count
        _search("one_query", 1_000_000, 128, 1, 128, 10, 20),
        # the benchmark's headline: 10,000 queries on 1M x 128, ordered by a pivot scan, norm terms with the rows
        _search("batch_1m_128", 1_000_000, 128, 10_000, 128, 10, 20, layout=2, pivots=256),
        # the smallest workload of the benchmark, in the order of Algorithm 1 (one expansion per step)
        _search("sequential_10k_128", 10_000, 128, 100, 64, 10, 20, clusters=100, mode=0),
        # long rows, 4-bit codes with a truncated range, a batch of a thousand, long rerank prefix
        _search("wide_960_4bit", 200_000, 960, 1000, 256, 10, 80, bits=4, coverage=0.99, aniso=0.5, clusters=100, layout=2),
        # unit-norm vectors, inner product: short rows, a full batch in the order it came
        _search("inner_product_96", 500_000, 96, 10_000, 128, 10, 20, metric="ip", sigma=0.25),
        # 4-bit traversal, 8-bit rescore, exact rerank, k = 100, 48 slots per row, the largest pool
        _search("cascade_768", 200_000, 768, 4000, 512, 100, 200, metric="ip", bits=4, fine_bits=8, coverage=0.99, degree=48,
                sigma=0.2, layout=2),
        # the edge filter of Section 4.3 (label bound and cap per expansion), odd sizes throughout
        _search("filtered_100", 50_021, 100, 513, 100, 7, 21, degree=27, mode=0, filtered=True),
        # ground truth of the headline workload: a dense contraction
        _truth("truth_1m_128", 1_000_000, 128, 10_000, 10),
        # ground truth with long rows and a long list
        _truth("truth_768_k100", 200_000, 768, 2000, 100, "ip"),
        # ground truth of the smallest workload (100 queries): launches and the host's waits count
        _truth("truth_10k_128", 10_000, 128, 100, 10),
        # codes of the headline's base set
        _build("codes_1m_128", "codes", 1_000_000, 128, 8, 1.0),
        # a whole index of long rows: truncated 4-bit codebook, codes, upload, row norms, pivots, release
        _build("index_960_4bit", "index", 200_000, 960, 4, 0.99, aniso=0.5, clusters=100),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["search", "search", "search", "truth", "truth", "codes", "index"])
    if kind == "search":
        bits = rng.choice([8, 8, 4])
        d = _log_int(rng, 24, 960)
        d += d % 2 if bits == 4 else 0
        n = _log_int(rng, 5000, max(5000, min(300_000, 120_000_000 // d)))
        metric = rng.choice(["l2", "l2", "ip"])
        ef = rng.choice([16, 32, 50, 64, 100, 128, 200, 256])
        k = rng.choice([1, 5, 10, 10, 16])
        mode = rng.choice([0, 1, 1])
        pivots = rng.choice([0, 256])
        filtered = rng.random() < 0.15
        return dict(_search("", n, d, _log_int(rng, 1, 10_000), ef, k, min(ef, k * rng.choice([2, 4])), metric=metric, bits=bits,
                            coverage=rng.choice([1.0, 0.99]), degree=rng.choice([16, 24, 32, 32, 48]), mode=mode,
                            layout=2 if metric == "l2" and mode == 1 and rng.random() < 0.6 else 0, pivots=pivots,
                            filtered=filtered), name="drawn")
    d = _log_int(rng, 24, 960)
    n = _log_int(rng, 5000, max(5000, min(1_000_000, 128_000_000 // d)))
    if kind == "truth":
        nq = _log_int(rng, 1, max(1, min(10_000, int(1.2e12 / n / d))))
        return dict(_truth("", n, d, nq, rng.choice([1, 10, 10, 16, 50, 100]), rng.choice(["l2", "l2", "ip"])), name="drawn")
    bits = rng.choice([8, 4])
    d += d % 2 if bits == 4 else 0
    if kind == "index":
        n = min(n, 300_000)
    return dict(_build("", kind, n, d, bits, rng.choice([1.0, 0.99]), degree=rng.choice([16, 32])), name="drawn")


# ------------------------------------------------------------------ inputs
def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _points(case, seed, nq):
    """Base vectors and queries of the case's mixture; node i belongs to cluster i % clusters."""
    g = _generator(seed)
    n, d, nc = case["n"], case["d"], case["clusters"]
    centres = torch.randn(nc, d, generator=g, device=DEV)
    scale = torch.exp(case["aniso"] * torch.randn(d, generator=g, device=DEV)) if case["aniso"] else None

    def sample(count, which):
        x = torch.randn(count, d, generator=g, device=DEV).mul_(case["sigma"]).add_(centres[which])
        if scale is not None:
            x.mul_(scale)
        if case.get("metric") == "ip":
            x.div_(x.norm(dim=1, keepdim=True))
        return x

    x = sample(n, torch.arange(n, device=DEV) % nc)
    q = sample(nq, torch.randint(nc, (nq,), generator=g, device=DEV)) if nq else None
    return x, q, g


def _graph(x, nc, degree, g):
    """Adjacency [n][degree] int32 with PAD, and the entry point (the node closest to the mean)."""
    n, d = x.shape
    size = -(-n // nc)
    n_near, n_same, n_far = (9, 4, 12) if degree >= 48 else (8, 2, 10) if degree >= 24 else (6, 2, 5)
    n_near = min(n_near, n // nc - 1)
    padded = torch.cat([x, x.new_zeros(size * nc - n, d)]) if size * nc != n else x
    by_cluster = padded.view(size, nc, d).transpose(0, 1)  # [nc][size][d]: node s * nc + c is (c, s)
    real = (torch.arange(size * nc, device=DEV) < n).view(size, nc).t()
    near = torch.empty(nc, size, n_near, dtype=torch.int64, device=DEV)
    step = max(1, 64_000_000 // (size * size))
    own = torch.arange(size, device=DEV)
    for c in range(0, nc, step):
        p = by_cluster[c:c + step].contiguous()
        dist = torch.baddbmm(p.square().sum(2)[:, None, :], p, p.transpose(1, 2).contiguous(), alpha=-2.0)
        dist.masked_fill_(~real[c:c + step, None, :], math.inf)
        dist[:, own, own] = math.inf
        near[c:c + step] = dist.topk(n_near, dim=2, largest=False).indices
    cluster = torch.arange(nc, device=DEV)[:, None, None]
    near = (near * nc + cluster).transpose(0, 1).reshape(size * nc, n_near)[:n]
    node = torch.arange(n, device=DEV)[:, None]
    same = torch.randint(n // nc, (n, n_same), generator=g, device=DEV) * nc + node % nc
    far = torch.randint(n, (n, n_far), generator=g, device=DEV)
    ids = torch.cat([near, same, far], 1)
    for t in range(ids.shape[1] - 1, 0, -1):  # a row names no neighbour twice, and not the node itself
        again = (ids[:, t:t + 1] == ids[:, :t]).any(1) | (ids[:, t] == node[:, 0])
        ids[:, t].masked_fill_(again, PAD)
    adj = torch.full((n, degree), PAD, dtype=torch.int32, device=DEV)
    adj[:, :ids.shape[1]] = ids.int()
    entry = int((x - x.mean(0)).square().sum(1).argmin())
    return adj, entry


def _row_bytes(d, bits):
    return d if bits == 8 else d // 2


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _quantizer_buffers(n, d, bits):
    return dict(lo=torch.empty(d, device=DEV), delta=torch.empty(d, device=DEV), norm=torch.empty(n, device=DEV),
                codes=torch.empty(n, _row_bytes(d, bits), dtype=torch.uint8, device=DEV))


def _quantize(x, bits, coverage, out):
    n, d = x.shape
    if coverage < 1.0:
        ann.ann_sq_train_truncated(x, n, d, bits, coverage, out["lo"], out["delta"], _stream())
    else:
        ann.ann_sq_train(x, n, d, bits, out["lo"], out["delta"], _stream())
    ann.ann_sq_encode(x, n, d, bits, out["lo"], out["delta"], out["codes"], out["norm"], _stream())
    return (bits, out["codes"], out["lo"], out["delta"], out["norm"])


class _Index:
    """An uploaded index that is released with the state that holds it."""

    def __init__(self, **desc):
        self.handle = ann.ann_upload_index(**desc)

    def release(self):
        if self.handle is not None:
            ann.ann_free_index(self.handle)
            self.handle = None

    def __del__(self):
        self.release()


def _metric(case):
    return ann.IP if case["metric"] == "ip" else ann.L2


def prepare(case, seed):
    s = dict(case=case)
    if case["kind"] == "truth":
        s["x"], s["q"], _ = _points(case, seed, case["nq"])
        s["ids"] = torch.empty(case["nq"], case["k"], dtype=torch.int32, device=DEV)
        s["dist"] = torch.empty(case["nq"], case["k"], device=DEV)
        return s
    if case["kind"] in ("codes", "index"):
        s["x"], _, g = _points(case, seed, 0)
        s["out"] = _quantizer_buffers(case["n"], case["d"], case["bits"])
        if case["kind"] == "index":
            s["adj"], s["entry"] = _graph(s["x"], case["clusters"], case["degree"], g)
        return s
    n, d, nq, ef, k = (case[f] for f in ("n", "d", "nq", "ef", "k"))
    x, s["q"], g = _points(case, seed, nq)
    adj, entry = _graph(x, case["clusters"], case["degree"], g)
    levels = [_quantize(x, b, case["coverage"], _quantizer_buffers(n, d, b)) for b in (case["bits"], case["fine_bits"]) if b]
    labels = torch.randint(10, 21, adj.shape, generator=g, device=DEV).float().div_(10.0) if case["filtered"] else None
    s["index"] = _Index(n=n, d=d, degree=case["degree"], metric=_metric(case), vectors=x, levels=levels, adjacency=adj,
                        entry_point=entry, edge_labels=labels, unit_norm_l2_keys=case["metric"] == "ip" and case["layout"] == 2,
                        stream=_stream())
    handle = s["index"].handle
    if case["layout"] == 2:
        ann.ann_build_row_norms(handle, _stream())
    if case["pivots"]:
        ann.ann_build_entry_table(handle, case["pivots"], _stream())
        s["scan"] = torch.empty(nq, dtype=torch.int32, device=DEV)
        s["order"] = torch.empty(nq, dtype=torch.int32, device=DEV)
    ann.ann_reserve_workspace(handle, nq, _stream())
    s["pool"] = torch.empty(nq, ef, dtype=torch.int32, device=DEV)
    s["keys"] = torch.empty(nq, ef, device=DEV)
    if case["fine_bits"]:
        s["fine_ids"] = torch.empty(nq, ef, dtype=torch.int32, device=DEV)
        s["fine_keys"] = torch.empty(nq, ef, device=DEV)
    s["ids"] = torch.empty(nq, k, dtype=torch.int32, device=DEV)
    s["dist"] = torch.empty(nq, k, device=DEV)
    return s


# ------------------------------------------------------------------ one pass
def _run_search(s):
    case, q, handle, stream = s["case"], s["q"], s["index"].handle, _stream()
    nq, ef, k = case["nq"], case["ef"], case["k"]
    extra = {}
    if case["pivots"]:
        ann.ann_entry_scan(handle, q, nq, 1, s["scan"], stream)
        ann.ann_schedule_queries(s["scan"], nq, case["n"], s["order"], stream)
        extra.update(query_order=s["order"], reuse_folded_queries=True)
    if case["filtered"]:
        extra.update(alpha_s=1.7, m_s=max(1, case["degree"] // 2))
    ann.ann_search_batch(handle, q, nq, k=k, ef=ef, out_ids=s["pool"], out_keys=s["keys"], mode=case["mode"],
                         layout=case["layout"], stream=stream, **extra)
    out = dict(pool=s["pool"], keys=s["keys"], ids=s["ids"], dist=s["dist"])
    cand = s["pool"]
    if case["fine_bits"]:
        ann.ann_rescore(handle, 1, q, nq, s["pool"], ef, ef, s["fine_ids"], s["fine_keys"], None, stream)
        cand = s["fine_ids"]
        out.update(fine_ids=cand, fine_keys=s["fine_keys"])
    ann.ann_rerank(handle, q, nq, cand, case["rerank"], ef, k, s["ids"], s["dist"], stream)
    return out


def run(state):
    case = state["case"]
    if case["kind"] == "search":
        return _run_search(state)
    if case["kind"] == "truth":
        ann.ann_bruteforce_topk(state["x"], case["n"], case["d"], state["q"], case["nq"], case["k"], _metric(case), state["ids"],
                                state["dist"], _stream())
        return dict(ids=state["ids"], dist=state["dist"])
    out = state["out"]
    level = _quantize(state["x"], case["bits"], case["coverage"], out)
    if case["kind"] == "index":
        index = _Index(n=case["n"], d=case["d"], degree=case["degree"], metric=_metric(case), vectors=state["x"], levels=[level],
                       adjacency=state["adj"], entry_point=state["entry"], stream=_stream())
        ann.ann_build_row_norms(index.handle, _stream())
        ann.ann_build_entry_table(index.handle, 256, _stream())
        index.release()
    return out


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    n, d = case["n"], case["d"]
    if case["kind"] == "truth":
        nq, k = case["nq"], case["k"]
        return {"bytes": 4 * d * (n + nq) + 8 * nq * k, "flops": 2 * nq * n * d}
    if case["kind"] in ("codes", "index"):
        size = 4 * n * d + n * _row_bytes(d, case["bits"]) + 4 * n + 8 * d
        if case["kind"] == "index":  # the arrays again, into the index, the rows with their norm terms beside them
            size += 2 * (4 * n * d + n * _row_bytes(d, case["bits"]) + 4 * n) + 4 * 4 * n * case["degree"]
        return {"bytes": size, "flops": 6 * n * d}
    nq, ef = case["nq"], case["ef"]
    expansions = min(n, ef + 40)   # measured on these graphs, one expansion per step
    evaluations = min(n, 14.0 * ef + 400)
    row = _row_bytes(d, case["bits"]) + (0 if case["metric"] == "ip" and case["layout"] != 2 else 4)
    per_query = expansions * 4 * case["degree"] + evaluations * row + 4 * d + 8 * ef + case["rerank"] * (4 * d + 4) + 8 * case["k"]
    if case["fine_bits"]:
        per_query += ef * (_row_bytes(d, case["fine_bits"]) + 4 + 8)
    return {"bytes": nq * per_query, "flops": 2 * nq * evaluations * d}


def tolerance(case):
    if case["kind"] == "search":
        # the traversal is integer work with a fixed rounding of the keys; the rerank sums in fp64 and rounds once
        return {"rel": 4e-7, "max": 1e-6, "differ": 1e-5}
    if case["kind"] == "truth":
        # fp64 distances rounded once; two neighbours closer than that may change places
        return {"rel": 4e-7, "max": 1e-6, "differ": 1e-4}
    return {"rel": 1e-7, "max": 2e-7, "differ": 0.0}  # codes are bytes; the norm is an fp64 sum rounded once


# ------------------------------------------------------------------ the same in 64 bits
def _exact_truth(case, seed):
    x, q, _ = _points(case, seed, case["nq"])
    x, q = x.double(), q.double()
    ids, dist = [], []
    xx = x.square().sum(1)
    step = max(1, 250_000_000 // case["n"])
    for i in range(0, case["nq"], step):
        b = q[i:i + step]
        dots = b @ x.t()
        score = -dots if case["metric"] == "ip" else xx - 2.0 * dots
        at = score.topk(case["k"], dim=1, largest=False).indices
        rows = x[at]
        exact_ = -(rows * b[:, None]).sum(2) if case["metric"] == "ip" else (rows - b[:, None]).square().sum(2)
        order = exact_.argsort(dim=1)
        ids.append(at.gather(1, order).int())
        dist.append(exact_.gather(1, order))
    return dict(ids=torch.cat(ids), dist=torch.cat(dist))


def _exact_range(x, coverage):
    if coverage >= 1.0:
        return x.amin(0), x.amax(0)
    n = x.shape[0]
    k = math.floor((1.0 - coverage) * (n - 1))
    lo, hi = [], []
    for j in range(0, x.shape[1], 64):
        col = x[:, j:j + 64].sort(0).values
        lo.append(col[k])
        hi.append(col[n - 1 - k])
    return torch.cat(lo), torch.cat(hi)


def _exact_codes(x, bits, coverage):
    """Codebook and codes; the code of a value is defined by single-precision arithmetic, the rest is in 64 bits."""
    top = (1 << bits) - 1
    mn, mx = _exact_range(x, coverage)
    # (a quotient of two floats taken in 64 bits and rounded once is the correctly rounded single-precision one)
    delta32 = torch.where(mx > mn, ((mx - mn).double() / top).float(), torch.ones_like(mx))
    delta = torch.where(mx > mn, (mx.double() - mn.double()) / top, torch.ones_like(mx, dtype=torch.float64))
    c = torch.empty(x.shape, dtype=torch.uint8, device=DEV)
    norm = torch.empty(x.shape[0], dtype=torch.float64, device=DEV)
    for i in range(0, x.shape[0], 100_000):
        steps = ((x[i:i + 100_000] - mn).double() / delta32.double()).float()
        part = (steps + 0.5).floor().clamp_(0, top)
        c[i:i + 100_000] = part.to(torch.uint8)
        norm[i:i + 100_000] = (mn.double() + delta * part.double()).square().sum(1)
    return dict(lo=mn.double(), delta=delta, codes=c, norm=norm)


def _exact_search(case, seed):
    """Algorithm 1 query by query (small batches, one code level)."""
    x, q, g = _points(case, seed, case["nq"])
    adj, entry = _graph(x, case["clusters"], case["degree"], g)
    lv = _exact_codes(x, case["bits"], case["coverage"])
    lo32, delta32 = lv["lo"].float().cpu().numpy(), lv["delta"].float().cpu().numpy()
    adj, codes, norm = adj.cpu().numpy(), lv["codes"].cpu().numpy(), lv["norm"].cpu().numpy()
    x, q = x.cpu().numpy(), q.cpu().numpy()
    top = np.float32(127.0)
    step = 1 if case["mode"] == 0 else ann.ann_default_expansions_per_step(case["ef"], case["degree"])
    l2_keys = case["metric"] == "l2" or case["layout"] == 2
    ef, k = case["ef"], case["k"]
    out = {f: [] for f in ("pool", "keys", "ids", "dist")}
    for v in q:
        a = delta32 * v
        amax = np.abs(a).max()
        scale = float(amax) / 127.0 if amax > 0 else 1.0
        t = np.clip(np.rint(a * (top / amax)), -127, 127).astype(np.int64) if amax > 0 else np.zeros(a.size, np.int64)
        qlo = float(np.dot(v.astype(np.float64), lo32.astype(np.float64)))

        def key(ids):
            dot = scale * (codes[ids].astype(np.int64) @ t)
            return norm[ids] - 2.0 * qlo - 2.0 * dot if l2_keys else -(dot + qlo)

        ids, keys, open_ = np.array([entry]), key(np.array([entry])), np.array([True])
        seen = {int(entry)}
        while open_.any():
            at = np.flatnonzero(open_)[:step]
            open_[at] = False
            new = []
            for u in ids[at]:
                for w in adj[u]:
                    if w != PAD and int(w) not in seen:
                        seen.add(int(w))
                        new.append(int(w))
            if new:
                new = np.array(new)
                ids, keys = np.concatenate([ids, new]), np.concatenate([keys, key(new)])
                open_ = np.concatenate([open_, np.ones(new.size, bool)])
                order = np.lexsort((ids, keys))[:ef]
                ids, keys, open_ = ids[order], keys[order], open_[order]
        pool, pool_keys = np.full(ef, PAD, np.int32), np.full(ef, np.inf)
        pool[:ids.size], pool_keys[:ids.size] = ids, keys
        c = ids[:case["rerank"]]
        rows, qd = x[c].astype(np.float64), v.astype(np.float64)
        dist = -(rows @ qd) if case["metric"] == "ip" else np.square(rows - qd).sum(1)
        order = np.lexsort((c, dist))[:k]
        top_ids, top_dist = np.full(k, PAD, np.int32), np.full(k, np.inf)
        top_ids[:order.size], top_dist[:order.size] = c[order], dist[order]
        for f, value in zip(("pool", "keys", "ids", "dist"), (pool, pool_keys, top_ids, top_dist)):
            out[f].append(value)
    return {f: np.stack(v) for f, v in out.items()}


def exact(case, seed):
    if case["kind"] == "truth":
        return _exact_truth(case, seed)
    if case["kind"] == "search":
        # a Python loop over the expansions: a few thousand of them
        return _exact_search(case, seed) if case["nq"] * case["ef"] <= 10_000 and not case["filtered"] else None
    x, _, _ = _points(case, seed, 0)
    found = _exact_codes(x, case["bits"], case["coverage"])
    if case["bits"] == 4:
        found["codes"] = found["codes"][:, 0::2] | (found["codes"][:, 1::2] << 4)
    return found
