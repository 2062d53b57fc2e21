"""Cases of the library's main paths for performance measurement: batched
range-filtered search in both entry modes and every row type, the exhaustive
filtered search, and the construction of the index on the GPU.

``listed()`` names the cases that stand for the library's use, ``draw(rng)``
gives further ones of the same ranges, ``prepare`` makes what a program has in
hand before a call (the uploaded index and the query batch, all from the
seed), ``run`` is one call through the Python binding, ``work`` the bytes and
operations no implementation can do without, ``tolerance`` the differences
another correct implementation may show, and ``exact`` the result in 64 bits
where the result is defined without the index's graph.

A case is a dict of plain values:

  do      "search", "exhaustive" (ground truth) or "build" (construction)
  n, d    base vectors and their dimension
  nq      queries of the batch
  k, L    results and pool size
  rows    storage of the rows: "fp32", "fp16" or "bf16"
  mode    entry mode: 0 each query its own stratified sample, 1 the sample
          shared by all queries
  cap     entry points per query: min(range, cap), or 16 for every query
          when cap is 0 (the method's default)
  budget  expansion budget
  n_inv   omitted layers of the index
  low     ranges have selectivity 2^-u, u uniform on [low, high]
  high    (equal: one fixed selectivity)
  data    "normal" (i.i.d.), "mixture" (Gaussian clusters, attribute a random
          permutation) or "slab" (unit vectors of a mixture, attribute the
          rank of a projection, so that a range selects a slab of space)
"""
import math

import numpy as np
import torch

import paper_2608_16491_amd as F

_KEYS = ("do", "n", "d", "nq", "k", "L", "rows", "mode", "cap", "budget", "n_inv", "low", "high", "data")


def _case(name=None, **kw):
    c = dict(do="search", n=100_000, d=128, nq=1000, k=10, L=64, rows="fp32", mode=1, cap=2560, budget=16, n_inv=7,
             low=0.0, high=10.0, data="mixture")
    c.update(kw)
    assert set(c) == set(_KEYS)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one user's query against a mid-sized collection, default parameters: latency
        _case("one_query", n=100_000, nq=1, mode=0, cap=0),
        # a handful of requests answered together, each with a thorough entry sample: latency
        _case("few_queries", n=200_000, nq=12, L=32, cap=2560),
        # the small unclustered workload of the tests: 100 queries, four selectivities' span, small rows
        _case("tiny", n=10_000, d=32, nq=100, L=64, cap=2000, high=6.7, data="normal"),
        # the headline workload at its pinned setting: throughput of a large batch
        _case("headline", n=1_000_000, nq=10_000, L=32, n_inv=5),
        # a large batch with each query's own stratified sample
        _case("stratified", n=250_000, nq=5000, L=32, budget=24, mode=0),
        # half-precision rows, small pool, as the 16-bit measurements of the benchmark
        _case("half_rows", n=300_000, d=96, nq=4000, L=24, budget=24, rows="fp16"),
        # bfloat16 rows of an odd dimension with the method's own 16 entry points
        _case("bf16_odd", n=150_001, d=100, nq=777, L=64, rows="bf16", mode=0, cap=0, data="normal"),
        # narrow filters of one selectivity: every range within the entry sample, so the result is exact
        _case("narrow", n=200_000, d=100, nq=2000, L=32, low=8.0, high=8.0),
        # hundred neighbours with the largest pool
        _case("hundred", n=300_000, nq=5000, k=100, L=256, cap=3072),
        # long vectors (64 lanes per row), the high-dimensional workload's setting
        _case("long_rows", n=40_000, d=960, nq=1000, L=128, mode=0, cap=1024, n_inv=6),
        # ground truth of a batch
        _case("exhaustive", do="exhaustive", n=300_000, nq=4000),
        # construction of an index on the GPU
        _case("build", do="build", n=60_000, d=96, nq=0, data="slab"),
    ]


def _log(rng, a, b):
    return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))


def draw(rng):
    kind = rng.choice(("shared", "shared", "shared", "own", "own", "exhaustive", "exhaustive", "build"))
    data = rng.choice(("normal", "mixture", "mixture", "slab"))
    if kind == "build":
        return _case(do="build", n=_log(rng, 5000, 60_000), d=_log(rng, 16, 96), nq=0, data=data)
    n = _log(rng, 10_000, 300_000)
    wide = rng.random() < 0.2
    if wide:
        n = min(n, 40_000)
        d = _log(rng, 129, 960)
    else:
        d = _log(rng, 20, 128)
    low = rng.choice((0.0, 0.0, 0.0, rng.uniform(0.0, 8.0)))
    high = low if low > 0.0 else rng.uniform(4.0, 10.0)
    k = rng.choice((1, 10, 10, 100, _log(rng, 1, 100)))
    if kind == "exhaustive":
        return _case(do="exhaustive", n=n, d=d, nq=_log(rng, 1, 500 if wide else 4000), k=k, data=data, low=low, high=high)
    return _case(n=n, d=d, nq=_log(rng, 1, 800 if wide else 5000), k=k, L=max(k, rng.choice((16, 24, 32, 64, 128, 256))),
                 rows="fp32" if wide else rng.choice(("fp32", "fp32", "fp32", "fp16", "bf16")),
                 mode=1 if kind == "shared" else 0, cap=rng.choice((0, _log(rng, 256, 3072), _log(rng, 256, 3072))),
                 budget=rng.choice((8, 16, 16, 24, 32)), n_inv=6 if d > 300 else rng.choice((5, 6, 7)), low=low, high=high,
                 data=data)


# ------------------------------------------------------------------ inputs

def _vectors(case, seed):
    """Base vectors, queries (on the GPU) and attribute (host) of a case."""
    n, d, nq = case["n"], case["d"], case["nq"]
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 2 + 1)

    def normal(rows):
        return torch.randn((rows, d), generator=g, device="cuda")

    X, Q = normal(n), normal(nq)
    if case["data"] != "normal":
        m = max(20, min(1000, n // 200))       # about 1000 vectors per cluster at the headline's size
        C = normal(m)
        X.mul_(0.3).add_(C[torch.randint(0, m, (n,), generator=g, device="cuda")])
        Q.mul_(0.3).add_(C[torch.randint(0, m, (nq,), generator=g, device="cuda")])
    if case["data"] == "slab":
        X = torch.nn.functional.normalize(X)
        Q = torch.nn.functional.normalize(Q)
        order = torch.argsort(X @ normal(1)[0])
    else:
        order = torch.randperm(n, generator=g, device="cuda")
    attr = torch.empty(n, dtype=torch.float64, device="cuda")
    attr[order] = torch.arange(n, dtype=torch.float64, device="cuda")
    return X, Q.contiguous(), attr.cpu().numpy()


def _ranges(case, seed):
    n, nq = case["n"], case["nq"]
    r = np.random.default_rng(int(seed) * 2 + 2)
    sigma = np.exp2(-(case["low"] + (case["high"] - case["low"]) * r.random(nq)))
    cnt = np.clip(np.rint(sigma * n), min(n, case["k"]), n).astype(np.int64)
    lo = r.integers(0, n - cnt + 1)
    return (torch.as_tensor(lo.astype(np.float64), device="cuda"),
            torch.as_tensor((lo + cnt - 1).astype(np.float64), device="cuda"))


def prepare(case, seed):
    X, Q, attr = _vectors(case, seed)
    host = X.cpu().numpy()
    del X
    if case["do"] == "build":
        return dict(case=case, X=host, attr=attr)
    ix = F.Index.build(host, attr, device=0, n_inv=case["n_inv"])
    if case["rows"] != "fp32":
        ix.upload(0, storage=case["rows"])
    if case["do"] == "search" and case["mode"] == 1:
        ix.prepare_sample(0)
    lo, hi = _ranges(case, seed)
    p = dict(entry_mode=case["mode"], budget=case["budget"])
    if case["cap"]:
        p.update(epn=16, epn_frac=1.0, epn_max=case["cap"])
    return dict(case=case, ix=ix, Q=Q, lo=lo, hi=hi, p=p)


def run(state):
    c = state["case"]
    if c["do"] == "build":
        ix = F.Index.build(state["X"], state["attr"], device=0, n_inv=c["n_inv"])
        out = ix.export()
        ix.free()
        return out
    if c["do"] == "exhaustive":
        return F.bruteforce(state["ix"], state["Q"], state["lo"], state["hi"], c["k"])
    return F.search(state["ix"], state["Q"], state["lo"], state["hi"], c["k"], c["L"], **state["p"])


# ------------------------------------------------------------------ what a result has to be

def _mean_range(case, most):
    """Mean over the selectivities of min(range, most)."""
    u = case["low"] + (case["high"] - case["low"]) * (np.arange(256) + 0.5) / 256
    return float(np.minimum(np.maximum(np.exp2(-u) * case["n"], case["k"]), most).mean())


def work(case):
    n, d, nq, k = case["n"], case["d"], case["nq"], case["k"]
    m = 16 if d <= 300 else 32
    H = max(1, math.ceil(math.log2(n)) + 1 - case["n_inv"])
    if case["do"] == "build":
        # the vectors once in, the candidate array once out; at least a full construction pool of
        # distances per vertex and layer
        ef = 128 if d <= 300 else 256
        return {"bytes": 4.0 * n * d + 8.0 * n + 4.0 * n * H * m, "flops": 3.0 * d * n * max(1, H - 1) * ef}
    io = nq * (4.0 * d + 16.0 + 8.0 * k)
    if case["do"] == "exhaustive":
        mean = _mean_range(case, n)
        return {"bytes": io + 4.0 * d * min(n, nq * mean), "flops": 2.0 * d * nq * mean}
    # the entry sample's distances; then at least L expansions a query, each reading a budget of
    # candidates and about three new vectors (ranges inside the sample hold no new ones)
    row = d * (4.0 if case["rows"] == "fp32" else 2.0)
    cap = case["cap"] or 16
    entry = nq * _mean_range(case, cap)
    u = case["low"] + (case["high"] - case["low"]) * (np.arange(256) + 0.5) / 256
    open_ = nq * float((np.exp2(-u) * n > cap).mean())
    fresh = open_ * case["L"] * 3.0
    rows = min(float(n), entry + fresh)
    enc = min(4.0 * n * H * m, nq * case["L"] * case["budget"] * 4.0)
    return {"bytes": io + rows * row + enc, "flops": 3.0 * d * (entry + fresh)}


def tolerance(case):
    if case["do"] == "build":
        return "exact"
    # squared distances summed in 64 bits and rounded once to fp32 (unit roundoff 6e-8): sums in another
    # order differ in the last bit of very few of them, and such a bit can order a near tie otherwise
    return {"rel": 2.5e-7, "differ": 1e-4}


def exact(case, seed):
    covered = case["do"] == "search" and case["cap"] and 2.0 ** -case["low"] * case["n"] <= case["cap"]
    if case["do"] == "build" or not (covered or case["do"] == "exhaustive"):
        return None     # the result depends on the index's graph
    X, Q, attr = _vectors(case, seed)
    lo, hi = _ranges(case, seed)
    a = torch.as_tensor(attr, device="cuda")
    X = {"fp32": X, "fp16": X.half(), "bf16": X.bfloat16()}[case["rows"]].double()
    Q, k = Q.double(), case["k"]
    xx = (X * X).sum(1)
    ids = torch.empty((len(Q), k), dtype=torch.int32, device="cuda")
    dists = torch.empty((len(Q), k), dtype=torch.float64, device="cuda")
    step = max(1, 400_000_000 // case["n"])
    for i in range(0, len(Q), step):
        q = Q[i:i + step]
        D = torch.addmm(xx[None, :], q, X.t(), alpha=-2.0)
        D.masked_fill_((a[None, :] < lo[i:i + step, None]) | (a[None, :] > hi[i:i + step, None]), math.inf)
        near = torch.topk(D, k, dim=1, largest=False).indices
        del D
        # the chosen ones again by differences, without the cancellation of the expanded square
        e = ((X[near.reshape(-1)].view(len(q), k, -1) - q[:, None, :]) ** 2).sum(2)
        e, at = torch.sort(e, dim=1)
        ids[i:i + step] = torch.gather(near, 1, at).int()
        dists[i:i + step] = e
    return (ids, dists, None) if case["do"] == "exhaustive" else (ids, dists)
