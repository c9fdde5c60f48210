"""Performance cases of the k-NN library: what a user's program has it do.

Each case is one pass through the public Python entry points (Handle.select_k,
graph, search, search_host_corpus, batch_search, pivot_grad) on inputs drawn
from a seed.  The listed cases span the range from calls bounded by launch
latency to whole k-NN graphs; draw() spreads further ones over the same ranges.
"""
import math

import numpy as np
import torch

import paper_1309_5478_amd as knn

DEVICE = "cuda"
SELECT_MAX = 1 << 30          # entries of the largest distance matrix
GRAPH_MAX = 2.0 * 131072.0 ** 2 * 1024  # flops of the largest graph


def listed():
    return [
        # A re-ranking step: the 10 best of a few thousand scores for a small
        # batch of queries.  The smallest call; launch latency is what counts.
        dict(name="select_small", kind="select", rows=64, cols=4096, k=10, data="dist", pivot="sample"),
        # The selection workload of the benchmark: a stored distance matrix
        # (squared distances of normal points), one long row per query.
        dict(name="select_matrix", kind="select", rows=16384, cols=65536, k=256, data="dist", pivot="sample"),
        # The paper's saturation workload at its low end: a handful of queries
        # against a million entries each (uniform values).
        dict(name="select_few_long", kind="select", rows=8, cols=1 << 20, k=32, data="uniform", pivot="sample"),
        # The smallest k-NN graph of the benchmark, launch- and latency-bound.
        dict(name="graph_small", kind="search", graph=True, m=4096, n=4096, d=128, k=16, precision="fp32",
             metric="sqeuclidean", data="uniform"),
        # The headline graph (d = 1024, k = 32, Gaussian mixture) on half its
        # points: the default precision, bounded by the distance product.
        dict(name="graph_fp32", kind="search", graph=True, m=131072, n=131072, d=1024, k=32, precision="fp32",
             metric="sqeuclidean", data="gmm"),
        # The same graph with the product in BF16.
        dict(name="graph_bf16", kind="search", graph=True, m=131072, n=131072, d=1024, k=32, precision="bf16",
             metric="sqeuclidean", data="gmm"),
        # The reduced-precision configuration (d = 256, k = 64) in FP8.
        dict(name="graph_fp8", kind="search", graph=True, m=262144, n=262144, d=256, k=64, precision="fp8",
             metric="sqeuclidean", data="gmm"),
        # Retrieval by cosine over embeddings whose sizes are multiples of
        # nothing, queries and corpus apart.
        dict(name="search_cosine", kind="search", graph=False, m=5003, n=150001, d=300, k=10, precision="fp32",
             metric="cosine", data="gmm"),
        # Online retrieval: one small batch of queries against a million
        # vectors; latency, and one read of the corpus.
        dict(name="search_few", kind="search", graph=False, m=16, n=1000000, d=128, k=10, precision="fp32",
             metric="sqeuclidean", data="gmm"),
        # The batched workload: uneven jobs (corpus sizes log-uniform, d 64, 128
        # or 768, k log-uniform up to 1024) in one call, replayed by a program
        # that keeps its buffers.
        dict(name="batch_uneven", kind="batch", jobs=96, m=1024, n_lo=1000, n_hi=200000, table=5, precision="fp32"),
        # A corpus in pinned host memory, streamed past resident queries.
        dict(name="host_corpus", kind="host", m=4096, n=1 << 20, d=256, k=32, part_rows=1 << 18, precision="fp32"),
        # Training the pivot network: loss and gradient of one batch (forward
        # and backward).
        dict(name="pivot_grad", kind="pivot", batch=4096, quantile=0.99),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["select", "select", "graph", "graph", "search", "search", "batch", "host", "pivot"])
    if kind == "select":
        cols = _log_int(rng, 300, 1 << 20)
        rows = min(_log_int(rng, 1, 16384), SELECT_MAX // cols)
        return dict(kind="select", rows=rows, cols=cols, k=min(_log_int(rng, 1, 1024), cols),
                    data=rng.choice(["dist", "uniform"]), pivot=rng.choice(["sample", "sample", "learned"]))
    if kind == "graph":
        prec = rng.choice(["fp32", "bf16", "fp8"])
        d = _log_int(rng, 16, 1024)
        top = int(min(262144.0 if prec != "fp32" else 131072.0, math.sqrt(GRAPH_MAX / (2.0 * d))))
        n = _log_int(rng, 2000, top)
        return dict(kind="search", graph=True, m=n, n=n, d=d, k=_log_int(rng, 4, 64), precision=prec,
                    metric=rng.choice(["sqeuclidean", "sqeuclidean", "cosine", "pearson"]),
                    data=rng.choice(["uniform", "gmm"]))
    if kind == "search":
        return dict(kind="search", graph=False, m=_log_int(rng, 1, 16384), n=_log_int(rng, 1000, 1000000),
                    d=_log_int(rng, 16, 768), k=_log_int(rng, 1, 100), precision=rng.choice(["fp32", "fp32", "bf16", "fp8"]),
                    metric=rng.choice(["sqeuclidean", "sqeuclidean", "cosine", "pearson"]),
                    data=rng.choice(["uniform", "gmm"]))
    if kind == "batch":
        return dict(kind="batch", jobs=rng.randint(4, 96), m=_log_int(rng, 32, 1024), n_lo=1000,
                    n_hi=_log_int(rng, 5000, 200000), table=rng.randint(100, 1 << 20),
                    precision=rng.choice(["fp32", "fp32", "bf16"]))
    if kind == "host":
        n = _log_int(rng, 1 << 17, 1 << 20)
        return dict(kind="host", m=_log_int(rng, 64, 4096), n=n, d=rng.choice([96, 128, 200, 256]),
                    k=_log_int(rng, 4, 64), part_rows=n // rng.randint(2, 5) + 1, precision="fp32")
    return dict(kind="pivot", batch=_log_int(rng, 256, 8192), quantile=rng.choice([0.9, 0.95, 0.99]))


# ---- inputs ---------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return g


def _points(g, count, d, data):
    """count x d points: uniform[0, 1), or the mixture of 64 unit Gaussians with
    means N(0, 4 I)."""
    if data == "uniform":
        return torch.rand((count, d), generator=g, device=DEVICE)
    means = 2.0 * torch.randn((64, d), generator=g, device=DEVICE)
    comp = torch.randint(0, 64, (count,), generator=g, device=DEVICE)
    x = torch.randn((count, d), generator=g, device=DEVICE)
    x += means[comp]
    return x


def _matrix(case, seed):
    """The stored matrix of a selection: squared distances of normal points in
    256 dimensions, or uniform values."""
    g = _gen(seed)
    rows, cols = case["rows"], case["cols"]
    if case["data"] == "uniform":
        return torch.rand((rows, cols), generator=g, device=DEVICE)
    q = torch.randn((rows, 256), generator=g, device=DEVICE)
    c = torch.randn((cols, 256), generator=g, device=DEVICE)
    out = torch.mm(q, c.t())
    out.mul_(-2.0).add_((c * c).sum(1)).add_((q * q).sum(1)[:, None])
    return out


def _search_points(case, seed):
    g = _gen(seed)
    n, m = case["n"], case["m"]
    x = _points(g, n if case.get("graph") else n + m, case["d"], case.get("data", "gmm"))
    return (x, x) if case.get("graph") else (x[n:].contiguous(), x[:n].contiguous())


def _jobs(case):
    """The job table: (n, d, k, data) per job, a function of the case alone."""
    rng = np.random.default_rng(case["table"])
    out = []
    for _ in range(case["jobs"]):
        n = int(round(math.exp(rng.uniform(math.log(case["n_lo"]), math.log(case["n_hi"])))))
        d = int((64, 128, 768)[int(rng.integers(0, 3))])
        k = int(round(math.exp(rng.uniform(0.0, math.log(1024.0)))))
        out.append((n, d, k, "uniform" if rng.random() < 0.5 else "gmm"))
    return out


def _job_points(case, seed):
    g = _gen(seed)
    m = case["m"]
    pts = []
    for n, d, k, data in _jobs(case):
        x = _points(g, n + m, d, data)
        pts.append((x[n:].contiguous(), x[:n].contiguous(), k))
    return pts


def _pivot_inputs(case, seed):
    """Feature rows and targets of the network's ranges, and He-initialised
    weights."""
    g = _gen(seed)
    B = case["batch"]
    x = torch.randn((B, 8), generator=g, device=DEVICE)
    x[:, 0] = 0.5 + 0.75 * torch.rand((B,), generator=g, device=DEVICE)   # log2(N) / 16
    x[:, 1] = torch.rand((B,), generator=g, device=DEVICE)                # log2(k) / 10
    x[:, 2] = -2.5 - 0.5 * x[:, 2].abs()                                  # sample minimum
    y = x[:, 2] + 0.3 * torch.randn((B,), generator=g, device=DEVICE)
    rng = np.random.default_rng(seed)
    w = np.zeros(4801, np.float32)
    w[:512] = rng.normal(0.0, math.sqrt(2.0 / 8), 512)
    w[576:4672] = rng.normal(0.0, math.sqrt(2.0 / 64), 4096)
    w[4736:4800] = rng.normal(0.0, math.sqrt(1.0 / 64), 64)
    w[4800] = -2.0
    return x.contiguous(), y.contiguous(), w


def prepare(case, seed):
    kind = case["kind"]
    if kind == "select":
        return dict(kind=kind, h=knn.handle(), x=_matrix(case, seed), k=case["k"], pivot=case["pivot"])
    if kind == "search":
        q, c = _search_points(case, seed)
        return dict(kind=kind, h=knn.handle(), q=q, c=c, graph=case["graph"], k=case["k"],
                    opt=dict(precision=case["precision"], metric=case["metric"]))
    if kind == "batch":
        # a program that replays a batch keeps its handle, its inputs and its
        # result buffers (here: slices of two arrays)
        jobs = _job_points(case, seed)
        total = sum(q.shape[0] * k for q, _, k in jobs)
        dist = torch.empty((total,), dtype=torch.float32, device=DEVICE)
        idx = torch.empty((total,), dtype=torch.int32, device=DEVICE)
        out, o = [], 0
        for q, _, k in jobs:
            e = o + q.shape[0] * k
            out.append((dist[o:e].view(-1, k), idx[o:e].view(-1, k)))
            o = e
        return dict(kind=kind, h=knn.Handle(0), jobs=jobs, out=out, dist=dist, idx=idx,
                    opt=dict(precision=case["precision"]))
    if kind == "host":
        q, c = _search_points(case, seed)
        host = torch.empty(c.shape, dtype=torch.float32, pin_memory=True)
        host.copy_(c)
        return dict(kind=kind, h=knn.handle(), q=q, c=host, k=case["k"], part_rows=case["part_rows"],
                    opt=dict(precision=case["precision"]))
    x, y, w = _pivot_inputs(case, seed)
    h = knn.Handle(0, pivot_weights=None)
    h.pivot_set_weights(w)
    return dict(kind=kind, h=h, x=x, y=y, quantile=case["quantile"])


def run(state):
    kind, h = state["kind"], state["h"]
    if kind == "select":
        return h.select_k(state["x"], state["k"], pivot=state["pivot"])
    if kind == "search":
        if state["graph"]:
            return h.graph(state["c"], state["k"], **state["opt"])
        return h.search(state["q"], state["c"], state["k"], **state["opt"])
    if kind == "batch":
        h.batch_search(state["jobs"], out=state["out"], **state["opt"])
        return state["dist"], state["idx"]
    if kind == "host":
        return h.search_host_corpus(state["q"], state["c"], state["k"], part_rows=state["part_rows"], **state["opt"])
    return h.pivot_grad(state["x"], state["y"], state["quantile"])


def work(case):
    """Inputs read once, outputs written once; 2 m n d flops per product."""
    kind = case["kind"]
    if kind == "select":
        return dict(bytes=4.0 * case["rows"] * case["cols"] + 8.0 * case["rows"] * case["k"], flops=0.0)
    if kind == "search":
        m, n, d = case["m"], case["n"], case["d"]
        pts = n if case["graph"] else n + m
        return dict(bytes=4.0 * pts * d + 8.0 * m * case["k"], flops=2.0 * m * n * d)
    if kind == "batch":
        m = case["m"]
        return dict(bytes=sum(4.0 * (n + m) * d + 8.0 * m * k for n, d, k, _ in _jobs(case)),
                    flops=sum(2.0 * m * n * d for n, d, k, _ in _jobs(case)))
    if kind == "host":
        m, n, d = case["m"], case["n"], case["d"]
        return dict(bytes=4.0 * (n + m) * d + 8.0 * m * case["k"], flops=2.0 * m * n * d)
    # forward, and the gradients of the weights and of the hidden layers
    return dict(bytes=case["batch"] * 36.0 + 4801 * 8.0, flops=case["batch"] * 2.0 * (2 * 8 * 64 + 3 * 64 * 64 + 3 * 64))


# ---- the same in 64 bits ---------------------------------------------------------
def _knn64(q, c, k, metric, graph):
    """Ascending distances to the k nearest corpus rows, FP64; rows beyond the
    corpus are +inf."""
    q64, c64 = q.double(), c.double()
    if metric == "pearson":
        q64, c64 = q64 - q64.mean(1, keepdim=True), c64 - c64.mean(1, keepdim=True)
    if metric != "sqeuclidean":
        q64, c64 = q64 / q64.norm(dim=1, keepdim=True), c64 / c64.norm(dim=1, keepdim=True)
    n = c64.shape[0]
    ct, cn = c64.t().contiguous(), (c64 * c64).sum(1)
    kk = min(k, n)
    out = torch.full((q64.shape[0], k), float("inf"), dtype=torch.float64, device=DEVICE)
    step = max(1, (1 << 28) // n)
    for i in range(0, q64.shape[0], step):
        b = q64[i:i + step]
        dist = torch.mm(b, ct).mul_(-2.0).add_(cn).add_((b * b).sum(1)[:, None])
        if graph:
            r = torch.arange(b.shape[0], device=DEVICE)
            dist[r, r + i] = float("inf")
        out[i:i + step, :kk] = torch.topk(dist, kk, dim=1, largest=False, sorted=True).values
    return out if metric == "sqeuclidean" else 0.5 * out


def exact(case, seed):
    kind = case["kind"]
    if kind == "select":
        x = _matrix(case, seed)
        step = max(1, (1 << 28) // case["cols"])
        vals = [torch.topk(x[i:i + step].double(), case["k"], dim=1, largest=False, sorted=True).values
                for i in range(0, case["rows"], step)]
        return torch.cat(vals), None
    if kind in ("search", "host"):
        q, c = _search_points(case, seed)
        return _knn64(q, c, case["k"], case.get("metric", "sqeuclidean"), case.get("graph", False)), None
    if kind == "batch":
        return torch.cat([_knn64(q, c, k, "sqeuclidean", False).reshape(-1)
                          for q, c, k in _job_points(case, seed)]), None
    x, y, w = _pivot_inputs(case, seed)
    w = torch.from_numpy(w).bfloat16().double().to(DEVICE)
    x, y, quantile = x.double(), y.double(), case["quantile"]
    w1, b1 = w[:512].view(64, 8), w[512:576]
    w2, b2 = w[576:4672].view(64, 64), w[4672:4736]
    w3, b3 = w[4736:4800], w[4800]
    z1 = torch.mm(x, w1.t()) + b1
    h1 = z1.clamp_min(0.0)
    z2 = torch.mm(h1, w2.t()) + b2
    h2 = z2.clamp_min(0.0)
    u = y - (torch.mv(h2, w3) + b3)
    loss = torch.where(u >= 0, quantile * u, (quantile - 1.0) * u).mean()
    dy = torch.where(u > 0, -quantile, torch.where(u < 0, 1.0 - quantile, 0.0)).double() / x.shape[0]
    d2 = dy[:, None] * w3 * (z2 > 0)
    d1 = torch.mm(d2, w2) * (z1 > 0)
    grad = torch.cat([torch.mm(d1.t(), x).reshape(-1), d1.sum(0), torch.mm(d2.t(), h1).reshape(-1), d2.sum(0),
                      torch.mv(h2.t(), dy), dy.sum()[None]])
    return grad, loss[None]
