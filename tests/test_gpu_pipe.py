"""The pipelined 256 x 256 product (gemm_pipe.hip) against the paths it stands
in for.

FP32 results are the exact k nearest by the FP32 direct-form distance whatever
product ranks the candidates, so the product on two-half operands and the FP32
matrix instruction (KNN_GEMM_SPLIT=0) must agree bit for bit, on every kind of
data.  BF16 and FP8 form the same key bits on either tile (KNN_GEMM_PIPE=0)."""
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def filtered():
    """Short corpora too on the filtered path (their distance rows are stored
    otherwise: test_gpu_dense.py)."""
    os.environ["KNN_DENSE"] = "0"
    yield
    del os.environ["KNN_DENSE"]


@pytest.fixture(scope="module")
def torch():
    import torch as t
    return t


@pytest.fixture(scope="module")
def h(torch):
    import paper_1309_5478_amd as knn
    return knn.Handle(0)


def points(kind, n, d, seed):
    r = np.random.default_rng(seed)
    if kind == "uniform":
        return r.random((n, d), dtype=np.float32)
    x = r.normal(0, 1, (n, d)).astype(np.float32)
    if kind == "gmm":
        mu = (2 * r.normal(0, 1, (16, d))).astype(np.float32)
        return x + mu[r.integers(0, 16, n)]
    if kind == "lognormal":              # magnitudes over many binades
        return (np.exp(3 * x) * np.sign(r.normal(0, 1, (n, d)))).astype(np.float32)
    if kind == "scales":                 # points of very different norms, zero points
        x *= np.exp2(r.integers(-40, 40, (n, 1))).astype(np.float32)
        x[::97] = 0.0
        return x
    if kind == "dups":                   # many exact duplicates
        return x[r.integers(0, max(n // 5, 1), n)]
    assert kind == "nonfinite"
    x[5, 3], x[n // 2, 0], x[n - 1, d - 1] = np.inf, np.nan, -np.inf
    return x


def both(env, off, fn):
    a = fn()
    was = os.environ.get(env)
    os.environ[env] = off
    try:
        b = fn()
    finally:
        if was is None:
            del os.environ[env]
        else:
            os.environ[env] = was
    return a, b


def same(a, b):
    for x, y in zip(a, b):
        assert np.array_equal(x.cpu().numpy().view(np.uint32), y.cpu().numpy().view(np.uint32))


# (m, n, d, k): row and column remainders of a tile, the smallest d and m, odd d,
# one k-chunk and a ragged last one, lists that overflow (k = 256 of 20011)
SHAPES = [(4096, 4099, 64, 5), (128, 49153, 65, 3), (129, 60001, 100, 10), (257, 30000, 128, 16),
          (4097, 5003, 96, 33), (1000, 20011, 64, 256), (700, 40000, 1000, 20)]


@pytest.mark.parametrize("kind", ["uniform", "gmm", "lognormal", "scales", "dups", "nonfinite"])
@pytest.mark.parametrize("m,n,d,k", SHAPES[:2])
def test_split_matches_fp32_kinds(h, torch, kind, m, n, d, k):
    print(f"split {kind} {m}x{n}x{d} k={k}", flush=True)
    Q = torch.from_numpy(points(kind, m, d, 1)).cuda()
    C = torch.from_numpy(points(kind, n, d, 2)).cuda()
    a, b = both("KNN_GEMM_SPLIT", "0", lambda: h.search(Q, C, k))
    same(a, b)


@pytest.mark.parametrize("m,n,d,k", SHAPES[2:])
def test_split_matches_fp32_shapes(h, torch, m, n, d, k):
    print(f"split {m}x{n}x{d} k={k}", flush=True)
    Q = torch.from_numpy(points("gmm", m, d, 3)).cuda()
    C = torch.from_numpy(points("gmm", n, d, 4)).cuda()
    for metric in ("sqeuclidean", "pearson"):
        a, b = both("KNN_GEMM_SPLIT", "0", lambda: h.search(Q, C, k, metric=metric))
        same(a, b)


@pytest.mark.parametrize("graph", [False, True])
def test_split_in_column_blocks(h, torch, graph):
    """Split operands capped at 5 blocks of the corpus's columns (with a ragged
    last one): the same result, own points excluded in every block."""
    n, d, k = 20011, 96, 12
    P = torch.from_numpy(points("dups", n, d, 5)).cuda()
    Q = torch.from_numpy(points("dups", 3000, d, 6)).cuda()
    run = (lambda: h.graph(P, k)) if graph else (lambda: h.search(Q, P, k))
    a, b = both("KNN_SPLIT_BYTES", str(4352 * 384), run)
    same(a, b)
    a, b = both("KNN_GEMM_SPLIT", "0", run)
    same(a, b)


@pytest.mark.parametrize("prec", ["bf16", "fp8"])
@pytest.mark.parametrize("n,d,k", [(4099, 64, 5), (5003, 129, 33), (20011, 200, 256), (9000, 700, 16)])
def test_low_precision_matches_small_tiles(h, torch, prec, n, d, k):
    print(f"{prec} graph {n}x{d} k={k}", flush=True)
    P = torch.from_numpy(points("gmm", n, d, 7)).cuda()
    a, b = both("KNN_GEMM_PIPE", "0", lambda: h.graph(P, k, precision=prec))
    same(a, b)


def test_batch_split_matches_fp32(torch):
    """Uneven FP32 jobs (graphs, odd d, few rows, tiny corpora among them) in one
    batch: the pipelined grouped products and the FP32 ones give the same bits,
    on the first call and on a replay with new values in the same buffers."""
    import paper_1309_5478_amd as knn
    shapes = [(300, 9000, 64, 7), (128, 30011, 96, 300), (1024, 5003, 65, 1), (50, 20000, 128, 10),
              (None, 4111, 72, 12), (257, 1500, 64, 16), (200, 700, 33, 900), (0, 5000, 64, 3)]

    def run(split):
        h = knn.Handle(0)
        jobs, res = [], []
        for s, (m, n, d, k) in enumerate(shapes):
            q = None if m is None else torch.from_numpy(points("gmm", m, d, 50 + s)).cuda()
            jobs.append((q, torch.from_numpy(points("gmm", n, d, 80 + s)).cuda(), k))
        out = [(torch.empty(((n if m is None else m), k), device="cuda"),
                torch.empty(((n if m is None else m), k), dtype=torch.int32, device="cuda"))
               for m, n, d, k in shapes]
        if not split:
            os.environ["KNN_GEMM_SPLIT"] = "0"
        try:
            for call in range(3):
                if call == 2:
                    for s, (q, c, k) in enumerate(jobs):
                        c.copy_(torch.from_numpy(points("gmm", c.shape[0], c.shape[1], 180 + s)))
                h.batch_search(jobs, out=out)
                res.append([(a.clone(), b.clone()) for a, b in out])
        finally:
            os.environ.pop("KNN_GEMM_SPLIT", None)
        return res

    for x, y in zip(run(True), run(False)):
        for a, b in zip(x, y):
            same(a, b)


# few tiles (24 and just above), more kept keys than a wave's list holds in one
# tile (kk = 1024 of 6145: a sixth or more of all), lists that stay open over many
# column tiles, and a last row tile of one row
@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp8"])
@pytest.mark.parametrize("m,n,d,k", [(130, 6145, 256, 256), (513, 2100, 64, 200), (140, 70001, 64, 3)])
def test_few_tiles_and_key_lists(h, torch, prec, m, n, d, k):
    import paper_1309_5478_amd as knn
    print(f"{prec} {m}x{n}x{d} k={k}", flush=True)
    Q = torch.from_numpy(points("gmm", m, d, 11)).cuda()
    C = torch.from_numpy(points("gmm", n, d, 12)).cuda()
    env = "KNN_GEMM_SPLIT" if prec == "fp32" else "KNN_GEMM_PIPE"
    a, b = both(env, "0", lambda: h.search(Q, C, k, precision=prec))
    same(a, b)
    same(h.search(Q, C, k, precision=prec, flags=knn.FLAG_AUTOTUNE), b)


@pytest.mark.parametrize("prec", ["bf16", "fp8"])
def test_batch_low_precision_matches_small_tiles(torch, prec):
    import paper_1309_5478_amd as knn
    shapes = [(300, 9000, 64, 7), (65, 30011, 96, 256), (64, 5003, 65, 1), (None, 4111, 200, 12), (200, 700, 33, 90)]
    jobs = [(None if m is None else torch.from_numpy(points("gmm", m, d, 21 + s)).cuda(),
             torch.from_numpy(points("gmm", n, d, 31 + s)).cuda(), k) for s, (m, n, d, k) in enumerate(shapes)]
    a, b = both("KNN_GEMM_PIPE", "0", lambda: knn.Handle(0).batch_search(jobs, precision=prec))
    for x, y in zip(a, b):
        same(x, y)


# resident rows: row tiles of 512 (remainders, fewer rows than a wave's), an XCD
# without columns, column remainders, both row lengths and a half-used one, lists
# that overflow in a step (kk = 1024 of 3000), d at the ends of each form
@pytest.mark.parametrize("prec,d", [("fp8", 128), ("fp8", 129), ("fp8", 256), ("fp8", 20), ("bf16", 64), ("bf16", 65),
                                    ("bf16", 128), ("bf16", 17)])
@pytest.mark.parametrize("m,n,k", [(513, 20011, 7), (40, 3000, 256), (5003, 2100, 60), (0, 9001, 12)])
def test_resident_rows_match_tiles(h, torch, prec, d, m, n, k):
    print(f"rows {prec} {m}x{n}x{d} k={k}", flush=True)
    C = points("scales" if d == 129 else "gmm", n, d, 41)
    Q = torch.from_numpy(points("gmm", m, d, 42)).cuda()
    C = torch.from_numpy(C).cuda()
    run = (lambda: h.search(Q, C, k, precision=prec)) if m else (lambda: h.graph(C, k, precision=prec))
    os.environ["KNN_GEMM_ROWS"] = "1"
    try:
        a, b = both("KNN_GEMM_ROWS", "0", run)
    finally:
        os.environ.pop("KNN_GEMM_ROWS", None)
    same(a, b)
