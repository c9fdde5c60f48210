"""FP32 searches on points whose mean is large against their spread, where the
rounding of the reduced keys is large against the gaps between them: the two-half
product leaves no more rows without a certificate than twice the error bound of
the FP32 matrix instruction would, and the rows that are re-run are exact."""
import os

import numpy as np
import pytest

from knn_check import compare

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


@pytest.fixture(scope="module")
def torch():
    import torch as t
    return t


@pytest.fixture(scope="module")
def h(torch):
    import paper_1309_5478_amd as knn
    return knn.Handle(0)


def points(kind, n, d, off, seed):
    r = np.random.default_rng(seed)
    x = r.random((n, d), dtype=np.float32) if kind == "uniform" else r.normal(0, 1, (n, d)).astype(np.float32)
    return x + np.float32(off)


def without_split(fn):
    os.environ["KNN_GEMM_SPLIT"] = "0"
    try:
        return fn()
    finally:
        del os.environ["KNN_GEMM_SPLIT"]


def same(a, b):
    for x, y in zip(a, b):
        assert np.array_equal(x.cpu().numpy().view(np.uint32), y.cpu().numpy().view(np.uint32))


def uncertain(torch, P, k):
    """Rows whose gap between the 4 k-th and the k-th reduced key (FP64, own point
    left out) is at most twice (g + 2u) c2 + 2 (g + 2u) |q| |c|, g = d u / (1 - d u)."""
    x = P.double()
    n, d = x.shape
    c2 = (x * x).sum(1)
    g = d * U / (1 - d * U) + 2 * U
    bad = 0
    for i in range(0, n, 4096):
        b = x[i:i + 4096]
        key = c2 - 2 * torch.mm(b, x.t().contiguous())
        r = torch.arange(b.shape[0], device="cuda")
        key[r, r + i] = float("inf")
        v = torch.topk(key, 4 * k, dim=1, largest=False, sorted=True).values
        E = 1.001 * (g * c2.max() + 2 * g * torch.sqrt(c2[i:i + 4096] * c2.max()))
        bad += int((v[:, -1] - v[:, k - 1] <= 2 * E).sum())
    return bad


# none, some and all rows beyond the bound; stored rows (8000 points) and lists
@pytest.mark.parametrize("n,d,k,kind,off", [(32768, 128, 16, "uniform", 8), (32768, 64, 16, "uniform", 16),
                                            (20000, 1024, 32, "uniform", 2), (20000, 300, 10, "normal", 12),
                                            (8000, 128, 16, "uniform", 8), (8000, 128, 16, "uniform", 24)])
def test_rerun_rows_and_results(h, torch, n, d, k, kind, off):
    host = points(kind, n, d, off, n + d)
    P = torch.from_numpy(host).cuda()
    a = h.graph(P, k)
    st = h.stats()
    most = uncertain(torch, P, k)
    print(f"{n}x{d} k={k} {kind}+{off}: re-run {st['rows_rerun']}, bound {most}", flush=True)
    same(a, without_split(lambda: h.graph(P, k)))
    rows = np.arange(0, n, n // 24)
    compare(host, host, k, a[0].cpu().numpy()[rows], a[1].cpu().numpy()[rows], rows, self_ids=np.arange(n))
    assert st["rows_rerun"] <= most


@pytest.mark.parametrize("d,off,qoff", [(128, 8, 8), (96, 8, 80), (65, 80, 8), (128, 40, 40)])
def test_queries_nearer_and_farther(h, torch, d, off, qoff):
    """Queries as far from the origin as the corpus, ten times nearer and farther,
    from a few to a batch's, forced re-runs among them."""
    import paper_1309_5478_amd as knn
    n, k = 20011, 12
    host, qh = points("normal", n, d, off, 3), points("normal", 300, d, qoff, 4)
    C, Q = torch.from_numpy(host).cuda(), torch.from_numpy(qh).cuda()
    for m in (300, 16):
        q = Q[:m].contiguous()
        a = h.search(q, C, k)
        print(f"{m} x {n} x {d}, {off}/{qoff}: re-run {h.stats()['rows_rerun']}", flush=True)
        same(a, without_split(lambda: h.search(q, C, k)))
        same(a, h.search(q, C, k, flags=knn.FLAG_FORCE_RERUN))
        rows = np.arange(0, m, max(m // 12, 1))
        compare(qh, host, k, a[0].cpu().numpy()[rows], a[1].cpu().numpy()[rows], rows)
        same(h.batch_search([(q, C, k), (q, C[:3000].contiguous(), k)])[0], a)


def test_cut_products(h, torch):
    """One large element per point over 127 small ones, with full mantissas, at
    the distance where the instruction cuts them off its sum."""
    r = np.random.default_rng(9)
    n, d, k = 12000, 128, 8
    for lo in (-9, -10, -11, -12, -13):
        x = np.float32(2.0 ** lo) * (1 + r.integers(0, 1 << 23, (n, d)) / 2.0 ** 23).astype(np.float32)
        x[:, 0] = 1 + r.integers(0, 8, n) / 2.0 ** 20
        P = torch.from_numpy(x).cuda()
        a = h.graph(P, k)
        print(f"2^{lo}: re-run {h.stats()['rows_rerun']}", flush=True)
        same(a, without_split(lambda: h.graph(P, k)))
        rows = np.arange(0, n, 1000)
        compare(x, x, k, a[0].cpu().numpy()[rows], a[1].cpu().numpy()[rows], rows, self_ids=np.arange(n))
