"""Short corpora, whose distance rows are stored and selected from, against the
filtered path (KNN_DENSE=0): FP32 results are the exact k nearest by the FP32
direct-form distance on either, and the reduced precisions select the same
candidates from the same keys, so the results agree bit for bit."""
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    return t


@pytest.fixture(scope="module")
def h(torch):
    import paper_1309_5478_amd as knn
    return knn.Handle(0)


def both(fn):
    a = fn()
    os.environ["KNN_DENSE"] = "0"
    try:
        b = fn()
    finally:
        del os.environ["KNN_DENSE"]
    for x, y in zip(a, b):
        assert np.array_equal(x.cpu().numpy().view(np.uint32), y.cpu().numpy().view(np.uint32))


# graphs (m = 0) and searches: just above a sample, at the longest corpus of a
# rule and beyond it, several blocks of rows (m n above 2^28 keys), corpora that are
# their own sample, one column above a tile, kk up to 1024, odd d
@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp8"])
@pytest.mark.parametrize("m,n,d,k", [(0, 2049, 64, 4), (0, 4099, 65, 16), (300, 8832, 128, 4), (300, 8833, 128, 4),
                                     (129, 20000, 37, 64), (70000, 4000, 64, 3), (5000, 2000, 200, 250),
                                     (131, 40000, 16, 256), (6000, 1500, 100, 7)])
def test_dense_matches_fused(h, torch, prec, m, n, d, k):
    print(f"dense {prec} {m}x{n}x{d} k={k}", flush=True)
    r = np.random.default_rng(n + d)
    C = r.normal(0, 1, (n, d)).astype(np.float32)
    C[n // 2:n // 2 + 50] = C[:50]                     # duplicates
    Q = r.normal(0, 1, (m, d)).astype(np.float32)
    C, Q = torch.from_numpy(C).cuda(), torch.from_numpy(Q).cuda()
    for kw in ({}, {"metric": "cosine"}, {"pivot": "plain"}):
        both(lambda: h.search(Q, C, k, precision=prec, **kw) if m else h.graph(C, k, precision=prec, **kw))


def test_dense_nonfinite_and_rerun(h, torch):
    import paper_1309_5478_amd as knn
    r = np.random.default_rng(5)
    C = r.normal(0, 1, (5000, 96)).astype(np.float32)
    C[7, 3], C[2500, 0], C[4999, 95] = np.inf, np.nan, -np.inf
    C = torch.from_numpy(C).cuda()
    both(lambda: h.graph(C, 9))
    both(lambda: h.graph(C[100:2400].contiguous(), 9, flags=knn.FLAG_FORCE_RERUN))
