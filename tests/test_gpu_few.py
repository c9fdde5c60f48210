"""A few queries against the corpus: their distance rows in one pass (few.hip)
against the fused path (KNN_FEW=0).  FP32 results are the exact k nearest by the
FP32 direct-form distance on either path, so they agree bit for bit."""
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# query tiles of 16 (remainders, each number of tiles, several passes), corpus
# rows not a multiple of a tile, d below a load, odd, at the ends of a step, long;
# rows that one workgroup selects and rows cut in parts; k up to 300
SHAPES = [(1, 2100, 1, 1), (1, 300001, 3, 10), (15, 4099, 17, 5), (16, 20011, 128, 300), (17, 70001, 129, 10),
          (33, 5000, 255, 64), (64, 100003, 48, 7), (65, 9001, 300, 16), (127, 30007, 100, 20), (50, 3001, 1030, 9),
          (96, 2600, 768, 3)]


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
    os.environ["KNN_FEW"] = "0"
    try:
        b = fn()
    finally:
        del os.environ["KNN_FEW"]
    for x, y in zip(a, b):
        assert np.array_equal(x.cpu().numpy().view(np.uint32), y.cpu().numpy().view(np.uint32))


@pytest.mark.parametrize("m,n,d,k", SHAPES)
def test_few_queries_match_fused(h, torch, m, n, d, k):
    import paper_1309_5478_amd as knn
    print(f"few {m}x{n}x{d} k={k}", flush=True)
    r = np.random.default_rng(n + d)
    C = r.normal(0, 1, (n, d)).astype(np.float32)
    C[n // 2:n // 2 + 40] = C[:40]                     # duplicates
    Q = np.concatenate([C[:m // 2], r.normal(0, 1, (m - m // 2, d)).astype(np.float32)])
    Q, C = torch.from_numpy(Q).cuda(), torch.from_numpy(C).cuda()
    both(lambda: h.search(Q, C, k))
    if d > 1:
        both(lambda: h.search(Q, C, k, metric="cosine"))
    both(lambda: h.search(Q, C, k, pivot="plain", flags=knn.FLAG_FORCE_RERUN))


def test_few_queries_nonfinite(h, torch):
    r = np.random.default_rng(3)
    Q, C = r.normal(0, 1, (20, 70)).astype(np.float32), r.normal(0, 1, (9000, 70)).astype(np.float32)
    C[5, 3], C[4000, 0], C[8999, 69], Q[7, 1], Q[19, 0] = np.inf, np.nan, -np.inf, np.nan, np.inf
    Q, C = torch.from_numpy(Q).cuda(), torch.from_numpy(C).cuda()
    both(lambda: h.search(Q, C, 6))


def test_few_queries_partition_of_larger_corpus(h, torch):
    """Rows of a corpus that do not begin on a 16-byte boundary."""
    r = np.random.default_rng(4)
    C = torch.from_numpy(r.normal(0, 1, (20001, 37)).astype(np.float32)).cuda()[1:]
    Q = torch.from_numpy(r.normal(0, 1, (9, 37)).astype(np.float32)).cuda()
    both(lambda: h.search(Q, C, 12))
