"""The re-rank reads only the candidates that can be among the k nearest.  With
k = n every corpus point is a candidate and none is left out, so the first k
columns of that result are what a smaller k must return, bit for bit: also for
queries so far from the corpus that the direct form's rounding decides the
order, and for duplicates and non-finite points."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["near", "far", "dups", "nonfinite"])
@pytest.mark.parametrize("n,d", [(1000, 64), (1024, 37), (700, 300)])
def test_pruned_rerank_is_a_prefix(kind, n, d):
    import torch
    import paper_1309_5478_amd as knn
    h = knn.Handle(0)
    r = np.random.default_rng(n + d)
    C = r.normal(0, 1, (n, d)).astype(np.float32)
    Q = r.normal(0, 1, (300, d)).astype(np.float32)
    if kind == "far":
        Q += 3000.0
    elif kind == "dups":
        C = C[r.integers(0, n // 8, n)]
        Q[:100] = C[:100]
    elif kind == "nonfinite":
        C[7, 1], Q[5, 0] = np.inf, np.nan
    Q, C = torch.from_numpy(Q).cuda(), torch.from_numpy(C).cuda()
    full = [x.cpu().numpy().view(np.uint32) for x in h.search(Q, C, n)]
    for k in (1, 8, 64):
        print(kind, n, d, k, flush=True)
        for flags in (0, 2):  # fused, unfused
            got = [x.cpu().numpy().view(np.uint32) for x in h.search(Q, C, k, flags=flags)]
            for f, g in zip(full, got):
                assert np.array_equal(f[:, :k], g)
