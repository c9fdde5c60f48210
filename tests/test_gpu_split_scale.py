"""Two-half operands of points at the ends of the FP32 range: the products rank
the corpus as the FP32 matrix instruction does (KNN_GEMM_SPLIT=0)."""
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("unit", [-146, -140, -130, -100, 40, 100])
def test_ranking_at_the_ends_of_the_range(unit):
    """One-hot queries, so that a reduced key is one corpus element (its norm
    underflows, or is the same for all points: one element dominates) and exact
    on either product; elements of 20 bits times 2^unit."""
    import torch
    import paper_1309_5478_amd as knn
    h = knn.Handle(0)
    r = np.random.default_rng(6)
    n, d, m, k = 20011, 64, 130, 4
    C = np.ldexp(r.integers(1 << 19, 1 << 20, (n, d)), unit).astype(np.float32)
    if unit > -130:
        C[:, 1:] = 0
    Q = np.zeros((m, d), np.float32)
    Q[np.arange(m), np.arange(m) % (d if unit <= -130 else 1)] = 1.0 if unit < 0 else np.ldexp(1.0, -unit)
    Q, C = torch.from_numpy(Q).cuda(), torch.from_numpy(C).cuda()
    a = h.search(Q, C, k)
    os.environ["KNN_GEMM_SPLIT"] = "0"
    try:
        b = h.search(Q, C, k)
    finally:
        del os.environ["KNN_GEMM_SPLIT"]
    for x, y in zip(a, b):
        assert np.array_equal(x.cpu().numpy().view(np.uint32), y.cpu().numpy().view(np.uint32))
