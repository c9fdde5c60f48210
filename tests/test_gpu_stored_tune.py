"""Autotuning a search over a short corpus: its rows stay stored, with the tile
shape of their product measured and recorded, and the results stay the same."""
import os

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


# graphs and searches, two-half operands and not, several blocks of rows, d odd (of
# lengths of their own: a choice is kept for the process)
@pytest.mark.parametrize("m,n,d,k,prec", [(0, 5003, 101, 16, "fp32"), (3000, 7001, 68, 8, "fp32"), (300, 9001, 35, 20, "fp32"),
                                          (70000, 4001, 66, 3, "fp32"), (500, 6007, 203, 7, "bf16"), (0, 4099, 79, 9, "fp8")])
def test_short_corpus(tmp_path, m, n, d, k, prec):
    import paper_1309_5478_amd as knn
    h = knn.Handle(0)
    r = np.random.default_rng(n)
    C = torch.from_numpy(r.normal(0, 1, (n, d)).astype(np.float32)).cuda()
    Q = torch.from_numpy(r.normal(0, 1, (max(m, 1), d)).astype(np.float32)).cuda()

    def run(**kw):
        out = h.search(Q, C, k, precision=prec, **kw) if m else h.graph(C, k, precision=prec, **kw)
        return [x.cpu().numpy().view(np.uint32) for x in out], h.stats()["candidates_total"]
    want, cands = run()
    assert cands == (m or n) * 4 * k                     # stored rows
    path = str(tmp_path / "tune.json")
    os.environ["KNN_AUTOTUNE_CACHE"] = path
    try:
        for rep in range(2):                             # measured, then looked up
            got, c = run(flags=knn.FLAG_AUTOTUNE)
            assert c == cands
            for a, b in zip(got, want):
                assert np.array_equal(a, b)
    finally:
        del os.environ["KNN_AUTOTUNE_CACHE"]
    assert any("|stored" in line for line in open(path))
