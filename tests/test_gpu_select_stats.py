"""Row statistics of selections held on chip whole (sample pivots, 1025 to 16384
columns) and of the parts of few long rows: the fields that the streamed
selection fills are filled."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def run(D, k):
    import torch
    import paper_1309_5478_amd as knn
    h = knn.Handle(0)
    h.select_k(torch.from_numpy(D).cuda(), k)
    return h.stats()


@pytest.mark.parametrize("rows,cols,k", [(300, 4096, 10), (70, 1500, 200), (2000, 16384, 64), (8, 300007, 32)])
def test_cycles_of_every_phase(rows, cols, k):
    D = np.random.default_rng(cols).random((rows, cols), dtype=np.float32)
    st = run(D, k)
    print(rows, cols, k, st, flush=True)
    assert st["rows"] == rows
    sorted_whole = cols <= 2016 and k > 128            # (no pivot)
    for i, c in enumerate(st["phase_cycles"]):
        assert c > 0 or (i == 0 and sorted_whole), (i, c)
    assert max(st["phase_cycles"]) < 1 << 50


def test_passes_over_rows_whose_survivors_do_not_fit():
    """Rows of distinct values need no pass beyond the first; a row of which half
    is the k-th value is counted over again."""
    r = np.random.default_rng(1)
    D = r.random((40, 8192), dtype=np.float32)
    assert run(D, 20)["passes_total"] == 0
    D[::2] = np.where(r.random((20, 8192)) < 0.5, np.float32(0), D[::2])
    st = run(D, 20)
    assert 20 <= st["passes_total"] <= 20 * 64 and 1 <= st["passes_max"] <= 64
    assert st["passes_total"] <= 20 * st["passes_max"]
