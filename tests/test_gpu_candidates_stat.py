"""candidates_total of searches whose keys are stored (few queries, short corpora):
the candidates that each row's selection hands on."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def pts(n, d, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn((n, d), generator=g, device="cuda")


@pytest.mark.parametrize("m,n,d,k,prec,want", [(16, 20011, 64, 10, "fp32", 40), (0, 5000, 96, 16, "fp32", 64),
                                               (3000, 8001, 32, 300, "fp32", 1024), (500, 6000, 200, 7, "bf16", 28)])
def test_stored_rows(m, n, d, k, prec, want):
    import paper_1309_5478_amd as knn
    h = knn.Handle(0)
    C, Q = pts(n, d, 1), pts(max(m, 1), d, 2)
    for rep in range(2):
        h.search(Q, C, k, precision=prec) if m else h.graph(C, k, precision=prec)
        assert h.stats()["candidates_total"] == (m or n) * want
    h.search(Q, C, k, precision=prec, flags=knn.FLAG_UNFUSED) if m else h.graph(C, k, precision=prec, flags=knn.FLAG_UNFUSED)
    assert h.stats()["candidates_total"] == 0


def test_batch_counts_every_job():
    import paper_1309_5478_amd as knn
    h = knn.Handle(0)
    jobs = [(pts(200, 64, 3), pts(6000, 64, 4), 8), (pts(100, 64, 5), pts(1000, 64, 6), 8), (None, pts(4000, 128, 7), 5)]
    for rep in range(2):                                 # (the second corpus is its own sample)
        h.batch_search(jobs)
        assert h.stats()["candidates_total"] == 200 * 32 + 4000 * 20
    jobs.append((pts(300, 64, 8), pts(70000, 64, 9), 8))
    h.batch_search(jobs)
    assert 300 * 32 <= h.stats()["candidates_total"] - (200 * 32 + 4000 * 20) <= 300 * 1024
