"""The products of short BF16 / FP8 rows (gemm_rows.hip, gemm_pipe.hip) against the
128 x 128 tiles (KNN_GEMM_PIPE=0): every form makes the same key bits, so the
results agree bit for bit; and against the oracle on points whose products are
exact."""
import os

import numpy as np
import pytest

import synth
from knn_check import compare

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    return t


@pytest.fixture(scope="module")
def h(torch):
    import paper_1309_5478_amd as knn
    return knn.Handle(0)


def run(h, torch, Q, C, k, prec, env):
    old = {v: os.environ.get(v) for v in env}
    os.environ.update(env)
    try:
        d, i = h.graph(C, k, precision=prec) if Q is None else h.search(Q, C, k, precision=prec)
        return d.cpu().numpy(), i.cpu().numpy()
    finally:
        for v, was in old.items():
            if was is None:
                del os.environ[v]
            else:
                os.environ[v] = was


ROWS, TILES = {"KNN_GEMM_ROWS": "1"}, {"KNN_GEMM_PIPE": "0"}


@pytest.mark.parametrize("prec,d", [("bf16", 256), ("bf16", 100), ("bf16", 128), ("fp8", 128), ("fp8", 77),
                                    ("fp8", 256), ("fp8", 200)])
@pytest.mark.parametrize("graph", [False, True])
def test_short_rows_equal_tiled(h, torch, prec, d, graph):
    """Rows no multiple of a tile, mixture data, k from 1 to 300; resident rows where
    the row length allows them (BF16 d <= 128, FP8), the pipelined tiles else."""
    m, n = 3001, 40000 + 37
    C = torch.from_numpy(synth.gmm_points(n, d, seed=71 + d)).cuda()
    Q = None if graph else torch.from_numpy(synth.gmm_points(m, d, seed=72 + d)).cuda()
    for k in (1, 16, 300):
        print(f"{prec} d={d} graph={graph} k={k}", flush=True)
        a = run(h, torch, Q, C, k, prec, ROWS)
        b = run(h, torch, Q, C, k, prec, TILES)
        assert np.array_equal(a[1], b[1])
        assert np.array_equal(a[0].view(np.uint32), b[0].view(np.uint32))


@pytest.mark.parametrize("prec,d", [("bf16", 64), ("bf16", 128), ("bf16", 192), ("fp8", 60), ("fp8", 250)])
def test_lattice_exact(h, torch, prec, d):
    """Integer points: every product is exact in BF16 and e4m3, so the sets and
    distances are the oracle's (massive ties)."""
    rng = np.random.default_rng(5)
    P = rng.integers(0, 8, size=(12000, d)).astype(np.float32)
    P[100:110] = P[5]                      # duplicates at distance 0
    os.environ["KNN_DENSE"] = "0"
    try:
        gd, gi = run(h, torch, None, torch.from_numpy(P).cuda(), 20, prec, ROWS)
    finally:
        del os.environ["KNN_DENSE"]
    rows = np.arange(0, 12000, 397)
    compare(P, P, 20, gd[rows], gi[rows], rows, self_ids=np.arange(12000))
