"""Rows of 1025 to 16384 columns (held on chip whole) and the parts of few long
rows, bit for bit against the oracle: at the edges of the instances (4096, 8192,
16384 columns), of the group counts (k = 128, 256, 512) and of the rows sorted
whole (2016), with ragged and misaligned rows, and with rows whose survivors do
not fit (ties at the pivot, NaN, signed zeros), which are cut at their exact k-th
key."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def check(D, k, offset=0, ld_pad=0, flags=0):
    import torch
    import paper_1309_5478_amd as knn
    h = knn.handle()
    R, C = D.shape
    print(f"select {R}x{C} k={k} offset={offset} pad={ld_pad}", flush=True)
    host = np.full(offset + R * (C + ld_pad), -1e30, np.float32)  # (a read beyond a row would win)
    host[offset:].reshape(R, C + ld_pad)[:, :C] = D
    dev = torch.from_numpy(host).cuda()
    v, i = h.select_k(dev[offset:].view(R, C + ld_pad)[:, :C], k, flags=flags)
    ov, oi = oracle.select_k(D, k)
    assert np.array_equal(i.cpu().numpy(), oi)
    assert np.array_equal(v.cpu().numpy().view(np.uint32), ov.view(np.uint32))
    st = h.stats()
    assert st["rows"] == R


@pytest.mark.parametrize("cols", [1025, 2016, 2017, 2048, 4095, 4096, 4099, 8192, 8193, 16381, 16384, 16385])
@pytest.mark.parametrize("ks", [(1, 4, 5, 64, 65), (127, 128, 129, 255), (256, 257, 511, 512, 513)])
def test_edges(cols, ks):
    r = np.random.default_rng(cols)
    D = r.normal(0, 1, (9, cols)).astype(np.float32)
    for k in ks:
        check(D, k)
    check(D, ks[0], offset=1, ld_pad=3)
    check(D, ks[-1], offset=3, ld_pad=0)


@pytest.mark.parametrize("cols", [1500, 4096, 10007, 16384])
def test_ties_and_classes(cols):
    rows = synth.adversarial_rows(cols, seed=cols)
    D = np.stack([rows[n] for n in sorted(rows)])
    for k in (1, 10, 128, 200, 512):
        check(D, k)


@pytest.mark.parametrize("rows,cols", [(1, 16385), (1, 70001), (5, 300007), (8, 1 << 20), (200, 40000)])
def test_few_long_rows(rows, cols):
    r = np.random.default_rng(cols)
    D = r.random((rows, cols), dtype=np.float32)
    D[0, 100:100 + cols // 2] = 0.25      # ties across parts
    for k in (1, 32, 512):
        check(D, k)
