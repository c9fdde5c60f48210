"""The tiled gradient pass of the pivot network at the edges of its tiles of 16
samples and of its grid of 256 workgroups, against the FP64 oracle.

Inputs and weights are small integers (BF16 holds them exactly), so that every
activation, the output and every back-propagated factor but 1 / B is exact in
FP32, and the masks and signs are the oracle's.  What rounds is 1 / B (the
quantile is 1/2), its products and the fixed-order sums: a tile's 16 samples, up to 17
tiles of a workgroup, 32 and 8 partial sums, one rounding each: below 80 * 2^-24
of the sum of the terms' magnitudes."""
import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 15, 16, 17, 4095, 4097, 16 * 256 * 16 + 5])
def test_gradient_tiles(B):
    import torch
    import paper_1309_5478_amd as knn
    h = knn.Handle(0, pivot_weights=None)
    rng = np.random.default_rng(B)
    theta = rng.integers(-1, 2, mlp.NPARAM).astype(np.float32)
    h.pivot_set_weights(theta)
    X = rng.integers(-2, 3, (B, 8)).astype(np.float32)
    y = rng.integers(-40, 41, B).astype(np.float32)
    g, loss = h.pivot_grad(torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda(), 0.5)
    g, loss = g.cpu().numpy().astype(np.float64), float(loss.cpu()[0])
    th = theta.astype(np.float64)
    want_loss, want = mlp.loss_and_grad(th, X, y, 0.5)
    W1, b1, W2, b2, w3, b3 = mlp.split(th)
    yh, (Xd, z1, h1, z2, h2) = mlp.forward(th, X)
    dy = np.where(y != yh, 0.5, 0.0) / B
    d2 = np.outer(dy, np.abs(w3)) * (z2 > 0)
    d1 = (d2 @ np.abs(W2)) * (z1 > 0)
    mag = np.concatenate([(d1.T @ np.abs(Xd)).ravel(), d1.sum(0), (d2.T @ h1).ravel(), d2.sum(0), h2.T @ dy,
                          [dy.sum()]])
    eps = 80 * 2.0 ** -24
    assert np.all(np.abs(g - want) <= eps * mag)
    assert abs(loss - want_loss) <= eps * want_loss
    # the sums are in a fixed order: the same call gives the same bits
    g2, _ = h.pivot_grad(torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda(), 0.5)
    assert np.array_equal(g2.cpu().numpy().astype(np.float64), g)
