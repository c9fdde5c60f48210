"""The tiled gradient pass of the pivot network at the edges of its tiles of 16
samples and of its grid of 256 workgroups, against the FP64 oracle.

Tolerance, per parameter: FP32 sums of at most 64 (units), 16 (a tile), 17
(tiles of a workgroup) and 40 (partial rows) terms in a fixed order, after
layers with relative errors of at most 73 roundings: below 256 * 2^-24 of the
sum of the terms' magnitudes."""
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
    theta = (rng.normal(0, 1, mlp.NPARAM) * 0.2).astype(np.float32)
    h.pivot_set_weights(theta)
    X = rng.normal(0, 1, (B, 8)).astype(np.float32)
    y = rng.normal(0, 2, B).astype(np.float32)
    g, loss = h.pivot_grad(torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda(), 0.9)
    g, loss = g.cpu().numpy().astype(np.float64), float(loss.cpu()[0])
    th = mlp.bf16_round(theta)
    want_loss, want = mlp.loss_and_grad(th, X, y, 0.9)
    # magnitudes of the summed terms
    W1, b1, W2, b2, w3, b3 = mlp.split(th)
    yh, (Xd, z1, h1, z2, h2) = mlp.forward(th, X)
    u = y - yh
    dy = np.where(u > 0, 0.9, 0.1) / B
    a2 = np.outer(dy, np.abs(w3)) * (z2 > 0)
    a1 = (a2 @ np.abs(W2)) * (z1 > 0)
    mag = np.concatenate([(a1.T @ np.abs(Xd)).ravel(), a1.sum(0), (a2.T @ h1).ravel(), a2.sum(0), h2.T @ dy,
                          [dy.sum()]])
    eps = 256 * 2.0 ** -24
    assert np.all(np.abs(g - want) <= eps * mag + 1e-30)
    mean_mag = np.mean(np.abs(u) + np.abs(yh) + np.abs(y))
    assert abs(loss - want_loss) <= eps * mean_mag
    # the sums are in a fixed order: the same call gives the same bits
    g2, _ = h.pivot_grad(torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda(), 0.9)
    assert np.array_equal(g2.cpu().numpy().astype(np.float64), g)
