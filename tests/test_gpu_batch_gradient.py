"""The batch gradient at its tile edges: batches of 1, around one block's 64
samples, around the 256 blocks' first round (16384) and the largest, and with
a non-finite row outside the batch.  Against FP64 autograd of the same
network: a sum of B products in FP32, in any order, is within B u sum|terms|
of the exact sum (u = 2^-24), the terms themselves (chains of at most 37 and
33 multiply-adds) within 128 u of their own magnitudes; the bar takes both on
the sum of magnitudes with the blocked order's chain length (64 rows, 16-row
matrix sums, 256 partials) instead of B."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def _weights(seed, bh):
    r = np.random.default_rng(seed)
    w = np.zeros(bh.MLP_NPARAM, np.float32)
    w[:1249] = 0.3 * r.standard_normal(1249)
    w[1249:1253] = r.standard_normal(4)
    w[1253:1257] = r.uniform(0.5, 2.0, 4)
    w[1257], w[1258] = -3.0, 2.0
    return w


def _reference(w, X, Y):
    """Gradient and loss in FP64, and the sum over the batch of the magnitudes of every parameter's terms
    (each factor replaced by the sum of the magnitudes that make it up)."""
    w = w.astype(np.float64)
    W1, b1, W2, b2, W3, b3 = (w[:128].reshape(32, 4), w[128:160], w[160:1184].reshape(32, 32), w[1184:1216],
                              w[1216:1248], w[1248])
    x = (X.astype(np.float64) - w[1249:1253]) * w[1253:1257]
    xa = (np.abs(X) + np.abs(w[1249:1253])) * w[1253:1257]
    z1, z1a = x @ W1.T + b1, xa @ np.abs(W1).T + np.abs(b1)
    h1 = np.maximum(z1, 0)
    z2, z2a = h1 @ W2.T + b2, z1a @ np.abs(W2).T + np.abs(b2)
    h2 = np.maximum(z2, 0)
    out, outa = h2 @ W3 + b3, z2a @ np.abs(W3) + np.abs(b3)
    r = out - (Y.astype(np.float64) - w[1257]) / w[1258]
    ra = outa + (np.abs(Y) + abs(w[1257])) / w[1258]
    B = X.shape[0]
    go, goa = 2 * r / B, 2 * ra / B
    g2, g2a = (z2 > 0) * go[:, None] * W3, (z2 > 0) * goa[:, None] * np.abs(W3)
    g1, g1a = (z1 > 0) * (g2 @ W2), (z1 > 0) * (g2a @ np.abs(W2))
    cat = lambda a, xx, b, h, hh, g: np.concatenate([(a.T @ xx).ravel(), a.sum(0), (b.T @ h).ravel(), b.sum(0),
                                                     hh.T @ g, [g.sum()]])
    return (cat(g1, x, g2, h1, h2, go), (r * r).mean(), cat(g1a, xa, g2a, z1a, z2a, goa), (ra * ra).mean())


@pytest.mark.parametrize("B", [1, 2, 63, 64, 65, 127, 4096, 16383, 16385, 65536])
def test_gradient_of_batch_sizes(B):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02289_amd import bh
    print(f"[gpu] batch gradient B={B}", flush=True)
    sys.stdout.flush()
    r = np.random.default_rng(B)
    w = _weights(3, bh)
    X = r.standard_normal((B, 4)).astype(np.float32)
    Y = r.standard_normal(B).astype(np.float32)
    ctx = bh.Context(criterion=bh.LEARNED, precision=bh.FP32_REL)
    ctx.mlp_weights(set=w)
    grad, loss = ctx.mlp_gradient(torch.as_tensor(X, device="cuda"), torch.as_tensor(Y, device="cuda"))
    g, l, mag, lmag = _reference(w, X, Y)
    # samples whose pre-activations lie within rounding of zero may take the other branch: none in these seeds
    tol = (128 + 64 + 16 + 64 + 16) * U * mag + 1e-30
    assert np.all(np.abs(grad.cpu().numpy() - g) <= tol), float(np.max(np.abs(grad.cpu().numpy() - g) / mag) / U)
    assert abs(float(loss.cpu()[0]) - l) <= 256 * U * lmag
    ctx.close()


def test_rows_outside_the_batch_do_not_matter():
    """Training of a batch smaller than a block with a non-finite first row that the shuffle leaves out."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02289_amd import bh
    print("[gpu] batch gradient: non-finite row outside the batch", flush=True)
    sys.stdout.flush()
    r = np.random.default_rng(8)
    X = r.standard_normal((40, 4)).astype(np.float32)
    Y = r.standard_normal(40).astype(np.float32)
    X[0] = np.inf
    ctx = bh.Context(criterion=bh.LEARNED, precision=bh.FP32_REL)
    ctx.mlp_weights(set=_weights(4, bh))
    left_out = 0
    for seed in range(6):
        ctx.mlp_set_dataset(X, Y)
        ctx.mlp_weights(set=_weights(4, bh))
        ctx.mlp_train(iters=1, batch=10, seed=seed, init=False)
        left_out += bool(np.all(np.isfinite(ctx.mlp_weights())))
    # a batch of 10 of 40 rows leaves row 0 out with probability 3/4: all six including it has probability 2e-4
    assert left_out >= 1
    ctx.close()
