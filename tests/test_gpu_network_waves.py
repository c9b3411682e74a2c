"""The learned rule's network evaluated for 64 inputs at once: counts around a
wave and a block, and weights and inputs with signed zeros, subnormals and very
large values.  Outputs bit-exact against the oracle's chain of fused
multiply-adds."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _weights(kind, rng):
    w = np.zeros(1259, np.float32)
    w[:1249] = rng.normal(0, 0.3, 1249)
    if kind == "scales":
        w[:1249] *= np.float32(2.0) ** rng.integers(-30, 20, 1249).astype(np.float32)
    if kind == "tiny":                    # products and sums in the subnormal range
        w[:1249] *= np.float32(2.0 ** -64)
        w[rng.integers(0, 1249, 100)] = np.float32(-0.0)
        w[rng.integers(128, 1249, 100)] = np.float32(3e-42)
    w[1253:1257] = 0.5
    w[1249:1253] = rng.normal(0, 1, 4)
    w[1257], w[1258] = 0.25, 1.5
    return w


@pytest.mark.parametrize("kind", ["plain", "scales", "tiny"])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 64, 65, 255, 256, 257, 70001])
def test_outputs_bit_exact(n, kind):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02289_amd import bh
    print(f"[gpu] network waves n={n} weights={kind}", flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(n)
    w = _weights(kind, rng)
    X = rng.normal(0, 4, (n, 4)).astype(np.float32)
    X[rng.integers(0, n, max(1, n // 8)), rng.integers(0, 4, max(1, n // 8))] = np.float32(-0.0)
    ctx = bh.Context(theta=0.5, eps=1e-3)
    ctx.mlp_weights(set=w)
    got = ctx.mlp_predict(torch.as_tensor(X, device="cuda")).cpu().numpy()
    np.testing.assert_array_equal(got, oracle.mlp_forward(w, X))
    ctx.close()
