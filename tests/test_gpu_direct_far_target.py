"""A target's direct sum does not depend on the other targets of the call: with
targets beyond the fast pair's range (2^400 and more), infinite or NaN
coordinates among the 64 that share a block, the others' results keep every bit."""
import sys

import numpy as np
import pytest

from paper_1907_02289_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps", [0.0, 1e-4])
@pytest.mark.parametrize("far", [2.0 ** 400, 2.0 ** 450, 1e200, np.inf, np.nan])
def test_far_target_beside_others(far, eps):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02289_amd import bh
    print(f"[gpu] direct sum with a target at {far:g}, eps={eps:g}", flush=True)
    sys.stdout.flush()
    # the far particle is the last of 4097: alone in its chunk's last tile, so that the others' tiles stay in range
    s = inputs.plummer(4097, 93)
    s.x[4096] = far
    s.m[4096] = 0.0
    dev = bh.to_device(s)
    ctx = bh.Context(theta=0.5, eps=eps)

    def run(tg):
        tg = np.asarray(tg, np.int64)
        out = {k: torch.zeros(tg.size, dtype=torch.float64, device="cuda") for k in ("ax", "ay", "az")}
        ctx.direct_sum(dev, torch.as_tensor(tg, device="cuda"), out)
        return np.stack([out[k].cpu().numpy() for k in ("ax", "ay", "az")])

    near = np.arange(0, 4000, 67)
    assert near.size < 64
    alone = run(near)
    beside = run(np.concatenate([near[:20], [4096], near[20:]]))
    np.testing.assert_array_equal(np.delete(beside, 20, axis=1), alone)
    ctx.close()
