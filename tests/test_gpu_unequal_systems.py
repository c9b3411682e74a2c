"""One large system among many small ones: each is loaded, and its root box
taken, by as many blocks as its own size asks for.  The time of keys, sort and
permutation against the large system alone, and keys and root boxes for sizes
around a block's share (1024 particles) against the oracle."""
import sys

import numpy as np
import pytest

import oracle
from paper_1907_02289_amd import inputs

pytestmark = pytest.mark.gpu


def _bh():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02289_amd import bh
    return torch, bh


def _keys_ms(torch, bh, systems):
    ctx = bh.Context(theta=0.5, eps=1e-3, n_leaf=64, n_group=256)
    ms = []
    for _ in range(6):
        ctx.build_tree(systems)
        torch.cuda.synchronize()
        ms.append(ctx.stage_times()["keys_sort"])
    ctx.close()
    return min(ms)


def test_time_of_one_large_system_among_many():
    torch, bh = _bh()
    print("[gpu] unequal systems, time", flush=True)
    sys.stdout.flush()
    big = bh.to_device(inputs.ring(1 << 20, 5))
    small = bh.to_device(inputs.ring(8000, 6))
    many = [{k: v[8 * j:8 * j + 8] for k, v in small.items()} for j in range(1000)]
    alone, beside = _keys_ms(torch, bh, [big]), _keys_ms(torch, bh, many[:500] + [big] + many[500:])
    print(f"    alone {alone:.3f} ms, among 1000 {beside:.3f} ms", flush=True)
    assert beside < 3.0 * alone


SIZES = [(1,), (1023, 1, 1025), (2047, 2048, 2049, 1), (5, 300000, 3, 1024, 70001), (1, 1, 1, 1, 40000)]


@pytest.mark.parametrize("sizes", SIZES, ids=["_".join(map(str, s)) for s in SIZES])
@pytest.mark.parametrize("cyl", [0.0, 1.05], ids=["cartesian", "cylindrical"])
def test_keys_and_boxes(sizes, cyl):
    torch, bh = _bh()
    print(f"[gpu] unequal systems {sizes} cyl={cyl}", flush=True)
    sys.stdout.flush()
    systems = [inputs.ring(n, 500 + k) for k, n in enumerate(sizes)]
    ctx = bh.Context(theta=0.5, eps=1e-3, n_group=64, cyl_radius=cyl, precision=bh.FP32_REL)
    dev = [bh.to_device(s) for s in systems]
    for step in range(2):            # from the caller's arrays, then from the sorted state
        if step == 0:
            ctx.build_tree(dev)
        else:
            ctx.step(dev, 0.0, 1)    # no time passes: the same positions, rebuilt
        keys, box, b = ctx.export("keys"), ctx.export("root_box"), 0
        for j, s in enumerate(systems):
            lo, S, _, k = oracle.keys_cyl(s.x, s.y, s.z, cyl) if cyl else oracle.keys(s.x, s.y, s.z)
            np.testing.assert_array_equal(keys[b:b + s.n], np.sort(k))
            np.testing.assert_array_equal(box[j], [*lo, 2.0 ** 21 / S])
            b += s.n
    ctx.close()
