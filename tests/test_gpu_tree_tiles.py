"""The octree built from all levels at once, at the edges of its tiles of 256
particles and of the 64 keys kept on either side: particle counts around
multiples of 256, leaf sizes around 64 and far above it, cells and runs of
equal keys that span several tiles, and levels around the 1024 nodes that the
single-block moment pass takes.  Keys, nodes, groups, boxes and lists bit-exact
against the oracle, moments within the FP64 summation bound (the checks of
test_gpu_parity)."""
import sys

import numpy as np
import pytest

import oracle
from paper_1907_02289_amd import inputs
from test_gpu_parity import _compare_structures

pytestmark = pytest.mark.gpu


def _ring(n, seed=60):
    return inputs.ring(n, seed)


def _equal(n, k, seed=61):
    """k of n particles at one point: equal keys over several tiles, a level-21 leaf above any leaf size."""
    s = inputs.ring(n, seed)
    for a in (s.x, s.y, s.z):
        a[n // 3:n // 3 + k] = a[0]
    return s


def _two_scales(n, seed=62):
    """Most particles in one cell 2^-12 of the box: deep narrow levels over many tiles."""
    s = inputs.plummer(n, seed)
    for a in (s.x, s.y, s.z):
        a[n // 8:] *= 2.0 ** -12
    return s


CASES = [(f"n{n}_leaf{nl}", lambda n=n: _ring(n), nl, max(nl, 32))
         for n, nl in ((2, 1), (255, 8), (256, 8), (257, 8), (513, 1), (1024, 63), (1025, 64), (1027, 65), (6000, 300),
                       (5000, 4096), (9000, 4096), (30000, 8))]
CASES += [("equal70", lambda: _equal(600, 70), 8, 32), ("equal700", lambda: _equal(2000, 700), 8, 64),
          ("equal700_leaf64", lambda: _equal(2000, 700), 64, 64), ("two_scales", lambda: _two_scales(7000), 8, 64)]


@pytest.mark.parametrize("name,make,n_leaf,n_grp", CASES, ids=[c[0] for c in CASES])
def test_tree_at_tile_edges(name, make, n_leaf, n_grp):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02289_amd import bh
    s = make()
    print(f"[gpu] tree tiles: {name} n={s.n} n_leaf={n_leaf} n_group={n_grp}", flush=True)
    sys.stdout.flush()
    ctx = bh.Context(theta=0.5, eps=1e-3, n_leaf=n_leaf, n_group=n_grp)
    ctx.build_tree([bh.to_device(s)])
    ctx.make_lists()
    _compare_structures(ctx, oracle.BHState(s.x, s.y, s.z, s.m, 0.5, n_leaf, n_grp), s.n)
    ctx.close()


def test_systems_across_tiles():
    """Systems whose boundaries fall at, before and inside tiles: each one's nodes are those of its own build."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02289_amd import bh
    sizes = [256, 1, 255, 40, 473, 8, 9, 700]
    print(f"[gpu] tree tiles: systems of {sizes}", flush=True)
    sys.stdout.flush()
    systems = [inputs.ring(n, 70 + k) for k, n in enumerate(sizes)]
    ctx = bh.Context(theta=0.5, eps=1e-3, n_leaf=8, n_group=32)
    ctx.build_tree([bh.to_device(s) for s in systems])
    nodes = ctx.export("nodes")
    off = np.concatenate([[0], np.cumsum(sizes)])
    assert np.all(np.diff(nodes[:, 0] * len(sizes) + nodes[:, 1]) >= 0)     # (level, system) ascending
    for k, s in enumerate(systems):
        t = oracle.BHState(s.x, s.y, s.z, s.m, 0.5, 8, 32).tree
        mine = nodes[nodes[:, 1] == k]
        for col, want in ((0, t["level"]), (2, t["prefix"].astype(np.int64)), (3, t["begin"] + off[k]),
                          (4, t["count"]), (6, t["n_child"])):
            np.testing.assert_array_equal(mine[:, col], want)
    ctx.close()
