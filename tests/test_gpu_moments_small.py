"""Moments of a whole tree in one block: node counts on either side of the 4096
that fit and particle counts on either side of 16384, leaves of one to many
particles, a single leaf, several systems, and the refresh of list-reusing steps
(which the drift monitor and the learned rule's second moments take through the
other launches).  Against the oracle as in test_gpu_parity."""
import sys

import numpy as np
import pytest

import oracle
from paper_1907_02289_amd import inputs
from test_gpu_parity import _compare_structures

pytestmark = pytest.mark.gpu

# particles and leaf size; 10400 to 12200 ring particles in leaves of 8 make 3770 to about 4300 nodes
CASES = [(1, 8), (7, 8), (9, 8), (1025, 1), (10400, 8), (10900, 8), (11600, 8), (12200, 8), (16384, 64), (16385, 64), (4096, 4096)]


def _bh():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02289_amd import bh
    return torch, bh


@pytest.mark.parametrize("n,n_leaf", CASES, ids=[f"n{n}_leaf{l}" for n, l in CASES])
def test_moments(n, n_leaf):
    torch, bh = _bh()
    print(f"[gpu] small moments n={n} n_leaf={n_leaf}", flush=True)
    sys.stdout.flush()
    s = inputs.ring(n, 97)
    n_grp = max(64, n_leaf)
    ctx = bh.Context(theta=0.5, eps=1e-3, n_leaf=n_leaf, n_group=n_grp)
    ctx.build_tree([bh.to_device(s)])
    ctx.make_lists()
    print(f"    {ctx.query()['n_nodes']} nodes", flush=True)
    _compare_structures(ctx, oracle.BHState(s.x, s.y, s.z, s.m, 0.5, n_leaf, n_grp), n)
    ctx.close()


def test_reuse_with_and_without_the_drift_monitor():
    """The same reused steps with the drift monitor on (its threshold never reached) and off: bit-identical states."""
    torch, bh = _bh()
    print("[gpu] small moments, reuse", flush=True)
    states = []
    for drift in (0.0, 1e6):
        systems = [bh.to_device(inputs.ring(700, 98)), bh.to_device(inputs.plummer(1300, 99))]
        ctx = bh.Context(theta=0.5, eps=1e-2, n_group=32, reuse_drift=drift)
        ctx.step(systems, 1e-3, 5, rebuild_every=8)
        torch.cuda.synchronize()
        states.append([getattr(s, k).cpu().numpy() if hasattr(s, k) else s[k].cpu().numpy()
                       for s in systems for k in ("x", "y", "z", "vx", "vy", "vz")])
        ctx.close()
    for a, b in zip(*states):
        np.testing.assert_array_equal(a, b)
