"""The cases of the GPU tests of small moments and of the walk's blocks are at
the edges that they are named for (no GPU: the oracle's trees): node counts on
either side of the 4096 of a one-block moment pass, and the group counts
around a block's and an XCD's share."""
import oracle
from paper_1907_02289_amd import inputs
from test_gpu_moments_small import CASES as MOMENTS
from test_gpu_walk_blocks import CASES as BLOCKS


def test_moment_cases_lie_on_both_sides_of_their_limits():
    nodes = {}
    for n, n_leaf in MOMENTS:
        s = inputs.ring(n, 97)
        nodes[n, n_leaf] = oracle.BHState(s.x, s.y, s.z, s.m, 0.5, n_leaf, max(64, n_leaf)).tree["begin"].size
    ring = sorted(v for (n, n_leaf), v in nodes.items() if n_leaf == 8 and 10000 < n < 13000)
    below, above = [v for v in ring if v <= 4096], [v for v in ring if v > 4096]
    assert below and above and max(below) > 3900 and min(above) < 4300, ring
    # 16384 and 16385 particles with few enough nodes that the particles decide
    assert nodes[16384, 64] <= 4096 and nodes[16385, 64] <= 4096
    assert nodes[4096, 4096] == 1 and nodes[1, 8] == 1


def test_walk_cases_have_the_group_counts_named():
    counts = []
    for n, n_grp in BLOCKS:
        s = inputs.ring(n, 50 + n_grp)
        counts.append(oracle.BHState(s.x, s.y, s.z, s.m, 0.5, min(8, n_grp), n_grp).gnode.size)
    assert counts == [1, 3, 7, 8, 9, 31, 32, 33, 222, 15392], counts
