"""The walk's distribution of groups over blocks and XCDs: group counts around
the edges of a block's and an XCD's share (counts below eight leave whole XCD
shares empty), and more groups than waves fit in one round.  Lists and interaction totals are
bit-exact against the oracle's."""
import sys

import numpy as np
import pytest

import oracle
from paper_1907_02289_amd import inputs

pytestmark = pytest.mark.gpu


# (particles, group size): 1, 3, 7, 8, 9, 31, 32, 33 and 222 groups; the last has 15,392, more than the 8192
# waves of one round
CASES = [(9, 64), (17, 16), (74, 16), (68, 16), (89, 16), (239, 16), (278, 16), (302, 16), (3000, 32), (20000, 2)]


@pytest.mark.parametrize("n,n_grp", CASES, ids=[f"n{n}_g{g}" for n, g in CASES])
def test_lists_for_group_counts(n, n_grp):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02289_amd import bh
    print(f"[gpu] walk blocks: ring n={n} n_group={n_grp}", flush=True)
    sys.stdout.flush()
    s = inputs.ring(n, 50 + n_grp)
    n_leaf = min(8, n_grp)
    ctx = bh.Context(theta=0.5, eps=1e-3, n_leaf=n_leaf, n_group=n_grp)
    ctx.build_tree([bh.to_device(s)])
    ctx.make_lists()
    st = oracle.BHState(s.x, s.y, s.z, s.m, 0.5, n_leaf, n_grp)
    pc_off, pc, pp_off, pp = ctx.export("lists")
    np.testing.assert_array_equal(pc_off, st.pc_off)
    np.testing.assert_array_equal(pp_off, st.pp_off)
    np.testing.assert_array_equal(pc, st.pc)
    np.testing.assert_array_equal(pp, st.pp)
    assert ctx.query()["interactions"] == st.interactions()
    ctx.close()
