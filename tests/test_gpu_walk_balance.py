"""The walk's groups spread over the chip whatever region needs the long walks.
A sphere alone, and with as many one-group systems beside it as it has groups:
its walk must not take longer for sharing the launch with walks of a few nodes
(dealt in contiguous shares, the sphere's groups would fall to half of the
chip).  And lists at group counts around a run of an XCD (32 groups), one run of
each (256) and the first rounds (8192 groups, 2048 with the learned rule),
against the oracle."""
import sys

import numpy as np
import pytest

from learned_ref import learned_inputs

import oracle
from paper_1907_02289_amd import inputs

pytestmark = pytest.mark.gpu


def _bh():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02289_amd import bh
    return torch, bh


def _walk_ms(torch, bh, systems):
    ctx = bh.Context(theta=0.15, eps=1e-3, n_group=256, precision=bh.FP32_REL)
    ctx.build_tree(systems)
    ms = []
    for _ in range(6):
        ctx.make_lists()
        torch.cuda.synchronize()
        ms.append(ctx.stage_times()["walk"])
    groups = ctx.query()["n_groups"]
    ctx.close()
    return min(ms), groups


def test_walk_time_beside_many_small_systems():
    torch, bh = _bh()
    print("[gpu] walk balance", flush=True)
    sys.stdout.flush()
    big = bh.to_device(inputs.plummer(1 << 20, 96))
    alone, groups = _walk_ms(torch, bh, [big])
    small = bh.to_device(inputs.ring(8 * groups, 97))
    many = [{k: v[8 * j:8 * j + 8] for k, v in small.items()} for j in range(groups)]
    beside, all_groups = _walk_ms(torch, bh, [big] + many)
    print(f"    {groups} groups {alone:.3f} ms, {all_groups} groups {beside:.3f} ms", flush=True)
    assert all_groups == 2 * groups
    assert beside < 1.4 * alone


# particles, group size, groups
CASES = [(140, 8, 31), (149, 8, 32), (143, 8, 33), (996, 8, 255), (1025, 8, 256), (1020, 8, 257), (10839, 2, 8191),
         (10854, 2, 8192), (10907, 2, 8193), (40000, 4, 21820)]


@pytest.mark.parametrize("n,n_grp,groups", CASES, ids=[f"{c[2]}groups" for c in CASES])
def test_lists_around_the_runs(n, n_grp, groups):
    torch, bh = _bh()
    s = inputs.ring(n, 60 + n_grp)
    st = oracle.BHState(s.x, s.y, s.z, s.m, 0.6, 2, n_grp)
    assert st.gnode.size == groups
    print(f"[gpu] walk runs: ring n={n} n_group={n_grp}, {groups} groups", flush=True)
    sys.stdout.flush()
    ctx = bh.Context(theta=0.6, eps=1e-3, n_leaf=2, n_group=n_grp)
    ctx.build_tree([bh.to_device(s)])
    ctx.make_lists()
    assert ctx.query()["n_groups"] == groups
    pc_off, pc, pp_off, pp = ctx.export("lists")
    np.testing.assert_array_equal(pc_off, st.pc_off)
    np.testing.assert_array_equal(pp_off, st.pp_off)
    np.testing.assert_array_equal(pc, st.pc)
    np.testing.assert_array_equal(pp, st.pp)
    assert ctx.query()["interactions"] == st.interactions()
    ctx.close()


def test_learned_lists_of_more_than_the_first_rounds():
    torch, bh = _bh()
    print("[gpu] learned walk over more than 2048 groups", flush=True)
    sys.stdout.flush()
    s = inputs.ring(9000, 98)
    r = np.random.default_rng(99)
    w = r.normal(0, 0.3, 1259).astype(np.float32)
    w[1249:] = [-6.0, -3.0, -12.0, -4.0, 0.5, 0.6, 0.3, 1.0, -8.0, 2.0]      # means, 1/std, label mean and std
    ctx = bh.Context(theta=0.3, eps=1e-3, n_group=4, n_leaf=4, precision=bh.FP64, criterion=bh.LEARNED, theta_min=0.1,
                     theta_max=0.6, tau=3e-3)
    ctx.mlp_weights(set=w)
    ctx.build_tree([bh.to_device(s)])
    ctx.make_lists()
    st, L = learned_inputs(s, 0.3, 1e-3, 4, n_leaf=4)
    assert st.gnode.size > 2048
    want = oracle.lists_learned(L["gbox"], L["gcen"], L["grad"], L["gamin"], L["t"], L["com4"], L["qn"], w,
                                L["S"], theta=0.3, theta_min=0.1, theta_max=0.6, tau=3e-3)
    for a, b in zip(ctx.export("lists"), want):
        np.testing.assert_array_equal(a, b)
    ctx.close()
