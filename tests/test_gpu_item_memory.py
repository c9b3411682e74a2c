"""The force kernel's work items keep their memory when the group count of the
same particles grows: nothing is freed or allocated (freeing waits for the
device), while the lists fit."""
import sys

import pytest

from paper_1907_02289_amd import inputs

pytestmark = pytest.mark.gpu


def test_more_groups_of_the_same_particles():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02289_amd import bh
    print("[gpu] memory of the work items", flush=True)
    sys.stdout.flush()
    dev = bh.to_device(inputs.ring(400000, 110))
    ctx = bh.Context(theta=0.05, eps=1e-3, n_group=512)
    ctx.build_tree([dev])
    ctx.make_lists()                       # few groups, long lists
    few = ctx.query()
    ctx.set_params(theta=1.2, n_group=8)
    ctx.build_tree([dev])
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    ctx.make_lists()                       # many groups, short lists
    torch.cuda.synchronize()
    many = ctx.query()
    print(f"    {few['n_groups']} and {many['n_groups']} groups, list entries {few['n_pc'], few['n_pp']} and "
          f"{many['n_pc'], many['n_pp']}", flush=True)
    assert many["n_groups"] > 10 * few["n_groups"]
    assert many["n_pc"] <= few["n_pc"] and many["n_pp"] <= few["n_pp"]
    assert torch.cuda.mem_get_info()[0] == free
    ctx.forces()
    ctx.close()
