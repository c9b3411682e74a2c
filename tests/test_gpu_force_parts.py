"""The force kernel's work items (256 particles of a group each) and its FP32
pair loop (four sources per turn): group sizes around one, two and three items,
a group of coincident particles far above the group limit, whose items wrap
around, and source counts that leave every remainder; with one mass and with
different masses.  Forces against the oracle on the same lists (FP64 within
1e-12 of the sum of the terms' magnitudes, FP32 within the FP32 bars or, for the
coincident particles, within the rounding of a sum of equal terms), and the same
bits from every further evaluation."""
import sys

import numpy as np
import pytest

from bars import fp32_bars

import oracle
from paper_1907_02289_amd import inputs

pytestmark = pytest.mark.gpu


def _plummer(n):
    return inputs.plummer(n, 70 + n)


def _coincident(n, k):
    s = inputs.plummer(n, 71)
    for a in (s.x, s.y, s.z):
        a[:k] = a[0]
    return s


# name, system, theta, particles per group: 1 to 13 and 67 sources for one group, then groups of up to 257, 300, 513
# and 900, and 1400 coincident particles in groups of at most 300 (two items) and 64 (one)
CASES = [(f"n{n}", lambda n=n: _plummer(n), 0.5, 64) for n in (2, 3, 5, 6, 7, 9, 12, 13, 67)]
CASES += [(f"n{n}_g{g}", lambda n=n: _plummer(n), 0.7, g)
          for n, g in ((255, 256), (256, 256), (257, 257), (2000, 300), (3000, 513), (4001, 900))]
CASES += [("coincident_g300", lambda: _coincident(3000, 1400), 0.5, 300),
          ("coincident_g64", lambda: _coincident(3000, 1400), 0.5, 64)]


@pytest.mark.parametrize("equal", [True, False], ids=["equal", "masses"])
@pytest.mark.parametrize("name,make,theta,n_grp", CASES, ids=[c[0] for c in CASES])
def test_forces_of_item_parts(name, make, theta, n_grp, equal):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02289_amd import bh
    s = make()
    if not equal:
        s.m[:] = s.m * np.random.default_rng(5).uniform(0.5, 1.5, s.n)
    eps = 1e-2
    st = oracle.BHState(s.x, s.y, s.z, s.m, theta, 8, n_grp, pack=True)
    ax, ay, az, _, mag = st.accel(s.x, s.y, s.z, s.m, eps)
    for prec in (bh.FP64, bh.FP32_REL):
        print(f"[gpu] force parts: {name} equal={equal} precision={prec}", flush=True)
        sys.stdout.flush()
        ctx = bh.Context(theta=theta, eps=eps, n_group=n_grp, precision=prec, pack_groups=True)
        ctx.build_tree([bh.to_device(s)])
        ctx.make_lists()
        first = None
        for _ in range(3):
            out = {k: torch.zeros(s.n, dtype=torch.float64, device="cuda") for k in ("ax", "ay", "az")}
            ctx.forces([out])
            g = [out[k].cpu().numpy() for k in ("ax", "ay", "az")]
            if first is None:
                first = g
            for a, b in zip(first, g):
                np.testing.assert_array_equal(a, b)
        err = np.sqrt((first[0] - ax) ** 2 + (first[1] - ay) ** 2 + (first[2] - az) ** 2)
        if prec == bh.FP64:
            assert np.all(err <= 1e-12 * mag + 1e-300), f"max err/mag {np.max(err / mag)}"
        elif name.startswith("coincident"):
            # the FP32 sum of 1400 equal terms rounds with one sign: up to 2^-24 of the sum for each of the s.n terms
            assert np.all(err <= s.n * 2.0 ** -24 * mag), f"max err/mag {np.max(err / mag)}"
        else:
            fp32_bars(err / np.sqrt(ax ** 2 + ay ** 2 + az ** 2), name)
        ctx.close()
