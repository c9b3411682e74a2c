"""Contacts at a radius beyond the massless entries that pad a source tile (at
1e18 in each coordinate): every listed particle is in contact, the padding is
not.  Groups of a few particles, whose chunks are sub-sliced over a padded
tile, and one of several hundred; against the oracle."""
import sys

import numpy as np
import pytest

from bars import fp32_bars

import oracle
from paper_1907_02289_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("n,n_grp", [(5, 64), (300, 512), (3001, 32), (3000, 300)])
def test_padding_has_no_contacts(n, n_grp, precision):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02289_amd import bh
    print(f"[gpu] contact radius beyond the padding: n={n} n_group={n_grp} precision={precision}", flush=True)
    sys.stdout.flush()
    s = inputs.ring(n, 95, v_disp=3e-3)
    rc, kappa, eta, theta, eps = 4e18, 1e-18, 0.5, 0.5, 1e-4
    ctx = bh.Context(theta=theta, eps=eps, n_group=n_grp, precision=precision, r_coll=rc, kappa=kappa, eta=eta)
    ctx.build_tree([bh.to_device(s)])
    ctx.make_lists()
    out = {k: torch.zeros(n, dtype=torch.float64, device="cuda") for k in ("ax", "ay", "az")}
    ctx.forces([out])
    st = oracle.BHState(s.x, s.y, s.z, s.m, theta, 8, n_grp)
    ax, ay, az, _, mag = st.accel(s.x, s.y, s.z, s.m, eps, vel=(s.vx, s.vy, s.vz), contact=(rc, kappa, eta))
    err = np.sqrt(sum((out[k].cpu().numpy() - a) ** 2 for k, a in (("ax", ax), ("ay", ay), ("az", az))))
    if precision == 0:
        assert np.all(err <= 1e-12 * mag), np.max(err / mag)
    else:
        fp32_bars(err / np.sqrt(ax ** 2 + ay ** 2 + az ** 2), f"n={n}")
    ctx.close()
