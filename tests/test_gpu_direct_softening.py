"""The FP64 direct sum where its fast pair's range ends from above: softening
lengths and distances whose cube overflows (m / (r^2 r) is 0 there, whatever the
mass), up to a square that is infinite, and large ones below; with and without
the collision branch."""
import sys

import numpy as np
import pytest

from paper_1907_02289_amd import inputs

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _run(s, eps, tg, **kw):
    torch = _torch()
    from paper_1907_02289_amd import bh
    ctx = bh.Context(theta=0.5, eps=eps, **kw)
    out = {k: torch.zeros(tg.size, dtype=torch.float64, device="cuda") for k in ("ax", "ay", "az")}
    ctx.direct_sum(bh.to_device(s), torch.as_tensor(tg, device="cuda"), out)
    g = np.stack([out[k].cpu().numpy() for k in ("ax", "ay", "az")])
    ctx.close()
    return g


@pytest.mark.parametrize("r_coll", [0.0, 1e-3], ids=["gravity", "contacts"])
@pytest.mark.parametrize("eps", [2.0 ** 342, 2.0 ** 399, 1e130, 2.0 ** 511, 1e154, 1.5e154, 1e200, 1.7e308])
def test_huge_softening_gives_no_force(eps, r_coll):
    print(f"[gpu] direct sum softening eps={eps:g} r_coll={r_coll}", flush=True)
    sys.stdout.flush()
    s = inputs.plummer(700, 91)
    s.m[:] = 2.0 ** 300
    g = _run(s, eps, np.array([0, 1, 350, 699], np.int64), r_coll=r_coll, kappa=0.0, eta=0.0)
    assert np.all(g == 0.0), g


@pytest.mark.parametrize("eps", [0.0, 1e-4])
@pytest.mark.parametrize("power", [342, 345, 399, 401])
def test_distance_whose_cube_overflows_gives_no_force(power, eps):
    print(f"[gpu] direct sum at a distance of 2^{power}, eps={eps:g}", flush=True)
    sys.stdout.flush()
    near, s = inputs.plummer(700, 94), inputs.plummer(700, 94)
    near.m[650] = 0.0
    s.x[650], s.m[650] = 2.0 ** power, 2.0 ** 300
    tg = np.array([0, 1, 350, 699], np.int64)
    np.testing.assert_allclose(_run(s, eps, tg), _run(near, eps, tg), rtol=1e-13, atol=0)


@pytest.mark.parametrize("eps", [1e20, 1e60, 1e90])
def test_large_softening(eps):
    """r^2 is eps^2 to all digits: the force is the mass-weighted distance over eps^3, m / eps^3 within the
    rounding of its own four operations and the sum's."""
    print(f"[gpu] direct sum softening eps={eps:g}", flush=True)
    sys.stdout.flush()
    s = inputs.plummer(700, 92)
    tg = np.array([0, 1, 350, 699], np.int64)
    g = _run(s, eps, tg).astype(np.longdouble)
    for k, i in enumerate(tg):
        for a, c in enumerate((s.x, s.y, s.z)):
            d = c.astype(np.longdouble) - np.longdouble(c[i])
            want, mag = (s.m * d).sum(), np.abs(s.m * d).sum()
            e3 = np.longdouble(eps) ** 3
            assert abs(g[a, k] * e3 - want) <= 150 * 2.0 ** -53 * mag
