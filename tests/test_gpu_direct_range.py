"""The FP64 direct sum's pair without the range handling of a square root and a
division: source counts around its tiles of 256 and chunks of 1024, no
softening (coincident particles, separations far below 2^-150), coordinates
and masses beyond 2^400, infinite ones.  Against sums in extended precision:
within the rounding of 64 terms of a tile and of the tiles, chunks and waves
that follow, 2^-53 each, plus 8 for a pair."""
import sys

import numpy as np
import pytest

from paper_1907_02289_amd import inputs

pytestmark = pytest.mark.gpu

L = np.longdouble


def _reference(s, eps, tg):
    """The sums and the sums of the terms' magnitudes, both in extended precision."""
    pos = np.stack([s.x, s.y, s.z]).astype(L)
    m = s.m.astype(L)
    acc, mag = np.zeros((3, tg.size), L), np.zeros(tg.size, L)
    for k, i in enumerate(tg):
        d = pos - pos[:, i:i + 1]
        r2 = (d * d).sum(0) + L(eps) ** 2
        with np.errstate(divide="ignore", invalid="ignore"):
            r3 = r2 * np.sqrt(r2)
            f = np.where((r2 > 0) & (r3 <= np.finfo(np.float64).max), m / r3, L(0))   # an overflowing r^3 gives no term
        acc[:, k] = (f * d).sum(1)
        mag[k] = (f * np.sqrt((d * d).sum(0))).sum()
    return acc, mag


def _run(s, eps, tg):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02289_amd import bh
    ctx = bh.Context(theta=0.5, eps=eps)
    out = {k: torch.zeros(tg.size, dtype=torch.float64, device="cuda") for k in ("ax", "ay", "az")}
    ctx.direct_sum(bh.to_device(s), torch.as_tensor(tg, device="cuda"), out)
    g = np.stack([out[k].cpu().numpy() for k in ("ax", "ay", "az")])
    ctx.close()
    return g


def _check(s, eps, tg, what):
    print(f"[gpu] direct sum range: {what}", flush=True)
    sys.stdout.flush()
    g = _run(s, eps, tg)
    acc, mag = _reference(s, eps, tg)
    tiles = (s.n + 255) // 256
    bound = (64 + tiles + 4 + 64 + 8) * 2.0 ** -53
    err = np.abs(g.astype(L) - acc).max(0)
    assert np.all(err <= bound * mag), f"{what}: {np.max(err / mag) / 2.0 ** -53} x 2^-53"


@pytest.mark.parametrize("eps", [0.0, 1e-4, 1e-100], ids=["eps0", "eps1e-4", "eps1e-100"])
@pytest.mark.parametrize("n", [2, 3, 255, 256, 257, 1023, 1024, 1025, 5000, 66000])
def test_source_counts(n, eps):
    s = inputs.plummer(n, 80 + n)
    tg = np.unique(np.array([0, n - 1, n // 2, n // 3], np.int64))
    _check(s, eps, tg, f"n={n} eps={eps}")


def test_unsoftened_close_and_coincident():
    s = inputs.plummer(700, 81)
    for a in (s.x, s.y, s.z):
        a[300] = a[10]                    # coincident: no term
        a[20] = a[21] = 0.0
    s.x[21] = 1e-100                      # r^2 = 1e-200: below 2^-300
    s.x[22] = s.y[22] = s.z[22] = 1e-60
    _check(s, 0.0, np.array([10, 300, 5, 21, 22, 20], np.int64), "close pairs")


def test_beyond_the_range():
    s = inputs.plummer(600, 82)
    s.x[400] = 2.0 ** 430                 # its square is finite, its cube is not
    s.m[401] = 2.0 ** 420
    _check(s, 1e-4, np.array([0, 300, 401, 599, 400], np.int64), "wide tile")


def test_overflowing_distance_adds_nothing():
    """A source so far away that its squared distance overflows gives no term, on any tile; a target that far gives 0."""
    s = inputs.plummer(600, 83)
    far = inputs.plummer(600, 83)
    far.y[550] = 1e200
    s.m[550] = 0.0
    tg = np.array([0, 100, 599], np.int64)
    np.testing.assert_allclose(_run(far, 1e-4, tg), _run(s, 1e-4, tg), rtol=1e-13, atol=0)
    assert np.all(_run(far, 1e-4, np.array([550], np.int64)) == 0.0)
