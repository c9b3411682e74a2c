"""The sample sort of several systems above 2^20 pairs, whose buckets hold 6144
pairs with their systems: keys and permutation against a stable numpy sort of
the library's own definition of the keys, for randomly ordered input up to the
largest size, and for an input that fills one bucket beyond that."""
import sys

import numpy as np
import pytest

import oracle
from paper_1907_02289_amd import inputs

pytestmark = pytest.mark.gpu


def _missed(n, total, seed):
    """n particles of total pairs: those at the places of a sample of 8 pairs in each of 1024 buckets form a
    ring, all others a clump that no splitter cuts."""
    s = inputs.ring(n, seed)
    m = 1024 * 8
    j = np.arange(m, dtype=np.uint64)
    stretch = (total << 32) // m
    a, b = (j * stretch) >> np.uint64(32), ((j + 1) * stretch) >> np.uint64(32)
    at = (a + ((b - a) * (((j + 1) * 2654435761) % 2 ** 32) >> np.uint64(32))).astype(np.int64)
    rest = np.setdiff1d(np.arange(n), at[at < n])
    r = np.random.default_rng(seed)
    for c in (s.x, s.y, s.z):
        c[rest] = c[at[0]] + 2.0 ** -12 * r.random(rest.size)
    return s


CASES = [("wide", lambda: [inputs.plummer(n, 100 + k) for k, n in enumerate((1 << 20, 1, 300, 70000))]),
         ("batch64", lambda: [inputs.plummer(32768, 200 + k) for k in range(64)]),
         ("largest", lambda: [inputs.ring(n, 300 + k) for k, n in enumerate((1 << 20, (5 << 18) - 5, 5, 1 << 18))]),
         ("missed", lambda: [_missed(1100000, 1100309, 400), inputs.ring(300, 401), inputs.ring(9, 402)])]


@pytest.mark.parametrize("name,make", CASES, ids=[c[0] for c in CASES])
def test_keys_and_permutation(name, make):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02289_amd import bh
    systems = make()
    total = sum(s.n for s in systems)
    assert (1 << 20) < total <= (5 << 19) and (name != "largest" or total == 5 << 19)
    print(f"[gpu] sort of several systems: {name}, {total} particles", flush=True)
    sys.stdout.flush()
    ctx = bh.Context(theta=0.5, eps=1e-3, n_leaf=64, n_group=256)
    ctx.build_tree([bh.to_device(s) for s in systems])
    keys, perm, b = ctx.export("keys"), ctx.export("perm"), 0
    for s in systems:
        k = oracle.keys(s.x, s.y, s.z)[3]
        order = np.argsort(k, kind="stable")
        np.testing.assert_array_equal(keys[b:b + s.n], k[order])
        np.testing.assert_array_equal(perm[b:b + s.n], order)
        b += s.n
    ctx.close()
