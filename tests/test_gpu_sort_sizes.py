"""The sort's three ways at the sizes where one takes over from another and at
the edges of their tiles, through bh_build_tree: keys and permutation against
a stable numpy sort of the library's own definition of the keys (equal keys
keep caller order), for one system and several, for rings, clumps, and inputs
in which many particles share a key (repeated splitters, a bucket beyond what
LDS holds)."""
import sys

import numpy as np
import pytest

import oracle
from paper_1907_02289_amd import inputs

pytestmark = pytest.mark.gpu


def _clump(n, k, seed):
    """k of n particles in a box 2^-18 of the ring: a few thousand distinct keys among them."""
    s = inputs.ring(n, seed)
    r = np.random.default_rng(seed)
    for a in (s.x, s.y, s.z):
        a[r.choice(n, k, replace=False)] = a[0] + 2.0 ** -18 * r.random(k)
    return s


def _same(n, k, seed):
    s = inputs.ring(n, seed)
    pick = np.random.default_rng(seed).choice(n, k, replace=False)
    for a in (s.x, s.y, s.z):
        a[pick] = a[pick[0]]
    return s


def _lattice(n, seed):
    """A repeated input order whose period divides the sample's stride: every sampled particle comes from one
    of 16 places unless the sample's places vary."""
    s = inputs.ring(n, seed)
    for a in (s.x, s.y, s.z):
        a[:] = np.where(np.arange(n) % 1024 < 16, a[0] + 1e-3 * (np.arange(n) % 16), a)
    return s


def _missed(n, seed):
    """Particles at the sample's places form a ring, all others a clump that no splitter cuts: one bucket holds
    nearly all pairs, more than LDS does."""
    s = inputs.ring(n, seed)
    buckets = min(1024, max(8, (n + 1023) // 1024))
    m = buckets * 8
    j = np.arange(m, dtype=np.uint64)
    a, b = (j * ((n << 32) // m)) >> np.uint64(32), ((j + 1) * ((n << 32) // m)) >> np.uint64(32)
    at = a + ((b - a) * (((j + 1) * 2654435761) % 2 ** 32) >> np.uint64(32))
    rest = np.setdiff1d(np.arange(n), at.astype(np.int64))
    r = np.random.default_rng(seed)
    for c in (s.x, s.y, s.z):
        c[rest] = c[at[0]] + 2.0 ** -12 * r.random(rest.size)
    return s


CASES = [(f"ring{n}", lambda n=n: [inputs.ring(n, 80)]) for n in
         (1, 2, 63, 64, 65, 1023, 1024, 1025, 2048, 2049, 4096, 4097, 8191, 8192, 8193, 9001, 12287, 12288, 12289,
          100003, (1 << 20) - 1, (1 << 20) + 1, (5 << 19), (5 << 19) + 1)]
CASES += [("clump", lambda: [_clump(150000, 60000, 81)]), ("same30000", lambda: [_same(100000, 30000, 82)]),
          ("all_same", lambda: [_same(20000, 20000, 83)]), ("same_in_small", lambda: [_same(5000, 4000, 84)]),
          ("missed", lambda: [_missed(100000, 88)]), ("missed_two", lambda: [_missed(60000, 89), inputs.ring(9, 90)]),
          ("lattice", lambda: [_lattice(262144, 85)]),
          ("systems_small", lambda: [inputs.ring(n, 86 + n) for n in (5, 700, 1, 64, 1300)]),
          ("systems_large", lambda: [inputs.plummer(n, 87 + n) for n in (30000, 3, 1, 12000, 257, 90000)]),
          ("systems_many", lambda: [inputs.ring(1 + k % 40, 3000 + k) for k in range(700)])]


@pytest.mark.parametrize("name,make", CASES, ids=[c[0] for c in CASES])
def test_keys_and_permutation(name, make):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1907_02289_amd import bh
    systems = make()
    print(f"[gpu] sort sizes: {name}, {sum(s.n for s in systems)} particles", flush=True)
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
