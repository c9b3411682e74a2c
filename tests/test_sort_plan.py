"""The sample sort's plan (no GPU): buckets that outgrow the LDS of their block
are rare in randomly ordered input, for every size and for one system and
several.  A bucket is `per` consecutive gaps of buckets * per sampled pairs, a
Beta(per, buckets per + 1 - per) share of the pairs; the expected number of
buckets above the capacity, checked against drawn samples where it is not
small."""
import ctypes
import os
import subprocess

import numpy as np
import pytest
from scipy.stats import beta

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "bh_sort_plan.hpp"
extern "C" void limits(uint32_t *o) { o[0] = bhk::SMALL_MAX; o[1] = bhk::SAMPLE_MAX; }
extern "C" void plan(uint32_t n, int several, uint32_t *o) {
    const bhk::SamplePlan p = bhk::sample_plan(n, several != 0);
    o[0] = p.buckets; o[1] = p.per; o[2] = p.capacity;
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, lib = d / "plan.cpp", d / "plan.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_1907_02289_amd", "csrc"), "-o", str(lib), str(src)], check=True)
    L = ctypes.CDLL(str(lib))
    o = (ctypes.c_uint32 * 3)()

    def call(n, several):
        L.plan(n, int(several), o)
        return tuple(o)

    L.limits(o)
    return call, o[0], o[1]


def _overfull(n, buckets, per, capacity):
    return buckets * beta.sf(capacity / n, per, buckets * per + 1 - per)


@pytest.mark.parametrize("several", [False, True], ids=["one", "several"])
def test_overfull_buckets_are_rare(plan, several):
    call, small, most = plan
    sizes = np.unique(np.concatenate([np.geomspace(small + 1, most, 200).astype(int),
                                      [1 << 20, (1 << 20) + 1, 1 << 21, 2190000, most]]))
    for n in sizes:
        buckets, per, capacity = call(int(n), several)
        assert buckets * per <= n                     # the sample is gathered into arrays of n
        assert buckets <= 1024 and capacity <= 8192   # ten-bit bucket numbers; thirteen-bit places in a block
        assert _overfull(n, buckets, per, capacity) <= 0.02, (n, several)


def test_the_distribution_is_that_of_drawn_samples():
    n, buckets, per, capacity = 5 << 19, 1024, 8, 6144
    r = np.random.default_rng(7)
    found = 0
    for _ in range(300):
        at = np.sort(r.random(buckets * per))[per - 1::per][:buckets - 1]
        found += int((np.diff(np.concatenate([[0.0], at, [1.0]])) > capacity / n).sum())
    want = 300 * _overfull(n, buckets, per, capacity)
    assert want > 100 and abs(found - want) < 5 * np.sqrt(want)
