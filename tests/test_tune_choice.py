"""The autotuner's choice from given times (no GPU): a group size takes the
256-source tile by its force times alone, when they are 2% below those of 512,
and group sizes are compared by their own force + walk / rebuild_every, without
a handicap for either tile."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "bh_tune.hpp"
extern "C" int tile(double f512, double f256, double walk) { return bhk::tune_tile({f512, f256, walk}); }
extern "C" double cost(double f512, double f256, double walk, int t, int every) {
    return bhk::tune_cost({f512, f256, walk}, t, every);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("tune")
    src, out = d / "tune.cpp", d / "tune.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_1907_02289_amd", "csrc"), "-o", str(out), str(src)], check=True)
    L = ctypes.CDLL(str(out))
    L.tile.argtypes = [ctypes.c_double] * 3
    L.cost.argtypes = [ctypes.c_double] * 3 + [ctypes.c_int] * 2
    L.cost.restype = ctypes.c_double
    return L


@pytest.mark.parametrize("walk", [0.0, 1.0, 100.0])
def test_the_tile_follows_from_the_force_times(lib, walk):
    assert lib.tile(1.0, 0.97, walk) == 256
    assert lib.tile(1.0, 0.99, walk) == 512           # within the timings' spread
    assert lib.tile(1.0, 1.0, walk) == 512
    assert lib.tile(1.0, 1.1, walk) == 512


def test_group_sizes_are_compared_by_their_own_times(lib):
    # 10.0 with a tile of 256 against 10.1 with one of 512: the first is faster
    a, b = (10.5, 9.0, 1.0), (9.1, 9.2, 1.0)
    ta, tb = lib.tile(*a), lib.tile(*b)
    assert (ta, tb) == (256, 512)
    assert lib.cost(*a, ta, 1) == 10.0 < lib.cost(*b, tb, 1) == 10.1
    assert lib.cost(9.1, 9.2, 1.0, 512, 4) == 9.1 + 0.25
