"""The kernels' index ranges (csrc/ranges.h), built for the host and checked against their meaning."""
import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2608_23245_amd", "csrc")

SOURCE = """
#include "ranges.h"
extern "C" int ring_block_meets(int jl, int jh, int jb, int n) { return fdtbx::ring_block_meets(jl, jh, jb, n); }
"""


@pytest.fixture(scope="module")
def ranges(tmp_path_factory):
    d = tmp_path_factory.mktemp("ranges")
    src = d / "ranges.cpp"
    src.write_text(SOURCE)
    lib = str(d / "ranges.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-ffp-contract=off", "-I", CSRC, str(src), "-o", lib],
                   check=True)
    return ctypes.CDLL(lib)


def test_ring_block_meets_a_lane_that_has_points_in_it(ranges):
    """Every small range, the empty one (1, 0) that a lane out of reach carries among them."""
    for n in (1, 8):
        for jl in range(-12, 13):
            for jh in range(jl - 1, 13):
                for jb in range(-24, 25):
                    want = any(jl <= j <= jh for j in range(jb, jb + n))
                    assert bool(ranges.ring_block_meets(jl, jh, jb, n)) == want, (jl, jh, jb, n)
