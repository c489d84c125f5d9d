"""The kernels' index ranges (csrc/ranges.h), built for the host and checked against their meaning."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2608_23245_amd", "csrc")

SOURCE = """
#include "ranges.h"
extern "C" int ring_block_meets(int jl, int jh, int jb, int n) { return fdtbx::ring_block_meets(jl, jh, jb, n); }
extern "C" int no_ring(int last) { return last ? fdtbx::kNoRingLast : fdtbx::kNoRingFirst; }
extern "C" double widened_extent(double rho, double r0) { return fdtbx::widened_extent(rho, r0); }
"""


@pytest.fixture(scope="module")
def ranges(tmp_path_factory):
    d = tmp_path_factory.mktemp("ranges")
    src = d / "ranges.cpp"
    src.write_text(SOURCE)
    lib = str(d / "ranges.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-ffp-contract=off", "-I", CSRC, str(src), "-o", lib],
                   check=True)
    lib = ctypes.CDLL(lib)
    lib.widened_extent.restype, lib.widened_extent.argtypes = ctypes.c_double, [ctypes.c_double, ctypes.c_double]
    return lib


def test_ring_block_meets_a_lane_that_has_points_in_it(ranges):
    """Every small range, and the empty one that a lane out of reach carries: it meets no block, and
    does not move the first or last index of a wave."""
    none = ranges.no_ring(0), ranges.no_ring(1)
    assert none[0] > 1 << 29 and none[1] < -(1 << 29)
    for n in (1, 8):
        for jb in [*range(-24, 25), 1 << 28, -(1 << 28)]:
            assert not ranges.ring_block_meets(*none, jb, n), (jb, n)
            for jl in range(-12, 13):
                for jh in range(jl, 13):
                    want = jb <= jh and jl <= jb + n - 1
                    assert want == any(jl <= j <= jh for j in range(jb, jb + n))
                    assert bool(ranges.ring_block_meets(jl, jh, jb, n)) == want, (jl, jh, jb, n)


F32 = np.float32


def f32(x):
    return np.asarray(x, dtype=np.float64).astype(F32)


def window(n, T, axes, R, Z, r0, rho):
    """The node window of a pixel (R, Z), in the float32 operations of pair_setup and
    node_window_ranges: axes are the (R, Z) coefficients of S, e1, e2, rho the record's extents."""
    inv_h, T32, r0 = f32(n / (2 * T)), f32(T), f32(r0)
    cmin = f32(1 / np.sqrt(1 + 2 * T * T))
    R, Z = f32(R), f32(Z)
    pS, p1, p2 = [(f32(c[0]) * R).astype(F32) + (f32(c[1]) * Z).astype(F32) for c in axes]
    rS, r1, r2 = [f32(r) * F32(1.0001) for r in rho]
    lo, hi = np.maximum(pS - rS, r0 * cmin * F32(0.9999)), np.minimum(pS + rS, r0 * F32(1.0001))
    inv_lo, inv_hi = (F32(1) / lo).astype(F32), (F32(1) / hi).astype(F32)
    big, out = F32(2) * T32, []
    for p, r in ((p1, r1), (p2, r2)):
        dl, dh = p - r, p + r
        dl = np.maximum(dl * np.where(dl >= 0, inv_hi, inv_lo), -big)
        dh = np.minimum(dh * np.where(dh >= 0, inv_lo, inv_hi), big)
        out.append(np.maximum(np.ceil((dl + T32) * inv_h - F32(0.625)), 0))
        out.append(np.minimum(np.floor((dh + T32) * inv_h - F32(0.375)), n - 1))
    assert all(v.dtype == F32 for v in (pS, rS, lo, hi, inv_lo, dl, dh))
    return lo <= hi, out


@pytest.mark.parametrize("lo,hi", [(-6, -5), (-5, -4), (-4, -3), (-3, -1.5), (-1.5, 0.3)])
def test_window_holds_every_node_in_reach(ranges, lo, hi):
    """Pixels that lie at the very edge of a node's reach, in binary64, for grids of half extent
    10^lo to 10^hi: the float32 window, with its margin of an eighth of a node, holds that node.  Supports of 10^-4 to 1 of the grid."""
    rng = np.random.default_rng(int(10 * lo) + 1000)
    N = 20000
    n, T = rng.choice([16, 24, 64, 96, 256], N), 10 ** rng.uniform(lo, hi, N)
    th, a, r0 = rng.uniform(0.05, np.pi - 0.05, N), rng.uniform(0, 2 * np.pi, N), 10 ** rng.uniform(-1.3, 0, N)
    zero, one = np.zeros(N), np.ones(N)
    # S in the (R, Z) half plane; e1, e2 turned about it by a
    S = np.stack([np.sin(th), zero, np.cos(th)], 1)
    u, v = np.stack([np.cos(th), zero, -np.sin(th)], 1), np.stack([zero, one, zero], 1)
    ca, sa = np.cos(a)[:, None], np.sin(a)[:, None]
    e1, e2 = ca * u + sa * v, ca * v - sa * u
    i1, i2 = rng.integers(0, n), rng.integers(0, n)
    h = 2 * T / n
    d1, d2 = -T + (i1 + 0.5) * h, -T + (i2 + 0.5) * h
    node = (r0 / np.sqrt(1 + d1 * d1 + d2 * d2))[:, None] * (S + d1[:, None] * e1 + d2[:, None] * e2)
    p = node * [1, 0, 1] + (T * r0 * 10 ** rng.uniform(-4, 0, N) * rng.choice([-1, 1], N))[:, None] * u
    # the reach along each axis: as far as the pixel lies from the node
    rho = [np.abs(((p - node) * e).sum(1)) * (1 + 1e-9) for e in (S, e1, e2)]
    rho[1:] = [np.array([ranges.widened_extent(*v) for v in zip(r, r0)]) for r in rho[1:]]
    ok, (l1, h1, l2, h2) = window(n, T, [(e[:, 0], e[:, 2]) for e in (S, e1, e2)], p[:, 0], p[:, 2], r0, rho)
    missed = ~ok | (i1 < l1) | (i1 > h1) | (i2 < l2) | (i2 > h2)
    assert not missed.any(), f"{missed.sum()} of {N}"
