// Index ranges of the kernels that the host can check as they stand: no HIP beyond the qualifiers.
#pragma once

#ifdef __HIPCC__
#define FDTBX_HD __host__ __device__
#else
#define FDTBX_HD
#endif

namespace fdtbx {

// Whether the ring indices jb .. jb + n - 1 of a block meet a lane's jl .. jh.  A lane without a ring
// point in reach carries the range below, which meets no block (as (1, 0) does not: that one counts as
// met by the blocks around 0): it must not widen the block's node window (a lane off the detector has
// R = Z = 0, which widens it to the origin).
constexpr int kNoRingFirst = 1 << 30, kNoRingLast = -(1 << 30);
FDTBX_HD inline bool ring_block_meets(int jl, int jh, int jb, int n) { return jb <= jh && jb + n > jl; }

// Extent of a support along e1 or e2, rho at a reflection of radius r0, as the node windows take it:
// widened by the float32 rounding of the query point's coordinate there, the sum of two products of
// rounded factors, which is off by up to 5 2^-24 of |p| ~ r0 however small it is, 3e-7 r0.  That is
// several nodes of a grid whose half extent is 1e-4 or less.
FDTBX_HD inline double widened_extent(double rho, double r0) { return rho + 1.0e-6 * r0; }

}  // namespace fdtbx
