// Index ranges of the kernels that the host can check as they stand: no HIP beyond the qualifiers.
#pragma once

#ifdef __HIPCC__
#define FDTBX_HD __host__ __device__
#else
#define FDTBX_HD
#endif

namespace fdtbx {

// Whether the ring indices jb .. jb + n - 1 of a block meet a lane's jl .. jh, which is empty where
// jl > jh: such a lane must not widen the block's node window (one off the detector has R = Z = 0,
// which widens it to the origin).
FDTBX_HD inline bool ring_block_meets(int jl, int jh, int jb, int n) { return jl <= jh && jb <= jh && jb + n > jl; }

// Margin of a node window on each side, in nodes of spacing 1/inv_h: what the float32 rounding of its
// bounds can move them by.  A bound is d = (p.e)/(p.S), with p.e the sum of two products of rounded
// factors, whose error is up to 5 2^-24 of |p| ~ p.S however small d is: 3e-7 in d, and 1e-6 here, which
// is 1e-6 inv_h nodes, a fraction of one where the grid is wide and several where it is narrow (half
// extents of 1e-4 and less).  The reciprocals and the place on the grid, a few parts in 10^7 of
// |d| <= 2 T, add less than 1e-3 of a node; the eighth of a node is for them.
FDTBX_HD inline float window_margin(float inv_h) { return 0.125f + 1.0e-6f * inv_h; }

}  // namespace fdtbx
