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

}  // namespace fdtbx
