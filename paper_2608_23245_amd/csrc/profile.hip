// Profile pattern: per pixel, the sum over the reflections of its tile list of
// W_hkl r0^2 sum_k omega_k Z(p* - s_k) (Eq. direct_sum with the lineshape's per-axis
// profile: Eq. I_shape with N -> N_eff, or its Gaussian or Hosemann (Eq. Z) form of the
// same integral breadth), times the Lorentz factor delta/(R + delta) (Eq. lorentz).
//
// Mapping: one to four 64-lane waves per pixel tile (tile_w x 64/tile_w pixels, 8x8 by
// default; the waves split the tile's list), one lane per pixel, pixel sums in
// registers.  Reflections of the tile list are uniform across the wave (their
// records come through scalar loads).  For each (tile, reflection) the wave
// bounds the node window that the tile's query points can reach, builds the
// per-node offsets for 64 window nodes at a time (one node per lane) into LDS, and
// then every lane walks those 64 nodes with broadcast LDS reads.
//
// Per (pixel, reflection) the lattice coordinates are written relative to D so
// that nothing of size h_i is cancelled in float32:
//   y_i = (N_i/2) a_i.(p* - s_k) = alpha_i - kappa_ik,
//   alpha_i = (N_i/2) [(R - R_D)(a_i.e_perp) + (Z - Z_D) a_i,z]           (per pixel)
//   kappa_ik = (N_i r0/2) [(c_k - 1) a_i.S + c_k d1 a_i.e1 + c_k d2 a_i.e2] (per node),
// so that N_i sinc^2(N_i u_i) = N_i sin^2(2 pi y_i)/(2 pi y_i)^2 with the hardware
// sine taking its argument in turns.  Support: max_i |y_i| <= m/2.  The Gaussian
// lineshape uses the same y (N exp(-pi N^2 u^2) = N exp(-4 pi y^2)); the Hosemann one
// writes the record with scale 1 instead of N_i/2 (y_i = u_i, support |y_i| <= 1/2).
#include <hip/hip_runtime.h>

#include <math.h>

#include "internal.h"
#include "profile_common.h"
#include "profile_tile.h"

namespace fdtbx {

// COUNT: counting pass (support test only, the same for every lineshape); LS: lineshape;
// WAVES: waves per tile (each its share of the tile's list).
template <bool COUNT, int LS, int WAVES>
__global__ void __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(7))) k_profile(ProfParams q, const float* __restrict__ refl,
                                                        const float* __restrict__ nodes, const double* __restrict__ pix,
                                                        const double* __restrict__ tile, const int64_t* __restrict__ offsets,
                                                        const int32_t* __restrict__ idx, float* __restrict__ image,
                                                        unsigned long long* __restrict__ counts,
                                                        const int32_t* __restrict__ order) {
  // per wave, the queues of window nodes that can be inside the support of some pixel of the
  // tile (candidates, then those inside the support of every pixel)
  __shared__ float4 qn[256 * WAVES];
  __shared__ int bq[64 * WAVES];
  __shared__ float xacc[WAVES > 1 ? 64 * (WAVES - 1) : 1];
  __shared__ int qk[LS == FDTBX_LINESHAPE_HOSEMANN ? 128 * WAVES : 1];  // node indices (support edge)
  const int t = order ? order[blockIdx.x] : tile_of_block(q, blockIdx.x);
  if (t < 0) return;  // uniform across the workgroup
  profile_tile<COUNT, LS, WAVES>(q, refl, nodes, pix, tile, offsets, idx, image, counts, t, qn, bq, xacc,
                                 LS == FDTBX_LINESHAPE_HOSEMANN ? qk : nullptr);
}

template <int WAVES>
static void launch_profile(const ProfParams& q, dim3 grid, hipStream_t s, const float* refl, const float* nodes,
                           const double* pix, const double* tile, const int64_t* offsets, const int32_t* idx,
                           const int32_t* order, float* image, int64_t* counts) {
  const dim3 block(64 * WAVES);
  unsigned long long* const nc = nullptr;
  if (counts)
    hipLaunchKernelGGL((k_profile<true, FDTBX_LINESHAPE_LAUE, WAVES>), grid, block, 0, s, q, refl, nodes, pix, tile, offsets,
                       idx, image, (unsigned long long*)counts, order);
  else if (q.lineshape == FDTBX_LINESHAPE_GAUSSIAN)
    hipLaunchKernelGGL((k_profile<false, FDTBX_LINESHAPE_GAUSSIAN, WAVES>), grid, block, 0, s, q, refl, nodes, pix, tile,
                       offsets, idx, image, nc, order);
  else if (q.lineshape == FDTBX_LINESHAPE_HOSEMANN)
    hipLaunchKernelGGL((k_profile<false, FDTBX_LINESHAPE_HOSEMANN, WAVES>), grid, block, 0, s, q, refl, nodes, pix, tile,
                       offsets, idx, image, nc, order);
  else
    hipLaunchKernelGGL((k_profile<false, FDTBX_LINESHAPE_LAUE, WAVES>), grid, block, 0, s, q, refl, nodes, pix, tile, offsets,
                       idx, image, nc, order);
}

// Batched models, persistent: every wave takes (model, tile) items from a shared counter
// until the list is exhausted (the exit every wave reaches).
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(6))) k_b_profile(const fdtbx_batch_entry* __restrict__ ent, const int64_t* __restrict__ items,
                                                  int64_t n_items, const float* __restrict__ refl,
                                                  const float* __restrict__ nodes, const double* __restrict__ pix,
                                                  const double* __restrict__ tile, const int64_t* __restrict__ rowptr,
                                                  const int32_t* __restrict__ idx, float* __restrict__ image,
                                                  unsigned long long* __restrict__ counter) {
  __shared__ float4 qn[128];
  __shared__ int bq[64];
  __shared__ int qk[128];  // node indices of the queue (the Hosemann support edge)
  for (int64_t it = blockIdx.x; it < n_items; it = next_item(counter, n_items)) {
    const int64_t packed = items[it];
    const int m = (int)(packed >> 40);
    const int t = (int)(packed & ((1ll << 40) - 1));
    const fdtbx_batch_entry& e = ent[m];
    ProfParams q;
    prof_params(&e.model, &q);
    const float* rf = refl + (int64_t)FDTBX_REFL_FLOATS * e.hkl_off;
    const float* nd = nodes + (int64_t)FDTBX_NODE_FLOATS * e.node_off;
    const double* px = pix + 2 * e.pix_off;
    const double* tb = tile + 8 * e.tile_off;
    const int64_t* rp = rowptr + e.rowptr_off;
    const int32_t* ix = idx + e.pair_off;
    float* im = image + e.pix_off;
    switch (q.lineshape) {  // uniform across the wave
      case FDTBX_LINESHAPE_GAUSSIAN:
        profile_tile<false, FDTBX_LINESHAPE_GAUSSIAN, 1, true, false>(q, rf, nd, px, tb, rp, ix, im, nullptr, t, qn, bq);
        break;
      case FDTBX_LINESHAPE_HOSEMANN:
        profile_tile<false, FDTBX_LINESHAPE_HOSEMANN, 1, true, false>(q, rf, nd, px, tb, rp, ix, im, nullptr, t, qn, bq,
                                                                      nullptr, qk);
        break;
      default:
        profile_tile<false, FDTBX_LINESHAPE_LAUE, 1, true, false>(q, rf, nd, px, tb, rp, ix, im, nullptr, t, qn, bq);
    }
  }
}

// ---------------------------------------------------------------- balanced launch
// The per-tile launch ends with a tail: a tile with a long list runs as one workgroup while
// the compute units around it have drained.  The balanced launch cuts every launched tile's
// list into units, which persistent waves take from queues, eight for each XCD: slot b of the
// per-tile launch order (the tile order of fdtbx_tile_order, whose slot b runs on XCD b % 8) puts
// its tile's units in the queues of XCD b % 8, in slot order (long lists first under the work
// order), so the units of neighbouring tiles still share an XCD's L2.  A wave whose queue is
// empty takes units from the others (for_units).  Each unit writes its 64 pixel sums
// to its own slot of the partial sums, and a second kernel adds a tile's units in unit order:
// the image does not depend on which wave ran which unit.
//
// A pair's share of the time: its set-up, and the nodes of its window, which are scanned and in
// part walked.  (Weights that grow faster with the window, n^1.5 and n^2, measured the same.)
constexpr int kWeightPair = 16;
__device__ inline int pair_weight(const ProfParams& q, const float* __restrict__ rec, const float* __restrict__ nodes,
                                  const TileBox& box) {
  int w01, w23;
  float lo[3], hi[3];
  if (!pair_setup<false>(q, rec, nodes, box, &w01, &w23, lo, hi)) return 2;
  const int n = ((w01 >> 16) - (w01 & 0xffff) + 1) * ((w23 >> 16) - (w23 & 0xffff) + 1);
  return kWeightPair + n;
}

// Whether the lists of n_pairs pairs are cut by weight.  Pairs of one pattern differ a
// hundredfold: a low-order reflection has every node in reach of a tile, most have a few.  Cut
// by their number alone, single units of heavy pairs ran on for 40 % of a launch of 490,639
// Hosemann pairs after the median wave had finished.  Weighing reads every pair's record twice,
// about 40 us per million pairs, and what it saves grows with the nodes of a heavy pair.  Forward
// + adjoint, cut by number / by weight, at 16 nodes per side: 28,657 pairs 0.120 + 0.148 / 0.109 +
// 0.117 ms, 485,808 pairs 0.378 + 0.632 / 0.391 + 0.539, 1.8 million 0.754 + 1.356 / 0.848 +
// 1.204, 7.2 million 2.36 + 4.37 / 2.65 + 4.22; at 64 nodes: 28,657 pairs 1.10 + 1.92 / 0.83 +
// 1.42, 485,808 pairs 3.60 + 7.63 / 2.92 + 6.17, 7.2 million 22.4 + 49.1 / 21.7 + 46.4.
// Longer lists of dense grids would still gain (28.9 million pairs 50.4 + 106 / 49.9 + 103.5, the
// large model 1024 / 1010), but are cut by number as a fixed unit_pairs cuts them: there, and up to
// 8192 pairs, a launch with unit_pairs 0 has the bits of one with fdtbx_unit_pairs, which callers of
// long lists compare.  Between the two limits bit equality needs the same nonzero unit_pairs on both.
static int64_t weigh_most(const ProfParams& q, int64_t fixed_U) {
  return fixed_U > 0 ? -1 : (int64_t)q.n * q.n * 2048;  // 2^19 pairs at 16 nodes per side, 2^23 at 64
}
// Up to 8192 pairs a unit is one pair whatever its weight.
__device__ inline bool weighed(const UnitTable& T, int64_t n_pairs) { return n_pairs > kUnitFew && n_pairs <= T.weigh_most; }

__device__ inline int64_t pairs_per_unit(const UnitTable& T, int64_t n_pairs) {
  return T.fixed_U > 0 ? T.fixed_U : default_unit_pairs(n_pairs);
}

__device__ inline TileBox tile_box(const double* __restrict__ tile, int t) {
  return {tile[8 * (int64_t)t + 0], tile[8 * (int64_t)t + 1], tile[8 * (int64_t)t + 2], tile[8 * (int64_t)t + 3]};
}

// The weight of each position's list, one wave each: its pairs, or where the lists are weighed
// the sum of their weights.  Also clears the queue counters.
__global__ void __launch_bounds__(256) k_unit_weight(ProfParams q, UnitTable T, const int64_t* __restrict__ offsets,
                                                     int64_t n_tiles, const float* __restrict__ refl,
                                                     const float* __restrict__ nodes, const double* __restrict__ tile,
                                                     const int32_t* __restrict__ idx) {
  const int64_t i = launch_index() * 256 + threadIdx.x;
  if (i < kQueues) T.ctr[i * kQueueStride] = 0;
  const int64_t p = i >> 6;
  const int lane = threadIdx.x & 63;
  if (p >= kXcds * T.nj) return;
  const int t = slot_tile(q, T, (p % T.nj) * kXcds + p / T.nj);
  int64_t w = 0;
  if (t >= 0) {
    const int64_t o = offsets[t], e = offsets[t + 1];
    if (weighed(T, offsets[n_tiles])) {
      const TileBox box = tile_box(tile, t);
      for (int64_t k = o + lane; k < e; k += 64) w += pair_weight(q, refl + (int64_t)FDTBX_REFL_FLOATS * idx[k], nodes, box);
      for (int s = 32; s >= 1; s >>= 1) w += __shfl_xor(w, s, 64);
    } else {
      w = e - o;
    }
  }
  if (lane == 0) T.weight[p] = w;
}

// One block: the weight W of a unit, that of as many mean pairs as a unit has, and the first
// unit of each position, which has ceil(weight / W) of them.
__global__ void __launch_bounds__(1024) k_unit_scan(UnitTable T, const int64_t* __restrict__ offsets, int64_t n_tiles) {
  __shared__ int64_t lds[16];
  const int64_t n = kXcds * T.nj, n_pairs = offsets[n_tiles], U = pairs_per_unit(T, n_pairs);
  int64_t W = U;
  if (weighed(T, n_pairs)) {
    int64_t sum = 0, total;
    for (int64_t i = threadIdx.x; i < n; i += 1024) sum += T.weight[i];
    block_exclusive_scan(sum, lds, &total);
    W = max64(1, ceil_div_dev(total, max64(1, n_pairs / U)));
  }
  constexpr int kPer = 8;
  int64_t carry = 0;  // the same in every thread
  for (int64_t b = 0; b < n; b += 1024 * kPer) {
    const int64_t i = b + (int64_t)threadIdx.x * kPer;
    int64_t x[kPer], sum = 0, tot;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      x[k] = i + k < n ? ceil_div_dev(T.weight[i + k], W) : 0;
      sum += x[k];
    }
    int64_t at = carry + block_exclusive_scan(sum, lds, &tot);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      if (i + k < n) T.qscan[i + k] = at;
      at += x[k];
    }
    carry += tot;
  }
  if (threadIdx.x == 0) {
    T.meta[0] = carry;
    T.meta[1] = U;
  }
}

// The number of units of position p.
__device__ inline int64_t units_at(const UnitTable& T, int64_t p) {
  return (p + 1 < kXcds * T.nj ? T.qscan[p + 1] : T.meta[0]) - T.qscan[p];
}

// Each position's units (within the capacity), one wave per position: U pairs each, or where the
// lists are weighed, with n units of a list of weight w, unit k from the first pair with
// n (weight of the pairs before it) >= k w.  The cut depends on the list alone, not on its place
// in the launch.
__global__ void __launch_bounds__(256) k_unit_fill(ProfParams q, UnitTable T, const int64_t* __restrict__ offsets,
                                                   int64_t n_tiles, const float* __restrict__ refl,
                                                   const float* __restrict__ nodes, const double* __restrict__ tile,
                                                   const int32_t* __restrict__ idx) {
  const int64_t p = (launch_index() * 256 + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (p >= kXcds * T.nj) return;
  const int64_t b = (p % T.nj) * kXcds + p / T.nj;
  const int t = slot_tile(q, T, b);
  if (t < 0) return;
  const int64_t s = T.qscan[p], U = T.meta[1], n = min64(units_at(T, p), T.max_units - s);
  const bool by_weight = weighed(T, offsets[n_tiles]);
  for (int64_t k = lane; k < n; k += 64) {
    T.unit_slot[s + k] = (int32_t)b;
    if (!by_weight || k == 0) T.unit_start[s + k] = (int32_t)(k * U);
  }
  if (!by_weight || n <= 1) return;
  const TileBox box = tile_box(tile, t);
  const double per = (double)units_at(T, p) / (double)T.weight[p];
  const int64_t o = offsets[t], len = offsets[t + 1] - o;
  int64_t before = 0;  // weight of the chunks before
  int last = 0;        // unit of the pair before
  for (int64_t k0 = 0; k0 < len; k0 += 64) {
    const int64_t k = k0 + lane;
    const int64_t w = k < len ? pair_weight(q, refl + (int64_t)FDTBX_REFL_FLOATS * idx[o + k], nodes, box) : 0;
    int64_t c = w;
    for (int d = 1; d < 64; d <<= 1) {
      const int64_t y = __shfl_up(c, d, 64);
      if (lane >= d) c += y;
    }
    const int unit = k < len ? (int)min((double)(n - 1), floor((double)(before + c - w) * per)) : (int)n - 1;
    int prev = __shfl_up(unit, 1, 64);
    if (lane == 0) prev = last;
    for (int v = prev + 1; v <= unit; ++v) T.unit_start[s + v] = (int32_t)(k < len ? k : len);
    last = __shfl(unit, 63, 64);
    before += __shfl(c, 63, 64);
  }
  for (int64_t v = last + 1 + lane; v < n; v += 64) T.unit_start[s + v] = (int32_t)len;
}

// Whether the launch splits its walk (SPLIT of pairs_sum): the second queue pays where a pair's
// queue is long, that is with dense node grids.  Forward launch split / not split at 32, 48, 56,
// 64, 96, 128 nodes per side (medium workload cut at 3 A): Laue 9.33/9.05, 17.4/17.2, 22.6/22.6,
// 28.7/28.7, 59.8/62.1, 104.2/108.2 ms; Gaussian 6.16/5.81, 10.41/10.46, 13.2/13.6, 16.4/17.3,
// 34.2/37.3, 58.8/64.7 ms; 0.600/0.571 ms for a draft of 24 nodes per side.  The Hosemann
// lineshape, whose support is one period, is never split (0.415/0.355 ms, the latter at 6 waves
// per SIMD).
constexpr int32_t kSplitNodes = 52;

// Persistent: every wave takes units until none is left (for_units).
template <int LS, bool SPLIT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(LS == FDTBX_LINESHAPE_HOSEMANN ? 6 : 7))) k_profile_units(ProfParams q, const float* __restrict__ refl,
                                                       const float* __restrict__ nodes, const double* __restrict__ pix,
                                                       const double* __restrict__ tile, const int64_t* __restrict__ offsets,
                                                       const int32_t* __restrict__ idx, UnitTable T,
                                                       float* __restrict__ partials) {
  constexpr int kQ = SPLIT ? 256 : 128;  // queue entries per wave
  __shared__ float4 qn[kQ * 4];
  __shared__ int bq[64 * 4];
  __shared__ int qk[LS == FDTBX_LINESHAPE_HOSEMANN ? 128 * 4 : 1];  // node indices (support edge)
  const int wv = (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63);
  const int64_t total = min(T.meta[0], T.max_units);
  for_units(T, total, [&](int64_t u) {
    int64_t p0, p1;
    const int t = unit_range(q, T, offsets, u, total, &p0, &p1);
    if (t < 0) return;
    const TilePixel px = tile_pixel(q, pix, tile, t, lane);
    unsigned long long cnt = 0;
    partials[u * 64 + lane] = pairs_sum<false, LS, false, SPLIT>(q, refl, nodes, idx, px.box, px.R, px.Z, p0, p1, 64, qn + kQ * wv,
                                                   bq + 64 * wv, cnt,
                                                   LS == FDTBX_LINESHAPE_HOSEMANN ? qk + 128 * wv : nullptr);
  });
}

// Per launched tile: its units' pixel sums, times the Lorentz factor, written with the mirror
// folds.  Four waves share a tile, wave w adding the units w, w + 4, ... in order and wave 0 the
// four sums: a tile of few pairs each has many units, and one wave waited for every eight of them
// (64 tiles of 37 units in the mean 20 -> 7 us, 4096 of 130 units 108 -> 39 us).
__global__ void __launch_bounds__(256) k_unit_reduce(ProfParams q, UnitTable T, const double* __restrict__ pix,
                                                     const double* __restrict__ tile, const float* __restrict__ partials,
                                                     float* __restrict__ image) {
  __shared__ float sum[3][64];
  const int64_t b = launch_index();
  const int t = slot_tile(q, T, b);
  if (t < 0) return;  // uniform
  const int lane = (int)threadIdx.x & 63, wv = (int)threadIdx.x >> 6;
  const TilePixel px = tile_pixel(q, pix, tile, t, lane);
  const int64_t n = units_at(T, queue_pos(b, T.nj)), s = T.qscan[queue_pos(b, T.nj)];
  const int64_t n_in = s < 0 ? 0 : (s + n < T.max_units ? n : T.max_units - s);  // within the capacity
  float acc = 0.0f;
#pragma unroll 8
  for (int64_t k = wv; k < n_in; k += 4) acc += partials[(s + k) * 64 + lane];
  if (wv > 0) sum[wv - 1][lane] = acc;
  __syncthreads();
  if (wv > 0 || !px.in) return;
  acc = (acc + sum[0][lane]) + (sum[1][lane] + sum[2][lane]);
  write_folded(q, image, px.i, px.j, px.tx, px.ty, (float)(q.delta / (px.R + q.delta)) * acc);
}

__global__ void k_zero_u64(unsigned long long* v, int n) {
  if ((int)threadIdx.x < n) v[threadIdx.x] = 0ull;
}

static constexpr unsigned kPersistentBlocks = 8192;

int launch_batch_profile(const fdtbx_batch_entry* ent, const int64_t* items, int64_t n_items, const float* refl,
                         const float* nodes, const double* pix, const double* tile, const int64_t* rowptr, const int32_t* idx,
                         float* image, int64_t* counter, hipStream_t s) {
  hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(64), 0, s, (unsigned long long*)counter, 1);
  FDTBX_LAUNCH_CHECK("batch profile counter");
  if (n_items <= 0) return FDTBX_OK;
  unsigned nb = n_items < (int64_t)kPersistentBlocks ? (unsigned)n_items : kPersistentBlocks;
  hipLaunchKernelGGL(k_b_profile, dim3(nb), dim3(64), 0, s, ent, items, n_items, refl, nodes, pix, tile, rowptr, idx, image,
                     (unsigned long long*)counter);
  FDTBX_LAUNCH_CHECK("batch profile");
  return FDTBX_OK;
}

// ---------------------------------------------------------------- batched models on stacked tiles
// Stacked tile s = sy tiles_x + sx holds tile rows 2 sy and 2 sy + 1 (the second when it is
// launched) of tile column sx; its box, row pointers and list start at the model's offsets in soff
// ([m][3]: first box, first row pointer, first list entry; the row pointers are relative to the
// model's first list entry).
struct StackedItem {
  ProfParams q;
  TilePixel a, b;  // the lane's pixels of the two tiles (b far from every reflection if there is one)
  TileBox box;
  const float *rf, *nd;
  const int32_t* ix;
  float* im;
  int64_t p0, p1;  // the stacked tile's list
};

__device__ __forceinline__ void stacked_item(const fdtbx_batch_entry* __restrict__ ent,
                                             const int64_t* __restrict__ soff, int64_t packed,
                                             const float* __restrict__ refl, const float* __restrict__ nodes,
                                             const double* __restrict__ pix, const double* __restrict__ tile,
                                             const double* __restrict__ stile, const int64_t* __restrict__ srowptr,
                                             const int32_t* __restrict__ sidx, float* __restrict__ image,
                                             StackedItem& it) {
  const int lane = threadIdx.x & 63;
  const int m = (int)(packed >> 40);
  const int st = (int)(packed & ((1ll << 40) - 1));
  const fdtbx_batch_entry& e = ent[m];
  prof_params(&e.model, &it.q);
  const double* px = pix + 2 * e.pix_off;
  const double* tb = tile + 8 * e.tile_off;
  const double* sbox = stile + 8 * (soff[3 * m] + st);
  const int64_t* rp = srowptr + soff[3 * m + 1];
  it.ix = sidx + soff[3 * m + 2];
  it.im = image + e.pix_off;
  const int sx = st % it.q.tiles_x, sy = st / it.q.tiles_x;
  const int ta = 2 * sy * it.q.tiles_x + sx;
  const bool two = 2 * sy + 1 < it.q.lrows;  // uniform
  it.a = tile_pixel(it.q, px, tb, ta, lane);
  it.b = tile_pixel(it.q, px, tb, two ? ta + it.q.tiles_x : ta, lane);
  if (!two) {
    it.b.in = false;
    it.b.R = 1.0e30;
    it.b.Z = 0.0;
  }
  it.box = {sbox[0], sbox[1], sbox[2], sbox[3]};
  it.rf = refl + (int64_t)FDTBX_REFL_FLOATS * e.hkl_off;
  it.nd = nodes + (int64_t)FDTBX_NODE_FLOATS * e.node_off;
  it.p0 = rp[st];
  it.p1 = rp[st + 1];
}

// The lane's two pixel sums over pairs p0 .. p1 of the item's list.
__device__ __forceinline__ void stacked_sums(const StackedItem& it, int64_t p0, int64_t p1, float4* qn, int* bq,
                                             int* qk, float* sa, float* sb) {
  switch (it.q.lineshape) {  // uniform across the wave
    case FDTBX_LINESHAPE_GAUSSIAN:
      pairs_sum_stacked<FDTBX_LINESHAPE_GAUSSIAN>(it.q, it.rf, it.nd, it.ix, it.box, it.a.R, it.a.Z, it.b.R, it.b.Z, p0,
                                                  p1, qn, bq, sa, sb);
      break;
    case FDTBX_LINESHAPE_HOSEMANN:
      pairs_sum_stacked<FDTBX_LINESHAPE_HOSEMANN>(it.q, it.rf, it.nd, it.ix, it.box, it.a.R, it.a.Z, it.b.R, it.b.Z, p0,
                                                  p1, qn, bq, sa, sb, qk);
      break;
    default:
      pairs_sum_stacked<FDTBX_LINESHAPE_LAUE>(it.q, it.rf, it.nd, it.ix, it.box, it.a.R, it.a.Z, it.b.R, it.b.Z, p0, p1,
                                              qn, bq, sa, sb);
  }
}

// The item's pixels from their sums, with the Lorentz factor and the mirror folds.
__device__ __forceinline__ void stacked_write(const StackedItem& it, float sa, float sb) {
  const TilePixel &a = it.a, &b = it.b;
  if (a.in) write_folded(it.q, it.im, a.i, a.j, a.tx, a.ty, (float)(it.q.delta / (a.R + it.q.delta)) * sa);
  if (b.in) write_folded(it.q, it.im, b.i, b.j, b.tx, b.ty, (float)(it.q.delta / (b.R + it.q.delta)) * sb);
}

// Every wave takes (model, stacked tile) items as k_b_profile takes tiles.
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(5))) k_b_profile_stacked(
    const fdtbx_batch_entry* __restrict__ ent, const int64_t* __restrict__ soff, const int64_t* __restrict__ items,
    int64_t n_items, const float* __restrict__ refl, const float* __restrict__ nodes, const double* __restrict__ pix,
    const double* __restrict__ tile, const double* __restrict__ stile, const int64_t* __restrict__ srowptr,
    const int32_t* __restrict__ sidx, float* __restrict__ image, unsigned long long* __restrict__ counter) {
  __shared__ float4 qn[128];
  __shared__ int bq[64];
  __shared__ int qk[128];  // node indices of the queue (the Hosemann support edge)
  for (int64_t k = blockIdx.x; k < n_items; k = next_item(counter, n_items)) {
    StackedItem it;
    stacked_item(ent, soff, items[k], refl, nodes, pix, tile, stile, srowptr, sidx, image, it);
    float sa = 0.0f, sb = 0.0f;
    stacked_sums(it, it.p0, it.p1, qn, bq, qk, &sa, &sb);
    stacked_write(it, sa, sb);
  }
}

// The same items cut into units of at most U pairs, one wave each: unit u is the
// (u - unit_ptr[k])-th of item k = unit_item[u] and writes its 128 pixel sums to a slot of its
// own; k_b_unit_reduce adds an item's units in their order.  A list longer than the others (a
// large model's tiles beside the beam hold 50 times the mean) then runs on many waves: with one
// wave per item the longest list took 120 ms, nearly half of a forward of 32 models.  MANY: this launch's
// units start at unit `first` (of a launch that kMaxUnits would not hold); without that scalar the kernel
// keeps its registers for the walk (nine models of up to 192 x 192 pixels 1.13 ms with it, 1.07 without).
constexpr int64_t kMaxUnits = (int64_t{1} << 26) - 1;  // 64 threads each, 2^32 along one dimension
template <bool MANY>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(5))) k_b_profile_units(
    const fdtbx_batch_entry* __restrict__ ent, const int64_t* __restrict__ soff, const int64_t* __restrict__ items,
    const int64_t* __restrict__ unit_ptr, const int32_t* __restrict__ unit_item, int64_t first, int64_t U,
    const float* __restrict__ refl, const float* __restrict__ nodes, const double* __restrict__ pix,
    const double* __restrict__ tile, const double* __restrict__ stile, const int64_t* __restrict__ srowptr,
    const int32_t* __restrict__ sidx, float* __restrict__ image, float* __restrict__ partials) {
  __shared__ float4 qn[128];
  __shared__ int bq[64];
  __shared__ int qk[128];  // node indices of the queue (the Hosemann support edge)
  const int64_t u = MANY ? first + blockIdx.x : blockIdx.x;
  const int k = unit_item[u];
  StackedItem it;
  stacked_item(ent, soff, items[k], refl, nodes, pix, tile, stile, srowptr, sidx, image, it);
  const int64_t p0 = it.p0 + (u - unit_ptr[k]) * U, p1 = p0 + U < it.p1 ? p0 + U : it.p1;
  float sa = 0.0f, sb = 0.0f;
  stacked_sums(it, p0, p1, qn, bq, qk, &sa, &sb);
  float* const o = partials + 128 * u + (threadIdx.x & 63);
  o[0] = sa;
  o[64] = sb;
}

__global__ void __launch_bounds__(64) k_b_unit_reduce(
    const fdtbx_batch_entry* __restrict__ ent, const int64_t* __restrict__ soff, const int64_t* __restrict__ items,
    const int64_t* __restrict__ unit_ptr, const double* __restrict__ pix, const double* __restrict__ tile,
    const double* __restrict__ stile, const int64_t* __restrict__ srowptr, float* __restrict__ image,
    const float* __restrict__ partials) {
  const int64_t k = blockIdx.x;
  StackedItem it;
  stacked_item(ent, soff, items[k], nullptr, nullptr, pix, tile, stile, srowptr, nullptr, image, it);
  float sa = 0.0f, sb = 0.0f;
  const int64_t u1 = unit_ptr[k + 1];
#pragma unroll 8
  for (int64_t u = unit_ptr[k]; u < u1; ++u) {
    const float* const o = partials + 128 * u + (threadIdx.x & 63);
    sa += o[0];
    sb += o[64];
  }
  stacked_write(it, sa, sb);
}

int launch_batch_profile_units(const fdtbx_batch_entry* ent, const int64_t* soff, const int64_t* items,
                               int64_t n_items, const int64_t* unit_ptr, const int32_t* unit_item, int64_t n_units,
                               int64_t unit_pairs, const float* refl, const float* nodes, const double* pix,
                               const double* tile, const double* stile, const int64_t* srowptr, const int32_t* sidx,
                               float* image, float* partials, hipStream_t s) {
  for (int64_t first = 0; first < n_units; first += kMaxUnits) {
    hipLaunchKernelGGL(n_units > kMaxUnits ? k_b_profile_units<true> : k_b_profile_units<false>,
                       dim3((unsigned)min64(n_units - first, kMaxUnits)), dim3(64), 0, s, ent, soff, items, unit_ptr,
                       unit_item, first, unit_pairs, refl, nodes, pix, tile, stile, srowptr, sidx, image, partials);
    FDTBX_LAUNCH_CHECK("batch profile units");
  }
  for (int64_t first = 0; first < n_items; first += kGridRow) {
    hipLaunchKernelGGL(k_b_unit_reduce, dim3((unsigned)min64(n_items - first, kGridRow)), dim3(64), 0, s, ent, soff,
                       items + first, unit_ptr + first, pix, tile, stile, srowptr, image, (const float*)partials);
    FDTBX_LAUNCH_CHECK("batch profile unit sums");
  }
  return FDTBX_OK;
}

int launch_batch_profile_stacked(const fdtbx_batch_entry* ent, const int64_t* soff, const int64_t* items,
                                 int64_t n_items, const float* refl, const float* nodes, const double* pix,
                                 const double* tile, const double* stile, const int64_t* srowptr, const int32_t* sidx,
                                 float* image, int64_t* counter, hipStream_t s) {
  hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(64), 0, s, (unsigned long long*)counter, 1);
  FDTBX_LAUNCH_CHECK("stacked batch profile counter");
  if (n_items <= 0) return FDTBX_OK;
  unsigned nb = n_items < (int64_t)kPersistentBlocks ? (unsigned)n_items : kPersistentBlocks;
  hipLaunchKernelGGL(k_b_profile_stacked, dim3(nb), dim3(64), 0, s, ent, soff, items, n_items, refl, nodes, pix, tile,
                     stile, srowptr, sidx, image, (unsigned long long*)counter);
  FDTBX_LAUNCH_CHECK("stacked batch profile");
  return FDTBX_OK;
}

// The persistent grid: as many 4-wave workgroups as the compute units hold at once.
template <int LS, bool SPLIT>
static int launch_units(const ProfParams& q, const float* refl, const float* nodes, const double* pix,
                        const double* tile, const int64_t* offsets, const int32_t* idx, const UnitTable& T,
                        float* partials, hipStream_t s) {
  int dev = 0, cus = 0, per_cu = 0;
  FDTBX_HIP(hipGetDevice(&dev));
  FDTBX_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  FDTBX_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(&k_profile_units<LS, SPLIT>),
                                                         256, 0));
  const unsigned n_wg = (unsigned)(cus > 0 ? cus : 1) * (unsigned)(per_cu > 0 ? per_cu : 1);
  hipLaunchKernelGGL((k_profile_units<LS, SPLIT>), dim3(n_wg), dim3(256), 0, s, q, refl, nodes, pix, tile, offsets, idx, T,
                     partials);
  FDTBX_LAUNCH_CHECK("balanced profile");
  return FDTBX_OK;
}

size_t balanced_workspace(const fdtbx_model* model, int64_t pair_cap) {
  ProfParams q;
  prof_params(model, &q);
  const int64_t U = model->geom.unit_pairs;
  const UnitLayout a = unit_layout(q, true, pair_cap, U), b = unit_layout(q, false, pair_cap, U);
  return a.total > b.total ? a.total : b.total;
}

int launch_balanced(const fdtbx_model* model, const float* refl, const float* nodes, const double* pix,
                    const double* tile, const int64_t* offsets, const int32_t* idx, const int32_t* order,
                    int64_t pair_cap, float* image, void* ws, size_t ws_bytes, hipStream_t s) {
  ProfParams q;
  prof_params(model, &q);
  const UnitLayout L = unit_layout(q, order != nullptr, pair_cap, model->geom.unit_pairs);
  if (ws_bytes < L.total) return fail(FDTBX_ERR_BUFFER_TOO_SMALL, "balanced profile workspace too small");
  if (L.max_units >= (int64_t{1} << 31) || L.n_slots >= (int64_t{1} << 31))
    return fail(FDTBX_ERR_UNSUPPORTED, "balanced profile: too many units or tiles");
  UnitTable T = unit_view(L, order, model->geom.unit_pairs, ws);
  T.weigh_most = min64(weigh_most(q, model->geom.unit_pairs), pair_cap);  // more pairs than idx holds are not read
  float* partials = (float*)((char*)ws + L.partials);
  const int64_t n_tiles = (int64_t)q.tiles_x * q.tiles_y;
  const dim3 gp = launch_grid(ceil_div(kXcds * L.nj, 4));
  hipLaunchKernelGGL(k_unit_weight, gp, dim3(256), 0, s, q, T, offsets, n_tiles, refl, nodes, tile, idx);
  FDTBX_LAUNCH_CHECK("balanced profile: unit weights");
  hipLaunchKernelGGL(k_unit_scan, dim3(1), dim3(1024), 0, s, T, offsets, n_tiles);
  FDTBX_LAUNCH_CHECK("balanced profile: unit scan");
  hipLaunchKernelGGL(k_unit_fill, gp, dim3(256), 0, s, q, T, offsets, n_tiles, refl, nodes, tile, idx);
  FDTBX_LAUNCH_CHECK("balanced profile: unit fill");
  auto launch = [&](auto units) { return units(q, refl, nodes, pix, tile, offsets, idx, T, partials, s); };
  const bool split = q.n >= kSplitNodes;
  int rc;
  if (q.lineshape == FDTBX_LINESHAPE_GAUSSIAN)
    rc = split ? launch(launch_units<FDTBX_LINESHAPE_GAUSSIAN, true>) : launch(launch_units<FDTBX_LINESHAPE_GAUSSIAN, false>);
  else if (q.lineshape == FDTBX_LINESHAPE_HOSEMANN)
    rc = launch(launch_units<FDTBX_LINESHAPE_HOSEMANN, false>);
  else
    rc = split ? launch(launch_units<FDTBX_LINESHAPE_LAUE, true>) : launch(launch_units<FDTBX_LINESHAPE_LAUE, false>);
  if (rc) return rc;
  hipLaunchKernelGGL(k_unit_reduce, launch_grid(L.n_slots), dim3(256), 0, s, q, T, pix, tile, (const float*)partials,
                     image);
  FDTBX_LAUNCH_CHECK("balanced profile: reduce");
  return FDTBX_OK;
}

}  // namespace fdtbx

using namespace fdtbx;

extern "C" int fdtbx_profile(const fdtbx_model* model, const float* refl, const float* nodes, const double* pix,
                             const double* tile, const int64_t* offsets, const int32_t* idx, const int32_t* order,
                             float* image, int64_t* counts, void* stream) {
  if (!model || !refl || !nodes || !pix || !tile || !offsets || !idx) return fail(FDTBX_ERR_INVALID_ARGUMENT, "null pointer");
  if (!counts && !image) return fail(FDTBX_ERR_INVALID_ARGUMENT, "image is NULL");
  int rc = check_model(model);
  if (rc) return rc;
  ProfParams q;
  prof_params(model, &q);
  hipStream_t s = (hipStream_t)stream;
  const dim3 grid((unsigned)(order ? order_grid(q.lcols, q.lrows) : tile_grid(q)));
  int waves = 1;
  rc = tile_waves(&model->geom, (int64_t)q.lcols * q.lrows, &waves);
  if (rc) return rc;
  if (waves == 4)
    launch_profile<4>(q, grid, s, refl, nodes, pix, tile, offsets, idx, order, image, counts);
  else if (waves == 2)
    launch_profile<2>(q, grid, s, refl, nodes, pix, tile, offsets, idx, order, image, counts);
  else
    launch_profile<1>(q, grid, s, refl, nodes, pix, tile, offsets, idx, order, image, counts);
  FDTBX_LAUNCH_CHECK("profile");
  return FDTBX_OK;
}

extern "C" int64_t fdtbx_unit_pairs(int64_t n_pairs) { return n_pairs < 0 ? 0 : default_unit_pairs(n_pairs); }

extern "C" size_t fdtbx_profile_balanced_workspace(const fdtbx_model* model, int64_t pair_cap) {
  if (!model || pair_cap < 0 || check_model(model)) return 0;
  if (model->geom.unit_pairs < 0) return 0;
  return balanced_workspace(model, pair_cap);
}

extern "C" int fdtbx_profile_balanced(const fdtbx_model* model, const float* refl, const float* nodes,
                                      const double* pix, const double* tile, const int64_t* offsets,
                                      const int32_t* idx, const int32_t* order, int64_t pair_cap, float* image,
                                      void* ws, size_t ws_bytes, void* stream) {
  if (!model || !refl || !nodes || !pix || !tile || !offsets || !idx || !image || !ws)
    return fail(FDTBX_ERR_INVALID_ARGUMENT, "null pointer");
  if (pair_cap < 0) return fail(FDTBX_ERR_INVALID_ARGUMENT, "pair_cap must be non-negative");
  int rc = check_model(model);
  if (rc) return rc;
  if (model->geom.unit_pairs < 0) return fail(FDTBX_ERR_INVALID_ARGUMENT, "unit_pairs must be non-negative");
  return launch_balanced(model, refl, nodes, pix, tile, offsets, idx, order, pair_cap, image, ws, ws_bytes,
                         (hipStream_t)stream);
}
