// Exact cylindrical average of the pattern (Eq. cyl-average): per pixel with ring
// coordinates (R, Z),
//   image = sum_h W_h (1/2 pi) sum_j dphi I_h(p_h(phi_j)),
//   p_h(phi) = R cos(phi) e_perp + R sin(phi) e_az + Z z,   e_az = z x e_perp,
// by the periodic trapezoid rule phi_j = j dphi, dphi = 2 pi/n, n = max(8, ceil(2 pi R/arc)),
// j = -floor(n/2) .. ceil(n/2) - 1, with I_h the shell quadrature of Eq. direct_sum.  Unlike the
// profile kernel (one query point per pixel at each reflection's own azimuth, weighted by the
// Lorentz factor of Eq. lorentz), every point of the ring is visited; no Lorentz factor enters.
//
// Mapping: one to four 64-lane waves per pixel tile (8x8 by default) over the tile's list under the cylindrical
// culling description (fdtbx_cyl_records); where a detector has few tiles, several such
// workgroups per tile.  Per (tile, reflection) each lane bounds the part
// of its ring that can reach the reflection's support (the ball of radius rho_B about D) and
// the wave steps a shared index j over the union of those ranges, kJB indices at a time; the
// 64 x kJB ring points of a step are treated like the splat's samples: node window from their
// coordinates, the node queue of the profile kernel, and kJB evaluations per lane and queued
// node.  cos and sin of j dphi come from a binary64 rotation recurrence per lane.
#include <hip/hip_runtime.h>

#include <math.h>

#include "internal.h"
#include "profile_common.h"
#include "profile_tile.h"
#include "ranges.h"

namespace fdtbx {

struct CylParams {
  ProfParams q;
  double arc;
  int32_t parts;  // workgroups per tile
};

// Ring indices evaluated together: they share the node window, queue and walk.
constexpr int kJB = 8;

// Workgroups per tile (cyl_parts): enough that a detector of few tiles, whose longest lists
// alone decide the time when each tile is one workgroup, still gives every SIMD several waves
// to choose from.  Measured with four waves per workgroup, ms with one / ceil(4096 / tiles) /
// ceil(16384 / tiles) / ceil(65536 / tiles) workgroups per tile: 64x64 pixels (64 tiles)
// 2.88 / 0.29 / 0.18 / 0.18, 224x224 (784) 1.44 / 0.37 / 0.33 / 0.36, 384x384 (2304)
// 4.06 / 2.29 / 1.74 / 1.79; 1024x1024 (16384) is better with one: 140 against 156 with four.
// At most kCylMaxParts: a list of 64x64 pixels has few pairs, and sharing the ring blocks of a
// pair repeats its setup (0.29 ms with 32 parts, 0.18 with 128).  (All measured with a longer
// set-up of a block of ring indices, whose bounds came from every ring point; with those of the
// arc's ends the chosen column is 0.18 / 0.29 / 1.30 ms and the 1024x1024 pixels take 123.)
constexpr int64_t kCylTarget = 16384;
constexpr int64_t kCylMaxParts = 128;

// Waves per SIMD that k_cyl is compiled for.  Its walk is a chain of transcendentals per
// evaluation, and the two waves that its 155 to 210 registers allowed left the SIMDs idle
// between them.  224x224 / 384x384 pixels / 300 reflections over 1024x1024 at three, four and five
// waves: Laue 0.295, 0.285, 0.289 / 1.36, 1.30, 1.34 / 129, 123, 123 ms; Gaussian 0.220, 0.202,
// 0.224 / 1.11, 1.03, 1.07; Hosemann, which spills most, 0.379, 0.395, 0.456 / 1.78, 1.81, 2.18.
__host__ __device__ constexpr int cyl_occupancy(int ls) { return ls == FDTBX_LINESHAPE_HOSEMANN ? 3 : 4; }

// The queue walk of walk_queue, each entry evaluated at the lane's kJB ring points.
template <bool COUNT, int LS>
__device__ __forceinline__ void walk_ring(const float4* qn, int cnt, const float (*al)[3], float half_m,
                                          const HoseK& hk, float& accr, unsigned long long& cnt_eval) {
  qn += threadIdx.y;
  float4 nxt = qn[0];
  float part = 0.0f;
  for (int jj = 0; jj < cnt; ++jj) {
    const float4 cur = nxt;
    nxt = qn[jj + 1];
#pragma unroll
    for (int u = 0; u < kJB; ++u) eval_node<COUNT, LS>(cur, al[u][0], al[u][1], al[u][2], half_m, hk, part, cnt_eval);
  }
  accr += part;
}

// walk_ring for the Hosemann lineshape with its support edge decided in binary64, in the two
// passes of the pattern walks (profile_tile.h): the walk adds the (node, ring point) terms with
// max|y_i| <= lo and marks the queue entries where some lane's ring point falls in the band
// (lo, hi); the second pass decides those in binary64 at ring point jb + u of the lane's ring
// (angle (jb + u) dphi from the reflection's azimuth), node index qk[jj].
__device__ __forceinline__ void walk_ring_edge(const ProfParams& q, const float4* qn, const int* qk, int cnt,
                                               const float (*al)[3], float lo, float hi, const HoseK& hk,
                                               const float* rec, double R, double Z, int jb, double dphi,
                                               float& accr) {
  const float4* const q0 = qn;
  qn += threadIdx.y;
  float4 nxt = qn[0];
  float part = 0.0f;
  unsigned long long um = 0;
  for (int jj = 0; jj < cnt; ++jj) {
    const float4 cur = nxt;
    nxt = qn[jj + 1];
    unsigned long long band = 0;
#pragma unroll
    for (int u = 0; u < kJB; ++u) {
      const float ya = al[u][0] - cur.x, yb = al[u][1] - cur.y, yc = al[u][2] - cur.z;
      const float mx = fmaxf(fmaxf(fabsf(ya), fabsf(yb)), fabsf(yc));
      const bool sure = mx <= lo;
      band |= __builtin_amdgcn_ballot_w64(mx < hi) & ~__builtin_amdgcn_ballot_w64(sure);
      if (sure) part = fmaf(cur.w, hose_prod(ya, yb, yc, hk), part);
    }
    um = band ? um | (1ull << jj) : um;
  }
  accr += part;
  float fix = 0.0f;
  const double RD = *(const double*)(rec + RS_RD), dZ = Z - *(const double*)(rec + RS_ZD);
  while (um) {  // uniform
    const int jj = (int)__builtin_ctzll(um);
    um &= um - 1;
    const float4 nd = q0[jj];
    const int k = qk[jj];
#pragma unroll 1
    for (int u = 0; u < kJB; ++u) {
      const float ya = al[u][0] - nd.x, yb = al[u][1] - nd.y, yc = al[u][2] - nd.z;
      const float mx = fmaxf(fmaxf(fabsf(ya), fabsf(yb)), fabsf(yc));
      if (hose_band(mx, lo, hi)) {
        const double ph = (double)(jb + u) * dphi;
        if (hose_inside64(q, rec, k, R * cos(ph) - RD, R * sin(ph), dZ)) fix = fmaf(nd.w, hose_prod(ya, yb, yc, hk), fix);
      }
    }
  }
  accr += fix;
}

// A tile's work is the pairs of its list times the blocks of kJB ring indices of each.
// p.parts workgroups share it: with L pairs, part k takes the pairs k, k + G, ... for
// G = min(parts, L), and where the list is shorter than the parts, parts / G workgroups share
// the ring blocks of a pair as well.  Within a part, wave w of its WAVES takes every
// (WAVES parts / G)-th block (its own LDS queue); wave 0 adds the others' pixel sums in wave
// order, and k_cyl_sum the parts in part order, so the result does not depend on the launch.
template <bool COUNT, int LS, int WAVES>
__global__ void __launch_bounds__(64 * WAVES, cyl_occupancy(LS)) k_cyl(CylParams p, const float* __restrict__ refl,
                                                    const float* __restrict__ nodes, const double* __restrict__ pix,
                                                    const int64_t* __restrict__ offsets, const int32_t* __restrict__ idx,
                                                    float* __restrict__ image, unsigned long long* __restrict__ counts,
                                                    const int32_t* __restrict__ order, float* __restrict__ sums) {
  // the Hosemann support edge is decided in binary64 (walk_ring_edge): the queue then carries
  // its node indices in qk
  constexpr bool EDGE = LS == FDTBX_LINESHAPE_HOSEMANN && !COUNT;
  __shared__ float4 qn_all[128 * WAVES];
  __shared__ int bq_all[64 * WAVES];
  __shared__ float xacc[WAVES > 1 ? 64 * (WAVES - 1) : 1];
  __shared__ int qk_all[EDGE ? 128 * WAVES : 1];
  const ProfParams& q = p.q;
  const int lane = threadIdx.x & 63;
  const int wv = WAVES > 1 ? (int)(threadIdx.x >> 6) : 0;
  float4* const qn = qn_all + 128 * wv;
  int* const bq = bq_all + 64 * wv;
  int* const qk = qk_all + (EDGE ? 128 * wv : 0);
  // the parts of a tile are consecutive, so that the tiles with the longest lists, first in the
  // order, also start first
  const int part = p.parts > 1 ? (int)(blockIdx.x % (unsigned)p.parts) : 0;
  const unsigned slot = p.parts > 1 ? blockIdx.x / (unsigned)p.parts : blockIdx.x;
  const int t = order ? order[slot] : tile_of_block(q, slot);
  if (t < 0) return;  // uniform across the workgroup
  const int tx = t % q.tiles_x, ty = t / q.tiles_x;
  const int pi_ = (tx << q.tlg) + (lane & ((1 << q.tlg) - 1));
  const int pj = ty * (64 >> q.tlg) + (lane >> q.tlg);
  const bool in = pi_ < q.W && pj < q.H;
  const double R = in ? pix[2 * ((int64_t)pj * q.W + pi_) + 0] : 0.0;
  const double Z = in ? pix[2 * ((int64_t)pj * q.W + pi_) + 1] : 0.0;
  // periodic trapezoid rule over this pixel's ring
  const double nf = ceil(2.0 * M_PI * R / p.arc);
  const int n = nf < 8.0 ? 8 : (int)nf;
  const double dphi = 2.0 * M_PI / (double)n;
  const int ring_lo = -(n / 2), ring_hi = n - n / 2 - 1;
  const double cd = cos(dphi), sd = sin(dphi);
  const float sag = (float)(R * (1.0 - cos(0.5 * (kJB - 1) * dphi)) * 1.0001);
  const int64_t p0 = offsets[t], p1 = offsets[t + 1];
  const int groups = p1 - p0 < p.parts ? (p1 > p0 ? (int)(p1 - p0) : 1) : p.parts;
  const int ring_parts = p.parts / groups;
  const int first = WAVES * (part / groups) + wv, stride = WAVES * ring_parts;  // in ring blocks
  const bool idle = part / groups >= ring_parts;
  // rotation over the blocks of the other waves
  const double cw = cos((double)(kJB * (stride - 1)) * dphi);
  const double sw = sin((double)(kJB * (stride - 1)) * dphi);
  float acc = 0.0f;
  unsigned long long cnt = 0;
  int64_t pp = p0 + (idle ? p1 - p0 : part % groups);
  int32_t r_next = pp < p1 ? idx[pp] : 0;
  for (; pp < p1; pp += groups) {
    const int32_t r = r_next;
    r_next = idx[pp + groups < p1 ? pp + groups : pp];
    const float* rec = refl + (int64_t)FDTBX_REFL_FLOATS * r;
    PairRec f;
    load_pair(rec, f);
    static_assert(RS_AZ == 31 && RS_TA == 34, "the load below reads slots 32..35 as e_az.e1, e_az.e2, TA_0, TA_1");
    const float4 x1 = *(const float4*)(rec + 32);
    const float az[3] = {f.at(RS_AZ), x1.x, x1.y};
    const float ta[3] = {x1.z, x1.w, rec[RS_TA + 2]};
    const double RD = f.at_f64(RS_RD), ZD = f.at_f64(RS_ZD);
    float Bv[3], G1[3], G2[3], tr[3], tz[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      Bv[a] = f.at(RS_B + a);
      G1[a] = f.at(RS_G1 + a);
      G2[a] = f.at(RS_G2 + a);
      tr[a] = f.at(RS_TR + a);
      tz[a] = f.at(RS_TZ + a);
    }
    // ring points within rho_B of D: |p(phi) - D|^2 = R^2 + R_D^2 + (Z - Z_D)^2 - 2 R R_D cos(phi)
    const float rS = f.at(RS_RHO), r1 = f.at(RS_RHO + 1), r2 = f.at(RS_RHO + 2);
    const float r0 = f.at(RS_R0);
    const double rhoB = ((double)(2.0f * r0 * sqrtf(0.5f * (1.0f - q.cmin))) + (double)sqrtf(rS * rS + r1 * r1 + r2 * r2)) *
                            1.001 + 1.0e-7;
    int jl = kNoRingFirst, jh = kNoRingLast;
    if (in) {
      const double dz = Z - ZD;
      const double num = ((R * R + RD * RD) + dz * dz) - rhoB * rhoB;
      const double den = 2.0 * R * RD;
      if (!(den > 0.0)) {
        if (num <= 0.0) {
          jl = ring_lo;
          jh = ring_hi;
        }
      } else {
        const double cmin = num / den;
        if (cmin <= -1.0) {
          jl = ring_lo;
          jh = ring_hi;
        } else if (cmin < 1.0) {
          const int jm = (int)floor(acos(cmin) / dphi) + 1;
          jl = max(ring_lo, -jm);
          jh = min(ring_hi, jm);
        }
      }
    }
    const int J0 = wave_min_i32(jl), J1 = wave_max_i32(jh);
    if (J0 > J1) continue;
    HoseK hk = {};
    if (LS == FDTBX_LINESHAPE_HOSEMANN && !COUNT) hose_constants(rec, hk);
    // the edge band (profile_tile.h) for y_i = T_R,i (R cos phi - R_D) + T_A,i R sin phi +
    // T_Z,i (Z - Z_D) - kappa_i, with |R cos phi - R_D| <= R + |R_D| and |R sin phi| <= R
    float elo = 0.0f, ehi = 0.0f;
    if (EDGE) {
      const float mX = wave_max(in ? (float)(R + fabs(RD)) : 0.0f), mY = wave_max(in ? (float)R : 0.0f);
      const float mZ = wave_max(in ? (float)fabs(Z - ZD) : 0.0f);
      float mag = 0.0f;
#pragma unroll
      for (int a = 0; a < 3; ++a)
        mag = fmaxf(mag, fabsf(tr[a]) * mX + fabsf(ta[a]) * mY + fabsf(tz[a]) * mZ + fabsf(Bv[a]) + fabsf(G1[a]) +
                             fabsf(G2[a]));
      const float band = fmaxf(1.0e-6f, mag * 0x1p-20f);
      elo = q.half_m - band;
      ehi = q.half_m + band;
    }
    double cj = cos((double)(J0 + kJB * first) * dphi), sj = sin((double)(J0 + kJB * first) * dphi);
    const float fZ = (float)(Z - ZD), fz = (float)Z;
    const float vz[3] = {tz[0] * fZ, tz[1] * fZ, tz[2] * fZ};
    float accp = 0.0f;
    // kJB consecutive ring indices share one node window, queue and walk.  With 64 lanes of
    // eight points a block's set-up is a large part of its time, so its bounds come from the arc's
    // ends alone (0.33 -> 0.29 ms at 224x224 pixels, 1.72 -> 1.30 at 384x384).
    for (int jb = J0 + kJB * first; jb <= J1; jb += kJB * stride) {
      float al[kJB][3];
      // the ends of the block's arc: al and the coordinates along S, e1, e2
      float ae[2][3], pe[2][3];
#pragma unroll
      for (int u = 0; u < kJB; ++u) {
        const int jj = jb + u;
        const bool act = jj >= jl && jj <= jh;  // jl > jh where the lane has no ring point in reach
        const double X = R * cj, Y = R * sj;
        const float fX = (float)(X - RD), fY = (float)Y;
        float v[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          v[a] = fmaf(tr[a], fX, fmaf(ta[a], fY, vz[a]));
          al[u][a] = LS == FDTBX_LINESHAPE_LAUE ? tag_alpha(v[a]) : v[a];
        }
        al[u][0] = act ? al[u][0] : 1.0e30f;
        if (u == 0 || u == kJB - 1) {
          const int e = u ? 1 : 0;
          const float Rc = (float)X;
          pe[e][0] = fmaf(Rc, f.at(RS_CS), fmaf(fY, az[0], fz * f.at(RS_CS + 1)));
          pe[e][1] = fmaf(Rc, f.at(RS_C1), fmaf(fY, az[1], fz * f.at(RS_C1 + 1)));
          pe[e][2] = fmaf(Rc, f.at(RS_C2), fmaf(fY, az[2], fz * f.at(RS_C2 + 1)));
#pragma unroll
          for (int a = 0; a < 3; ++a) ae[e][a] = v[a];
        }
        const double cn = fma(cj, cd, -(sj * sd));
        sj = fma(sj, cd, cj * sd);
        cj = cn;
      }
      if (stride > 1) {
        const double cn = fma(cj, cw, -(sj * sw));
        sj = fma(sj, cw, cj * sw);
        cj = cn;
      }
      // a coordinate of the ring is a sinusoid of the azimuth: over an arc of half-angle d it stays
      // within its amplitude times 1 - cos d of its values at the arc's ends
      const bool reach = ring_block_meets(jl, jh, jb, kJB);
      float lo[3], hi[3], pl[3], ph[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const float da = sag * (fabsf(tr[a]) + fabsf(ta[a]));
        lo[a] = wave_min(reach ? fminf(ae[0][a], ae[1][a]) - da : INFINITY) - q.half_m - q.margin;
        hi[a] = wave_max(reach ? fmaxf(ae[0][a], ae[1][a]) + da : -INFINITY) + q.half_m + q.margin;
        pl[a] = wave_min(reach ? fminf(pe[0][a], pe[1][a]) - sag : INFINITY);
        ph[a] = wave_max(reach ? fmaxf(pe[0][a], pe[1][a]) + sag : -INFINITY);
      }
      Window w;
      if (node_window_ranges(q, r0, pl[0], ph[0], pl[1], ph[1], pl[2], ph[2], rS, r1, r2, &w)) {
        float accr = 0.0f;
        int qlen = 0;  // uniform
        scan_window(q, nodes, w, Bv, G1, G2, lo, hi, bq, [&](bool keep, int k, float4 e) {
          const unsigned long long bal = __ballot(keep);
          if (keep) {
            const int pos = qlen + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(bal >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0u));
            qn[pos] = LS == FDTBX_LINESHAPE_LAUE ? tag_kappa4(e) : e;
            if (EDGE) qk[pos] = k;
          }
          qlen += __popcll(bal);
          wave_sync();
          if (qlen >= 64) {
            if (EDGE)
              walk_ring_edge(q, qn, qk, 64, al, elo, ehi, hk, rec, R, Z, jb, dphi, accr);
            else
              walk_ring<COUNT, LS>(qn, 64, al, q.half_m, hk, accr, cnt);
            qlen -= 64;
            wave_sync();
            if (lane < qlen) {
              qn[lane] = qn[64 + lane];
              if (EDGE) qk[lane] = qk[64 + lane];
            }
            wave_sync();
          }
        });
        if (EDGE)
          walk_ring_edge(q, qn, qk, qlen, al, elo, ehi, hk, rec, R, Z, jb, dphi, accr);
        else
          walk_ring<COUNT, LS>(qn, qlen, al, q.half_m, hk, accr, cnt);
        wave_sync();
        accp += accr;
      }
    }
    acc = fmaf(f.at(RS_WK), accp, acc);
  }
  if (COUNT) {
    for (int o = 32; o >= 1; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
    if (lane == 0 && cnt) atomicAdd(counts, cnt);
  } else {
    if (WAVES > 1) {
      if (wv > 0) xacc[64 * (wv - 1) + lane] = acc;
      __syncthreads();
      if (wv > 0) return;
      for (int k = 1; k < WAVES; ++k) acc += xacc[64 * (k - 1) + lane];
    }
    acc *= (float)(dphi / (2.0 * M_PI));
    if (p.parts > 1)
      sums[64 * ((int64_t)part * q.lcols * q.lrows + (int64_t)ty * q.lcols + tx) + lane] = acc;
    else if (in)
      write_folded(q, image, pi_, pj, tx, ty, acc);
  }
}

// The parts' sums of each launched tile (one lane per pixel), added in part order.
__global__ void __launch_bounds__(256) k_cyl_sum(ProfParams q, int parts, const float* __restrict__ sums,
                                                 float* __restrict__ image) {
  const int64_t n = 64 * (int64_t)q.lcols * q.lrows, i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int tile = (int)(i >> 6), lane = (int)(i & 63);
  const int tx = tile % q.lcols, ty = tile / q.lcols;
  const int pi_ = (tx << q.tlg) + (lane & ((1 << q.tlg) - 1));
  const int pj = ty * (64 >> q.tlg) + (lane >> q.tlg);
  if (pi_ >= q.W || pj >= q.H) return;
  float acc = 0.0f;
#pragma unroll 8
  for (int k = 0; k < parts; ++k) acc += sums[n * k + i];
  write_folded(q, image, pi_, pj, tx, ty, acc);
}

// Workgroups per tile: a rule on the detector's tiles, folded or not, so that a folded image
// has the sums of the unfolded one.
static int cyl_parts(const fdtbx_geometry* g) {
  const int64_t tiles = (int64_t)tiles_x_of(g) * tiles_y_of(g);
  const int64_t want = ceil_div(kCylTarget, tiles);
  return (int)(want < kCylMaxParts ? want : kCylMaxParts);
}

__global__ void k_zero_count(unsigned long long* c) {
  if (threadIdx.x == 0) *c = 0ull;
}

template <int WAVES>
static void launch_cyl(const CylParams& p, dim3 grid, hipStream_t s, const float* refl, const float* nodes,
                       const double* pix, const int64_t* offsets, const int32_t* idx, const int32_t* order, float* image,
                       unsigned long long* counts, float* sums) {
  const dim3 block(64 * WAVES);
  if (counts)
    hipLaunchKernelGGL((k_cyl<true, FDTBX_LINESHAPE_LAUE, WAVES>), grid, block, 0, s, p, refl, nodes, pix, offsets, idx, image,
                       counts, order, sums);
  else if (p.q.lineshape == FDTBX_LINESHAPE_GAUSSIAN)
    hipLaunchKernelGGL((k_cyl<false, FDTBX_LINESHAPE_GAUSSIAN, WAVES>), grid, block, 0, s, p, refl, nodes, pix, offsets, idx,
                       image, counts, order, sums);
  else if (p.q.lineshape == FDTBX_LINESHAPE_HOSEMANN)
    hipLaunchKernelGGL((k_cyl<false, FDTBX_LINESHAPE_HOSEMANN, WAVES>), grid, block, 0, s, p, refl, nodes, pix, offsets, idx,
                       image, counts, order, sums);
  else
    hipLaunchKernelGGL((k_cyl<false, FDTBX_LINESHAPE_LAUE, WAVES>), grid, block, 0, s, p, refl, nodes, pix, offsets, idx, image,
                       counts, order, sums);
}

}  // namespace fdtbx

using namespace fdtbx;

static int profile_cyl(const fdtbx_model* model, const float* refl, const float* nodes, const double* pix,
                       const int64_t* offsets, const int32_t* idx, const int32_t* order, double arc, float* image,
                       int64_t* counts, int parts, float* sums, void* stream) {
  if (!(arc >= 1.0e-5 && arc < 1.0)) return fail(FDTBX_ERR_INVALID_ARGUMENT, "arc must be in [1e-5, 1) 1/A");
  CylParams p;
  prof_params(model, &p.q);
  p.arc = arc;
  p.parts = parts;
  // without an order: the plain tile order (the ring work of a few reflections concentrates on
  // a few superblocks, which the spatially grouped order would pile onto few XCDs)
  p.q.sbw = 0;
  hipStream_t s = (hipStream_t)stream;
  const int64_t tiles = (int64_t)p.q.lcols * p.q.lrows;
  const dim3 grid((unsigned)(parts * (order ? order_grid(p.q.lcols, p.q.lrows) : tile_grid(p.q))));
  unsigned long long* cp = (unsigned long long*)counts;
  if (counts) {
    hipLaunchKernelGGL(k_zero_count, dim3(1), dim3(64), 0, s, cp);
    FDTBX_LAUNCH_CHECK("cylindrical average counter");
  }
  int waves = 1;
  const int rc = tile_waves(&model->geom, tiles, &waves);
  if (rc) return rc;
  if (waves == 4)
    launch_cyl<4>(p, grid, s, refl, nodes, pix, offsets, idx, order, image, cp, sums);
  else if (waves == 2)
    launch_cyl<2>(p, grid, s, refl, nodes, pix, offsets, idx, order, image, cp, sums);
  else
    launch_cyl<1>(p, grid, s, refl, nodes, pix, offsets, idx, order, image, cp, sums);
  FDTBX_LAUNCH_CHECK("cylindrical average");
  if (!counts && parts > 1) {
    hipLaunchKernelGGL(k_cyl_sum, dim3((unsigned)ceil_div(64 * tiles, 256)), dim3(256), 0, s, p.q, parts, sums, image);
    FDTBX_LAUNCH_CHECK("cylindrical average sum");
  }
  return FDTBX_OK;
}

extern "C" int fdtbx_profile_cyl(const fdtbx_model* model, const float* refl, const float* nodes, const double* pix,
                                 const int64_t* offsets, const int32_t* idx, const int32_t* order, double arc, float* image,
                                 int64_t* counts, void* stream) {
  if (!model || !refl || !nodes || !pix || !offsets || !idx) return fail(FDTBX_ERR_INVALID_ARGUMENT, "null pointer");
  if (!counts && !image) return fail(FDTBX_ERR_INVALID_ARGUMENT, "image is NULL");
  const int rc = check_model(model);
  if (rc) return rc;
  return profile_cyl(model, refl, nodes, pix, offsets, idx, order, arc, image, counts, 1, nullptr, stream);
}

extern "C" size_t fdtbx_cyl_workspace(const fdtbx_geometry* geom) {
  if (!geom || check_geometry(geom) != FDTBX_OK) return 0;
  const int parts = cyl_parts(geom);
  return parts > 1 ? (size_t)parts * lcols_of(geom) * lrows_of(geom) * 64 * sizeof(float) : 0;
}

extern "C" int fdtbx_profile_cyl_split(const fdtbx_model* model, const float* refl, const float* nodes, const double* pix,
                                       const int64_t* offsets, const int32_t* idx, const int32_t* order, double arc,
                                       float* image, void* ws, size_t ws_bytes, void* stream) {
  if (!model || !refl || !nodes || !pix || !offsets || !idx || !image)
    return fail(FDTBX_ERR_INVALID_ARGUMENT, "null pointer");
  const int rc = check_model(model);
  if (rc) return rc;
  const size_t need = fdtbx_cyl_workspace(&model->geom);
  if (ws_bytes < need || (need && !ws)) return fail(FDTBX_ERR_BUFFER_TOO_SMALL, "cylindrical average workspace too small");
  return profile_cyl(model, refl, nodes, pix, offsets, idx, order, arc, image, nullptr, cyl_parts(&model->geom), (float*)ws,
                     stream);
}
