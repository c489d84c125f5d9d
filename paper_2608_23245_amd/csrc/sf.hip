// Direct structure factors (Eq. structure_factor with the isotropic Debye-Waller
// factor):  F_hkl = sum_j occ_j f_t(j)(s) exp(-B_j s^2) exp(2 pi i (h x_j + k y_j + l z_j)).
//
// A thread takes one or two reflections, atoms streamed through LDS in groups of 256; the atom
// range is split over gridDim.y so that small reflection lists still fill the chip.
// The phase h x + k y + l z is formed in binary64 (exact: integer times float32),
// reduced modulo one turn there and only then rounded to float32, so the argument
// of the hardware sine/cosine (which take revolutions) carries ~1.5e-8 turns of error
// whatever the size of h.  The sums of each atom chunk are reduced in a fixed order
// in binary64: deterministic, no atomics.
//
// F(-h) = conj F(h): an enumerated list is symmetric, reflection n - 1 - i being the Friedel
// mate of reflection i, so a block of the first half writes the second half's sums too after it
// has compared the indices; where a block's mates are not mates, it evaluates them as well, or
// where the launch is short a second block does (blockIdx.z).
//
// Bound: the vector instructions of a term, 6 binary64 ones of 5 cycles per wave and SIMD, 3
// transcendentals of 8.4 and 7 float32 ones of 2.6, or 73 cycles; 73 are reached.  The inner
// loop reads the coordinates from LDS as binary64, converted once per atom and block.
// 293298 reflections of 50000 atoms take 3.4 ms, 6.4 when every reflection was evaluated; one
// binary64 operation less, the phase's fraction in [0, 1) by v_fract_f64, takes 3.2 ms, but the
// gradients of a small refinement step are then a fifth further off.
#include <hip/hip_runtime.h>

#include <math.h>

#include "internal.h"

namespace fdtbx {

static constexpr int kSFThreads = 256;
static constexpr int kMaxTypes = 16;
// Atoms summed in float32 before they are added in binary64.  The float32 sums of a whole chunk
// were most of the error: 1.7e-7 to 6.4e-7 of |F| for 160 to 30000 atoms, 1.0e-7 to 1.6e-7 so.
static constexpr int kSFGroup = 8;
static constexpr int64_t kSFBlocks = 2048;  // eight blocks on each of the chip's 256 compute units
// Up to here the blocks of both halves fit on the chip together, and the second half has blocks of
// its own, which end at once where the mates are mates.  One after the other / side by side, the
// mates no mates: 1000 reflections of 5000 atoms 21.1 / 18.4 us (with mates 18.0 / 17.8), 10000 of
// 1000 21.4 / 17.8, 5000 of 5000 36.0 / 31.9; with 2051 blocks the ended ones cost more than they
// gain (150000 of 5000, with mates: 214 / 224).
static constexpr int64_t kSFBothHalves = kSFBlocks / 2;

struct SFParams {
  double as[9];          // reciprocal basis rows a*, b*, c*
  int64_t n_hkl, n_atoms, chunk;
  int32_t n_types, n_chunks;
};

// The group of atoms in LDS: 36 bytes per atom, read as two 16-byte words and the type.
struct AtomsLds {
  double2 xy[kSFThreads];
  struct alignas(16) {
    double z;
    float nBl2e, occ;
  } zb[kSFThreads];
  int type[kSFThreads];  // its row of the form-factor table

  __device__ __forceinline__ void put(int i, const float* x, const float* y, const float* z, const float* B, const float* o,
                                      const int32_t* ty, int64_t j, int n_types, int row) {
    int t = ty[j];
    t = t < 0 ? 0 : (t >= n_types ? n_types - 1 : t);
    xy[i] = make_double2((double)x[j], (double)y[j]);
    zb[i] = {(double)z[j], -B[j] * 1.4426950408889634f, o[j]};
    type[i] = t * row;
  }
};

// The phase of a term, h x + k y + l z to the nearest turn: at most half a turn either way, so that
// its float32 rounding is half that of a phase in [0, 1).
__device__ __forceinline__ float sf_phase(double h, double k, double l, double2 xy, double z) {
  const double ph = fma(h, xy.x, fma(k, xy.y, l * z));
  return (float)(ph - rint(ph));
}

__device__ __forceinline__ float form_factor(const float* c, double s2) {
  double f = c[8];
  for (int g = 0; g < 4; ++g) f += (double)c[g] * exp(-(double)c[4 + g] * s2);
  return (float)f;
}

// K reflections per thread, 256 apart, of the list's first half: block b, thread t takes
// 256 K b + 256 k + t, and their mates.
template <int K>
__global__ void __launch_bounds__(kSFThreads) k_sf_partial(SFParams p, const float* __restrict__ x, const float* __restrict__ y,
                                                           const float* __restrict__ z, const float* __restrict__ B,
                                                           const float* __restrict__ occ, const int32_t* __restrict__ type,
                                                           const float* __restrict__ ff, const int32_t* __restrict__ hkl,
                                                           float2* __restrict__ part) {
  __shared__ AtomsLds at;
  extern __shared__ float ftab[];  // [n_types][256][K]
  const int64_t half = (p.n_hkl + 1) / 2;
  const int64_t i0 = (int64_t)blockIdx.x * (K * kSFThreads) + threadIdx.x;
  part += (int64_t)blockIdx.y * p.n_hkl;
  bool mates = true;
  for (int k = 0; k < K; ++k) {
    const int64_t i = i0 + k * kSFThreads, j = p.n_hkl - 1 - i;
    if (i < half && j != i)
      for (int c = 0; c < 3; ++c) mates = mates && (int64_t)hkl[3 * i + c] + (int64_t)hkl[3 * j + c] == 0;
  }
  mates = __syncthreads_and(mates);
  const int64_t a0 = (int64_t)blockIdx.y * p.chunk;
  const int64_t a1 = a0 + p.chunk < p.n_atoms ? a0 + p.chunk : p.n_atoms;
  for (int second = (int)blockIdx.z; second < (mates ? 1 : 2); second += (int)gridDim.z) {  // uniform
    double h[K], kk[K], l[K];
    float s2[K];
    double re[K], im[K];
    bool any = false;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int64_t i = i0 + k * kSFThreads, r = second ? p.n_hkl - 1 - i : i;
      const bool have = i < half && !(second && r == i);
      any = any || have;
      h[k] = have ? hkl[3 * r + 0] : 0;
      kk[k] = have ? hkl[3 * r + 1] : 0;
      l[k] = have ? hkl[3 * r + 2] : 0;
      double D[3];
      for (int j = 0; j < 3; ++j) D[j] = (h[k] * p.as[j] + kk[k] * p.as[3 + j]) + l[k] * p.as[6 + j];
      const double s2d = 0.25 * ((D[0] * D[0] + D[1] * D[1]) + D[2] * D[2]);
      s2[k] = (float)s2d;
      re[k] = im[k] = 0.0;
      for (int t = 0; t < p.n_types; ++t) ftab[(t * kSFThreads + threadIdx.x) * K + k] = form_factor(ff + 9 * t, s2d);
    }
    for (int64_t g0 = a0; g0 < a1; g0 += kSFThreads) {
      __syncthreads();
      if (g0 + threadIdx.x < a1) at.put(threadIdx.x, x, y, z, B, occ, type, g0 + threadIdx.x, p.n_types, kSFThreads * K);
      __syncthreads();
      const int cnt = (int)((a1 - g0) < kSFThreads ? (a1 - g0) : kSFThreads);
      if (any) {
        float gr[K], gi[K];
        auto term = [&](int i) {
          const double2 xy = at.xy[i];
          const auto zb = at.zb[i];
          const float* f = ftab + at.type[i] + threadIdx.x * K;
#pragma unroll
          for (int k = 0; k < K; ++k) {
            const float fr = sf_phase(h[k], kk[k], l[k], xy, zb.z);
            const float amp = zb.occ * f[k] * __builtin_amdgcn_exp2f(zb.nBl2e * s2[k]);
            gr[k] = fmaf(amp, __builtin_amdgcn_cosf(fr), gr[k]);
            gi[k] = fmaf(amp, __builtin_amdgcn_sinf(fr), gi[k]);
          }
        };
        auto clear = [&] {
#pragma unroll
          for (int k = 0; k < K; ++k) gr[k] = gi[k] = 0.0f;
        };
        auto add = [&] {
#pragma unroll
          for (int k = 0; k < K; ++k) {
            re[k] += (double)gr[k];
            im[k] += (double)gi[k];
          }
        };
        const int full = cnt / kSFGroup * kSFGroup;
        for (int i0 = 0; i0 < full; i0 += kSFGroup) {
          clear();
#pragma unroll 4
          for (int i = i0; i < i0 + kSFGroup; ++i) term(i);
          add();
        }
        if (full < cnt) {
          clear();
#pragma unroll 1
          for (int i = full; i < cnt; ++i) term(i);
          add();
        }
      }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int64_t i = i0 + k * kSFThreads, j = p.n_hkl - 1 - i;
      if (i >= half) continue;
      const float r32 = (float)re[k], i32 = (float)im[k];
      if (!second) part[i] = make_float2(r32, i32);
      if (j != i && (second || mates)) part[j] = make_float2(r32, second ? i32 : -i32);
    }
  }
}

// The chunks' sums, added in order, eight loads in flight (one at a time waited 0.25 us for each:
// 50 reflections of 50000 atoms, 782 chunks, 205 us with the sums before it, 46 so).
__global__ void k_sf_final(int64_t n_hkl, int32_t n_chunks, const float2* __restrict__ part, float* __restrict__ F,
                           float* __restrict__ F2) {
  int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n_hkl) return;
  double re = 0.0, im = 0.0;
#pragma unroll 8
  for (int c = 0; c < n_chunks; ++c) {
    float2 v = part[(int64_t)c * n_hkl + r];
    re += v.x;
    im += v.y;
  }
  if (F) {
    F[2 * r + 0] = (float)re;
    F[2 * r + 1] = (float)im;
  }
  if (F2) F2[r] = (float)(re * re + im * im);
}

// Batched models: an item of refl_blocks covers reflections [first, first + 256) of one model,
// SPLIT blocks of 256 / SPLIT of them, and a block loops over all of that model's atoms (binary64
// accumulation, no partials), thread t with reflection t % (256 / SPLIT) and the share
// t / (256 / SPLIT) of every group of 256 atoms; the shares are added in order.  Six models of a
// few hundred atoms: 33 us with one thread per reflection, 8 us with sixteen.
template <int SPLIT>
__global__ void __launch_bounds__(kSFThreads) k_b_sf(const fdtbx_batch_entry* __restrict__ ent, const int64_t* __restrict__ blocks,
                                                     const float* __restrict__ x, const float* __restrict__ y,
                                                     const float* __restrict__ z, const float* __restrict__ B,
                                                     const float* __restrict__ occ, const int32_t* __restrict__ type,
                                                     const float* __restrict__ ff, const int32_t* __restrict__ hkl,
                                                     float* __restrict__ F, float* __restrict__ F2) {
  constexpr int kRefl = kSFThreads / SPLIT;
  __shared__ AtomsLds at;
  __shared__ float ftab[kMaxTypes * kRefl];
  const int64_t item = blocks[blockIdx.x / SPLIT];
  const int m = (int)(item >> 40);
  const fdtbx_batch_entry& e = ent[m];
  const int share = (int)threadIdx.x / kRefl, col = (int)threadIdx.x % kRefl;
  const int64_t first = (item & ((1ll << 40) - 1)) + kRefl * (int)(blockIdx.x % SPLIT);
  if (first >= e.n_hkl) return;  // uniform across the workgroup
  const int64_t r = first + col;
  const bool have = r < e.n_hkl;
  const int64_t g = e.hkl_off + r;
  // fdtbx_batch_entries_check keeps n_types in 1..kMaxTypes; clamped here as well, so that the
  // LDS table is never indexed past its end
  const int n_types = e.n_types < 1 ? 1 : (e.n_types > kMaxTypes ? kMaxTypes : e.n_types);
  const float* ffm = ff + 9 * e.ff_off;
  double h = 0, k = 0, l = 0;
  float s2 = 0.0f;
  if (have) {
    h = hkl[3 * g + 0];
    k = hkl[3 * g + 1];
    l = hkl[3 * g + 2];
    double D[3];
    for (int j = 0; j < 3; ++j) D[j] = (h * e.frame[9 + j] + k * e.frame[12 + j]) + l * e.frame[15 + j];
    double q = (D[0] * D[0] + D[1] * D[1]) + D[2] * D[2];
    double s2d = 0.25 * q;
    s2 = (float)s2d;
    for (int t = share; t < n_types; t += SPLIT) ftab[t * kRefl + col] = form_factor(ffm + 9 * t, s2d);
  }
  const int64_t a0 = e.atom_off, a1 = e.atom_off + e.n_atoms;
  double re = 0.0, im = 0.0;
  for (int64_t g0 = a0; g0 < a1; g0 += kSFThreads) {
    __syncthreads();
    const int64_t j = g0 + threadIdx.x;
    if (j < a1) at.put(threadIdx.x, x, y, z, B, occ, type, j, n_types, kRefl);
    __syncthreads();
    const int cnt = (int)((a1 - g0) < kSFThreads ? (a1 - g0) : kSFThreads);
    if (have) {
      const int end = min(cnt, (share + 1) * kRefl);
      for (int i = share * kRefl; i < end; ++i) {
        const auto zb = at.zb[i];
        const float frac = sf_phase(h, k, l, at.xy[i], zb.z);
        const float amp = zb.occ * ftab[at.type[i] + col] * __builtin_amdgcn_exp2f(zb.nBl2e * s2);
        re = fma((double)amp, (double)__builtin_amdgcn_cosf(frac), re);
        im = fma((double)amp, (double)__builtin_amdgcn_sinf(frac), im);
      }
    }
  }
  if (SPLIT > 1) {
    __shared__ double gs[SPLIT][2][kRefl];
    gs[share][0][col] = re;
    gs[share][1][col] = im;
    __syncthreads();
    if (share > 0) return;
#pragma unroll
    for (int k = 1; k < SPLIT; ++k) {
      re += gs[k][0][col];
      im += gs[k][1][col];
    }
  }
  if (have) {
    if (F) {
      F[2 * g + 0] = (float)re;
      F[2 * g + 1] = (float)im;
    }
    if (F2) F2[g] = (float)(re * re + im * im);
  }
}

int launch_batch_sf(const fdtbx_batch_entry* ent, const int64_t* blocks, int64_t n_rb, const float* x, const float* y,
                    const float* z, const float* B, const float* occ, const int32_t* type, const float* ff, const int32_t* hkl,
                    float* F, float* F2, hipStream_t s) {
  if (n_rb <= 0) return FDTBX_OK;
  auto launch = [&](auto kernel, int split) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)(n_rb * split)), dim3(kSFThreads), 0, s, ent, blocks, x, y, z, B, occ, type, ff,
                       hkl, F, F2);
  };
  const int split = batch_split(n_rb);
  if (split == 16)
    launch(k_b_sf<16>, 16);
  else if (split == 4)
    launch(k_b_sf<4>, 4);
  else
    launch(k_b_sf<1>, 1);
  FDTBX_LAUNCH_CHECK("batch structure factors");
  return FDTBX_OK;
}

// Reflections per thread, atom chunks and their length.  Two reflections per thread share the
// atom's LDS reads (293298 reflections of 50000 atoms: 8 % less time than with one, whose 40
// bytes a term keep the LDS busy longer than the vector unit; four gain another 2 %), but a chunk then
// starts with twice the form factors, so they are taken where chunks of 1024 atoms fill the chip
// (9692 reflections of 50000 atoms: 0.20 ms with one, 0.26 with two).
static int sf_split(int64_t n_hkl, int64_t n_atoms, int32_t* n_chunks, int64_t* chunk) {
  const int64_t half = (n_hkl + 1) / 2, maxc = ceil_div(n_atoms, 64);
  const int k = ceil_div(half, 2 * kSFThreads) * ceil_div(n_atoms, 1024) >= kSFBlocks ? 2 : 1;
  const int64_t nb = ceil_div(half, k * kSFThreads);
  // fill the chip: with one reflection per thread eight blocks of a compute unit run at once, and the
  // 2051 blocks that ceil makes of 293 leave it a ninth: 150000 reflections of 5000 atoms 0.214 ms,
  // 0.202 with the 1758 of floor, and 0.420 / 0.395 where no mates are mates.  From 410 blocks floor
  // leaves too few (489 blocks: 0.171 / 0.172), and so it does with two per thread, whose blocks are
  // fewer and longer (290000 of 50000 3.34 / 3.41).
  int64_t nc = k == 1 && nb <= kSFBlocks / 5 ? kSFBlocks / nb : ceil_div(kSFBlocks, nb);
  if (nc > maxc) nc = maxc;
  if (nc < 1) nc = 1;
  *chunk = ceil_div(n_atoms, nc);
  *n_chunks = (int32_t)ceil_div(n_atoms, *chunk);
  return k;
}

}  // namespace fdtbx

using namespace fdtbx;

extern "C" size_t fdtbx_sf_workspace(int64_t n_hkl, int64_t n_atoms) {
  if (n_hkl <= 0 || n_atoms <= 0) return 0;
  int32_t nc;
  int64_t chunk;
  sf_split(n_hkl, n_atoms, &nc, &chunk);
  return (size_t)nc * n_hkl * sizeof(float2);
}

extern "C" int fdtbx_structure_factors(const fdtbx_cell* cell, int64_t n_atoms, const float* x, const float* y,
                                       const float* z, const float* B, const float* occ, const int32_t* type,
                                       const float* ff, int32_t n_types, const int32_t* hkl, int64_t n_hkl, float* F,
                                       float* F2, void* ws, size_t ws_bytes, void* stream) {
  if (!cell) return fail(FDTBX_ERR_INVALID_ARGUMENT, "null pointer");
  if (n_atoms < 0 || n_hkl < 0) return fail(FDTBX_ERR_INVALID_ARGUMENT, "n_atoms and n_hkl must be non-negative");
  if (n_hkl == 0) return FDTBX_OK;
  if (!F && !F2) return fail(FDTBX_ERR_INVALID_ARGUMENT, "F and F2 both NULL");
  if (n_atoms == 0) {  // no atoms: F = 0
    int r0 = fill(F, 2 * n_hkl, 0.0f, (hipStream_t)stream);
    if (r0) return r0;
    return fill(F2, n_hkl, 0.0f, (hipStream_t)stream);
  }
  if (!x || !y || !z || !B || !occ || !type || !ff || !hkl || !ws) return fail(FDTBX_ERR_INVALID_ARGUMENT, "null pointer");
  if (n_types < 1 || n_types > kMaxTypes) return fail(FDTBX_ERR_INVALID_ARGUMENT, "n_types must be in 1..16");
  if (n_hkl > (int64_t)0x7fffffff * kSFThreads) return fail(FDTBX_ERR_UNSUPPORTED, "too many reflections");
  int rc = check_cell(cell);
  if (rc) return rc;
  if (ws_bytes < fdtbx_sf_workspace(n_hkl, n_atoms)) return fail(FDTBX_ERR_BUFFER_TOO_SMALL, "sf workspace too small");
  SFParams p;
  {
    // reciprocal basis of the laboratory frame, the same construction as the exact unit
    double ca = cos(cell->alpha), cb = cos(cell->beta), cg = cos(cell->gamma), sa = sin(cell->alpha);
    double cv[3] = {0.0, 0.0, cell->c};
    double bv[3] = {0.0, cell->b * sa, cell->b * ca};
    double az = cell->a * cb, ay = cell->a * (cg - ca * cb) / sa;
    double av[3] = {sqrt(cell->a * cell->a - ay * ay - az * az), ay, az};
    auto cross = [](const double* u, const double* v, double* w) {
      w[0] = u[1] * v[2] - u[2] * v[1];
      w[1] = u[2] * v[0] - u[0] * v[2];
      w[2] = u[0] * v[1] - u[1] * v[0];
    };
    double bxc[3], cxa[3], axb[3];
    cross(bv, cv, bxc);
    cross(cv, av, cxa);
    cross(av, bv, axb);
    double V = (av[0] * bxc[0] + av[1] * bxc[1]) + av[2] * bxc[2];
    for (int j = 0; j < 3; ++j) {
      p.as[j] = bxc[j] / V;
      p.as[3 + j] = cxa[j] / V;
      p.as[6 + j] = axb[j] / V;
    }
  }
  p.n_hkl = n_hkl;
  p.n_atoms = n_atoms;
  p.n_types = n_types;
  const int per_thread = sf_split(n_hkl, n_atoms, &p.n_chunks, &p.chunk);
  hipStream_t s = (hipStream_t)stream;
  float2* part = (float2*)ws;
  const unsigned nb = (unsigned)ceil_div((n_hkl + 1) / 2, per_thread * kSFThreads);
  const dim3 grid(nb, (unsigned)p.n_chunks, (int64_t)nb * p.n_chunks <= kSFBothHalves ? 2 : 1);
  const size_t lds = (size_t)n_types * kSFThreads * per_thread * sizeof(float);
  if (per_thread == 2)
    hipLaunchKernelGGL(k_sf_partial<2>, grid, dim3(kSFThreads), lds, s, p, x, y, z, B, occ, type, ff, hkl, part);
  else
    hipLaunchKernelGGL(k_sf_partial<1>, grid, dim3(kSFThreads), lds, s, p, x, y, z, B, occ, type, ff, hkl, part);
  FDTBX_LAUNCH_CHECK("structure factors");
  hipLaunchKernelGGL(k_sf_final, dim3((unsigned)ceil_div(n_hkl, 256)), dim3(256), 0, s, n_hkl, p.n_chunks, part, F, F2);
  FDTBX_LAUNCH_CHECK("structure factor reduce");
  return FDTBX_OK;
}
