// Spectral heat current (Sec. II.C): the virial-velocity correlation of
// Eq. 21 accumulated in float64, and its transform (Eq. 22).
//
//   K^{mu nu}(tau) += sum_{t in block} sum_i Wmu[s0 + t - tau][nu Np + i] V[t][nu Np + i]
//
// Dofs are stored direction-major, column j = nu * Np + i (Np = N rounded up
// to 32, zero padded): Wmu[s][nu Np + i] = W_i^{mu nu}(s) in a ring of the
// last n_lags - 1 + T steps and V[t][nu Np + i] = v_i^nu(s0 + t).  Every
// work-group's dof range lies inside one direction segment, so its partial
// sums belong to one motion direction nu (the split of Sec. II, remark after
// Eq. 10) and Eq. 21 itself is the sum over nu.  The products of the float32
// inputs are formed exactly in float64 and summed in float64 in a fixed
// order, so the result is reproducible bit for bit.
#include "mhc_common.h"
#include "mhc_numeric.h"

namespace mhc {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------- ring fill
// ring[(s % ring_len) * 3 + mu][nu Np + i] = W[t][i][mu][nu] and
// vt[t][nu Np + i] = v[t][i][nu] for the block's steps s = s0 + t, t < t_count
// (ld = 3 Np).  One thread per (t, i): 12 floats in, 12 out, consecutive
// atoms to consecutive columns.
__device__ __forceinline__ void shc_ring_atom(const float* __restrict__ W, const float* __restrict__ v,
                                              int t_count, int64_t N, int64_t Np, float* __restrict__ ring,
                                              int64_t ring_len, int64_t ld, int64_t s0, float* __restrict__ vt,
                                              int t, int64_t i) {
  if (t >= t_count || i >= N) return;
  const float* src = W + ((int64_t)t * N + i) * 9;
  float w[9];
#pragma unroll
  for (int c = 0; c < 9; ++c) w[c] = src[c];
  const float* vs = v + ((int64_t)t * N + i) * 3;
  const float v0 = vs[0], v1 = vs[1], v2 = vs[2];
  float* row = ring + ((s0 + t) % ring_len) * 3 * ld + i;
#pragma unroll
  for (int mu = 0; mu < 3; ++mu)
#pragma unroll
    for (int nu = 0; nu < 3; ++nu) row[mu * ld + nu * Np] = w[3 * mu + nu];
  float* vr = vt + (int64_t)t * ld + i;
  vr[0] = v0;
  vr[Np] = v1;
  vr[2 * Np] = v2;
}

__global__ void __launch_bounds__(256) k_shc_ring(const float* __restrict__ W, const float* __restrict__ v,
                                                 int t_count, int64_t N, int64_t Np, float* __restrict__ ring,
                                                 int64_t ring_len, int64_t ld, int64_t s0, float* __restrict__ vt) {
  shc_ring_atom(W, v, t_count, N, Np, ring, ring_len, ld, s0, vt, blockIdx.y, (int64_t)blockIdx.x * 256 + threadIdx.x);
}

// The system of work-group (or block) b of a grouped launch: the last
// descriptor whose first index is <= b.
__device__ __forceinline__ int shc_system_of(const ShcBlockDesc* __restrict__ d, int n_sys, int64_t b, int which) {
  // 64 candidates at a time, one per lane (whole waves call this): one load's
  // latency for up to 64 systems.  A scan over the systems waited for a load
  // each, 3 us per work-group of 32 systems.
  const int lane = threadIdx.x & 63;
  int lo = 0, len = n_sys;
  while (len > 1) {
    const int step = (len + 63) / 64;
    const ShcBlockDesc& e = d[lo + min(lane * step, len - 1)];
    const int64_t f = which == 0 ? e.ring_blk0 : (which == 1 ? e.gram_wg0 : e.acc_blk0);
    const unsigned long long m = __ballot(lane * step < len && f <= b);
    const int k = __builtin_popcountll(m) - 1;   // the first system starts at 0
    lo += k * step;
    len = min(step, len - k * step);
  }
  return lo;
}

__global__ void __launch_bounds__(256) k_shc_ring_group(const ShcBlockDesc* __restrict__ d, int n_sys) {
  const int q = shc_system_of(d, n_sys, blockIdx.x, 0);
  const ShcBlockDesc& e = d[q];
  shc_ring_atom(e.W, e.v, e.t_count, e.N, e.Np, e.ring, e.ring_len, e.ld, e.s0, e.vt, blockIdx.y,
                (int64_t)(blockIdx.x - e.ring_blk0) * 256 + threadIdx.x);
}

hipError_t launch_shc_ring_group(hipStream_t s, const ShcBlockDesc* d, int n_sys, int64_t n_blocks, int t_count) {
  if (t_count <= 0 || n_blocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_shc_ring_group, dim3((unsigned)n_blocks, (unsigned)t_count), dim3(256), 0, s, d, n_sys);
  return hipGetLastError();
}

hipError_t launch_shc_ring(hipStream_t s, const float* W, const float* v, int t_count, int64_t N, int64_t Np,
                           float* ring, int64_t ring_len, int64_t ld, int64_t s0, float* vt) {
  if (t_count <= 0) return hipSuccess;
  dim3 grid((unsigned)((N + 255) / 256), (unsigned)t_count);
  hipLaunchKernelGGL(k_shc_ring, grid, dim3(256), 0, s, W, v, t_count, N, Np, ring, ring_len, ld, s0, vt);
  return hipGetLastError();
}

// ---------------------------------------------------------------- products
// The partial sums on the FP64 matrix cores, in Gram form.  Work-group
// (kc, mu, a, b) covers steps t in [64a, 64a + 64), lags tau in
// [128b, 128b + 128) and one component mu over the dof range of kc (a 1-D
// grid; consecutive ids go to different XCDs, so ids are remapped to give
// each XCD a contiguous range, and the tiles of one dof range are adjacent,
// sharing that XCD's L2).  Its origins s' = s0 + t - tau are 192 consecutive
// ring rows R (origin row0 + R); wave w takes steps 64a + 16w + c (c < 16)
// and rows R = 16w + rho, rho < 144 (9 blocks of 16), and accumulates
//   G[rho][c] = sum_j Wmu[row0 + 16w + rho][j] V[64a + 16w + c][j]
// with v_mfma_f64_16x16x4f64: A = a block of virial rows, B = velocity rows,
// 4 dofs per product (lane l supplies row or step l % 16 at dof l / 16 of the
// product's 4), and lane l's register i of the result is entry
// [4i + l / 16][l % 16].  The entry with lag tau = 128b + lambda lies at
// rho = 127 + c - lambda, so a work-group's partial for lambda is the sum of
// G along that diagonal over the 4 waves and 16 steps, taken in a fixed order
// after the dof loop.  Of the 9 x 256 products per wave and dof, the 16 x 128
// on those diagonals are used.  Dofs are staged 32 at a time in LDS (float32,
// double-buffered; rows padded to 36 floats) and converted to float64 as the
// operands are read; the products of float32 inputs are exact in float64.
// Loads are unconditional, from a valid row, and masked to zero outside the
// sampled rows and the block's steps.  The operands of a half chunk are read
// while the other half's products run, and the one barrier per chunk stands
// between products, so that neither the LDS latency nor the wait for the other
// waves empties the matrix cores.  G is summed in the LDS of the staging
// buffers, so two work-groups fit on a CU.  Measured, 8000 atoms, 250 lags,
// T = 256 (152 us of products): 215 -> 198 us.  Operands read from the L2 by
// every wave for itself, without LDS and barriers, took 265 us; converted to
// float64 on the way into LDS, 16 dofs at a time, 215 us.
constexpr int SM_T = 64, SM_L = 128, SM_DC = 32;
constexpr int SM_RB = (SM_L + 16) / 16;                 // 9 row blocks per wave
constexpr int SM_ROWS = SM_T - 16 + 16 * SM_RB;         // 192 staged rows
constexpr int SM_WS = SM_DC + 4;                        // LDS row stride (floats)
constexpr int SM_GS = 17;                               // LDS row stride of G (doubles)

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// Loads and stores of the tile go through pointers in the global address
// space: a pointer read from a descriptor in memory (grouped launches) is
// otherwise generic to the compiler, whose flat loads also count against the
// LDS wait counter, so that every LDS wait of the loop would wait for the
// next chunk's loads as well.
typedef __attribute__((address_space(1))) const f32x4 gcf32x4;
typedef __attribute__((address_space(1))) double gdouble;

// One work-group's tile; v = its index among the launch's work-groups of this
// system after the XCD remapping.
__device__ __forceinline__ void shc_gram_tile(const float* __restrict__ vt, const float* __restrict__ ring,
                                              int64_t ring_len, int64_t ld, int64_t N, int64_t Np, int t_count,
                                              int64_t s0, int64_t dk, int n_kcs, int n_ttiles, int n_lags_pad,
                                              double* __restrict__ part, int v) {
  // staging buffers (192 rows of W, then 64 of V), and after the products the
  // G of the 4 waves
  constexpr int BUF = (SM_ROWS + SM_T) * SM_WS;                             // floats
  constexpr int RED = 4 * 16 * SM_RB * SM_GS;                               // doubles
  constexpr int SMEM = 2 * BUF * 4 > RED * 8 ? 2 * BUF * 4 : RED * 8;
  __shared__ __attribute__((aligned(16))) unsigned char smem[SMEM];
  float* const stage = reinterpret_cast<float*>(smem);
  double (*red)[16 * SM_RB][SM_GS] = reinterpret_cast<double (*)[16 * SM_RB][SM_GS]>(smem);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane & 15, g = lane >> 4;
  const int n_ab = n_ttiles * (n_lags_pad / SM_L);
  const int kc = v / (3 * n_ab);
  const int mu = (v / n_ab) % 3;
  const int a = (v % n_ab) % n_ttiles;
  const int b = (v % n_ab) / n_ttiles;
  const int64_t seg0 = (int64_t)(kc / n_kcs) * Np;
  const int64_t j0 = seg0 + (int64_t)(kc % n_kcs) * dk;
  const int64_t j1 = min(seg0 + N, j0 + dk);
  const int64_t row0 = s0 + (int64_t)SM_T * a - (int64_t)SM_L * b - (SM_L - 1);
  const int64_t s_last = s0 + t_count - 1;
  if (row0 + SM_ROWS <= 0) {   // every origin lies before the first sample
    if (tid < SM_L)
      ((gdouble*)part)[(((int64_t)kc * n_ttiles + a) * n_lags_pad + (int64_t)SM_L * b + tid) * 3 + mu] = 0.0;
    return;
  }

  // staging of one 32-dof chunk: thread (r, q) takes float4 q of rows r + 32 k
  // of W (k < 6) and of steps r + 32 k of V (k < 2); the columns past the last
  // atom are the zero pads of the rows
  constexpr int WPT = SM_ROWS / 32, VPT = SM_T / 32;
  static_assert(WPT * 256 == SM_ROWS * (SM_DC / 4) && VPT * 256 == SM_T * (SM_DC / 4), "staging shape");
  const int sr = tid / (SM_DC / 4), sq = tid % (SM_DC / 4);
  gcf32x4* src[WPT + VPT];
  uint32_t keep = 0;                                          // bit k: row k is a sample
  // ring slots in 32 bits: row0 - s0 > -(n_lags + 191) >= -(ring_len + 128) and
  // ring_len >= 64, so four ring lengths more are never negative
  const uint32_t rl = (uint32_t)ring_len;
  const uint32_t slot0 = (uint32_t)(s0 % ring_len) + 4 * rl + (uint32_t)(int32_t)(row0 - s0);
#pragma unroll
  for (int k = 0; k < WPT; ++k) {
    const int64_t sp = row0 + sr + 32 * k;
    const bool ok = sp >= 0 && sp <= s_last;
    keep |= (ok ? 1u : 0u) << k;
    src[k] = (gcf32x4*)(ring + (int64_t)((slot0 + sr + 32 * k) % rl) * 3 * ld + mu * ld + j0 + 4 * sq);
  }
#pragma unroll
  for (int k = 0; k < VPT; ++k) {
    const int t = SM_T * a + sr + 32 * k;
    keep |= (t < t_count ? 1u : 0u) << (WPT + k);
    src[WPT + k] = (gcf32x4*)(vt + (int64_t)min(t, t_count - 1) * ld + j0 + 4 * sq);
  }
  f32x4 st[WPT + VPT];
  const int n_chunks = (int)((j1 - j0 + SM_DC - 1) / SM_DC);
  auto load = [&](int ch) {
    const int64_t o = (int64_t)min(ch, n_chunks - 1) * (SM_DC / 4);
#pragma unroll
    for (int k = 0; k < WPT + VPT; ++k) st[k] = src[k][o];
  };
  float* const dst = stage + sr * SM_WS + 4 * sq;
  auto store = [&](int buf) {
#pragma unroll
    for (int k = 0; k < WPT + VPT; ++k) {
      const uint32_t m = (keep >> k) & 1u ? ~0u : 0u;
      *reinterpret_cast<u32x4*>(dst + buf * BUF + 32 * k * SM_WS) = __builtin_bit_cast(u32x4, st[k]) & m;
    }
  };

  f64x4 acc[SM_RB];
#pragma unroll
  for (int rb = 0; rb < SM_RB; ++rb) acc[rb] = f64x4{0.0, 0.0, 0.0, 0.0};
  // lane (c, g) supplies dofs 16 h + 4 g .. + 3 of half chunk h
  const float* const wp = stage + (16 * wave + c) * SM_WS + 4 * g;
  const float* const vp = wp + SM_ROWS * SM_WS;
  auto read = [&](f32x4 (&f)[SM_RB + 1], int buf, int h) {
#pragma unroll
    for (int rb = 0; rb < SM_RB; ++rb)
      f[rb] = *reinterpret_cast<const f32x4*>(wp + buf * BUF + 16 * rb * SM_WS + 16 * h);
    f[SM_RB] = *reinterpret_cast<const f32x4*>(vp + buf * BUF + 16 * h);
  };
  auto products = [&](const f32x4 (&f)[SM_RB + 1], int x0, int x1) {
    // the 9 independent accumulators between two products on the same one
#pragma unroll
    for (int x = x0; x < x1; ++x) {
      const double vb = (double)f[SM_RB][x];
#pragma unroll
      for (int rb = 0; rb < SM_RB; ++rb)
        acc[rb] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)f[rb][x], vb, acc[rb], 0, 0, 0);
    }
  };
  f32x4 f0[SM_RB + 1], f1[SM_RB + 1];
  load(0);
  store(0);
  load(1);
  __syncthreads();
  read(f0, 0, 0);
  for (int ch = 0; ch < n_chunks; ++ch) {
    const int buf = ch & 1;
    read(f1, buf, 1);
    __builtin_amdgcn_sched_barrier(0);
    products(f0, 0, 4);
    __builtin_amdgcn_sched_barrier(0);
    store(buf ^ 1);                      // last read before the previous barrier
    load(ch + 2);
    __builtin_amdgcn_sched_barrier(0);
    products(f1, 0, 2);
    __syncthreads();
    read(f0, buf ^ 1, 0);
    __builtin_amdgcn_sched_barrier(0);
    products(f1, 2, 4);
    __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();                       // the last reads, before G takes the buffers
  // lane (c, g) holds G[16 rb + 4 i + g][c] in acc[rb][i]
#pragma unroll
  for (int rb = 0; rb < SM_RB; ++rb)
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wave][16 * rb + 4 * i + g][c] = acc[rb][i];
  __syncthreads();
  if (tid < SM_L) {
    const int lam = tid;
    double s = 0.0;
    for (int w = 0; w < 4; ++w)
      for (int cc = 0; cc < 16; ++cc) s += red[w][(SM_L - 1) + cc - lam][cc];
    ((gdouble*)part)[(((int64_t)kc * n_ttiles + a) * n_lags_pad + (int64_t)SM_L * b + lam) * 3 + mu] = s;
  }
}

// Consecutive work-group ids go to different XCDs: ids are remapped so that
// each XCD takes a contiguous range (the tiles of one dof range are adjacent
// and share that XCD's L2).
__device__ __forceinline__ int shc_xcd_remap(int b, int G) { return (G % 8 == 0) ? (b % 8) * (G / 8) + b / 8 : b; }

__global__ void __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(2, 2)))
k_shc_gram(const float* __restrict__ vt, const float* __restrict__ ring, int64_t ring_len, int64_t ld, int64_t N,
           int64_t Np, int t_count, int64_t s0, int64_t dk, int n_kcs, int n_ttiles, int n_lags_pad,
           double* __restrict__ part) {
  shc_gram_tile(vt, ring, ring_len, ld, N, Np, t_count, s0, dk, n_kcs, n_ttiles, n_lags_pad, part,
                shc_xcd_remap(blockIdx.x, gridDim.x));
}

// Several systems' products in one launch: the remapped id picks the system
// (systems in order, each its work-groups in the single-system order).  Ids
// are dealt to the XCDs `grain` at a time, in turn.
__device__ __forceinline__ int shc_xcd_deal(int b, int G, int grain) {
  const int full = G / (8 * grain) * (8 * grain);   // the rest in order
  return b < full ? (b / 8 / grain * 8 + b % 8) * grain + b / 8 % grain : b;
}

__global__ void __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(2, 2)))
k_shc_gram_group(const ShcBlockDesc* __restrict__ d, int n_sys, int grain) {
  const int v = shc_xcd_deal(blockIdx.x, gridDim.x, grain);
  const int q = shc_system_of(d, n_sys, v, 1);
  const ShcBlockDesc& e = d[q];
  shc_gram_tile(e.vt, e.ring, e.ring_len, e.ld, e.N, e.Np, e.t_count, e.s0, e.dk, e.n_kcs, e.n_ttiles,
                e.n_lags_pad, e.part, (int)(v - e.gram_wg0));
}

// Fixed-order sum of the partials of one block into the running float64 sums
// of each motion direction (Neumaier): one thread per (nu, tau, mu), summing
// the n_kcs dof ranges of segment nu and the step tiles in order;
// ksum[nu][tau][mu].
__device__ __forceinline__ void shc_accum_one(const double* __restrict__ part, int n_kcs, int n_ttiles, int n_lags,
                                              int n_lags_pad, double* __restrict__ ksum, double* __restrict__ kcomp,
                                              int q) {
  if (q >= 3 * n_lags * 3) return;
  const int nu = q / (n_lags * 3);
  const int r = q - nu * n_lags * 3;
  const int tau = r / 3, m = r % 3;
  // partials (kc, a) of segment nu, kc-major: loads eight at a time, added in that order
  const int n_p = n_kcs * n_ttiles;
  const double* base = part + ((int64_t)nu * n_p * n_lags_pad + tau) * 3 + m;
  const int64_t stride = (int64_t)n_lags_pad * 3;
  double s = 0.0;
  for (int p0 = 0; p0 < n_p; p0 += 8) {
    double x[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = base[(int64_t)min(p0 + k, n_p - 1) * stride];
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (p0 + k < n_p) s += x[k];
  }
  neumaier_add(ksum[q], kcomp[q], s);
}

__global__ void __launch_bounds__(256) k_shc_accum(const double* __restrict__ part, int n_kcs, int n_ttiles,
                                                  int n_lags, int n_lags_pad, double* __restrict__ ksum,
                                                  double* __restrict__ kcomp) {
  shc_accum_one(part, n_kcs, n_ttiles, n_lags, n_lags_pad, ksum, kcomp, blockIdx.x * 256 + threadIdx.x);
}

__global__ void __launch_bounds__(256) k_shc_accum_group(const ShcBlockDesc* __restrict__ d, int n_sys) {
  const int q = shc_system_of(d, n_sys, blockIdx.x, 2);
  const ShcBlockDesc& e = d[q];
  shc_accum_one(e.part, e.n_kcs, e.n_ttiles, e.n_lags, e.n_lags_pad, e.ksum, e.kcomp,
                (int)(blockIdx.x - e.acc_blk0) * 256 + threadIdx.x);
}

hipError_t launch_shc_products(hipStream_t s, const float* vt, const float* ring, int64_t ring_len, int64_t ld,
                               int64_t N, int64_t Np, int t_count, int64_t s0, int n_lags, int64_t dk, int n_kcs,
                               double* part) {
  if (t_count <= 0) return hipSuccess;
  const int n_ttiles = (t_count + SM_T - 1) / SM_T;
  const int n_lags_pad = (n_lags + SM_L - 1) / SM_L * SM_L;
  const int n_ltiles = n_lags_pad / SM_L;
  hipLaunchKernelGGL(k_shc_gram, dim3((unsigned)(9 * n_kcs * n_ttiles * n_ltiles)), dim3(256), 0, s, vt, ring,
                     ring_len, ld, N, Np, t_count, s0, dk, n_kcs, n_ttiles, n_lags_pad, part);
  return hipGetLastError();
}

hipError_t launch_shc_gram_group(hipStream_t s, const ShcBlockDesc* d, int n_sys, int64_t n_wgs, int grain) {
  if (n_wgs <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_shc_gram_group, dim3((unsigned)n_wgs), dim3(256), 0, s, d, n_sys, grain);
  return hipGetLastError();
}

hipError_t launch_shc_accum_group(hipStream_t s, const ShcBlockDesc* d, int n_sys, int64_t n_blocks) {
  if (n_blocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_shc_accum_group, dim3((unsigned)n_blocks), dim3(256), 0, s, d, n_sys);
  return hipGetLastError();
}

// Work-groups of one system's product launch and blocks of its accumulation
// launch for a block of t_count steps (the grouped launches concatenate them).
int64_t shc_gram_wgs(int t_count, int n_lags, int n_kcs) {
  const int n_ttiles = (t_count + SM_T - 1) / SM_T;
  const int n_ltiles = (n_lags + SM_L - 1) / SM_L;
  return (int64_t)9 * n_kcs * n_ttiles * n_ltiles;
}
int64_t shc_accum_blocks(int n_lags) { return (3 * (int64_t)n_lags * 3 + 255) / 256; }

hipError_t launch_shc_accum(hipStream_t s, const double* part, int t_count, int n_lags, int n_kcs, double* ksum,
                            double* kcomp) {
  if (t_count <= 0) return hipSuccess;
  const int n_ttiles = (t_count + SM_T - 1) / SM_T;
  const int n_lags_pad = (n_lags + SM_L - 1) / SM_L * SM_L;
  hipLaunchKernelGGL(k_shc_accum, dim3((unsigned)((3 * n_lags * 3 + 255) / 256)), dim3(256), 0, s, part, n_kcs,
                     n_ttiles, n_lags, n_lags_pad, ksum, kcomp);
  return hipGetLastError();
}

// ---------------------------------------------------------------- read-out
// Kd[tau][mu][nu] = (ksum + kcomp)[nu][tau][mu] / (S - tau) and
// K[tau][mu] = (Kd[..][0] + Kd[..][1]) + Kd[..][2]; zero for lags with no origin.
__global__ void k_shc_finish(const double* __restrict__ ksum, const double* __restrict__ kcomp, int n_lags,
                             int64_t S, double* __restrict__ K, double* __restrict__ Kd) {
  const int q = blockIdx.x * 256 + threadIdx.x;
  if (q >= n_lags * 3) return;
  const int tau = q / 3;
  double k = 0.0;
#pragma unroll
  for (int nu = 0; nu < 3; ++nu) {
    const int e = nu * n_lags * 3 + q;
    const double d = (S > tau) ? (ksum[e] + kcomp[e]) / (double)(S - tau) : 0.0;
    if (Kd) Kd[q * 3 + nu] = d;
    k += d;
  }
  if (K) K[q] = k;
}

// Eq. 22 on the sampled lags, even extension, trapezoid rule, optional Hann
// window: Kw[w][m] = dt sum_tau c_tau K[tau][m] cos(omega_w tau dt), for the NC
// components m of each lag (3, or 9 for the split).  One wave per omega: lane l
// takes lags l, l + 64, ... for all components, so that each cosine is
// computed once and the lags run side by side; the lanes are added by a fixed
// butterfly (one thread per (omega, m) walked the lags alone: 240 frequencies
// x 9 components, 250 lags took 129 us, the whole call 156 us and now 34 us).
template <int NC>
__global__ void __launch_bounds__(256) k_shc_spectrum(const double* __restrict__ K, int n_lags,
                                                      const double* __restrict__ omega, int n_omega, double dt,
                                                      int window, double* __restrict__ Kw) {
  const int w = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (w >= n_omega) return;
  const double om = omega[w];
  double s[NC];
#pragma unroll
  for (int m = 0; m < NC; ++m) s[m] = 0.0;
  for (int tau = lane; tau < n_lags; tau += 64) {
    double c = (tau == 0 || tau == n_lags - 1) ? 1.0 : 2.0;
    if (window && n_lags > 1) c *= 0.5 * (1.0 + cos(M_PI * (double)tau / (double)(n_lags - 1)));
    const double cw = cos(om * (double)tau * dt);
#pragma unroll
    for (int m = 0; m < NC; ++m) s[m] += c * K[tau * NC + m] * cw;
  }
#pragma unroll
  for (int m = 0; m < NC; ++m) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s[m] += __shfl_xor(s[m], off);
    if (lane == m) Kw[(int64_t)w * NC + m] = dt * s[m];
  }
}

hipError_t launch_shc_finish(hipStream_t s, const double* ksum, const double* kcomp, int n_lags, int64_t S,
                             double* K, double* Kd) {
  hipLaunchKernelGGL(k_shc_finish, dim3((unsigned)((n_lags * 3 + 255) / 256)), dim3(256), 0, s, ksum, kcomp, n_lags,
                     S, K, Kd);
  return hipGetLastError();
}

hipError_t launch_shc_spectrum(hipStream_t s, const double* K, int n_lags, int nc, const double* omega, int n_omega,
                               double dt, int window, double* Kw) {
  if (n_omega <= 0) return hipSuccess;
  const dim3 grid((unsigned)((n_omega + 3) / 4)), block(256);
  if (nc == 3)
    hipLaunchKernelGGL(k_shc_spectrum<3>, grid, block, 0, s, K, n_lags, omega, n_omega, dt, window, Kw);
  else if (nc == 9)
    hipLaunchKernelGGL(k_shc_spectrum<9>, grid, block, 0, s, K, n_lags, omega, n_omega, dt, window, Kw);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace mhc
