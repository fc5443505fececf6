// Frequency binning, float64 time accumulation and the GKMA correlation.
//
//   J_b^mu(t) = sum_{n in b} J_n^mu(t)                 (frequency bins, Sec. III.A)
//   HNEMA:  S_b^mu += sum_t J_b^mu(t), S^mu += sum_t J^mu(t)   (Eq. 19 numerator)
//   GKMA:   C_b^{mu nu}(tau) += sum_t J_b^mu(t) J^nu(t - tau)  (Eq. 17 integrand)
// Modes are stored in bin-sorted slots, so bin b is the contiguous slot range
// [bin_off[b], bin_off[b+1]).  All sums are float64 in a fixed order (no
// atomics), so results are reproducible bit for bit; long running sums use
// Neumaier compensation.
#include "mhc_common.h"
#include "mhc_back_group.h"
#include "mhc_numeric.h"

namespace mhc {

// Neumaier update of three running sums by the fixed-order sums over a 256-thread
// work-group of x[0..2]: threads t and t + 128, then t + 64, through LDS, the
// last 64 by shuffles of one wave (the pairs of a tree over the work-group).
// One barrier for the three; a tree of barriers each, with the running sums
// loaded behind it, took 2 us of the bin sums' 5.4 (64 atoms, 100 bins: 3.3
// us now).  The sums' old values come from sums3_load, early in the kernel.
struct Sums3 { double s, c; };   // of component min(thread, 2)
__device__ __forceinline__ Sums3 sums3_load(const double* sum, const double* comp) {
  const int m = min((int)threadIdx.x, 2);
  return {sum[m], comp[m]};
}
__device__ __forceinline__ void sums3_add(const double (&x)[3], double (*sh)[256], Sums3 old, double* sum, double* comp) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int m = 0; m < 3; ++m) sh[m][tid] = x[m];
  __syncthreads();
  if (tid >= 64) return;
  double r[3];
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    r[m] = (sh[m][tid] + sh[m][tid + 128]) + (sh[m][tid + 64] + sh[m][tid + 192]);
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) r[m] += __shfl_down(r[m], w);
    r[m] = __shfl(r[m], 0);
  }
  if (tid < 3) {
    neumaier_add(old.s, old.c, tid == 0 ? r[0] : (tid == 1 ? r[1] : r[2]));
    sum[tid] = old.s;
    comp[tid] = old.c;
  }
}

// Eq. 10 summed over atoms: one wave per step adds the float64 partials of
// the atom chunks in a fixed order.
__device__ __forceinline__ void total_body(const double* __restrict__ jt_part, int n_chunks,
                                           double* __restrict__ jtot, int t, int lane) {
  double j0 = 0.0, j1 = 0.0, j2 = 0.0;
  const double* p = jt_part + (int64_t)t * n_chunks * 3;
  for (int c = lane; c < n_chunks; c += 64) {
    j0 += p[c * 3 + 0];
    j1 += p[c * 3 + 1];
    j2 += p[c * 3 + 2];
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    j0 += __shfl_xor(j0, off);
    j1 += __shfl_xor(j1, off);
    j2 += __shfl_xor(j2, off);
  }
  if (lane == 0) {
    jtot[t * 3 + 0] = j0;
    jtot[t * 3 + 1] = j1;
    jtot[t * 3 + 2] = j2;
  }
}

// ------------------------------------------------------------------ reduce
__device__ __forceinline__ void reduce_body(ReduceArgs a, int b) {
  __shared__ double sh[3][256];
  const int tid = threadIdx.x;
  if (a.t0_dev) a.t0 = *a.t0_dev;
  if (b < a.nb) {
    Sums3 old{0.0, 0.0};
    if (a.hsum) old = sums3_load(a.hsum + b * 3, a.hcomp + b * 3);
    const int64_t lo = a.bin_off[b], hi = a.bin_off[b + 1];
    const int64_t n = hi - lo;
    if (!a.layout_g) {
      // HNEMA-only: parts [p][sub][slot][mu], already summed over each part's steps
      double s3[3] = {0.0, 0.0, 0.0};
      const int per_part = (int)(n * 3);
      if (a.slot_sum) {                         // already summed over the parts
        int mu = tid % 3;
        for (int e = tid; e < per_part; e += 256) {
          const double val = a.slot_sum[lo * 3 + e];
          if (mu == 0) s3[0] += val; else if (mu == 1) s3[1] += val; else s3[2] += val;
          mu = (mu == 2) ? 0 : mu + 1;
        }
      } else if (per_part <= 256 && a.n_sub == 1) {
        // one value of a part per thread: eight parts' loads at a time
        double s = 0.0;
        if (tid < per_part)
          for (int p0 = 0; p0 < a.n_parts; p0 += 8) {
            float x[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) x[k] = a.in[((int64_t)min(p0 + k, a.n_parts - 1) * a.M_pad + lo) * 3 + tid];
#pragma unroll
            for (int k = 0; k < 8; ++k)
              if (p0 + k < a.n_parts) s += (double)x[k];
          }
        const int mu = tid % 3;
        s3[0] = mu == 0 ? s : 0.0;
        s3[1] = mu == 1 ? s : 0.0;
        s3[2] = mu == 2 ? s : 0.0;
      } else {
        for (int p = 0; p < a.n_parts; ++p) {
          const float* base = a.in + ((int64_t)p * a.n_sub * a.M_pad + lo) * 3;
          int mu = tid % 3;                       // e % 3, and 256 % 3 == 1
          for (int e = tid; e < per_part; e += 256) {
            float part = base[e];
            if (a.n_sub > 1)
              for (int q = 1; q < a.n_sub; ++q) part += base[(int64_t)q * a.M_pad * 3 + e];
            const double val = (double)part;
            if (mu == 0) s3[0] += val; else if (mu == 1) s3[1] += val; else s3[2] += val;
            mu = (mu == 2) ? 0 : mu + 1;
          }
        }
      }
      sums3_add(s3, sh, old, a.hsum + b * 3, a.hcomp + b * 3);
    } else {
      // GKMA: X[(b*3+mu)][t] = sum over the bin's segment rows in segment order
      // (from k_reduce_seg); thread t of the work-group, steps strided by 256.
      const int64_t P = (int64_t)a.n_seg + a.nb;
      const int64_t sg0 = lo / REDUCE_SEG, sg1 = (hi - 1) / REDUCE_SEG;
      const int64_t xo = a.xoff_dev ? *a.xoff_dev : a.xoff;
      double h3[3] = {0.0, 0.0, 0.0};
      for (int t = tid; t < a.t_count; t += 256) {
#pragma unroll
        for (int mu = 0; mu < 3; ++mu) {
          double s = 0.0;
          if (n > 0)
            for (int64_t sg = sg0; sg <= sg1; ++sg) s += a.seg_part[((int64_t)mu * P + sg + b) * a.ld + t];
          a.X[((int64_t)b * 3 + mu) * a.ldx + xo + t] = s;
          if (a.bring) a.bring[((int64_t)b * a.ring_len + (a.t0 + t) % a.ring_len) * 3 + mu] = s;
          h3[mu] += s;
        }
      }
      if (a.hsum) sums3_add(h3, sh, old, a.hsum + b * 3, a.hcomp + b * 3);
    }
    return;
  }
  // last work-group: per-step total current of Eq. 10, summed over atoms here
  // (a wave per step) or by an earlier kernel
  if (a.jt_part) {
    for (int t = tid >> 6; t < a.t_count; t += 4) total_body(a.jt_part, a.n_chunks, a.jtot, t, tid & 63);
    __syncthreads();
  }
  Sums3 t_old{0.0, 0.0}, td_old{0.0, 0.0};
  if (a.tsum) t_old = sums3_load(a.tsum, a.tcomp);
  if (a.tdsum) td_old = sums3_load(a.tdsum, a.tdcomp);
  double h3[3] = {0.0, 0.0, 0.0};
  const int64_t xo = a.X ? (a.xoff_dev ? *a.xoff_dev : a.xoff) : 0;
  for (int t = tid; t < a.t_count; t += 256) {
#pragma unroll
    for (int mu = 0; mu < 3; ++mu) {
      const double j = a.jtot[t * 3 + mu];
      h3[mu] += j;
      if (a.X) {
        a.X[((int64_t)a.nb * 3 + mu) * a.ldx + xo + t] = j;
        a.ring[((a.t0 + t) % a.ring_len) * 3 + mu] = j;
      }
    }
  }
  if (a.tsum) sums3_add(h3, sh, t_old, a.tsum, a.tcomp);
  if (a.tdsum) {   // motion-direction split of the Eq. 10 total
    double d3[3] = {0.0, 0.0, 0.0};
    for (int t = tid; t < a.t_count; t += 256)
#pragma unroll
      for (int mu = 0; mu < 3; ++mu) d3[mu] += a.jdtot[t * 3 + mu];
    __syncthreads();   // the totals' reads of sh
    sums3_add(d3, sh, td_old, a.tdsum, a.tdcomp);
  }
}

// grid y: direction region of the one-contraction split
__global__ void __launch_bounds__(256) k_reduce(ReduceArgs a) {
  const int d = blockIdx.y;
  if (d > 0) {
    a.in += d * a.in_region;
    a.hsum += (int64_t)d * a.nb * 3;
    a.hcomp += (int64_t)d * a.nb * 3;
    a.tsum = nullptr;
    if (a.tdsum) {
      a.jdtot += d * a.jdtot_region;
      a.tdsum += 3 * d;
      a.tdcomp += 3 * d;
    }
  }
  reduce_body(a, blockIdx.x);
}

// grid y: 0 the totals, d + 1 the split totals of direction region d
__global__ void __launch_bounds__(64) k_total(TotalArgs a) {
  const int d = (int)blockIdx.y - 1;
  if (d < 0) total_body(a.jt_part, a.n_chunks, a.jtot, blockIdx.x, threadIdx.x);
  else
    total_body(a.jd_part + d * a.jd_region, a.n_chunks, a.jdtot + d * a.jdtot_region, blockIdx.x, threadIdx.x);
}

hipError_t launch_total(hipStream_t s, const TotalArgs& a, int t_count) {
  if (t_count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_total, dim3((unsigned)t_count, (unsigned)(1 + a.n_dir)), dim3(64), 0, s, a);
  return hipGetLastError();
}

// GKMA segment pass: TT = 64, 128 or 256 lanes per segment (the smallest that
// covers t_count; steps strided by TT), 256 / TT segments per work-group.  A
// segment's REDUCE_SEG slots are summed in slot order, bin by bin, into
// seg_part[mu][seg + b][t] (every bin the segment touches).
__device__ __forceinline__ void reduce_seg_body(const ReduceArgs& a, int blk) {
  const int tid = threadIdx.x;
  const int TT = a.t_count <= 64 ? 64 : (a.t_count <= 128 ? 128 : 256);
  const int G = 256 / TT;
  // one segment per wave: the branches on its bins are scalar (they
  // waited for an LDS read per slot: 1500 modes, 96 steps 14 -> 10 us)
  const int g = __builtin_amdgcn_readfirstlane(tid / TT), tl = tid % TT;
  const int64_t seg = (int64_t)blk * G + g;
  const int64_t slot0 = seg * REDUCE_SEG;
  if (seg >= a.n_seg) return;
  // lane q holds slot q's bin; bit q of first: slot q is its bin's first here
  static_assert(REDUCE_SEG == 64 && M_ALIGN % REDUCE_SEG == 0, "a segment is a wave's lanes, all inside M_pad");
  const int lane = tid & 63;
  const int bin = a.slot_bin[slot0 + lane];
  const unsigned long long first = __ballot(bin != __shfl_up(bin, 1));
  const int64_t P = (int64_t)a.n_seg + a.nb;
  const float* __restrict__ in = a.in;
  double* __restrict__ out = a.seg_part;
  for (int t = tl; t < a.t_count; t += TT) {
#pragma unroll
    for (int mu = 0; mu < 3; ++mu) {
      // all of the segment's values first (independent, unconditional loads:
      // padding rows exist in the contraction output and hold zeros), then
      // the bin-by-bin sums in slot order
      const float* col = in + ((int64_t)mu * a.M_pad + slot0) * a.ld + t;
      float x[REDUCE_SEG];
#pragma unroll
      for (int q = 0; q < REDUCE_SEG; ++q) x[q] = col[(int64_t)q * a.ld];
      asm volatile("" ::: "memory");   // no load moves behind the branches below
      double s = 0.0;
      int cur = __builtin_amdgcn_readlane(bin, 0);
#pragma unroll
      for (int q = 0; q < REDUCE_SEG; ++q) {
        if (q > 0 && (first >> q & 1)) {
          if (cur >= 0) out[((int64_t)mu * P + seg + cur) * a.ld + t] = s;
          cur = __builtin_amdgcn_readlane(bin, q);
          s = 0.0;
        }
        s += (double)x[q];   // (sums of padding are not stored)
      }
      if (cur >= 0) out[((int64_t)mu * P + seg + cur) * a.ld + t] = s;
    }
  }
}

// The work-groups from tot_blk0 on sum the steps' totals, a wave each.
__global__ void __launch_bounds__(256) k_reduce_seg(ReduceArgs a, int tot_blk0) {
  if ((int)blockIdx.x >= tot_blk0) {
    const int t = ((int)blockIdx.x - tot_blk0) * 4 + (threadIdx.x >> 6);
    if (t < a.t_count) total_body(a.jt_part, a.n_chunks, a.jtot, t, threadIdx.x & 63);
    return;
  }
  reduce_seg_body(a, blockIdx.x);
}

// Per-step path, several steps: the parts (one per step) of every (slot, mu)
// summed in step order, one thread each, every load of a step's row
// contiguous.  Left to the bins, a bin of 25 modes kept 74 threads of its
// work-group walking the steps one load at a time (64 steps of 12288 modes,
// 500 bins: 118 us, now 15 us for both kernels).
// The work-groups from tot_blk0 on sum the steps' totals as in k_reduce_seg.
__global__ void __launch_bounds__(256) k_reduce_parts(ReduceArgs a, int64_t n, int tot_blk0) {
  if ((int)blockIdx.x >= tot_blk0) {
    const int t = ((int)blockIdx.x - tot_blk0) * 4 + (threadIdx.x >> 6);
    if (t < a.t_count) total_body(a.jt_part, a.n_chunks, a.jtot, t, threadIdx.x & 63);
    return;
  }
  const float* __restrict__ in = a.in;
  const int n_parts = a.n_parts;
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= n) return;
  double s = 0.0;
  for (int p0 = 0; p0 < n_parts; p0 += 8) {
    float x[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = in[(int64_t)min(p0 + k, n_parts - 1) * n + e];
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (p0 + k < n_parts) s += (double)x[k];
  }
  a.slot_sum[e] = s;
}

// Where the sums over atoms run: with a kernel that precedes the bin sums, in
// work-groups of its own, if there is one; in the last work-group of the bin
// sums for at most 4 steps (one per wave: 1 us there, against 2 us and a
// launch's gap); in k_total otherwise (the last work-group alone would read
// every step's partials).
hipError_t launch_reduce(hipStream_t s, ReduceArgs a, const TotalArgs& tot) {
  const bool parts = !a.layout_g && a.slot_sum;
  const bool seg = a.layout_g && a.t_count > 0 && a.n_seg > 0;
  const bool with = tot.jt_part && tot.n_dir == 0 && (parts || seg || a.t_count <= 4);
  hipError_t e;
  if (tot.jt_part && !with && (e = launch_total(s, tot, a.t_count)) != hipSuccess) return e;
  a.n_chunks = tot.n_chunks;
  a.jt_part = with ? tot.jt_part : nullptr;
  const int tot_blks = with ? (a.t_count + 3) / 4 : 0;
  if (parts) {
    const int64_t n = a.M_pad * 3;
    const int blks = (int)((n + 255) / 256);
    hipLaunchKernelGGL(k_reduce_parts, dim3((unsigned)(blks + tot_blks)), dim3(256), 0, s, a, n, blks);
  } else if (seg) {
    const int TT = a.t_count <= 64 ? 64 : (a.t_count <= 128 ? 128 : 256);
    const int G = 256 / TT;
    const int blks = (a.n_seg + G - 1) / G;
    hipLaunchKernelGGL(k_reduce_seg, dim3((unsigned)(blks + tot_blks)), dim3(256), 0, s, a, blks);
  }
  if (parts || seg) {
    if ((e = hipGetLastError()) != hipSuccess) return e;
    a.jt_part = nullptr;
  }
  hipLaunchKernelGGL(k_reduce, dim3((unsigned)(a.nb + 1), (unsigned)a.n_dir), dim3(256), 0, s, a);
  return hipGetLastError();
}

// -------------------------------------------------------------- correlation
// Sums are stored lag-contiguous: C[(r*3 + nu)*L + tau].
// Work-group tile: 64 rows r x 64 lags tau (x 3 nu); X and the needed window
// of the history ring are staged in LDS per chunk of 64 steps.  The update of
// one chunk is a float64 matrix product on the matrix cores: with the window
// entry q = j + 63 - lambda holding the total at step j of the chunk minus lag
// tau0 + lambda,
//   C[r][lambda][nu] += sum_j X[r][j] * window[nu][j + 63 - lambda],
// done by v_mfma_f64_16x16x4f64 over 4 steps at a time (A = 16 rows x 4
// steps of X, B = 4 steps x 16 lags of the window, its lane (k, c) reading
// entry j + k + 63 - lambda_c).  Wave w owns rows 16w .. 16w + 15 and all 64
// lags (4 blocks of 16) for the 3 nu: 12 accumulators; lane l's register i of
// an accumulator is row 4i + l / 16, lag l % 16 of its block.  Steps past the
// block's end are staged as zeros, so every 4-step product is complete.
// Up to CORR_FILL tiles (four to a CU) a tile is 16 lags instead: the wave's
// chain of products is a quarter, X is staged four times as often.  Measured
// 64 / 16 lags per tile: 376 tiles, 1024 steps 217 / 170 us; 752 tiles 458 /
// 382 us; 1504 tiles 709 / 738 us.  Each sum takes its products in the same
// order.  With the loads of a chunk in flight together (see fetch) and the
// small tiles: 114 rows x 150 lags x 231 steps 59 -> 19 us, 1503 rows x 500
// lags x 1024 steps 261 -> 131 us.
constexpr int CT = 64;   // steps per chunk
constexpr int CR = 64;   // rows per tile
constexpr int CORR_FILL = 1024;

typedef double f64x4 __attribute__((ext_vector_type(4)));

template <int LB>   // lag blocks of 16 per tile
__device__ __forceinline__ void corr_body(const double* __restrict__ X, int64_t ldx, int t_count, int64_t R3,
                                          int L, const double* __restrict__ ring, int64_t ring_len, int64_t t0,
                                          double* __restrict__ csum, double* __restrict__ ccomp,
                                          const int64_t* __restrict__ t0_dev, const int64_t* __restrict__ tbuf_dev,
                                          int bx, int by) {
  if (tbuf_dev) {
    // buffered steps ending with this block (the same value in every thread)
    const int64_t tb = *tbuf_dev;
    if (tb <= 0) return;
    t0 = *t0_dev + t_count - tb;
    t_count = (int)tb;
  } else if (t0_dev) {
    t0 = *t0_dev;
  }
  constexpr int CL = 16 * LB;                // lags per tile
  __shared__ double xs[CR][CT + 2];          // xs[r][t]
  __shared__ double rs[3][CT + CL + 2];      // ring window, rs[nu][q]
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int c = lane & 15, g = lane >> 4;
  const int64_t r0 = (int64_t)bx * CR;
  const int tau0 = by * CL;
  f64x4 acc[LB][3];                          // [lag block][nu]
#pragma unroll
  for (int lb = 0; lb < LB; ++lb)
#pragma unroll
    for (int n = 0; n < 3; ++n) acc[lb][n] = f64x4{0.0, 0.0, 0.0, 0.0};

  // Staging of a chunk: X rows r0.. and the ring window (q in [0, CT + CL) <->
  // global time t0 + tc - tau0 - (CL - 1) + q).  The next chunk's values are
  // loaded into registers while the current chunk's products run, and written
  // to LDS after them.  Loads are unconditional, from clamped in-range
  // addresses, and the zeros for what lies outside are selected on the way to
  // LDS: selected at the load, the compiler turned each into a branch around
  // it, and a chunk's 16 loads of a thread waited for one another.
  constexpr int XPT = CR * CT / 256;                    // X values per thread
  constexpr int RPT = ((CT + CL) * 3 + 255) / 256;      // ring values per thread
  const int uwave = __builtin_amdgcn_readfirstlane(wave);
  const int rl = (int)ring_len, t0m = (int)(t0 % ring_len);
  double xr[XPT], rr[RPT];
  auto fetch = [&](int tc) {
    const int col = min(tc + lane, t_count - 1);
#pragma unroll
    for (int k = 0; k < XPT; ++k) {
      const double* row = X + min(r0 + uwave + 4 * k, R3 - 1) * ldx;   // one per wave
      xr[k] = row[col];
    }
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int idx = min(tid + 256 * k, (CT + CL) * 3 - 1);
      // steps from t0, no further back than the last lag needs (a lag past the
      // last is never stored) and no further on than the block
      int off = min(max(tc - tau0 - (CL - 1) + idx / 3, 1 - L), t_count - 1) + t0m;
      off += off < 0 ? rl : 0;
      off -= off >= rl ? rl : 0;
      rr[k] = ring[(int64_t)off * 3 + idx % 3];
    }
  };
  auto stage = [&](int tc) {
#pragma unroll
    for (int k = 0; k < XPT; ++k)
      xs[wave + 4 * k][lane] = (r0 + uwave + 4 * k < R3 && tc + lane < t_count) ? xr[k] : 0.0;
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int idx = tid + 256 * k;
      const int off = tc - tau0 - (CL - 1) + idx / 3;
      if (idx < (CT + CL) * 3) rs[idx % 3][idx / 3] = (t0 + off >= 0 && off < t_count) ? rr[k] : 0.0;
    }
  };
  fetch(0);
  for (int tc = 0; tc < t_count; tc += CT) {
    stage(tc);
    __syncthreads();
    if (tc + CT < t_count) fetch(tc + CT);
    const int jmax = min(CT, t_count - tc);
    // JU products' operands at a time (the reads stay inside the chunk)
    constexpr int JU = LB == 1 ? 4 : 2;
    for (int j0 = 0; j0 < jmax; j0 += 4 * JU) {
      double av[JU], bv[JU][LB][3];
#pragma unroll
      for (int u = 0; u < JU; ++u) {
        const int j = j0 + 4 * u + g;
        av[u] = xs[16 * wave + c][j];
#pragma unroll
        for (int lb = 0; lb < LB; ++lb)
#pragma unroll
          for (int n = 0; n < 3; ++n) bv[u][lb][n] = rs[n][j + (CL - 1) - (16 * lb + c)];
      }
#pragma unroll
      for (int u = 0; u < JU; ++u) {
        if (j0 + 4 * u >= jmax) break;
#pragma unroll
        for (int lb = 0; lb < LB; ++lb)
#pragma unroll
          for (int n = 0; n < 3; ++n)
            acc[lb][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u], bv[u][lb][n], acc[lb][n], 0, 0, 0);
      }
    }
    __syncthreads();
  }
  // Neumaier update of the lane's 4 rows x LB lags x 3: every load issues
  // from a clamped in-range address, only the stores are conditional
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t r = r0 + 16 * wave + 4 * i + g;
    const int64_t rc = min(r, R3 - 1);
#pragma unroll
    for (int n = 0; n < 3; ++n) {
      double sm[LB], cp[LB];
#pragma unroll
      for (int lb = 0; lb < LB; ++lb) {
        const int64_t o = (rc * 3 + n) * L + min(tau0 + 16 * lb + c, L - 1);
        sm[lb] = csum[o];
        cp[lb] = ccomp[o];
      }
#pragma unroll
      for (int lb = 0; lb < LB; ++lb) {
        const int tau = tau0 + 16 * lb + c;
        neumaier_add(sm[lb], cp[lb], acc[lb][n][i]);
        if (r < R3 && tau < L) {
          const int64_t o = (r * 3 + n) * L + tau;
          csum[o] = sm[lb];
          ccomp[o] = cp[lb];
        }
      }
    }
  }
}

template <int LB>
__global__ void __launch_bounds__(256) k_corr(const double* __restrict__ X, int64_t ldx, int t_count, int64_t R3,
                                              int L, const double* __restrict__ ring, int64_t ring_len, int64_t t0,
                                              double* __restrict__ csum, double* __restrict__ ccomp,
                                              const int64_t* __restrict__ t0_dev, const int64_t* __restrict__ tbuf_dev,
                                              int64_t ring_zs, int64_t out_zs) {
  // grid z: one history ring of 3 columns and one slice of sums per z
  corr_body<LB>(X, ldx, t_count, R3, L, ring + (int64_t)blockIdx.z * ring_zs, ring_len, t0,
            csum + (int64_t)blockIdx.z * out_zs, ccomp + (int64_t)blockIdx.z * out_zs, t0_dev, tbuf_dev, blockIdx.x,
            blockIdx.y);
}

hipError_t launch_corr(hipStream_t s, const double* X, int64_t ldx, int t_count, int64_t R3, int L,
                       const double* ring, int64_t ring_len, int64_t t0, double* csum, double* ccomp,
                       const int64_t* t0_dev, const int64_t* tbuf_dev, int nz, int64_t ring_zs, int64_t out_zs) {
  if (t_count <= 0 || nz <= 0) return hipSuccess;
  const int64_t rows = (R3 + CR - 1) / CR;
  const bool small = rows * ((L + 63) / 64) * nz < CORR_FILL;
  const dim3 grid((unsigned)rows, (unsigned)(small ? (L + 15) / 16 : (L + 63) / 64), (unsigned)nz);
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, X, ldx, t_count, R3, L, ring, ring_len, t0, csum, ccomp, t0_dev,
                       tbuf_dev, ring_zs, out_zs);
  };
  if (small) launch(k_corr<1>); else launch(k_corr<4>);
  return hipGetLastError();
}

// ----------------------------------------------------------------- read-out
// Work-group = 16 series q = (r, nu) over all lags, 64 lags at a time: the sums
// come in along the lags (contiguous), the running integral of a series is
// taken by one thread in LDS while the next lags' sums load, and both go out
// along the series (128 bytes contiguous).  One thread per series read its sums
// L doubles apart from its neighbours' and stored every lag by itself: 200 lags
// x 909 series 171 us, now 16 us.
constexpr int CF_S = 16, CF_T = 64;   // series and lags per tile
__global__ void __launch_bounds__(256) k_corr_finish(const double* __restrict__ csum, const double* __restrict__ ccomp,
                                                     const double* __restrict__ psum, const double* __restrict__ pcomp,
                                                     int64_t n_binned, int L, int64_t S, double dt,
                                                     double* __restrict__ corr, double* __restrict__ integral,
                                                     double* __restrict__ hcacf) {
  constexpr int V = CF_S * CF_T / 256;                        // values per thread
  __shared__ double cs[CF_S][CF_T + 1], gs[CF_S][CF_T + 1];   // [series][lag]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t n_q = n_binned + 9, q0 = (int64_t)blockIdx.x * CF_S;
  // the pending sums are read from csum where there are none, and not added
  const double* __restrict__ p0 = psum ? psum : csum;
  const double* __restrict__ p1 = psum ? pcomp : ccomp;
  double v[4][V];
  auto fetch = [&](int t0) {
    const int tau = min(t0 + lane, L - 1);
#pragma unroll
    for (int k = 0; k < V; ++k) {
      const int64_t src = min(q0 + wave + 4 * k, n_q - 1) * L + tau;
      v[0][k] = csum[src];
      v[1][k] = ccomp[src];
      v[2][k] = p0[src];
      v[3][k] = p1[src];
    }
  };
  fetch(0);
  double G = 0.0, prev = 0.0;                                 // of series q0 + tid (tid < 16)
  for (int t0 = 0; t0 < L; t0 += CF_T) {
    const int64_t cnt = S - min(t0 + lane, L - 1);
#pragma unroll
    for (int k = 0; k < V; ++k) {
      double sum = v[0][k] + v[1][k];
      if (psum) sum += v[2][k] + v[3][k];                     // steps not yet in the running sums
      cs[wave + 4 * k][lane] = (cnt > 0) ? sum / (double)cnt : 0.0;
    }
    __syncthreads();
    if (t0 + CF_T < L) fetch(t0 + CF_T);
    if (tid < CF_S) {
#pragma unroll 8
      for (int t = 0; t < CF_T; ++t) {
        const double c = cs[tid][t];
        if (t0 + t > 0) G += dt * 0.5 * (prev + c);
        gs[tid][t] = G;
        prev = c;
      }
    }
    __syncthreads();
    const int64_t q = q0 + (tid & (CF_S - 1));
#pragma unroll
    for (int k = 0; k < V; ++k) {
      const int t = tid / CF_S + k * (256 / CF_S);
      const int64_t lag = t0 + t;
      if (q >= n_q || lag >= L) continue;
      if (q < n_binned) {
        corr[lag * n_binned + q] = cs[tid & (CF_S - 1)][t];
        integral[lag * n_binned + q] = gs[tid & (CF_S - 1)][t];
      } else {
        hcacf[lag * 9 + q - n_binned] = cs[tid & (CF_S - 1)][t];
      }
    }
    __syncthreads();
  }
}

hipError_t launch_corr_finish(hipStream_t s, const double* csum, const double* ccomp, const double* psum,
                              const double* pcomp, int64_t nb, int L, int64_t S, double dt, double* corr,
                              double* integral, double* hcacf) {
  hipLaunchKernelGGL(k_corr_finish, dim3((unsigned)((nb * 9 + 9 + CF_S - 1) / CF_S)), dim3(256), 0, s, csum, ccomp, psum,
                     pcomp, nb * 9, L, S, dt, corr, integral, hcacf);
  return hipGetLastError();
}

// The bin sums, then the Eq. 10 totals, then (tdsum) their direction split.
__global__ void __launch_bounds__(256) k_hnema_finish(const double* __restrict__ hsum, const double* __restrict__ hcomp,
                                                      int64_t n, const double* __restrict__ tsum,
                                                      const double* __restrict__ tcomp,
                                                      const double* __restrict__ tdsum,
                                                      const double* __restrict__ tdcomp, int64_t S,
                                                      double* __restrict__ avg) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t k = i - n;
  double v;
  if (k < 0) v = hsum[i] + hcomp[i];
  else if (k < 3) v = tsum[k] + tcomp[k];
  else if (k < 12 && tdsum) v = tdsum[k - 3] + tdcomp[k - 3];
  else return;
  avg[i] = (S > 0) ? v / (double)S : 0.0;
}

hipError_t launch_hnema_finish(hipStream_t s, const double* hsum, const double* hcomp, int64_t n, const double* tsum,
                               const double* tcomp, const double* tdsum, const double* tdcomp, int64_t S, double* avg) {
  hipLaunchKernelGGL(k_hnema_finish, dim3((unsigned)((n + 12 + 255) / 256)), dim3(256), 0, s, hsum, hcomp, n, tsum, tcomp,
                     tdsum, tdcomp, S, avg);
  return hipGetLastError();
}

// ------------------------------------------------------- grouped back end
// The back end of every system of a group in four launches (totals, segment
// sums, bin sums, correlations); work-group w belongs to the last system i
// with wg0[i] <= w (systems with no work-groups in a launch are skipped).
__device__ __forceinline__ int back_system(const int* __restrict__ wg0, int n, int w) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (wg0[mid] <= w) lo = mid; else hi = mid - 1;
  }
  return lo;
}

__global__ void __launch_bounds__(64) k_total_group(const BackDesc* __restrict__ d, int t_count) {
  const BackDesc& s = d[blockIdx.x / t_count];
  total_body(s.jt_part, s.n_chunks, s.jtot, blockIdx.x % t_count, threadIdx.x);
}

__global__ void __launch_bounds__(256) k_reduce_seg_group(const ReduceArgs* __restrict__ a,
                                                          const int* __restrict__ wg0, int n) {
  const int i = back_system(wg0, n, blockIdx.x);
  reduce_seg_body(a[i], blockIdx.x - wg0[i]);
}

__global__ void __launch_bounds__(256) k_reduce_group(const ReduceArgs* __restrict__ a, const int* __restrict__ wg0,
                                                      int n) {
  const int i = back_system(wg0, n, blockIdx.x);
  reduce_body(a[i], blockIdx.x - wg0[i]);
}

// Tiles of 64 lags: a group's systems fill the GPU together (16 uneven systems
// with 500 bins and 1000 lags: 3072 tiles), where 64 lags are the faster tile.
__global__ void __launch_bounds__(256) k_corr_group(const BackDesc* __restrict__ d, const int* __restrict__ wg0, int n,
                                                    int t_count) {
  const int i = back_system(wg0, n, blockIdx.x);
  const BackDesc& s = d[i];
  const int local = blockIdx.x - wg0[i];
  corr_body<4>(s.X, s.ldx, t_count, s.R3, s.L, s.ring, s.ring_len, 0, s.csum, s.ccomp, s.t0_dev, s.tbuf_dev,
            local % s.n_rt, local / s.n_rt);
}

hipError_t launch_back_group(hipStream_t s, const BackGroup& b, int n, int t_count) {
  hipLaunchKernelGGL(k_total_group, dim3((unsigned)(n * t_count)), dim3(64), 0, s, b.d, t_count);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (b.n_wg_seg > 0) {
    hipLaunchKernelGGL(k_reduce_seg_group, dim3((unsigned)b.n_wg_seg), dim3(256), 0, s, b.red, b.wg0_seg, n);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_reduce_group, dim3((unsigned)b.n_wg_red), dim3(256), 0, s, b.red, b.wg0_red, n);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (b.n_wg_corr > 0) {
    hipLaunchKernelGGL(k_corr_group, dim3((unsigned)b.n_wg_corr), dim3(256), 0, s, b.d, b.wg0_corr, n, t_count);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace mhc
