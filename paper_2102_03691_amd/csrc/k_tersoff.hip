// Per-atom virial, forces and HNEMD driving force of Tersoff's bond-order
// potential on the device (float64), following Sec. II.A of the paper:
//   F_ij  = dU_i/dr_ij - dU_j/dr_ji                           (Eq. 4)
//   W_i   = sum_{j != i} r_ij (x) dU_j/dr_ji                   (Eq. 8)
//   F_ext = E_i F_e + F_e . W_i                                 (Eq. 12)
// with the site energies
//   U_i     = 1/2 sum_j f_C(r_ij) [A exp(-l1 r_ij) - b_ij B exp(-l2 r_ij)]
//   b_ij    = (1 + beta^n zeta_ij^n)^(-1/(2n))
//   zeta_ij = sum_{k != j} f_C(r_ik) g(cos theta_ijk) exp(l3^m (r_ij - r_ik)^m)
//   g(c)    = gamma (1 + c0^2/d^2 - c0^2/(d^2 + (c - h)^2)).
//
// Pipeline (deterministic: fixed summation orders, sorted lists):
//   neighbours (every few MD steps): cell of each atom (counting sort with
//     atomics), exclusive scan of the cell counts, the atoms and their
//     positions by cell, per atom a scan of the 27 surrounding cells by
//     sixteen lanes (minimum image, r < R + D + skin), list sorted by atom
//     index (so the result does not depend on the order the atomics filled the
//     cells), reverse slots (where i sits in j's list);
//   per evaluation, LPA lanes per atom (one per neighbour slot, LPA the
//     next power of two >= the largest neighbour count, at least 4; where LPA
//     is 8, 4 lanes x 2 slots), the pair values of an atom shared through LDS:
//     k_tersoff_site -- pair vector, f_C, the two exponentials, zeta_ij,
//       b_ij, db_ij/dzeta_ij; U_i (summed in slot order by the first lane);
//       the partial dU_i/dr_ij of the lane's pair;
//     k_tersoff_gather -- per pair dU_i/dr_ij - dU_j/dr_ji and
//       r_ij (x) dU_j/dr_ji (the second partial read from j's list through the
//       reverse slot), summed in slot order into F_i and W_i (Eq. 8), then
//       E_i, F_ext (Eq. 12) and the float32 copy of W_i in the layout the
//       modal-current push takes.
// Pair arrays are slot-major, [slot][N]: the lanes of a wave read 64/LPA
// consecutive atoms of each slot.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "mhc_tersoff.h"

namespace mhc {

// Minimum-image difference; iL = 1 / L.  For every pair closer than L / 2 by
// more than rounding (all listed pairs: each box edge exceeds twice the list
// cutoff) the shift is the same integer as with d / L, so the result is too.
__device__ __forceinline__ double min_image(double d, double L, double iL) { return d - L * rint(d * iL); }

__device__ __forceinline__ int cell_coord(double x, double L, int nc) {
  const double w = x - L * floor(x / L);
  int c = (int)(w * nc / L);
  return c < 0 ? 0 : (c >= nc ? nc - 1 : c);
}

// ------------------------------------------------------------- neighbour lists
__global__ void k_set_i32(int* __restrict__ p, int value) {
  if (threadIdx.x == 0) *p = value;
}

__global__ void k_fill_zero_i32(int* __restrict__ p, int n) {
  const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i < n) p[i] = 0;
}

// Cell of every atom and its place among the cell's atoms (in the order the
// atomics served them; the sorted lists do not depend on it).
__global__ void __launch_bounds__(256) k_cell_count(const double* __restrict__ pos, int64_t N, CellGrid cg,
                                                    int* __restrict__ cell_of, int* __restrict__ place,
                                                    int* __restrict__ count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const int cx = cell_coord(pos[3 * i], cg.box[0], cg.nc[0]);
  const int cy = cell_coord(pos[3 * i + 1], cg.box[1], cg.nc[1]);
  const int cz = cell_coord(pos[3 * i + 2], cg.box[2], cg.nc[2]);
  const int c = (cx * cg.nc[1] + cy) * cg.nc[2] + cz;
  cell_of[i] = c;
  place[i] = atomicAdd(&count[c], 1);
}

// Exclusive scan of n counts into start[0..n] (start[n] = total) over tiles
// of SCAN_TILE counts: per-tile sums, then every tile's own scan plus the sum
// of the tiles before it, which each work-group adds up itself while there are
// few tiles (an exclusive scan of the tile sums by one work-group in between
// where there are more than SCAN_DIRECT of them).
// Up to SCAN_SELF tiles each adds the counts before it for itself instead, and
// k_scan_tile_sums does not run either (2 to 3 us less up to 8 tiles, 0.5 us
// less at 36).
constexpr int SCAN_TILE = 1024, SCAN_DIRECT = 2048, SCAN_SELF = 40;

// Inclusive scan of one value per thread over a 1024-thread work-group: each
// wave by shuffles, then the sums of the waves before.
__device__ __forceinline__ int block_scan_incl(int v, int* sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int w = __shfl_up(v, off);
    if (lane >= off) v += w;
  }
  if (lane == 63) sh[wave] = v;
  __syncthreads();
  for (int w = 0; w < wave; ++w) v += sh[w];
  __syncthreads();
  return v;
}

__global__ void __launch_bounds__(1024) k_scan_tile_sums(const int* __restrict__ count, int n, int* __restrict__ sums) {
  __shared__ int sh[16];
  const int c = blockIdx.x * SCAN_TILE + threadIdx.x;
  const int v = block_scan_incl(c < n ? count[c] : 0, sh);
  if (threadIdx.x == SCAN_TILE - 1) sums[blockIdx.x] = v;
}

// Exclusive scan of the tile sums in place (n_tiles values, any count).
__global__ void __launch_bounds__(1024) k_scan_tile_offsets(int* __restrict__ sums, int n_tiles) {
  __shared__ int sh[16];
  __shared__ int total;
  int run = 0;
  for (int base = 0; base < n_tiles; base += SCAN_TILE) {
    const int c = base + threadIdx.x;
    const int v = c < n_tiles ? sums[c] : 0;
    const int incl = block_scan_incl(v, sh);
    if (c < n_tiles) sums[c] = run + incl - v;
    if (threadIdx.x == SCAN_TILE - 1) total = incl;
    __syncthreads();
    run += total;
    __syncthreads();
  }
}

// start, and zero in flags[1] for the search that follows.  sums (null: the
// counts themselves) holds the sums of the tiles, or with scanned their offsets.
__global__ void __launch_bounds__(1024) k_scan_apply(const int* __restrict__ count, int n,
                                                     const int* __restrict__ sums, bool scanned,
                                                     int* __restrict__ start, int* __restrict__ flags) {
  __shared__ int sh[16];
  __shared__ int before;
  const int t = threadIdx.x;
  if (blockIdx.x == 0 && t == 0) flags[1] = 0;
  if (!scanned) {
    int s = 0;
    const int tiles = blockIdx.x;
    if (sums) {
      for (int k = t; k < tiles; k += SCAN_TILE) s += sums[k];
    } else {
      for (int k0 = 0; k0 < tiles; k0 += 16) {   // sixteen loads at a time
        int x[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) x[q] = count[min(k0 + q, tiles - 1) * SCAN_TILE + t];
#pragma unroll
        for (int q = 0; q < 16; ++q) s += k0 + q < tiles ? x[q] : 0;
      }
    }
    s = block_scan_incl(s, sh);
    if (t == SCAN_TILE - 1) before = s;
  } else if (t == 0) {
    before = sums[blockIdx.x];
  }
  const int c = blockIdx.x * SCAN_TILE + t;
  const int v = c < n ? count[c] : 0;
  const int own = block_scan_incl(v, sh);   // synchronizes: `before` is there
  const int incl = own + before;
  if (c < n) start[c] = incl - v;
  if (c == n - 1) start[n] = incl;
}

// The atoms by cell, and their positions in that order.
__global__ void __launch_bounds__(256) k_cell_fill(const double* __restrict__ pos, int64_t N,
                                                   const int* __restrict__ cell_of, const int* __restrict__ place,
                                                   const int* __restrict__ start, int* __restrict__ atoms,
                                                   double* __restrict__ cpos) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const int64_t k = start[cell_of[i]] + place[i];
  atoms[k] = (int)i;
  cpos[3 * k] = pos[3 * i];
  cpos[3 * k + 1] = pos[3 * i + 1];
  cpos[3 * k + 2] = pos[3 * i + 2];
}

// The lists: NL lanes per atom, NA atoms per work-group.  The candidates of
// an atom are the atoms of up to nine rows of cells along z (the three cells
// of a row are consecutive, and so are their atoms; at the ends of the row two
// pieces); lane r sets up row r, then the lanes walk all candidates NL at a
// time, reading consecutive entries of the cell-ordered positions.  The pairs
// found go to LDS in any order; each then counts the smaller indices among
// them, which is its slot (ascending j, whatever order the cells were filled
// in), and the work-group writes 16 consecutive atoms of a slot at a time.
// Bound: latency of the dependent loads (row -> candidates).  Measured against
// one thread per atom with an insertion sort in global memory: 64000 Si atoms
// without skin 63.5 -> 17.6 us.  The largest counts go out per work-group and
// k_reverse takes their maximum: an atomic maximum on one address costs every
// work-group its turn (64000 atoms 69 us, 512000 atoms 540 us).
// most[work-group] = its largest counts inside rc (which may exceed max_nb:
// only max_nb are kept) and inside rb.  clear: cell counts to zero for the
// next search (n_clear: at most the launch's lanes).
constexpr int NB_LANES = 16, NB_ATOMS = 16, NB_MAX = 64;
__global__ void __launch_bounds__(NB_LANES * NB_ATOMS) k_neighbors(
    const double* __restrict__ pos, int64_t N, CellGrid cg, double rc2, double rb2, const int* __restrict__ cell_of,
    const int* __restrict__ start, const int* __restrict__ atoms, const double* __restrict__ cpos, int max_nb,
    int* __restrict__ nbr, int* __restrict__ n_nb, int2* __restrict__ most, int* __restrict__ clear, int64_t n_clear) {
  constexpr int NL = NB_LANES, NA = NB_ATOMS;
  __shared__ int first[NA][9], len[NA][9], wrap[NA][9], upto[NA][10];   // row: main piece, its length, second piece
  __shared__ int found[NA][NB_MAX], sorted[NA][NB_MAX];
  __shared__ int cnt[NA], cntb[NA];
  const int tid = threadIdx.x, l = tid & (NL - 1), a = tid / NL;
  const int64_t i0 = (int64_t)blockIdx.x * NA, i = i0 + a;
  const int64_t q0 = (int64_t)blockIdx.x * (NL * NA) + tid;
  if (q0 < n_clear) clear[q0] = 0;
  const bool act = i < N;
  const int c = act ? cell_of[i] : 0;
  int n_row = 0, f = 0, m = 0, w = 0;
  if (act && l < 9) {
    const int cz0 = c % cg.nc[2], cy0 = (c / cg.nc[2]) % cg.nc[1], cx0 = c / (cg.nc[2] * cg.nc[1]);
    const int dx = l / 3 - 1, dy = l % 3 - 1;
    // an axis of one cell has no neighbouring cells
    if ((dx == 0 || cg.nc[0] >= 3) && (dy == 0 || cg.nc[1] >= 3)) {
      const int cx = (cx0 + dx + cg.nc[0]) % cg.nc[0], cy = (cy0 + dy + cg.nc[1]) % cg.nc[1];
      const int row = (cx * cg.nc[1] + cy) * cg.nc[2];
      int z0 = cz0, z1 = cz0 + 1, zw = -1;
      if (cg.nc[2] >= 3) {
        z0 = cz0 - 1;
        z1 = cz0 + 2;
        if (z0 < 0) zw = cg.nc[2] - 1, z0 = 0;
        if (z1 > cg.nc[2]) zw = 0, z1 = cg.nc[2];
      }
      f = start[row + z0];
      m = start[row + z1] - f;
      n_row = m;
      if (zw >= 0) {
        w = start[row + zw];
        n_row += start[row + zw + 1] - w;
      }
    }
  }
  int up = n_row;   // inclusive sum over the rows
#pragma unroll
  for (int off = 1; off < NL; off <<= 1) {
    const int o = __shfl_up(up, off, NL);
    if (l >= off) up += o;
  }
  if (l < 9) {
    first[a][l] = f;
    len[a][l] = m;
    wrap[a][l] = w;
    upto[a][l + 1] = up;
  }
  if (l == 9) upto[a][0] = 0;
  if (l == 10) cnt[a] = 0;
  if (l == 11) cntb[a] = 0;
  __syncthreads();
  if (act) {
    const double xi = pos[3 * i], yi = pos[3 * i + 1], zi = pos[3 * i + 2];
    const int total = upto[a][9];
    int r = 0;
    for (int k = l; k < total; k += NL) {
      while (k >= upto[a][r + 1]) ++r;
      const int o = k - upto[a][r];
      const int64_t q = o < len[a][r] ? first[a][r] + o : wrap[a][r] + (o - len[a][r]);
      const int j = atoms[q];
      const double ddx = min_image(cpos[3 * q] - xi, cg.box[0], cg.ibox[0]);
      const double ddy = min_image(cpos[3 * q + 1] - yi, cg.box[1], cg.ibox[1]);
      const double ddz = min_image(cpos[3 * q + 2] - zi, cg.box[2], cg.ibox[2]);
      const double d2 = ddx * ddx + ddy * ddy + ddz * ddz;
      if (j != (int)i && d2 < rc2) {
        const int p = atomicAdd(&cnt[a], 1);
        if (p < max_nb) found[a][p] = j;
        if (d2 < rb2) atomicAdd(&cntb[a], 1);
      }
    }
  }
  __syncthreads();
  const int n = act ? min(cnt[a], max_nb) : 0;
  for (int p = l; p < n; p += NL) {
    const int j = found[a][p];
    int rank = 0;
    for (int q = 0; q < n; ++q) rank += found[a][q] < j;
    sorted[a][rank] = j;
  }
  __syncthreads();
  // slot-major rows, consecutive atoms of a slot by consecutive lanes
  const int wa = tid % NA;
  const int wn = i0 + wa < N ? min(cnt[wa], max_nb) : 0;
  for (int s = tid / NA; s < wn; s += NL) nbr[(int64_t)s * N + i0 + wa] = sorted[wa][s];
  if (tid < NA && i0 + tid < N) n_nb[i0 + tid] = min(cnt[tid], max_nb);
  if (tid < 64) {
    int mc = tid < NA ? cnt[tid] : 0, mb = tid < NA ? cntb[tid] : 0;
#pragma unroll
    for (int o = NA / 2; o > 0; o >>= 1) {
      mc = max(mc, __shfl_xor(mc, o, 64));
      mb = max(mb, __shfl_xor(mb, o, 64));
    }
    if (tid == 0) most[blockIdx.x] = make_int2(mc, mb);
  }
}

// rev[s][i] = slot of i in the list of j = nbr[s][i] (-1 if absent, which a
// symmetric distance test rules out; the host checks).  Lists are ascending
// (k_neighbors sorts them), so the slot is found by bisection.
// One lane per (atom, slot): threadIdx.x runs over 64 consecutive atoms (so a
// wave's list reads and writes are contiguous) and threadIdx.y over the slots
// y, y + REV_SLOTS, ...; each lane finds i in j's sorted list by bisection.
constexpr int REV_SLOTS = 16;
__global__ void __launch_bounds__(64 * REV_SLOTS) k_reverse(int64_t N, const int* __restrict__ nbr,
                                                            const int* __restrict__ n_nb, int* __restrict__ rev,
                                                            int* __restrict__ flags, const int2* __restrict__ most,
                                                            int n_most) {
  if (blockIdx.x == 0) {   // the search's largest counts: flags[0] and flags[2]
    __shared__ int sh[2][REV_SLOTS];
    const int t = threadIdx.y * 64 + threadIdx.x;
    int mc = 0, mb = 0;
    for (int k = t; k < n_most; k += 64 * REV_SLOTS) {
      mc = max(mc, most[k].x);
      mb = max(mb, most[k].y);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      mc = max(mc, __shfl_xor(mc, o, 64));
      mb = max(mb, __shfl_xor(mb, o, 64));
    }
    if (threadIdx.x == 0) sh[0][threadIdx.y] = mc, sh[1][threadIdx.y] = mb;
    __syncthreads();
    if (t < 2) {
      int m = 0;
      for (int w = 0; w < REV_SLOTS; ++w) m = max(m, sh[t][w]);
      flags[2 * t] = m;
    }
  }
  const int64_t i = (int64_t)blockIdx.x * 64 + threadIdx.x;
  if (i >= N) return;
  const int n = n_nb[i];
  for (int s = threadIdx.y; s < n; s += REV_SLOTS) {
    const int j = nbr[(int64_t)s * N + i];
    const int nj = n_nb[j];
    int lo = 0, hi = nj;   // first slot of j's list whose entry is >= i
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (nbr[(int64_t)mid * N + j] < (int)i) lo = mid + 1;
      else hi = mid;
    }
    const int r = lo < nj && nbr[(int64_t)lo * N + j] == (int)i ? lo : -1;
    rev[(int64_t)s * N + i] = r;
    if (r < 0) flags[1] = 1;
  }
}

// --------------------------------------------------------------- potential
__device__ __forceinline__ void cutoff_fn(const TersoffParams& p, double r, double* fc, double* dfc) {
  if (r < p.R - p.D) {
    *fc = 1.0;
    *dfc = 0.0;
  } else if (r > p.R + p.D) {
    *fc = 0.0;
    *dfc = 0.0;
  } else {
    double s, c;
    sincos(0.5 * M_PI * (r - p.R) / p.D, &s, &c);
    *fc = 0.5 - 0.5 * s;
    *dfc = -0.25 * M_PI / p.D * c;
  }
}

// 1 / x for a positive normal x whose reciprocal is normal too: the hardware
// estimate refined by two Newton steps, within about an ulp of the rounded
// quotient (a full IEEE division adds scaling for the extremes of the range
// and a final correctly rounded step)
__device__ __forceinline__ double recip(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  r = fma(r, fma(-x, r, 1.0), r);
  return r;
}

// Natural logarithm of a positive x (normal or subnormal): x = m 2^e with m in
// [sqrt(1/2), sqrt(2)), log m = 2 atanh(s) with s = (m - 1) / (m + 1) summed as
// its odd power series (Abramowitz and Stegun 4.1.27; |s| < 0.1716, so the
// terms up to s^23 leave less than 1e-18), e ln 2 with ln 2 in two parts (the
// first with 21 significant bits, so e times it is exact).  Within 3 ulps of
// the true value from the subnormals up, at a fraction of the cost of the
// library routine, which carries double-length sums.
__device__ __forceinline__ double log_pos(double x) {
  int e;
  double m = frexp(x, &e);   // [0.5, 1)
  if (m < 0.70710678118654752440) {
    m += m;
    --e;
  }
  const double s = (m - 1.0) * recip(m + 1.0);
  const double s2 = s * s;
  double t = 1.0 / 23.0;
  t = fma(t, s2, 1.0 / 21.0);
  t = fma(t, s2, 1.0 / 19.0);
  t = fma(t, s2, 1.0 / 17.0);
  t = fma(t, s2, 1.0 / 15.0);
  t = fma(t, s2, 1.0 / 13.0);
  t = fma(t, s2, 1.0 / 11.0);
  t = fma(t, s2, 1.0 / 9.0);
  t = fma(t, s2, 1.0 / 7.0);
  t = fma(t, s2, 1.0 / 5.0);
  t = fma(t, s2, 1.0 / 3.0);
  const double lm = fma(2.0 * s * s2, t, 2.0 * s);
  const double de = (double)e;
  return fma(de, 0.6931467056274414, fma(de, 4.7493250390316726e-07, lm));
}

// log(1 + x) for x >= 0 by Goldberg's form x log(u) / (u - 1), u = 1 + x
// rounded (exact where u = 1): within 5 ulps for x below 2^1020
__device__ __forceinline__ double log1p_pos(double x) {
  const double u = 1.0 + x;
  return u == 1.0 ? x : (x * recip(u - 1.0)) * log_pos(u);
}

// g(cos theta) with t = cos theta - h, as gamma (1 + (c^2/d^2) t^2 / (d^2 + t^2)):
// the same function as gamma (1 + c^2/d^2 - c^2 / (d^2 + t^2)) without the
// cancellation of its two large terms (c^2/d^2 is about 4e7 for Si, g about 1e4)
__device__ __forceinline__ double angle_g(const TersoffParams& p, double cs) {
  const double t = cs - p.h;
  const double t2 = t * t;
  return fma(p.gc2d2 * t2, recip(p.d2 + t2), p.gamma);
}

// g and dg / dcos theta = 2 gamma c^2 t / (d^2 + t^2)^2
__device__ __forceinline__ void angle_fn(const TersoffParams& p, double cs, double* g, double* dg) {
  const double t = cs - p.h;
  const double t2 = t * t;
  const double inv = recip(p.d2 + t2);
  *g = fma(p.gc2d2 * t2, inv, p.gamma);
  *dg = p.g2c2 * t * inv * inv;
}

// exp(l3^m x^m) and its derivative in x (m = 1 or 3); L3 = false: lambda3 = 0
template <bool L3>
__device__ __forceinline__ void exp_fn(const TersoffParams& p, double x, double* e, double* de) {
  if (!L3) {
    *e = 1.0;
    *de = 0.0;
    return;
  }
  const double xm1 = p.m == 3 ? x * x : 1.0;
  *e = exp(p.l3m * xm1 * x);
  *de = *e * p.m * p.l3m * xm1;
}

// zeta + (f_C g) e with f_C g rounded first, also where e = 1 (left to itself the
// compiler would then fuse the product f_C g into the sum)
template <bool L3>
__device__ __forceinline__ double zeta_add(double fg, double e, double zeta) {
  if (L3) return fma(fg, e, zeta);
  asm("" : "+v"(fg));
  return zeta + fg;
}

// List slot of the s-th kept pair of a bond mask (bit f: list slot f is kept).
__device__ __forceinline__ int kept_slot(unsigned long long m, int s) {
  for (int c = 0; c < s; ++c) m &= m - 1;
  return __builtin_ctzll(m);
}

// LPA lanes per atom, SPL list slots per lane: lane s0 of the group handles
// the pairs (i, j = nbr[s][i]) of the slots s = s0 + k LPA, k < SPL.  Each
// pair's values go to LDS (field-major, sh[field][atom base + slot]) and
// every lane reads them after a barrier.  All sums run over the slots in list
// order, so the results do not depend on LPA and SPL.  With SPL = 2 a wave
// whose atoms all have at most LPA pairs skips the second slot of every lane.
// One wavefront per work-group: an atom's lanes never span two (LPA <= 64), so
// the barriers only order the wave's own LDS traffic, and waves of unequal
// length (atoms with more pairs) do not wait for each other.  L3: lambda3 is
// not 0 (without it the exponentials of a triplet and their derivatives go).
// Bound: float64 instructions (216000 atoms), the chain of loads and
// arithmetic of one pair (8000 atoms).  Measured, other pairs one after the
// other with a test each and lists loaded after their counts: 216000 Si atoms
// 33.5 -> 28.8 us, 8000 atoms 7.0 -> 6.2 us.
constexpr int SITE_WG = 64;
template <int LPA, int SPL, bool L3>
__global__ void __launch_bounds__(SITE_WG) k_tersoff_site(TersoffArgs a, TersoffParams p) {
  __shared__ double sh[8][SITE_WG * SPL];
  const int tid = threadIdx.x;
  const int s0 = tid & (LPA - 1);
  const int gb = (tid - s0) * SPL;   // this atom's slot 0 in LDS
  const int64_t N = a.N;
  const int64_t i = ((int64_t)blockIdx.x * SITE_WG + tid) / LPA;
  const int64_t ic = i < N ? i : N - 1;
  // the count, the first list entry and the atom's position in flight together
  // (and with the rebuild flag): an entry past the count, or of a list about
  // to be rebuilt, is not used
  int n = a.n_nb[ic];
  int j0 = a.nbr[(int64_t)min(s0, a.max_nb - 1) * N + ic];
  const double xi = a.pos[3 * ic], yi = a.pos[3 * ic + 1], zi = a.pos[3 * ic + 2];
  const bool build = a.bond_need && *a.bond_need;   // one value for the whole grid
  asm volatile("" ::: "memory");                    // no load moves behind the branches below
  if (a.bond_clear && blockIdx.x == 0 && tid == 0) *a.bond_clear = 0;
  if (i >= N) n = 0;
  if (build) {
    // bond lists out of the skin lists (BondBufs): the listed pairs closer
    // than rb in list order, LPA list slots at a time; their reverse slots
    // need every atom's mask and come from the gather kernel
    const int full = i < N ? a.full_n[i] : 0;
    unsigned long long m = 0;
    for (int f0 = 0; __ballot(f0 < full) != 0; f0 += LPA) {
      bool keep = false;
      if (f0 + s0 < full) {
        const int64_t j = a.full_nbr[(int64_t)(f0 + s0) * N + i];
        const double dx = min_image(a.pos[3 * j] - xi, a.box[0], a.ibox[0]);
        const double dy = min_image(a.pos[3 * j + 1] - yi, a.box[1], a.ibox[1]);
        const double dz = min_image(a.pos[3 * j + 2] - zi, a.box[2], a.ibox[2]);
        keep = dx * dx + dy * dy + dz * dz < a.bond_rb2;
      }
      const unsigned long long hits = __ballot(keep) >> (tid - s0);
      m |= (LPA == 64 ? hits : hits & ((1ull << (LPA & 63)) - 1ull)) << f0;
    }
    const int found = __builtin_popcountll(m);
    n = found < a.max_nb ? found : a.max_nb;
    if (i < N && s0 == 0) {
      a.bond_n[i] = n;
      a.bond_mask[i] = m;
      a.bond_ref[3 * i] = xi;
      a.bond_ref[3 * i + 1] = yi;
      a.bond_ref[3 * i + 2] = zi;
      if (found > a.max_nb) {
        atomicMax(&a.bond_flags[0], found);
        a.bond_flags[1] = 1;
      }
    }
#pragma unroll
    for (int k = 0; k < SPL; ++k) {
      const int s = s0 + k * LPA;
      if (s < n) {
        const int j = a.full_nbr[(int64_t)kept_slot(m, s) * N + i];
        a.bond_nbr[(int64_t)s * N + i] = j;
        if (k == 0) j0 = j;
      }
    }
  }
  double x[SPL], y[SPL], z[SPL], r[SPL], ir[SPL], fc[SPL], dfc[SPL], er[SPL], ea[SPL];
#pragma unroll
  for (int k = 0; k < SPL; ++k) {
    const int s = s0 + k * LPA;
    x[k] = y[k] = z[k] = 0.0;
    r[k] = ir[k] = 1.0;
    fc[k] = dfc[k] = er[k] = ea[k] = 0.0;
    if (s < n) {
      const int64_t j = k == 0 ? j0 : a.nbr[(int64_t)s * N + i];
      x[k] = min_image(a.pos[3 * j] - xi, a.box[0], a.ibox[0]);
      y[k] = min_image(a.pos[3 * j + 1] - yi, a.box[1], a.ibox[1]);
      z[k] = min_image(a.pos[3 * j + 2] - zi, a.box[2], a.ibox[2]);
      r[k] = sqrt(x[k] * x[k] + y[k] * y[k] + z[k] * z[k]);
      ir[k] = 1.0 / r[k];
      cutoff_fn(p, r[k], &fc[k], &dfc[k]);
      if (fc[k] != 0.0) {                    // a pair beyond R + D (listed with a skin) needs neither
        er[k] = p.A * exp(-p.l1 * r[k]);     // f_R
        ea[k] = p.B * exp(-p.l2 * r[k]);     // f_A (the attractive term enters as -b f_A)
      }
    }
    sh[0][gb + s] = x[k];
    sh[1][gb + s] = y[k];
    sh[2][gb + s] = z[k];
    sh[3][gb + s] = r[k];
    sh[4][gb + s] = ir[k];
    sh[5][gb + s] = fc[k];
  }
  __syncthreads();
  // Listed pairs beyond R + D (f_C = 0: lists built with a skin) add exact
  // zeros to every sum below, so they are skipped, and such a pair's own
  // slot has nothing to compute (its energy, bracket weight and partials are
  // zero).
  //
  // The other pairs q != s of a bond go three at a time (a bond of an atom with
  // four has three), o-th other = slot o + (o >= s): their LDS reads and angle
  // terms are independent, only the sums chain.
  constexpr int OTH = 3;
  double b[SPL], adb[SPL];
#pragma unroll
  for (int k = 0; k < SPL; ++k) {
    const int s = s0 + k * LPA;
    b[k] = 1.0;
    adb[k] = 0.0;
    double u = 0.0;
    if (s < n && fc[k] != 0.0) {
      double zeta = 0.0;
      for (int o0 = 0; o0 < n - 1; o0 += OTH) {
        double term[OTH], e[OTH], fq[OTH];
#pragma unroll
        for (int v = 0; v < OTH; ++v) {
          const int l = gb + min(o0 + v + (o0 + v >= s ? 1 : 0), n - 1);
          fq[v] = o0 + v < n - 1 ? sh[5][l] : 0.0;
          const double cs = (x[k] * sh[0][l] + y[k] * sh[1][l] + z[k] * sh[2][l]) * (ir[k] * sh[4][l]);
          double de;
          term[v] = angle_g(p, cs);
          exp_fn<L3>(p, r[k] - sh[3][l], &e[v], &de);
        }
#pragma unroll
        for (int v = 0; v < OTH; ++v)
          if (fq[v] != 0.0) zeta = zeta_add<L3>(fq[v] * term[v], e[v], zeta);
      }
      // (beta zeta)^n and (1 + bz)^(-1/(2n)) through exp and log (bz = 0 where beta zeta = 0)
      const double bzeta = p.beta * zeta;
      const double bz = bzeta > 0.0 ? exp(p.n * log_pos(bzeta)) : 0.0;
      b[k] = exp(p.ninv2 * log1p_pos(bz));
      // db/dzeta = -1/2 beta^n zeta^(n-1) (1 + (beta zeta)^n)^(-1/(2n) - 1) = -b bz / (2 zeta (1 + bz))
      const double db = zeta == 0.0 ? 0.0 : -0.5 * b[k] * bz / (zeta * (1.0 + bz));
      adb[k] = fc[k] * ea[k] * db;
      u = fc[k] * (er[k] - b[k] * ea[k]);
    }
    sh[6][gb + s] = adb[k];
    sh[7][gb + s] = u;
  }
  __syncthreads();
  if (i < N && s0 == 0) {
    double acc = 0.0;
    for (int q = 0; q < n; ++q) acc += sh[7][gb + q];
    a.U[i] = 0.5 * acc;
  }
#pragma unroll
  for (int k = 0; k < SPL; ++k) {
    const int s = s0 + k * LPA;
    if (s >= n) continue;
    double* dd = a.dd + 3 * ((int64_t)s * N + i);
    if (fc[k] == 0.0) {
      dd[0] = 0.0;
      dd[1] = 0.0;
      dd[2] = 0.0;
      continue;
    }
    // dU_i/dr_ij for this slot's pair j
    const double ux = x[k] * ir[k], uy = y[k] * ir[k], uz = z[k] * ir[k];
    // (one association of the sum, so that its value does not depend on the build)
    const double radial = 0.5 * fma(dfc[k], er[k] - b[k] * ea[k], fc[k] * (-p.l1 * er[k] + p.l2 * b[k] * ea[k]));
    const double ir2 = ir[k] * ir[k];
    double zx = 0.0, zy = 0.0, zz = 0.0;   // d zeta_ij / d r_ij
    double kx = 0.0, ky = 0.0, kz = 0.0;   // sum_{k != j} a_ik db_ik d zeta_ik / d r_ij
    for (int o0 = 0; o0 < n - 1; o0 += OTH) {
#pragma unroll
      for (int v = 0; v < OTH; ++v) {
        const int l = gb + min(o0 + v + (o0 + v >= s ? 1 : 0), n - 1);
        const double fcq = o0 + v < n - 1 ? sh[5][l] : 0.0;
        const double qx = sh[0][l], qy = sh[1][l], qz = sh[2][l], rq = sh[3][l];
        const double iri = ir[k] * sh[4][l];   // 1 / (r_ij r_ik)
        const double cs = (x[k] * qx + y[k] * qy + z[k] * qz) * iri;
        // d cos theta / d r_ij = r_ik / (r_ij r_ik) - cos theta r_ij / r_ij^2
        const double cr = cs * ir2;
        const double cx = fma(qx, iri, -x[k] * cr);
        const double cy = fma(qy, iri, -y[k] * cr);
        const double cz = fma(qz, iri, -z[k] * cr);
        double g, dg, e1, de1, e2, de2;
        angle_fn(p, cs, &g, &dg);
        exp_fn<L3>(p, r[k] - rq, &e1, &de1);
        exp_fn<L3>(p, rq - r[k], &e2, &de2);
        // zeta_ij's term: f_C(r_ik) (g' e1 dcos/dr_ij + g e1' u_ij)
        const double za = fcq * dg * e1, zb = fcq * g * de1;
        // zeta_ik's term through f_C(r_ij), g and e2 = exp(l3^m (r_ik - r_ij)^m), weighted by a_ik db_ik
        const double w = sh[6][l];
        const double ka = w * fc[k] * dg * e2, kb = w * g * (dfc[k] * e2 - fc[k] * de2);
        if (fcq != 0.0) {
          zx = fma(za, cx, L3 ? fma(zb, ux, zx) : zx);   // zb = 0 without lambda3
          zy = fma(za, cy, L3 ? fma(zb, uy, zy) : zy);
          zz = fma(za, cz, L3 ? fma(zb, uz, zz) : zz);
          kx = fma(ka, cx, fma(kb, ux, kx));
          ky = fma(ka, cy, fma(kb, uy, ky));
          kz = fma(ka, cz, fma(kb, uz, kz));
        }
      }
    }
    dd[0] = radial * ux - 0.5 * (adb[k] * zx + kx);
    dd[1] = radial * uy - 0.5 * (adb[k] * zy + ky);
    dd[2] = radial * uz - 0.5 * (adb[k] * zz + kz);
  }
}

// Orders a wave's own LDS traffic (its LDS operations complete in order; this
// keeps the compiler from moving them).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Per pair dU_i/dr_ij - dU_j/dr_ji (Eq. 4) and r_ij (x) dU_j/dr_ji (Eq. 8),
// LPA lanes per atom and SPL slots per lane as in the site kernel.  A round of
// LPA slots goes through the wave's own part of LDS, from which each of the
// atom's lanes adds its share of the twelve sums (F, then W row by row) in
// slot order; rounds that no atom of the wave has are skipped.  The sums go
// back to LDS, so that the three lanes of an atom finish one component each
// (E_i, F_ext of Eq. 12, with o.kick_vel the second half kick and thermostat
// scale of the step) and W leaves in whole lines.  Bound: the scattered reads
// of the partners' partials (24 contiguous bytes each).  Measured against one
// lane summing and storing for its atom, partials in three planes, 8 lanes
// for 4 bonds: 216000 Si atoms in MD 24.2 -> 16.0 us, 8000 atoms 6.2 -> 4.9 us.
// The rest of an NVE step (half kicks, drift, displacement test) runs here
// too, a component per lane: 216000 atoms 22 us instead of 16 + 7.3 us in a
// kernel of its own, and one launch fewer (a step of 8000 atoms 20.4 -> 15.3 us
// with the bond build in the site kernel instead of one that mostly exits).
// A step's two kernels are chains of dependent loads, so every load that needs
// no other goes first, and the partials of bond lists with the positions: an
// MD step of 216000 atoms 59.8 -> 54.9 us, of 512000 117 -> 108 us, of 8000
// under the thermostat 17.4 -> 17.0 us.
constexpr int GATHER_WG = 256;
template <int LPA, int SPL>
__global__ void __launch_bounds__(GATHER_WG) k_tersoff_gather(TersoffArgs a, GatherArgs o) {
  constexpr int APW = 64 / LPA, APB = GATHER_WG / LPA;   // atoms per wave, per work-group
  constexpr int QL = LPA >= 12 ? 1 : (12 + LPA - 1) / LPA;   // sums per lane
  constexpr int ROW = 66;                                // padded: the lanes of an atom read different rows
  __shared__ double pair[GATHER_WG / 64][12 * ROW];
  __shared__ double tot[GATHER_WG / 64][APW * 12];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int s0 = lane & (LPA - 1), g = lane / LPA;       // slot of round 0; atom within the wave
  double* sh = pair[wave];
  double* tt = tot[wave];
  const int64_t N = a.N;
  const int64_t i0 = (int64_t)blockIdx.x * APB + (int64_t)wave * APW, i = i0 + g;
  // Every load that needs no other goes first, without a branch (what a call
  // does not use is read from an array that is there): the count, the first
  // round's list entry and reverse slot (the rows below max_nb exist; entries
  // at or past n are not used) and what component s0 needs at the end.
  const int64_t ic = i < N ? i : N - 1;
  const int64_t e0 = (int64_t)min(s0, a.max_nb - 1) * N + ic, qc = 3 * ic + min(s0, 2);
  const bool ext = o.Fext || o.add_ext, comp = i < N && s0 < 3;
  const int n_i = a.n_nb[ic];
  int jl = a.nbr[e0], rl = a.rev[e0];
  const int need = *(a.bond_need ? a.bond_need : a.n_nb);
  const double x_q = a.pos[qc], e_i = (ext ? a.U : a.pos)[ic];
  const double m_i = (o.vel || o.kick_vel ? o.mass : a.pos)[ic];
  const double* pv = o.vel ? o.vel : a.pos;
  const double va[3] = {pv[3 * ic], pv[3 * ic + 1], pv[3 * ic + 2]};
  const double v_q = (o.kick_vel ? o.kick_vel : a.pos)[qc], ref_q = (o.drift_ref ? o.drift_ref : a.pos)[qc];
  const double scale = (o.kick_scale ? o.kick_scale : a.pos)[2];
  asm volatile("" ::: "memory");   // the loads stay up here
  const int n = i < N ? n_i : 0;
  const bool built = a.bond_need && need;   // bond lists just built by the site kernel
  // the reverse slots of new bond lists: bond s of i sits at the s-th kept
  // slot f of i's skin list, which is slot t = full_rev[f][i] in the list of
  // j; its bond slot in j's list is the number of j's kept slots below t
  const unsigned long long mi = built && i < N ? a.bond_mask[i] : 0ull;
  auto reverse_slot = [&](int s, int64_t j) -> int {
    const int t = a.full_rev[(int64_t)kept_slot(mi, s) * N + i];
    const unsigned long long mj = t >= 0 ? a.bond_mask[j] : 0ull;
    const int r = t >= 0 && ((mj >> t) & 1ull) ? __builtin_popcountll(mj & ((1ull << t) - 1ull)) : -1;
    a.bond_rev[(int64_t)s * N + i] = r < 0 ? 0 : r;   // the call fails at its end; no read out of range until then
    if (r < 0) a.bond_flags[2] = 1;
    return r < 0 ? 0 : r;
  };
  double sum[QL];
#pragma unroll
  for (int q = 0; q < QL; ++q) sum[q] = 0.0;
#pragma unroll
  for (int k = 0; k < SPL; ++k) {
    if (k > 0 && __ballot(n > k * LPA) == 0) break;
    const int s = s0 + k * LPA;
    double c[12];
#pragma unroll
    for (int q = 0; q < 12; ++q) c[q] = 0.0;
    if (s < n) {
      const int64_t es = (int64_t)s * N + i;
      if (k > 0) jl = a.nbr[es], rl = a.rev[es];
      const int64_t j = jl;
      if (__builtin_expect(built, 0)) rl = reverse_slot(s, j);
      double dij[3], dji[3];
      auto partials = [&]() {
        const double* p = a.dd + 3 * es;
        const double* q = a.dd + 3 * ((int64_t)rl * N + j);
#pragma unroll
        for (int mu = 0; mu < 3; ++mu) dij[mu] = p[mu], dji[mu] = q[mu];
      };
      // bond lists: nearly every pair is near, its partials are loaded with the
      // positions
      if (a.bond_need) partials();
      const double pj[3] = {a.pos[3 * j], a.pos[3 * j + 1], a.pos[3 * j + 2]};
      const double pi[3] = {a.pos[3 * i], a.pos[3 * i + 1], a.pos[3 * i + 2]};
      asm volatile("" ::: "memory");
      const double r[3] = {min_image(pj[0] - pi[0], a.box[0], a.ibox[0]),
                           min_image(pj[1] - pi[1], a.box[1], a.ibox[1]),
                           min_image(pj[2] - pi[2], a.box[2], a.ibox[2])};
      // a pair beyond R + D has zero partials both ways (written so by the site
      // kernel): nothing to load or add
      if (r[0] * r[0] + r[1] * r[1] + r[2] * r[2] < o.rcut2) {
        if (!a.bond_need) partials();
#pragma unroll
        for (int mu = 0; mu < 3; ++mu) {
          c[mu] = dij[mu] - dji[mu];
#pragma unroll
          for (int nu = 0; nu < 3; ++nu) c[3 + 3 * mu + nu] = r[mu] * dji[nu];
        }
      }
    }
    if (k > 0) wave_lds_fence();
#pragma unroll
    for (int q = 0; q < 12; ++q) sh[q * ROW + lane] = c[q];
    wave_lds_fence();
    const int m = min(n - k * LPA, LPA);
    if (s0 * QL < 12) {
      for (int t = 0; t < m; ++t)
#pragma unroll
        for (int q = 0; q < QL; ++q) sum[q] += sh[(s0 * QL + q) * ROW + g * LPA + t];
    }
  }
  if (s0 * QL < 12) {
#pragma unroll
    for (int q = 0; q < QL; ++q) tt[g * 12 + s0 * QL + q] = sum[q];
  }
  wave_lds_fence();
  double mv2 = 0.0, d2 = 0.0;
  if (comp) {   // component s0 of atom i
    const double* t = tt + g * 12;
    double f = t[s0];
    if (ext) {
      double e = e_i;
      if (o.vel) e += 0.5 * m_i * (va[0] * va[0] + va[1] * va[1] + va[2] * va[2]) * o.ke_unit;
      const double fx = e * o.fe[s0] + (o.fe[0] * t[3 + s0] + o.fe[1] * t[6 + s0] + o.fe[2] * t[9 + s0]);
      if (o.Fext) o.Fext[3 * i + s0] = fx;
      if (o.add_ext) f += fx;
    }
    if (o.F) o.F[3 * i + s0] = f;
    if (o.kick_vel) {
      // The rest of the step (the loads of v above, E_i's too, precede every store)
      double v = v_q;
      if (o.kick2) {   // end of a step: v += c F / m, under a thermostat v *= exp(-xi dt / 2)
        v = v + o.kick_c * f / m_i;
        if (o.kick_scale) v = v * scale;
        if (o.kick_v32) o.kick_v32[3 * i + s0] = (float)v;
        mv2 = m_i * v * v;
      }
      if (o.drift_pos) {   // start of the next: as k_md_step, into the other positions
        v = v + o.kick_c * f / m_i;
        const double L = a.box[s0];
        double x = x_q + o.drift_dt * v;
        x -= floor(x / L) * L;
        if (x >= L) x -= L;
        if (x < 0.0) x += L;
        o.drift_pos[3 * i + s0] = x;
        if (o.drift_ref) {
          double d = x - ref_q;
          d -= L * rint(d / L);
          d2 = d * d;
        }
      }
      o.kick_vel[3 * i + s0] = v;
    }
  }
  if (o.drift_ref) {   // the bond lists' displacement test
    const double y = __shfl(d2, lane + 1), z = __shfl(d2, lane + 2);
    if (s0 == 0 && d2 + y + z > o.drift_thr2) *o.drift_need = 1;
  }
  // W of the wave's atoms, consecutive values by consecutive lanes
  const int64_t left = N - i0 < APW ? N - i0 : APW;
  const int nw = left > 0 ? (int)left * 9 : 0;
  if (o.W)
    for (int e = lane; e < nw; e += 64) o.W[9 * i0 + e] = tt[e / 9 * 12 + 3 + e % 9];
  if (o.W32)
    for (int e = lane; e < nw; e += 64) o.W32[9 * i0 + e] = (float)tt[e / 9 * 12 + 3 + e % 9];
  if (o.ke_part) {   // the work-group's partial sum of m v^2 after the kick (uniform over the launch)
    // (with two slots per lane a work-group's atoms make two sums: the order
    // of the total does not depend on the lanes per atom a list asks for)
    constexpr int H = APB / SPL;
    __shared__ double kp[APB];
    const double y = __shfl(mv2, lane + 1), z = __shfl(mv2, lane + 2);
    if (s0 == 0) kp[tid / LPA] = (mv2 + y) + z;
    __syncthreads();
#pragma unroll
    for (int w = H / 2; w > 0; w >>= 1) {
      if (tid < SPL * w) kp[tid / w * H + tid % w] += kp[tid / w * H + tid % w + w];
      __syncthreads();
    }
    if (tid < SPL && (int64_t)blockIdx.x * APB + tid * H < N) o.ke_part[(int64_t)blockIdx.x * SPL + tid] = kp[tid * H];
  }
}

// ------------------------------------------------------------- launchers
static inline unsigned blocks_of(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

hipError_t launch_zero_i32(hipStream_t s, int* p, int n) {
  hipLaunchKernelGGL(k_fill_zero_i32, dim3(blocks_of(n, 256)), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

hipError_t launch_set_i32(hipStream_t s, int* p, int value) {
  hipLaunchKernelGGL(k_set_i32, dim3(1), dim3(64), 0, s, p, value);
  return hipGetLastError();
}

hipError_t launch_neighbors(hipStream_t s, const double* pos, int64_t N, const CellGrid& cg, double rc, double rb,
                            int max_nb, NeighborBufs b) {
  if (max_nb > NB_MAX) return hipErrorInvalidValue;
  const int n_cells = cg.nc[0] * cg.nc[1] * cg.nc[2];
  const int n_tiles = (n_cells + SCAN_TILE - 1) / SCAN_TILE;
  const bool scanned = n_tiles > SCAN_DIRECT;
  // the cell counts are zero between searches (k_neighbors clears them)
  hipLaunchKernelGGL(k_cell_count, dim3(blocks_of(N, 256)), dim3(256), 0, s, pos, N, cg, b.cell_of, b.place, b.count);
  const bool self = n_tiles <= SCAN_SELF;
  if (!self)
    hipLaunchKernelGGL(k_scan_tile_sums, dim3((unsigned)n_tiles), dim3(SCAN_TILE), 0, s, b.count, n_cells, b.tile_sums);
  if (scanned)
    hipLaunchKernelGGL(k_scan_tile_offsets, dim3(1), dim3(SCAN_TILE), 0, s, b.tile_sums, n_tiles);
  hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)n_tiles), dim3(SCAN_TILE), 0, s, b.count, n_cells,
                     self ? nullptr : b.tile_sums, scanned, b.start, b.flags);
  hipLaunchKernelGGL(k_cell_fill, dim3(blocks_of(N, 256)), dim3(256), 0, s, pos, N, b.cell_of, b.place, b.start,
                     b.atoms, b.cpos);
  hipLaunchKernelGGL(k_neighbors, dim3(blocks_of(N, NB_ATOMS)), dim3(NB_LANES * NB_ATOMS), 0, s, pos, N, cg, rc * rc,
                     rb * rb * (1.0 + 1e-12), b.cell_of, b.start, b.atoms, b.cpos, max_nb, b.nbr, b.n_nb, b.most,
                     b.count, (int64_t)n_cells);
  hipLaunchKernelGGL(k_reverse, dim3(blocks_of(N, 64)), dim3(64, REV_SLOTS), 0, s, N, b.nbr, b.n_nb, b.rev,
                     b.flags, b.most, (int)blocks_of(N, NB_ATOMS));
  return hipGetLastError();
}

template <int LPA>
static hipError_t launch_pair_kernels(hipStream_t s, const TersoffArgs& a, const TersoffParams& p, const GatherArgs& o,
                                      hipEvent_t e1) {
  // 5..8 pairs: 4 lanes x 2 slots (most atoms of a crystal have 4 bonds, so
  // most waves run one slot round)
  constexpr int SL = LPA == 8 ? 4 : LPA, SPL = LPA / SL;
  const dim3 grid(blocks_of(a.N * SL, SITE_WG));
  if (p.l3m == 0.0) hipLaunchKernelGGL((k_tersoff_site<SL, SPL, false>), grid, dim3(SITE_WG), 0, s, a, p);
  else
    hipLaunchKernelGGL((k_tersoff_site<SL, SPL, true>), grid, dim3(SITE_WG), 0, s, a, p);
  if (e1) {
    hipError_t e = hipEventRecord(e1, s);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_tersoff_gather<SL, SPL>), dim3(blocks_of(a.N * SL, GATHER_WG)), dim3(GATHER_WG), 0, s, a, o);
  return hipSuccess;
}

// ------------------------------------------------ velocity Verlet (NVE)
// First half kick of a step and its drift in place, where they do not run in
// the gather kernel (GatherArgs): v += c F / m with c = dt / (2 KE) (a = F /
// (m KE) in A/fs^2), x += dt v wrapped into [0, L) per axis (x - floor(x / L) L,
// then one correction step against rounding at the edges), and, with ref, the
// bond lists' displacement test: *need = 1 if the atom is farther than
// sqrt(thr2) from ref (its position at the last bond build).
// One thread per atom component, 64 atoms (192 components, contiguous in
// memory) per work-group; the displacement test sums each atom's three
// squared components in LDS.
constexpr int MD_ATOMS = 64;

__global__ void __launch_bounds__(3 * MD_ATOMS) k_md_step(double* __restrict__ pos, double* __restrict__ vel,
                                                          const double* __restrict__ F,
                                                          const double* __restrict__ mass, double c, double dt,
                                                          double Lx, double Ly, double Lz, int64_t N,
                                                          const double* __restrict__ ref, double thr2,
                                                          int* __restrict__ need) {
  __shared__ double sh[3 * MD_ATOMS];
  const int t = threadIdx.x;
  const int64_t q = (int64_t)blockIdx.x * (3 * MD_ATOMS) + t;
  double d2 = 0.0;
  if (q < 3 * N) {
    const int a = (int)(q % 3);
    double v = vel[q];
    v = v + c * F[q] / mass[q / 3];
    const double L = a == 0 ? Lx : (a == 1 ? Ly : Lz);
    double x = pos[q] + dt * v;
    x -= floor(x / L) * L;
    if (x >= L) x -= L;
    if (x < 0.0) x += L;
    pos[q] = x;
    vel[q] = v;
    if (ref) {
      double d = x - ref[q];
      d -= L * rint(d / L);
      d2 = d * d;
    }
  }
  if (!ref) return;   // uniform over the launch
  sh[t] = d2;
  __syncthreads();
  if (t < MD_ATOMS && sh[3 * t] + sh[3 * t + 1] + sh[3 * t + 2] > thr2) *need = 1;
}

hipError_t launch_md_step(hipStream_t s, double* pos, double* vel, const double* F, const double* mass, double c,
                          double dt, const double box[3], int64_t N, const double* ref, double thr2, int* need) {
  hipLaunchKernelGGL(k_md_step, dim3(blocks_of(N, MD_ATOMS)), dim3(3 * MD_ATOMS), 0, s, pos, vel, F, mass, c, dt,
                     box[0], box[1], box[2], N, ref, thr2, need);
  return hipGetLastError();
}

// ------------------------------------------------ Nose-Hoover thermostat
// Thermostat state on the device: st[0] = xi (1/fs), st[1] = eta (its time
// integral), st[2] = exp(-xi dt / 2), the velocity scale of the current step,
// st[3] = the last kinetic energy (eV).  Kinetic energies are summed in a fixed
// order: per work-group of 64 atoms in an LDS tree, then the work-groups'
// partials by one work-group.

// Sum of the 3 MD_ATOMS values in sh[] (every thread of the work-group calls it).
__device__ __forceinline__ double block_sum_192(double* sh) {
  const int t = threadIdx.x;
  __syncthreads();
  if (t < 64) sh[t] += sh[t + 64] + sh[t + 128];
  __syncthreads();
  for (int w = 32; w > 0; w >>= 1) {
    if (t < w) sh[t] += sh[t + w];
    __syncthreads();
  }
  return sh[0];
}

// Partial sums of m v^2, one per work-group of 64 atoms (the thermostat's
// kinetic energy at the entry of an NVT call; later steps take theirs from
// the gather kernel).
__global__ void __launch_bounds__(3 * MD_ATOMS) k_md_ke_partial(const double* __restrict__ vel,
                                                                const double* __restrict__ mass, int64_t N,
                                                                double* __restrict__ part) {
  __shared__ double sh[3 * MD_ATOMS];
  const int t = threadIdx.x;
  const int64_t q = (int64_t)blockIdx.x * (3 * MD_ATOMS) + t;
  double mv2 = 0.0;
  if (q < 3 * N) mv2 = mass[q / 3] * vel[q] * vel[q];
  sh[t] = mv2;
  const double s = block_sum_192(sh);
  if (t == 0) part[blockIdx.x] = s;
}

// Thermostat update of the state from the kinetic energy K = ke_unit / 2 sum
// of m v^2: mode & 1 (end of a step): eta += dt/2 xi, xi += dt/2 G; mode & 2
// (start of a step): xi += dt/2 G, scale = exp(-xi dt / 2), eta += dt/2 xi;
// G = (2K - gkt) / Q.
__device__ __forceinline__ void thermostat_update(double sum, double st[4], const ThermostatArgs& th, int mode) {
  const double K = 0.5 * sum * th.ke_unit;
  const double G = (2.0 * K - th.gkt) / th.Q;
  double xi = st[0], eta = st[1];
  if (mode & 1) {
    eta += 0.5 * th.dt * xi;
    xi += 0.5 * th.dt * G;
  }
  if (mode & 2) {
    xi += 0.5 * th.dt * G;
    st[2] = exp(-0.5 * th.dt * xi);
    eta += 0.5 * th.dt * xi;
  }
  st[0] = xi;
  st[1] = eta;
  st[3] = K;
}

// The update by one work-group of 256 threads, from state `from` into `to`.
__global__ void __launch_bounds__(256) k_thermostat(const double* __restrict__ part, int64_t n_part,
                                                    const double* from, double* to, ThermostatArgs th, int mode) {
  __shared__ double sh[256];
  const int t = threadIdx.x;
  double acc = 0.0;
  for (int64_t k0 = t; k0 < n_part; k0 += 8 * 256) {   // eight loads at a time, added in order
    double x[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) x[q] = part[k0 + 256 * q < n_part ? k0 + 256 * q : n_part - 1];
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (k0 + 256 * q < n_part) acc += x[q];
  }
  sh[t] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w) sh[t] += sh[t + w];
    __syncthreads();
  }
  if (t != 0) return;
  double st[4] = {from[0], from[1], from[2], from[3]};
  thermostat_update(sh[0], st, th, mode);
  for (int q = 0; q < 4; ++q) to[q] = st[q];
}

// Start of a step under the thermostat: the scale st[2], the first half kick,
// the drift and the bond lists' displacement test, as k_md_step.  With n_part
// > 0 every work-group first takes the thermostat update itself (the same sum
// in the same order in each, work-group 0 writes the state to `to`), which
// saves a launch of one work-group per step: an MD step of 8000 atoms is a
// chain of short kernels.  n_part = 0: the update is already in `to`.
__global__ void __launch_bounds__(3 * MD_ATOMS) k_md_nvt_start(double* __restrict__ pos, double* __restrict__ vel,
                                                               const double* __restrict__ F,
                                                               const double* __restrict__ mass, double c, double dt,
                                                               double Lx, double Ly, double Lz, int64_t N,
                                                               const double* __restrict__ part, int n_part,
                                                               const double* __restrict__ from, double* to,
                                                               ThermostatArgs th, int mode,
                                                               const double* __restrict__ ref, double thr2,
                                                               int* __restrict__ need) {
  __shared__ double sh[3 * MD_ATOMS];
  __shared__ double new_scale;
  const int t = threadIdx.x;
  const int64_t q = (int64_t)blockIdx.x * (3 * MD_ATOMS) + t;
  const bool act = q < 3 * N;
  // every load first: the kernel is one chain of latencies
  const int64_t qc = act ? q : 0;
  double v = vel[qc], x = pos[qc], f = F[qc], m = mass[qc / 3], rq = 0.0;
  if (ref) rq = ref[qc];
  const double* state = n_part > 0 ? from : to;
  const double st0 = state[0], st1 = state[1], st2 = state[2], st3 = state[3];
  asm volatile("" ::: "memory");
  double scale;
  if (n_part > 0) {
    if (t < 64) {   // one wave; k_thermostat's sum: its threads' values, then its tree
      double p[4] = {0.0, 0.0, 0.0, 0.0};
      for (int k0 = 0; k0 < n_part; k0 += 256)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int k = k0 + 64 * q + t;
          p[q] += k < n_part ? part[k] : 0.0;
        }
      double sum = (p[0] + p[2]) + (p[1] + p[3]);
#pragma unroll
      for (int w = 32; w > 0; w >>= 1) sum += __shfl_down(sum, w);
      if (t == 0) sh[0] = sum;
    }
    if (t == 0) {
      double st[4] = {st0, st1, st2, st3};
      thermostat_update(sh[0], st, th, mode);
      new_scale = st[2];
      if (blockIdx.x == 0)
        for (int k = 0; k < 4; ++k) to[k] = st[k];
    }
    __syncthreads();
    scale = new_scale;
  } else {
    scale = st2;
  }
  double d2 = 0.0;
  if (act) {
    const int a = (int)(q % 3);
    v = v * scale;
    v = v + c * f / m;
    const double L = a == 0 ? Lx : (a == 1 ? Ly : Lz);
    x = x + dt * v;
    x -= floor(x / L) * L;
    if (x >= L) x -= L;
    if (x < 0.0) x += L;
    pos[q] = x;
    vel[q] = v;
    if (ref) {
      double d = x - rq;
      d -= L * rint(d / L);
      d2 = d * d;
    }
  }
  if (!ref) return;   // uniform over the launch
  __syncthreads();
  sh[t] = d2;
  __syncthreads();
  if (t < MD_ATOMS && sh[3 * t] + sh[3 * t + 1] + sh[3 * t + 2] > thr2) *need = 1;
}

__global__ void k_thermostat_set(double* st, double xi, double eta) {
  if (threadIdx.x == 0) {
    st[0] = xi;
    st[1] = eta;
    st[2] = 1.0;
    st[3] = 0.0;
  }
}

int64_t md_nvt_parts(int64_t N) { return (N + MD_ATOMS - 1) / MD_ATOMS; }

hipError_t launch_md_ke_partial(hipStream_t s, const double* vel, const double* mass, int64_t N, double* part) {
  hipLaunchKernelGGL(k_md_ke_partial, dim3((unsigned)md_nvt_parts(N)), dim3(3 * MD_ATOMS), 0, s, vel, mass, N, part);
  return hipGetLastError();
}

hipError_t launch_thermostat(hipStream_t s, const double* part, int64_t n_part, const double* from, double* to,
                             const ThermostatArgs& th, int mode) {
  hipLaunchKernelGGL(k_thermostat, dim3(1), dim3(256), 0, s, part, n_part, from, to, th, mode);
  return hipGetLastError();
}

int64_t gather_parts(int64_t N, int lpa) { return (int64_t)blocks_of(N * lpa, GATHER_WG); }

hipError_t launch_md_nvt_start(hipStream_t s, double* pos, double* vel, const double* F, const double* mass, double c,
                               double dt, const double box[3], int64_t N, const double* part, int64_t n_part,
                               const double* from, double* to, const ThermostatArgs& th, int mode, const double* ref,
                               double thr2, int* need) {
  // Summing the partials in every work-group is cheaper than a launch while
  // there are few of them; the reads grow with the square of the size.  An NVT
  // step with the launch / without, us: 512 atoms (16 partials) 16.1 / 14.1,
  // 8000 (250) 18.7 / 16.8, 16224 (507) 19.2 / 17.4, 32768 (1024) 22.2 / 21.3,
  // 64000 (2000) 29.8 / 30.1, 216000 (6750) 58 / 68.  The line is short of the
  // crossing, which lies between 1024 and 2000.
  constexpr int64_t INLINE_PARTS = 512;
  if (n_part > INLINE_PARTS) {
    const hipError_t e = launch_thermostat(s, part, n_part, from, to, th, mode);
    if (e != hipSuccess) return e;
    n_part = 0;
  }
  hipLaunchKernelGGL(k_md_nvt_start, dim3((unsigned)md_nvt_parts(N)), dim3(3 * MD_ATOMS), 0, s, pos, vel, F, mass, c,
                     dt, box[0], box[1], box[2], N, part, (int)n_part, from, to, th, mode, ref, thr2, need);
  return hipGetLastError();
}

hipError_t launch_thermostat_set(hipStream_t s, double* st, double xi, double eta) {
  hipLaunchKernelGGL(k_thermostat_set, dim3(1), dim3(64), 0, s, st, xi, eta);
  return hipGetLastError();
}

int tersoff_lanes(int max_count) {
  int l = 4;
  while (l < max_count) l *= 2;
  return l;
}

hipError_t launch_tersoff(hipStream_t s, const TersoffArgs& a, const TersoffParams& p, const GatherArgs& o, int lpa,
                          hipEvent_t e0, hipEvent_t e1, hipEvent_t e2) {
  hipError_t e = hipSuccess;
  if (e0 && (e = hipEventRecord(e0, s)) != hipSuccess) return e;
  switch (lpa) {
    case 4: e = launch_pair_kernels<4>(s, a, p, o, e1); break;
    case 8: e = launch_pair_kernels<8>(s, a, p, o, e1); break;
    case 16: e = launch_pair_kernels<16>(s, a, p, o, e1); break;
    case 32: e = launch_pair_kernels<32>(s, a, p, o, e1); break;
    case 64: e = launch_pair_kernels<64>(s, a, p, o, e1); break;
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (e2) e = hipEventRecord(e2, s);
  return e;
}

}  // namespace mhc
