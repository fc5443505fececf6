// Internal declarations of the per-atom virial kernels (k_tersoff.hip) used
// by the host side in mhc_virial.cpp.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mhc {

// Cell grid of the neighbour search: nc cells per axis (1, or at least 3, so
// that the 27 surrounding cells never repeat), each at least the cutoff wide.
struct CellGrid {
  double box[3];
  double ibox[3];   // 1 / box: the minimum-image shift multiplies instead of dividing
  int nc[3];
};

// Device buffers of the neighbour lists: nbr, rev [max_nb][N] (slot-major),
// n_nb [N]; cell_of, place [N] (an atom's cell and its place in it); atoms [N]
// and cpos [N][3] (the atoms by cell and their positions); count [n_cells]
// (zero between searches), start [n_cells + 1]; tile_sums [ceil(n_cells / 1024)]
// (scan workspace); most [ceil(N / 16)] (largest counts of the search's
// work-groups); flags (host memory) [0] = largest neighbour count found, flags[1] = 1 if a
// reverse slot was missing, flags[2] = largest count inside the bond lists'
// cutoff.
struct NeighborBufs {
  int* nbr;
  int* rev;
  int* n_nb;
  int* cell_of;
  int* place;
  int* atoms;
  double* cpos;
  int* count;
  int* start;
  int* tile_sums;
  int2* most;
  int* flags;
};

// Bond lists (the listed pairs inside R + D + delta, delta the bond lists'
// own skin): nbr, rev [max_b][N] (slot-major), n_nb [N], mask [N] (bit s:
// list slot s is kept), ref [N][3] (positions at their build); flags[0] =
// largest count found, flags[1] = 1 if an atom had more than max_b, flags[2] =
// 1 if a reverse slot was missing; need [2]: the rebuild flags of alternate
// evaluations.
struct BondBufs {
  int* nbr;
  int* rev;
  int* n_nb;
  unsigned long long* mask;
  int* flags;
  double* ref;
  int* need;
};

// Tersoff parameters as the kernels use them: l3m = lambda3^m, c2 = c^2, d2 = d^2,
// c2d2 = c^2 / d^2, gc2d2 = gamma c^2 / d^2, g2c2 = 2 gamma c^2, ninv2 = -1 / (2n).
struct TersoffParams {
  double A, B, l1, l2, l3m, beta, n, c2, d2, c2d2, h, gamma, R, D, gc2d2, g2c2, ninv2;
  int m;
};

// Per-evaluation buffers: positions (device, [N][3]); neighbour lists; the
// partials dd [max_nb][N][3] (dU_i/dr_ij); site energies U [N].
struct TersoffArgs {
  const double* pos;
  int64_t N;
  double box[3];
  double ibox[3];   // 1 / box
  const int* nbr;
  const int* n_nb;
  const int* rev;
  int max_nb;
  double* dd;
  double* U;
  // Bond lists (nbr, n_nb, rev above): when bond_need is not null and
  // *bond_need != 0 the site kernel first builds them out of the skin lists
  // (full_n, full_nbr, full_rev: the pairs closer than sqrt(bond_rb2), at most
  // max_nb per atom, and the positions at the build) and the gather kernel
  // their reverse slots, through the views below (which nbr, n_nb and rev then
  // point to).  bond_flags[0] = largest count and [1] = 1 if an atom had more
  // than max_nb, [2] = 1 if a reverse slot is missing.  bond_clear (may be
  // null): the other evaluation's rebuild flag, zeroed by the site kernel.
  const int* bond_need;
  int* bond_clear;
  double bond_rb2;
  const int* full_n;
  const int* full_nbr;
  const int* full_rev;
  int* bond_nbr;
  int* bond_n;
  int* bond_rev;
  unsigned long long* bond_mask;
  double* bond_ref;
  int* bond_flags;
};

// Outputs of the gather kernel (any may be null): F [N][3], W [N][3][3] float64
// and W32 float32 (W[i][mu][nu]), Fext [N][3]; vel [N][3] and mass [N] give the
// kinetic part of E_i (vel null: E_i = U_i).
struct GatherArgs {
  const double* vel;
  const double* mass;
  double fe[3];
  double ke_unit;
  double rcut2;               // (R + D)^2 slightly widened: pairs beyond have zero partials
  double* F;
  double* W;
  float* W32;
  double* Fext;
  bool add_ext;               // F = interatomic force + F_ext (needs fe; vel for E_i)
  // The steps between two evaluations on the fly (kick_vel null: none), on
  // kick_vel after E_i has read vel.  kick2: the end of a step, v += kick_c
  // F / m, with kick_scale v *= kick_scale[2], the float32 copy to kick_v32
  // (may be null) and per work-group the sum of m v^2 to ke_part (may be null).
  // drift_pos (null: none): the start of the next step, v += kick_c F / m and
  // drift_pos = the evaluation's positions + drift_dt v, wrapped into the box
  // (another array: the launch still reads the positions), and with drift_ref
  // *drift_need = 1 if the atom is farther than sqrt(drift_thr2) from it.
  double* kick_vel;
  double kick_c;
  bool kick2;
  const double* kick_scale;
  float* kick_v32;
  double* ke_part;
  double* drift_pos;
  double drift_dt;
  const double* drift_ref;
  double drift_thr2;
  int* drift_need;
};

// Lists of the pairs closer than rc; also counts, per atom, those closer
// than rb (flags[2]: the largest such count).
hipError_t launch_neighbors(hipStream_t s, const double* pos, int64_t N, const CellGrid& cg, double rc, double rb,
                            int max_nb, NeighborBufs b);
// Zero n ints (n > 0).
hipError_t launch_zero_i32(hipStream_t s, int* p, int n);
hipError_t launch_set_i32(hipStream_t s, int* p, int value);
// Lanes per atom of the evaluation kernels for a largest neighbour count:
// the next power of two, at least 4 (64 at most: max_nb <= 64).
int tersoff_lanes(int max_count);
// Queues the site and gather kernels with lpa lanes per atom; the optional
// events are recorded before the site kernel (e0), between the two (e1) and
// after the gather kernel (e2).
hipError_t launch_tersoff(hipStream_t s, const TersoffArgs& a, const TersoffParams& p, const GatherArgs& o, int lpa,
                          hipEvent_t e0, hipEvent_t e1, hipEvent_t e2);

// First half kick of a velocity-Verlet step and its drift, in place on [N][3]
// float64 arrays: vel += c F / mass, pos += dt vel wrapped into the box, and
// with ref (NULL: none) *need = 1 if an atom is farther than sqrt(thr2) from
// its position in ref.  (Elsewhere they run in the gather kernel.)
hipError_t launch_md_step(hipStream_t s, double* pos, double* vel, const double* F, const double* mass, double c,
                          double dt, const double box[3], int64_t N, const double* ref, double thr2, int* need);

// Nose-Hoover thermostat steps (states of 4 doubles on the device: xi, eta,
// the velocity scale exp(-xi dt/2), the last kinetic energy; an update reads
// one and writes the other).  ke_partial: sums of m v^2, one per 64 atoms
// (md_nvt_parts of them); thermostat: mode 1 end-of-step, 2 start-of-step, 3
// both, from n_part partials; start: the update (mode 2 or 3), then the scale,
// the first half kick and the drift (ref, thr2, need as for launch_md_step).
// The end of a step runs in the gather kernel (GatherArgs.kick_vel).
struct ThermostatArgs {
  double dt, Q, gkt, ke_unit;
};
int64_t md_nvt_parts(int64_t N);
hipError_t launch_md_ke_partial(hipStream_t s, const double* vel, const double* mass, int64_t N, double* part);
hipError_t launch_thermostat(hipStream_t s, const double* part, int64_t n_part, const double* from, double* to,
                             const ThermostatArgs& th, int mode);
// m v^2 sums that the gather kernel writes to ke_part for lists of lpa lanes per atom.
int64_t gather_parts(int64_t N, int lpa);
hipError_t launch_md_nvt_start(hipStream_t s, double* pos, double* vel, const double* F, const double* mass, double c,
                               double dt, const double box[3], int64_t N, const double* part, int64_t n_part,
                               const double* from, double* to, const ThermostatArgs& th, int mode, const double* ref,
                               double thr2, int* need);
hipError_t launch_thermostat_set(hipStream_t s, double* st, double xi, double eta);

}  // namespace mhc
