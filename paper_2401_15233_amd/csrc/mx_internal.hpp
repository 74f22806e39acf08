// Internal interface between the C-ABI runtime and the gfx950 kernels.
#pragma once
#include <cmath>
#include <cstddef>
#include <hip/hip_runtime.h>

namespace mx {

// Device-resident control block: time step, time and status live on the device so that a
// sequence of steps needs no host round trip, and every step's first stage launch works out the
// step's dt itself (no launch of its own: the separate one-wavefront kernel that did it cost 2 to
// 4 us and a launch gap per step: 9.9 us against 5.9 for a first-order step of 1000 5-moment cells,
// with the face algebra of that time).  What a step
// reads and what it leaves for the next one stand in different slots, picked by the host's step
// counter `slot`, because the workgroups of one launch read and write in any order:
//   t, step      read from [slot & 1], written to [(slot + 1) & 1] by one workgroup of the first
//                stage
//   RatePart     rate read from [slot % 3]; the last stage reduces the new state's rate into
//                [(slot + 1) % 3], which the step before had cleared; the first stage clears
//                [(slot + 2) % 3]
//   fail_step    a step runs while no earlier step failed: a failure of the running step does
//                not stop its own later workgroups
struct DevCtrl {
  double dt;                     // time step of the running step (0: the step is a no-op), for
                                 // its second stage
  double dt_last;
  double t[2];                   // time
  long long step[2];             // steps taken
  long long n_fallback;          // positivity fallbacks
  long long fail_step;           // first failing step (1-based; 0: the loaded state; NO_FAILURE: none)
  int status;                    // bit 1 non-finite, bit 2 unrealizable
  long long n_fp64;              // mixed precision: face states re-evaluated in FP64
  long long n_states;            // mixed precision: face states evaluated
  long long n_sigma_limited;     // cells with sigma < sigma_lim (set by the counting kernel)
  int asym_z, asym_y;            // set to 1 by the ingest kernel: a z-odd moment (u_z, P_xz, P_yz,
                                 // q_z) / a y-odd one (u_y, P_xy, P_yz, q_y) is non-zero somewhere
};

// Whether the step after `step` steps runs: no earlier one failed.  64 bits, as the count of steps:
// a run of small tubes takes 2^31 steps in a few hours.
constexpr long long NO_FAILURE = 0x7fffffffffffffffLL;
__host__ __device__ constexpr bool step_runs(long long fail_step, long long step) { return fail_step > step; }
// the failing step as the reports carry it (0: none)
constexpr int reported_fail_step(long long fail_step) {
  return fail_step == NO_FAILURE ? 0 : (fail_step < 0x7fffffff ? (int)fail_step : 0x7fffffff);
}

// 1D tiles: a workgroup of NT threads owns NT - 4 cells, so that the cells plus the two-cell
// halo on each side (NT), the limiter items (NT - 2) and the faces (NT - 3) each take a single
// round over the threads.
constexpr int tile_1d(int nt) { return nt - 4; }

// the factor of 1 / tau that a run keeps (inv_tau; mode 0: local tau, 1: constant)
inline double inv_tau_constant(int mode, double tau_ref, double rho_ref, double T_ref) {
  return mode == 0 ? 1.0 / (tau_ref * rho_ref * std::sqrt(T_ref)) : 1.0 / tau_ref;
}

// Reductions over a wavefront; every lane gets the result.  Within rows of 16 lanes by DPP moves
// (pairs, quads, half rows, rows), the four rows by scalar reads: a chain of about 20
// instructions without LDS, where six ds_bpermute steps would each wait for LDS.
template <int CTRL> __device__ __forceinline__ int dpp_move(int x) {
  return __builtin_amdgcn_mov_dpp(x, CTRL, 0xf, 0xf, true);
}
template <int CTRL> __device__ __forceinline__ double dpp_move(double x) {
  const long long b = __double_as_longlong(x);
  return __longlong_as_double(((long long)dpp_move<CTRL>((int)(b >> 32)) << 32) | (unsigned)dpp_move<CTRL>((int)b));
}
__device__ __forceinline__ int read_lane(int x, int l) { return __builtin_amdgcn_readlane(x, l); }
__device__ __forceinline__ double read_lane(double x, int l) {
  const long long b = __double_as_longlong(x);
  return __longlong_as_double(((long long)read_lane((int)(b >> 32), l) << 32) | (unsigned)read_lane((int)b, l));
}
template <class T, class F> __device__ __forceinline__ T row_reduce(T v, F f) {
  v = f(v, dpp_move<0xB1>(v));    // lane ^ 1
  v = f(v, dpp_move<0x4E>(v));    // lane ^ 2
  v = f(v, dpp_move<0x141>(v));   // mirrored in half rows
  return f(v, dpp_move<0x140>(v));  // mirrored in rows
}
template <class T, class F> __device__ __forceinline__ T wave_reduce(T v, F f) {
  v = row_reduce(v, f);
  return f(f(read_lane(v, 0), read_lane(v, 16)), f(read_lane(v, 32), read_lane(v, 48)));
}
__device__ __forceinline__ double wave_max(double v) {
  return wave_reduce(v, [](double x, double y) { return fmax(x, y); });
}
__device__ __forceinline__ int wave_or(int v) {
  return wave_reduce(v, [](int x, int y) { return x | y; });
}
__device__ __forceinline__ int wave_sum(int v) {
  return wave_reduce(v, [](int x, int y) { return x + y; });
}

// raise a maximum kept as the bit pattern of a non-negative double.  Device-wide atomics on one
// address take their turn; a load first leaves out those that would change nothing, which is
// nearly all of them once the largest rates have been seen.
__device__ __forceinline__ void raise_max(unsigned long long* word, double m) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(m);
  if (b > __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(word, b);
}

enum { MODE_EULER = 0, MODE_HEUN2 = 1, MODE_MID2 = 2 };
enum { ST_NONFINITE = 1, ST_UNREALIZABLE = 2 };

// New value of a component from its residual L (modes MODE_EULER, MODE_HEUN2, MODE_MID2): explicit
// fused operations, so that every kernel rounds alike whatever surrounds the expression.
__device__ __forceinline__ double stage_update(int mode, double cdt, double dt, double L, double Ub, double Ua) {
  if (mode == MODE_EULER) return __builtin_fma(cdt * dt, L, Ub);
  if (mode == MODE_HEUN2) return __builtin_fma(0.5, Ua, 0.5 * __builtin_fma(dt, L, Ub));
  return __builtin_fma(dt, L, Ua);
}

// The maximum CFL rate, in RATE_PARTS parts on cache lines of their own: device-wide atomics on
// one address take their turn (about 25 ns each), and the workgroups of a small grid end
// together.  A workgroup raises the part of its index; every wavefront of the next step's first
// stage reads them all and takes the largest.  A step of 800 1D tiles: one word 19.1 us (5
// moments) and 23.1 (7), 16 parts 15.0 and 20.0 (64 parts 0.7 to 0.8 more than 16); on large grids
// 64 lines per wavefront cost as much L2 traffic as the tile (2048 x 2048 2 per cent slower), 16
// nothing that can be measured.
constexpr int RATE_PARTS = 16;   // one row of lanes reads them
struct alignas(128) RatePart {
  unsigned long long rate[3];    // bit patterns of non-negative doubles, a slot of the step each
};
constexpr size_t CTRL_BYTES = 256;                                            // DevCtrl's place ...
constexpr size_t RATE_BYTES = RATE_PARTS * sizeof(RatePart);                  // ... and the parts'
static_assert(sizeof(DevCtrl) <= CTRL_BYTES, "the control block fits its place");

struct StageParams {
  const double* Ub;        // stage input, read with its neighbourhood
  const double* Ua;        // U^n for the second-stage combinations (may equal Uout)
  double* Uout;
  int nx, ny, pitch;
  long long plane;         // ny * pitch
  double x0, y0, dx, dy, inv_dx, inv_dy;
  int bc[4];
  int n_jets;
  double jet_yc[4], jet_w[4], jet_ang[4];   // centre along the jet's wall, width, angle
  int jet_wall[4];         // 0 x-low, 1 x-high, 2 y-low, 3 y-high
  double jet_mach, jet_rho, jet_T;
  int use_source, tau_mode;
  int src_implicit;        // BGK source by backward Euler on the transported state (EULER mode)
  double tau_ref, rho_ref, T_ref;
  double inv_tau_ref;      // inv_tau_constant of the three
  double sigma_lim, kws;
  int limiter, flux, fallback;
  int mode;
  double cdt;              // stage step = cdt * dt (EULER mode)
  int do_cfl;
  int copy_on_idle;        // dt == 0: copy Ub to Uout (forward-Euler ping-pong) instead of skipping
  int ntx, nty;            // tile grid
  int nblk;                // real number of tiles
  double dt_replay;        // > 0: the step's dt (a replayed recorded step)
  int head;                // this launch is its step's first stage: it works out dt
  unsigned slot;           // the step's slots in the control block
  double dt_fixed, t_end, cfl;   // head: fixed dt (> 0) or CFL, end time (> 0)
  double* tape_dt;         // head: where to record the step's dt (null: nowhere)
  DevCtrl* ctrl;
  RatePart* rates;
};

struct CflParams {
  const double* U;
  int nx, ny, pitch;
  long long plane;
  double dx, dy;
  double sigma_lim, kws;
  RatePart* rates;
  int slot;                // of the step that reads the rate
};

struct BatchInst;
// src: unpadded [nv][ny][nx], primitive (repr 0) or conserved (1); U: padded [nv][ny][pitch]
struct IngestParams {
  const double* src;
  double* U;
  int repr;
  int nx, ny, pitch;
  double dx, dy;
  double sigma_lim, kws;
  DevCtrl* ctrl;
  RatePart* rates;         // the rate goes to slot 0
  const int* cell_inst;    // batched tubes: the tube of every cell, and the tubes' records
  BatchInst* inst;         // (their maxrate, zero before); null otherwise
};

// launchers (mx_kernels.hip)
// reduced (14 moments): the state is symmetric and the stage carries only the moments that can
// be non-zero -- 2D planar (u_z = P_xz = P_yz = q_z = 0; ten moments, Sys14P), 1D axial (also
// u_y = P_xy = q_y = 0; seven moments, Sys14A)
hipError_t launch_stage(int system, int dim, int order, int precision, bool reduced,
                        const StageParams& p, hipStream_t s);
hipError_t launch_cfl(int system, int dim, const CflParams& p, hipStream_t s);
// rates: null for a control block whose rate is not used
hipError_t launch_ctrl_reset(DevCtrl* c, RatePart* rates, double t0, hipStream_t s);
// zero the planes a reduced kernel never writes (2, 3, 5, 6, 8, 11, 12: u_y, u_z, P_xy, P_xz,
// P_yz, q_y, q_z) of a 14-moment field of `plane` doubles per plane (a kernel, no memset);
// nothing for nv != 14
hipError_t launch_zero_planes(double* U, long long plane, int nv, hipStream_t s);
// loads a field into U, checks it, and reduces its CFL rate into slot 0 of the parts (or the
// tubes' records); ctrl is reset before
hipError_t launch_ingest(int system, int dim, const IngestParams& p, hipStream_t s);
// dst: unpadded [components][ny][nx]
// repr 0 primitive, 1 conserved, 2 sigma, 3 closing moments (19 values per 14-moment cell)
hipError_t launch_egress(int system, int repr, const double* U, double* dst, int nx, int ny,
                         int pitch, double sigma_lim, hipStream_t s);
// zero ctrl->n_sigma_limited first; adds the cells of U with sigma < sigma_lim
hipError_t launch_count_sigma_limited(int system, const double* U, int nx, int ny, int pitch,
                                      double sigma_lim, DevCtrl* c, hipStream_t s);

}  // namespace mx
