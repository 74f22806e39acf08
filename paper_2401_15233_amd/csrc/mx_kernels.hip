// gfx950 kernels of the finite-volume step (FP64; FP32 / mixed face evaluation by template).
//
// One fused kernel per Runge-Kutta stage.  A workgroup owns a TX x TY tile of cells and
//   1. loads the tile plus a G-cell halo of the stage input U (structure of arrays, x
//      fastest), applying the boundary conditions while loading (ghost cells are never
//      stored), converts to primitives and keeps them in LDS;
//   2. computes the common (most stringent) limiter factor of every cell that feeds a face
//      of the tile (Section 3.2), with the positivity fallback;
//   3. evaluates every face of the tile once: both reconstructed states, their closure
//      (Sections 2.3-2.4, Appendix A), wave speeds (Section 5.1), physical fluxes and the
//      HLL / Rusanov combination (Section 3.1);
//   4. updates each cell with the flux differences and the BGK source at the cell centre,
//      writes the result, checks it (non-finite, rho <= 0, P not SPD) and, in the last
//      stage of a step, reduces the CFL rate of the new state for the next step.
// The 2D tile is 16 x 15 cells: 255 x-faces and 256 y-faces, one of each for 256 threads.  The 1D
// tile is 60 cells: cells plus halo fill one 64-wide wavefront exactly.  Small FP64 grids run
// the same tiles with twice the threads (512 in 2D, 128 in 1D) and two lanes per face.
#include <algorithm>

#include "mx_internal.hpp"
#include "mx_batch.hpp"
#include "mx_physics.hpp"
#include "mx_scheme.hpp"
#include "mx_bc.hpp"
#include "mx_planar.hpp"
#include "mx_axial.hpp"

namespace mx {

// The time step of a step from the control block (its first stage launch; every workgroup
// and wavefront comes to the same value): fixed or CFL, clipped to t_end; 0 once the end time is reached or
// an earlier step failed.
__device__ __forceinline__ double step_dt(const StageParams& p, int dim) {
  const DevCtrl* c = p.ctrl;
  const double t = c->t[p.slot & 1];
  double dt = 0.0;
  if (step_runs(c->fail_step, c->step[p.slot & 1])) {
    if (p.dt_fixed > 0.0) {
      dt = p.dt_fixed;
    } else {
      const double part = __longlong_as_double((long long)p.rates[threadIdx.x % RATE_PARTS].rate[p.slot % 3]);
      const double m = read_lane(row_reduce(part, [](double x, double y) { return fmax(x, y); }), 0);
      dt = (dim == 1) ? p.cfl * p.dx / m : p.cfl / m;
      if (!(m > 0.0)) dt = 0.0;
    }
    if (p.t_end > 0.0) {
      if (t >= p.t_end * (1.0 - 1e-14)) dt = 0.0;
      else dt = fmin(dt, p.t_end - t);
    }
  }
  return dt;
}

// what the step leaves for the next one (one wavefront of its first stage launch); a step that
// does nothing hands time, step count and rate on
__device__ __forceinline__ void step_advance(const StageParams& p, double dt) {
  DevCtrl* c = p.ctrl;
  RatePart* part = p.rates + threadIdx.x;
  const unsigned now = p.slot & 1, next = now ^ 1;
  const bool go = dt > 0.0;
  if (!go) part->rate[(p.slot + 1) % 3] = part->rate[p.slot % 3];
  part->rate[(p.slot + 2) % 3] = 0ull;
  if (threadIdx.x != 0) return;
  c->t[next] = go ? c->t[now] + dt : c->t[now];
  c->step[next] = c->step[now] + (go ? 1 : 0);
  c->dt = dt;
  if (go) c->dt_last = dt;
  if (p.tape_dt) *p.tape_dt = dt;
}

// CFL rate of a cell state
template <class SYS, int DIM>
__device__ __forceinline__ double cell_rate(const double* W, double sigma_lim, double kws, double dx, double dy) {
  if constexpr (DIM == 1) return SYS::template cell_lambda<0>(W, sigma_lim, kws);
  else return SYS::cell_rate2d(W, sigma_lim, kws, dx, dy);
}
// the same for a loaded field (1D, 14 moments: whether it is a tube is not known yet)
template <class SYS, int DIM>
__device__ __forceinline__ double field_rate(const double* W, double sigma_lim, double kws, double dx, double dy) {
  if constexpr (DIM == 1 && SYS::NV == 14) return SYS::tube_lambda(W, sigma_lim, kws);
  else return cell_rate<SYS, DIM>(W, sigma_lim, kws, dx, dy);
}

// ------------------------------------------------------------------ stage kernel
// One stage of a tile: primitives of the tile and its halo in LDS, limiter factors, face fluxes,
// update, checks and (last stage) the CFL rate of the new state.  Bound by FP64 VALU work; the
// planar system runs 3200 VALU instructions per cell and stage on large grids at 84 per cent
// of the issue rate (2048 x 2048 developed crossed jets: 0.45 to 0.47 ms per launch, the mean of both
// stages, over runs and cards).  LPF lanes share a face: one, or (grids that leave the chip partly idle, where a tile's latency is the time of the
// stage) two, each with the state of one side, in twice as many threads.
//
// Waves per SIMD the kernel is compiled for.  Planar 2D (ten moments), one lane per face: three
// 256-thread workgroups per CU fit in LDS (52 KB each), so three, which caps the kernel at 168
// VGPRs (no spills at second order, two registers at first).  Two lanes per face: a 512-thread
// workgroup is two waves per SIMD, and four (two workgroups per CU) cap it at 128 VGPRs: the
// planar kernel uses 114, the one with all 14 moments spills 20 (first order 18).
constexpr int stage_min_waves(int nv, int dim, int lanes) {
  if (dim == 1) return 1;
  return lanes == 2 ? 4 : (nv <= 10 ? 3 : 1);
}

template <class SYS, int DIM, int ORDER, int PREC, int TX, int TY, int NT, int LPF>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(stage_min_waves(SYS::NV, DIM, LPF))))
void stage_kernel(StageParams p) {
  constexpr int NV = SYS::NV;
  constexpr int G = (ORDER == 2) ? 2 : 1;
  constexpr int LX = TX + 2 * G;
  constexpr int LY = (DIM == 2) ? TY + 2 * G : 1;
  constexpr int NL = LX * LY;
  constexpr int NFX = (TX + 1) * TY;
  constexpr int NFY = (DIM == 2) ? TX * (TY + 1) : 0;
  constexpr int NPX = (ORDER == 2) ? (TX + 2) * TY : 1;
  constexpr int NPY = (ORDER == 2 && DIM == 2) ? TX * (TY + 2) : 1;
  // Where the fluxes go.  SEP (two lanes per face, planar): x and y fluxes in arrays of their
  // own beside the primitive tile, one barrier between faces and update (76 KB, two 512-thread
  // workgroups per CU).  XREG (one lane per face, planar): no separate x-flux array; the
  // x-flux components v >= XK go to LDS at once, past the primitive tile (free during the face
  // phases); the first XK stay in registers through the y-face phase, and all of them
  // overwrite the primitive tile after a barrier.  XK = 1: the largest LDS footprint that still
  // fits three 256-thread workgroups per CU (52 KB each; all ten components would take 54 KB).
  // Otherwise (14 moments in 2D) x fluxes have their array and y fluxes stay in registers until
  // they overwrite the primitive tile.
  constexpr bool SEP = (DIM == 2 && NV <= 10 && LPF == 2);
  constexpr bool XREG = (DIM == 2 && NV <= 10 && LPF == 1);
  constexpr int NFL = XREG ? NV * (NFX + NFY) : NV * NFY;
  constexpr int XK = XREG ? 1 : NV;
  constexpr int NW0 = XREG ? NV * NL + (NV - XK) * NFX : NV * NL;
  constexpr int NW = (SEP || NW0 > NFL) ? NW0 : NFL;
  constexpr int XH = NW - (NV - XK) * NFX;      // where the LDS-held x-flux components start
  static_assert(!XREG || XH >= NV * NL, "x-flux slots past the primitive tile");
  static_assert(!XREG || XK * NFX + NV * NFY <= XH, "fluxes after the barrier fit below them");
  static_assert(LPF * NFX <= NT, "one x-face (side) per thread");
  static_assert(LPF * NFY <= NT, "one y-face (side) per thread");

  __shared__ double sW[NW];        // primitives of the tile + halo; later the face fluxes
  __shared__ double sFx[XREG ? 1 : NV * NFX];
  __shared__ double sFyOwn[SEP ? NV * NFY : 1];
  __shared__ double sPx[NPX];
  __shared__ double sPy[NPY];
  __shared__ double sRed[NT / 64];
  __shared__ int sFlag[3];

  const int b = blockIdx.x;
  int n64 = 0;      // FP64 re-evaluations of face states (mixed precision)
  int nfb = 0;      // positivity fallbacks
  int flag = 0;     // failed checks of the new state
  double rate = 0.0;

  // XCD-aware tile order: hardware deals consecutive workgroups round-robin to the 8 XCDs;
  // give each XCD a contiguous band of tiles so halos are shared in its L2.
  const int nb8 = (p.nblk + 7) / 8;
  const int tile = (b % 8) * nb8 + b / 8;
  if (b / 8 >= nb8 || tile >= p.nblk) return;
  const int t = threadIdx.x;
  const int i0 = (tile % p.ntx) * TX;
  const int j0 = (tile / p.ntx) * TY;
  // Which wavefronts have work in a phase is a scalar test on their first thread; inside, spare
  // lanes repeat the phase's last item (same values to the same place, or not stored), so the
  // phases hold no divergent branch.
  const int t0 = __builtin_amdgcn_readfirstlane(t);
  // the cell this thread updates
  constexpr int NC = TX * TY;
  const int cc = min(t, NC - 1);
  const int ci = cc % TX, cj = cc / TX;
  const int gi = min(i0 + ci, p.nx - 1), gj = min(j0 + cj, p.ny - 1);
  const bool own = (t < NC) && (i0 + ci < p.nx) && (j0 + cj < p.ny);
  const long long off = (long long)gj * p.pitch + gi;
  // The step's dt, and whether there is anything to do.  Two lanes per face (small grids): asked
  // for after the tile's loads are on their way, so that the latency of the control block and
  // that of the tile overlap (with the early update inputs below, 1000 cells with 14 moments 18.9 ->
  // 18.3 us per step; the tubes' kernels are as fast either way at 1000 cells, 12.9 and 16.2, and 2 per
  // cent slower at 96000); otherwise before, so that an idle step on a large grid reads no field.
  double dt;
  auto begin = [&]() {
    if (p.dt_replay > 0.0) {
      dt = p.dt_replay;
    } else if (p.head) {
      dt = step_dt(p, DIM);
      if (b == 0 && threadIdx.x < RATE_PARTS) step_advance(p, dt);
    } else {
      dt = p.ctrl->dt;
    }
    return dt > 0.0 || p.copy_on_idle;   // uniform: time end reached or a failure stopped the run
  };
  if constexpr (LPF == 1) {
    if (!begin()) return;
  }

  // Issue priority by phase: first loads, conversion and limiters, then the update, the face
  // phase last.  A workgroup passes its short, waiting phases as soon as they can issue and the
  // long face phases of its neighbours on the CU fill what is left, instead of all of them
  // waiting for memory or a barrier together (2048 x 2048 1440 -> 1364 us per step with load and
  // read, 1200 x 1200 of four steps 937 -> 873, 14 moments 515 x 387 267 -> 256; the face phase first:
  // nothing gained).
  __builtin_amdgcn_s_setprio(3);
  // 1. tile + halo -> primitives in LDS
  // (a thread issues the loads of all its cells before it converts any)
  constexpr int NR = (NL + NT - 1) / NT;
  double Uh[NR][NV];
  HaloSrc hs[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    if (t0 + r * NT < NL) {
      const int c = min(t + r * NT, NL - 1);
      const int li = c % LX, lj = c / LX;
      hs[r] = load_cons<SYS>(p, p.Ub, i0 + li - G, (DIM == 2) ? j0 + lj - G : 0, Uh[r]);
    }
  }
  if constexpr (LPF == 2) {
    asm volatile("" ::: "memory");   // the loads stay above
    if (!begin()) return;
  }
  if (threadIdx.x < 3) sFlag[threadIdx.x] = 0;
  if (!(dt > 0.0)) {
    if (own) {
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const long long o = SYS::plane_of(v) * p.plane + off;
        p.Uout[o] = p.Ub[o];
      }
    }
    return;
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    if (t0 + r * NT < NL) {
      const int c = min(t + r * NT, NL - 1);
      const int li = c % LX, lj = c / LX;
      double W[NV];
      finish_prims<SYS>(p, hs[r], i0 + li - G, (DIM == 2) ? j0 + lj - G : 0, Uh[r], W);
#pragma unroll
      for (int v = 0; v < NV; ++v) sW[v * NL + c] = W[v];
    }
  }
  __syncthreads();

  auto lds = [&](int ti, int tj, double* W) {
    int c = (DIM == 2) ? (tj + G) * LX + (ti + G) : (ti + G);
#pragma unroll
    for (int v = 0; v < NV; ++v) W[v] = sW[v * NL + c];
  };

  // 2. common limiter factors of x items (cells -1 .. TX of each row) and y items
  if constexpr (ORDER == 2) {
    auto limiter = [&](int ti, int tj, int di, int dj, const double* Wc, bool mine) {
      double Wm[NV], Wp[NV];
      lds(ti - di, tj - dj, Wm); lds(ti + di, tj + dj, Wp);
      double phi = cell_limiter<SYS>(Wm, Wc, Wp, p.limiter);
      if (p.fallback && phi > 0.0 && !faces_admissible<SYS>(Wm, Wc, Wp, phi)) {
        phi = 0.0;
        if (mine && i0 + ti < p.nx && j0 + tj < p.ny) ++nfb;
      }
      return phi;
    };
    if constexpr (DIM == 2 && LPF == 1) {
      // a thread takes both items of its cell, whose natural scales they share, and the 62
      // items of the ring go to one wavefront: 5 wavefront rounds, two of them double, where one
      // sweep over all 542 items takes 9 (2048 x 2048 with load and read 1357 -> 1341 us, 515 x 387
      // with 14 moments 251 -> 247)
      if (t0 < NC) {
        double Wc[NV];
        lds(ci, cj, Wc);
        const double px = limiter(ci, cj, 1, 0, Wc, t < NC);
        const double py = limiter(ci, cj, 0, 1, Wc, t < NC);
        sPx[cj * (TX + 2) + ci + 1] = px;
        sPy[(cj + 1) * TX + ci] = py;
      }
      constexpr int RING = 2 * (TX + TY);
      static_assert(RING <= 64 && NT >= 64, "the ring is one wavefront's");
      if (t0 == NT - 64) {
        const int h = min(t - t0, RING - 1), g = h - 2 * TY;
        const bool isx = g < 0;
        const int ti = isx ? ((h & 1) ? TX : -1) : g % TX, tj = isx ? h >> 1 : (g < TX ? -1 : TY);
        double Wc[NV];
        lds(ti, tj, Wc);
        const double phi = limiter(ti, tj, isx ? 1 : 0, isx ? 0 : 1, Wc, false);
        if (isx) sPx[tj * (TX + 2) + ti + 1] = phi;
        else sPy[(tj + 1) * TX + ti] = phi;
      }
    } else {
      // x and y items in one sweep (two lanes per face: 542 items on 512 threads)
      constexpr int NPT = (DIM == 2) ? NPX + NPY : NPX;
#pragma unroll 1
      for (int r0 = 0; t0 + r0 < NPT; r0 += NT) {
        const int c = min(t + r0, NPT - 1);
        const bool isx = c < NPX;
        const int cy = c - NPX;
        const int ti = isx ? c % (TX + 2) - 1 : cy % TX, tj = isx ? c / (TX + 2) : cy / TX - 1;
        double Wc[NV];
        lds(ti, tj, Wc);
        const bool mine = t + r0 < NPT && (isx ? (ti >= 0 && ti < TX) : (tj >= 0 && tj < TY));
        const double phi = limiter(ti, tj, isx ? 1 : 0, isx ? 0 : 1, Wc, mine);
        if (isx) sPx[c] = phi;
        else sPy[cy] = phi;
      }
    }
    __syncthreads();
  }

  // the update's inputs from memory: U of the stage and (second-stage combinations) U^n.  Few
  // registers are in use in the two-lane 1D kernel, so there they are in flight during the faces.
  constexpr bool EARLY = DIM == 1 && LPF == 2;
  double Ub[NV], Ua[NV];
  auto load_own = [&]() {
    if (t0 < NC) {
#pragma unroll
      for (int v = 0; v < NV; ++v) Ub[v] = p.Ub[SYS::plane_of(v) * p.plane + off];
      if (p.mode != MODE_EULER) {
#pragma unroll
        for (int v = 0; v < NV; ++v) Ua[v] = p.Ua[SYS::plane_of(v) * p.plane + off];
      }
    }
  };
  if constexpr (EARLY) load_own();

  __builtin_amdgcn_s_setprio(0);
  // 3a. x faces: face f lies between tile cells (fi-1, fj) and (fi, fj)
  double Fx[NV];
  if (t0 < LPF * NFX) {
    const int f = min(t / LPF, NFX - 1);
    const int fi = f % (TX + 1), fj = f / (TX + 1);
    double Fh[NV];
    if constexpr (LPF == 2) {
      const int side = t & 1;
      double W[NV];
      if constexpr (ORDER == 2) {
        double A[NV], B[NV], C[NV];
        lds(fi - 2 + side, fj, A); lds(fi - 1 + side, fj, B); lds(fi + side, fj, C);
        face_state<SYS>(A, B, C, sPx[fj * (TX + 2) + fi + side], side ? -1.0 : 1.0, W);
      } else {
        lds(fi - 1 + side, fj, W);
      }
      face_flux_pair<SYS, 0>(W, side != 0, p.sigma_lim, p.kws, p.flux, Fh);
    } else {
      double WL[NV], WR[NV];
      if constexpr (ORDER == 2) {
        double A[NV], B[NV], C[NV], D[NV];
        lds(fi - 2, fj, A); lds(fi - 1, fj, B); lds(fi, fj, C); lds(fi + 1, fj, D);
        face_state<SYS>(A, B, C, sPx[fj * (TX + 2) + fi], 1.0, WL);
        face_state<SYS>(B, C, D, sPx[fj * (TX + 2) + fi + 1], -1.0, WR);
      } else {
        lds(fi - 1, fj, WL); lds(fi, fj, WR);
      }
      const int n64_before = n64;
      if constexpr (PREC == 0) face_flux<SYS, 0>(WL, WR, p.sigma_lim, p.kws, p.flux, Fh);
      else if constexpr (PREC == 1) face_flux_mixed<SYS, 0>(WL, WR, p.sigma_lim, p.kws, p.flux, Fh, n64);
      else face_flux_fp32<SYS, 0>(WL, WR, p.sigma_lim, p.kws, p.flux, Fh);
      if (PREC == 1 && t >= NFX) n64 = n64_before;
    }
    if constexpr (XREG) {
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        if (v < XK) Fx[v] = Fh[v];
        else sW[XH + (v - XK) * NFX + f] = Fh[v];
      }
    } else if (LPF == 1 || (t & 1) == 1) {
#pragma unroll
      for (int v = 0; v < NV; ++v) sFx[v * NFX + f] = Fh[v];
    }
  }

  // 3b. y faces: face f lies between tile cells (fi, fj-1) and (fi, fj)
  double Fy[NV];
  const int fy = min(t / LPF, NFY > 0 ? NFY - 1 : 0);
  if constexpr (DIM == 2) {
    static_assert((LPF * NFY) % 64 == 0, "whole wavefronts of y faces");
    if (t0 < LPF * NFY) {
      const int fi = fy % TX, fj = fy / TX;
      if constexpr (LPF == 2) {
        const int side = t & 1;
        double W[NV];
        if constexpr (ORDER == 2) {
          double A[NV], B[NV], C[NV];
          lds(fi, fj - 2 + side, A); lds(fi, fj - 1 + side, B); lds(fi, fj + side, C);
          face_state<SYS>(A, B, C, sPy[(fj + side) * TX + fi], side ? -1.0 : 1.0, W);
        } else {
          lds(fi, fj - 1 + side, W);
        }
        face_flux_pair<SYS, 1>(W, side != 0, p.sigma_lim, p.kws, p.flux, Fy);
        if constexpr (SEP) {
          if (side == 1) {
#pragma unroll
            for (int v = 0; v < NV; ++v) sFyOwn[v * NFY + fy] = Fy[v];
          }
        }
      } else {
        double WL[NV], WR[NV];
        if constexpr (ORDER == 2) {
          double A[NV], B[NV], C[NV], D[NV];
          lds(fi, fj - 2, A); lds(fi, fj - 1, B); lds(fi, fj, C); lds(fi, fj + 1, D);
          face_state<SYS>(A, B, C, sPy[fj * TX + fi], 1.0, WL);
          face_state<SYS>(B, C, D, sPy[(fj + 1) * TX + fi], -1.0, WR);
        } else {
          lds(fi, fj - 1, WL); lds(fi, fj, WR);
        }
        if constexpr (PREC == 0) face_flux<SYS, 1>(WL, WR, p.sigma_lim, p.kws, p.flux, Fy);
        else if constexpr (PREC == 1) face_flux_mixed<SYS, 1>(WL, WR, p.sigma_lim, p.kws, p.flux, Fy, n64);
        else face_flux_fp32<SYS, 1>(WL, WR, p.sigma_lim, p.kws, p.flux, Fy);
      }
    }
  }
  // 3c. the update's inputs, gathered before the barriers so that the global loads overlap
  // the waits: the cell's stage input and (second-stage combinations) U^n from memory, its
  // primitives from the tile in LDS (converted by the load phase, so no second primitive
  // recovery) and the BGK source at the cell centre
  const bool implicit_src = p.use_source && p.src_implicit;
  double Cs[NV];
  if constexpr (!EARLY) load_own();
  if (t0 < NC) {
    if (p.use_source && !implicit_src) {
      double W[NV];
      lds(ci, cj, W);
      if constexpr (SYS::TUBE) SYS::source(W, 1.0 / tau_tube<SYS>(W, p.tau_mode, p.tau_ref, p.rho_ref, p.T_ref), Cs);
      else SYS::source(W, inv_tau<SYS>(W, p.tau_mode, p.inv_tau_ref), Cs);
    } else {
#pragma unroll
      for (int v = 0; v < NV; ++v) Cs[v] = 0.0;
    }
  }
  __syncthreads();
  // y-face fluxes (XREG: and the x-face fluxes) over the primitive tile
  constexpr int Y0 = XREG ? XK * NFX : 0;
  if constexpr (DIM == 2 && !SEP) {
    if constexpr (XREG) {
      const int f = min(t, NFX - 1);
#pragma unroll
      for (int v = 0; v < XK; ++v) sW[v * NFX + f] = Fx[v];
    }
    if (t0 < LPF * NFY && (LPF == 1 || (t & 1) == 1)) {
#pragma unroll
      for (int v = 0; v < NV; ++v) sW[Y0 + v * NFY + fy] = Fy[v];
    }
    __syncthreads();
  }
  const double* sFy = SEP ? sFyOwn : sW + Y0;

  __builtin_amdgcn_s_setprio(1);
  // 4. update
  if (t0 < NC) {
    double Un[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const double* fx = XREG ? sW : sFx;
      const int xb = (XREG && v >= XK) ? XH + (v - XK) * NFX : v * NFX;
      double L = Cs[v];
      if constexpr (DIM == 2) L = tfma(sFy[v * NFY + cj * TX + ci] - sFy[v * NFY + (cj + 1) * TX + ci], p.inv_dy, L);
      L = tfma(fx[xb + cj * (TX + 1) + ci] - fx[xb + cj * (TX + 1) + ci + 1], p.inv_dx, L);
      Un[v] = stage_update(p.mode, p.cdt, dt, L, Ub[v], Ua[v]);
    }
    if (implicit_src) {
      // backward-Euler BGK relaxation of the transported state (forward-Euler stages only):
      // the source keeps rho, rho u and the energy, so the Maxwellian and tau of the new
      // state are those of the transported state, and U_new = (U_t + h U_eq) / (1 + h),
      // h = dt / tau
      double Wt[NV], We[NV], Ue[NV];
      SYS::cons_to_prim(Un, Wt);
      double h, w;
      if constexpr (SYS::TUBE) {   // (the roundings are fixed)
        h = (p.cdt * dt) / tau_tube<SYS>(Wt, p.tau_mode, p.tau_ref, p.rho_ref, p.T_ref);
        w = 1.0 / (1.0 + h);
        SYS::equilibrium_cons(Wt, Ue);
      } else {
        h = (p.cdt * dt) * inv_tau<SYS>(Wt, p.tau_mode, p.inv_tau_ref);
        w = mrcp(1.0 + h);
        SYS::equilibrium(Wt, We);
        SYS::prim_to_cons(We, Ue);
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) Un[v] = (Un[v] + h * Ue[v]) * w;
    }
    bool fin = true;
#pragma unroll
    for (int v = 0; v < NV; ++v) fin = fin && isfinite(Un[v]);
    if (own) {
#pragma unroll
      for (int v = 0; v < NV; ++v) p.Uout[SYS::plane_of(v) * p.plane + off] = Un[v];
    }
    int bad = 0;
    double r = 0.0;
    if (p.do_cfl) {
      // the last stage of a step: the new state's primitives also give its CFL rate
      double Wn[NV];
      if constexpr (SYS::TUBE) SYS::cons_to_prim(Un, Wn, false);
      else SYS::cons_to_prim(Un, Wn);
      if (!SYS::admissible(Wn)) bad = ST_UNREALIZABLE;
      r = cell_rate<SYS, DIM>(Wn, p.sigma_lim, p.kws, p.dx, p.dy);
    } else if (!SYS::admissible_cons(Un)) {
      bad = ST_UNREALIZABLE;
    }
    if (!fin) bad = ST_NONFINITE;
    // a failed cell's rate does not count; a NaN is passed over, as by the maximum before
    if (own) {
      flag |= bad;
      rate = fmax(rate, bad ? 0.0 : r);
    }
  }
  // block reductions: status, fallback count, CFL rate
  flag = wave_or(flag);
  nfb = wave_sum(nfb);
  if constexpr (PREC == 1) n64 = wave_sum(n64);
  const int lane = t & 63, wid = t >> 6;
  if (lane == 0) {
    if (flag) atomicOr(&sFlag[0], flag);
    if (nfb) atomicAdd(&sFlag[1], nfb);
    if (PREC == 1 && n64) atomicAdd(&sFlag[2], n64);
  }
  if (p.do_cfl) {
    rate = wave_max(rate);
    if (lane == 0) sRed[wid] = rate;
  }
  __syncthreads();
  if (t == 0) {
    if (sFlag[0]) {
      atomicOr(&p.ctrl->status, sFlag[0]);
      // this step's 1-based index, from whichever slot holds it
      atomicMin((unsigned long long*)&p.ctrl->fail_step,
                (unsigned long long)(p.head ? p.ctrl->step[p.slot & 1] + 1 : p.ctrl->step[(p.slot + 1) & 1]));
    }
    if (sFlag[1]) atomicAdd((unsigned long long*)&p.ctrl->n_fallback, (unsigned long long)sFlag[1]);
    if (PREC != 0) {
      if (sFlag[2]) atomicAdd((unsigned long long*)&p.ctrl->n_fp64, (unsigned long long)sFlag[2]);
      // every tile evaluates the same number of face states: counted once per launch
      if (b == 0)
        atomicAdd((unsigned long long*)&p.ctrl->n_states, (unsigned long long)p.nblk * (2 * (NFX + NFY)));
    }
    if (p.do_cfl) {
      double m = sRed[0];
      for (int k = 1; k < NT / 64; ++k) m = fmax(m, sRed[k]);
      raise_max(&p.rates[b % RATE_PARTS].rate[(p.slot + 1) % 3], m);
    }
  }
}

// ------------------------------------------------------------------ whole-field kernels
// Cell k of an nx x ny field in a plane of row pitch `pitch`.  A field holds at most 2^31
// cells, so the division is a 32-bit one, and a field without row padding needs none.
__device__ __forceinline__ long long padded_index(unsigned k, unsigned nx, int ny, int pitch) {
  if (ny == 1 || (unsigned)pitch == nx) return k;
  const unsigned j = k / nx;
  return (long long)j * pitch + (k - j * nx);
}

// Workgroups of a whole-field kernel: eight per CU (256 CUs), each striding over the field, so
// that the reductions at their ends cost at most 2048 atomics.
static int field_grid(long long n) { return (int)std::min<long long>((n + 255) / 256, 2048); }

// maximum of a workgroup's rates (256 threads) into its part
__device__ __forceinline__ void block_max_rate(double rate, RatePart* rates, int slot) {
  __shared__ double sRed[4];
  rate = wave_max(rate);
  if ((threadIdx.x & 63) == 0) sRed[threadIdx.x >> 6] = rate;
  __syncthreads();
  if (threadIdx.x == 0)
    raise_max(&rates[blockIdx.x % RATE_PARTS].rate[slot % 3], fmax(fmax(sRed[0], sRed[1]), fmax(sRed[2], sRed[3])));
}

// ------------------------------------------------------------------ CFL rate of a state
template <class SYS, int DIM>
__global__ __launch_bounds__(256) void cfl_kernel(CflParams p) {
  constexpr int NV = SYS::NV;
  const unsigned n = (unsigned)p.nx * (unsigned)p.ny;
  double rate = 0.0;
  for (unsigned c = blockIdx.x * 256 + threadIdx.x; c < n; c += gridDim.x * 256) {
    const long long off = padded_index(c, p.nx, p.ny, p.pitch);
    double U[NV], W[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) U[v] = p.U[v * p.plane + off];
    SYS::cons_to_prim(U, W);
    rate = fmax(rate, field_rate<SYS, DIM>(W, p.sigma_lim, p.kws, p.dx, p.dy));
  }
  block_max_rate(rate, p.rates, p.slot);
}

// ------------------------------------------------------------------ control block
__global__ void ctrl_reset_kernel(DevCtrl* c, RatePart* rates, double t0) {
  if (rates) rates[threadIdx.x] = RatePart{};
  if (threadIdx.x == 0) {
    DevCtrl z = {};
    z.t[0] = t0;
    z.fail_step = NO_FAILURE;
    *c = z;
  }
}

// zero the planes no reduced kernel writes (u_y, u_z, P_xy, P_xz, P_yz, q_y, q_z) of a
// 14-moment field
__global__ __launch_bounds__(256) void zero_planes_kernel(double* U, long long plane) {
  const long long n = 7 * plane;
  for (long long k = (long long)blockIdx.x * 256 + threadIdx.x; k < n; k += (long long)gridDim.x * 256) {
    const int w = (int)(k / plane);
    const long long o = k - w * plane;
    const int v = w == 0 ? 2 : (w == 1 ? 3 : (w == 2 ? 5 : (w == 3 ? 6 : (w == 4 ? 8 : (w == 5 ? 11 : 12)))));
    U[v * plane + o] = 0.0;
  }
}

// ------------------------------------------------------------------ state in / out
// Load a field: conserved moments, the checks of every cell, the symmetry of a 14-moment state
// and the first CFL rate, in one pass (bound by HBM: the source read once, the state written
// once).  The rate of a batch goes to each tube's own record: the lanes of a wavefront that
// share a tube reduce among themselves first (nearly all wavefronts lie in one tube).
template <class SYS, int DIM, bool BATCH>
__global__ __launch_bounds__(256) void ingest_kernel(IngestParams p) {
  constexpr int NV = SYS::NV;
  const unsigned n = (unsigned)p.nx * (unsigned)p.ny;
  const long long plane = (long long)p.ny * p.pitch;
  int bad = 0, np = 0;
  double rate = 0.0;
  // a thread's next cell is on its way while it works on one (spare lanes read the last cell;
  // 1200 x 1200: loading, four steps and reading 864 -> 850 us, although the registers leave three
  // wavefronts per SIMD instead of four)
  double A[NV], next[NV];
  auto load = [&](unsigned long long k) {
    const unsigned c = k < n ? (unsigned)k : n - 1;
#pragma unroll
    for (int v = 0; v < NV; ++v) next[v] = p.src[(long long)v * n + c];
  };
  load(blockIdx.x * 256 + threadIdx.x);
  // whole wavefronts stay in the loop (the batch reduces across their lanes)
  for (unsigned long long w = blockIdx.x * 256 + (threadIdx.x & ~63u); w < n; w += gridDim.x * 256) {
    const unsigned k = (unsigned)w + (threadIdx.x & 63);
    const bool in = k < n;
    double r = 0.0;
    int inst = 0;
#pragma unroll
    for (int v = 0; v < NV; ++v) A[v] = next[v];
    if (w + gridDim.x * 256 < n) load(w + gridDim.x * 256 + (threadIdx.x & 63));
    if (in) {
      const long long off = padded_index(k, p.nx, p.ny, p.pitch);
      double Uc[NV], W[NV];
      if (p.repr == 0) {
        SYS::prim_to_cons(A, Uc);
#pragma unroll
        for (int v = 0; v < NV; ++v) W[v] = A[v];
      } else {
#pragma unroll
        for (int v = 0; v < NV; ++v) Uc[v] = A[v];
        SYS::cons_to_prim(Uc, W);
      }
      bool fin = true;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        fin = fin && isfinite(Uc[v]);
        p.U[v * plane + off] = Uc[v];
      }
      if (!fin) bad |= ST_NONFINITE;
      else if (!SYS::admissible(W)) bad |= ST_UNREALIZABLE;
      // symmetry (14 moments): z-odd moments u_z, P_xz, P_yz, q_z and y-odd moments u_y, P_xy,
      // P_yz, q_y exactly zero
      if constexpr (NV == 14) {
        if (Uc[3] != 0.0 || Uc[6] != 0.0 || Uc[8] != 0.0 || Uc[12] != 0.0) np |= 1;
        if (Uc[2] != 0.0 || Uc[5] != 0.0 || Uc[8] != 0.0 || Uc[11] != 0.0) np |= 2;
      }
      if constexpr (DIM == 1) SYS::cons_to_prim(Uc, W);
      r = fmax(field_rate<SYS, DIM>(W, p.sigma_lim, p.kws, p.dx, p.dy), 0.0);
      if constexpr (BATCH) inst = p.cell_inst[k];
    }
    if constexpr (BATCH) {
      const int first = __builtin_amdgcn_readfirstlane(inst);   // lane 0 is inside the field
      if (__all(!in || inst == first)) {
        const double m = wave_max(r);
        if ((threadIdx.x & 63) == 0) atomicMax(&p.inst[first].maxrate, (unsigned long long)__double_as_longlong(m));
      } else if (in) {
        atomicMax(&p.inst[inst].maxrate, (unsigned long long)__double_as_longlong(r));
      }
    } else {
      rate = fmax(rate, r);
    }
  }
  bad = wave_or(bad);
  if ((threadIdx.x & 63) == 0 && bad) {
    atomicOr(&p.ctrl->status, bad);
    p.ctrl->fail_step = 0;   // no step runs from a state that failed its check
  }
  // plain stores of one value: any number of wavefronts may set a flag (an atomic each took
  // their turn at one address, 0.2 ms for a 2048 x 2048 field)
  if constexpr (NV == 14) {
    np = wave_or(np);
    if ((threadIdx.x & 63) == 0) {
      if (np & 1) p.ctrl->asym_z = 1;
      if (np & 2) p.ctrl->asym_y = 1;
    }
  }
  if constexpr (!BATCH) block_max_rate(rate, p.rates, 0);
}

// Closing moments of a cell state (dimensional, at sigma_bar = max(sigma, sigma_lim)):
// 14 moments: Q_ijk (10: xxx xxy xxz xyy xyz xzz yyy yyz yzz zzz), R_ijkk (6: xx xy xz yy yz zz),
// S_ijjkk (3: x y z); 5 moments: s.
constexpr int NCLOSE14 = 19;

MX_HD void closing14(const double* W, double sigma_lim, double* out) {
  Sys14::Core<double> k;
  Sys14::core(W, sigma_lim, k);
  double Q[6], R[3], S;
  Sys14::closure_dir<0>(k, Q, R, S);   // Q_ijx: xxx xyx xzx yyx yzx zzx
  out[0] = Q[0]; out[1] = Q[1]; out[2] = Q[2]; out[3] = Q[3]; out[4] = Q[4]; out[5] = Q[5];
  out[10] = R[0]; out[11] = R[1]; out[12] = R[2];
  out[16] = S;
  Sys14::closure_dir<1>(k, Q, R, S);   // Q_ijy: ... yyy yzy zzy
  out[6] = Q[3]; out[7] = Q[4]; out[8] = Q[5];
  out[13] = R[1]; out[14] = R[2];
  out[17] = S;
  Sys14::closure_dir<2>(k, Q, R, S);   // Q_zzz
  out[9] = Q[5];
  out[15] = R[2];
  out[18] = S;
}

// Read a field back in one representation (0 primitive, 1 conserved, 2 sigma, 3 closing
// moments): one kernel each, so that none carries another's registers (one kernel for all four
// spilled, and ran the plain copies at half the wavefronts).
template <class SYS, int REPR>
__global__ __launch_bounds__(256) void egress_kernel(const double* U, double* dst, int nx, int ny, int pitch,
                                                     double sigma_lim) {
  constexpr int NV = SYS::NV;
  const unsigned n = (unsigned)nx * (unsigned)ny;
  const long long plane = (long long)ny * pitch;
  for (unsigned k = blockIdx.x * 256 + threadIdx.x; k < n; k += gridDim.x * 256) {
    const long long off = padded_index(k, nx, ny, pitch);
    double Uc[NV], W[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) Uc[v] = U[v * plane + off];
    if constexpr (REPR == 1) {
#pragma unroll
      for (int v = 0; v < NV; ++v) dst[(long long)v * n + k] = Uc[v];
    } else {
      SYS::cons_to_prim(Uc, W);
      if constexpr (REPR == 0) {
#pragma unroll
        for (int v = 0; v < NV; ++v) dst[(long long)v * n + k] = W[v];
      } else if constexpr (REPR == 2) {
        dst[k] = SYS::sigma(W);
      } else if constexpr (NV == 14) {
        double c[NCLOSE14];
        closing14(W, sigma_lim, c);
#pragma unroll
        for (int m = 0; m < NCLOSE14; ++m) dst[(long long)m * n + k] = c[m];
      } else {
        typename SYS::template Core<double> kc;
        SYS::core(W, sigma_lim, kc);
        dst[k] = SYS::closing_s(kc);
      }
    }
  }
}

// cells of a state whose unlimited sigma is below sigma_lim (the closure evaluates them at
// sigma_bar = sigma_lim), added to ctrl->n_sigma_limited
template <class SYS>
__global__ __launch_bounds__(256) void count_sigma_limited_kernel(const double* U, int nx, int ny,
                                                                  int pitch, double sigma_lim,
                                                                  DevCtrl* c) {
  constexpr int NV = SYS::NV;
  const unsigned n = (unsigned)nx * (unsigned)ny;
  const long long plane = (long long)ny * pitch;
  int cnt = 0;
  for (unsigned k = blockIdx.x * 256 + threadIdx.x; k < n; k += gridDim.x * 256) {
    const long long off = padded_index(k, nx, ny, pitch);
    double Uc[NV], W[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) Uc[v] = U[v * plane + off];
    SYS::cons_to_prim(Uc, W);
    cnt += (SYS::sigma(W) < sigma_lim) ? 1 : 0;
  }
  cnt = wave_sum(cnt);
  if ((threadIdx.x & 63) == 0 && cnt)
    atomicAdd((unsigned long long*)&c->n_sigma_limited, (unsigned long long)cnt);
}

// ------------------------------------------------------------------ launchers
template <class SYS, int DIM, int ORDER, int PREC, int LPF>
static hipError_t launch_stage_l(const StageParams& p, hipStream_t s) {
  const int grid = ((p.nblk + 7) / 8) * 8;
  constexpr int TX = DIM == 2 ? 16 : tile_1d(64), TY = DIM == 2 ? 15 : 1, NT = (DIM == 2 ? 256 : 64) * LPF;
  hipLaunchKernelGGL((stage_kernel<SYS, DIM, ORDER, PREC, TX, TY, NT, LPF>), dim3(grid), dim3(NT), 0, s, p);
  return hipGetLastError();
}

// Tiles up to which two lanes share a face: while the doubled workgroups all run at once.  2D
// planar: two 512-thread workgroups on each of the 256 CUs (two stages and their gaps, one
// lane -> two: 64 x 64 30.2 -> 27.0 us, 224 x 224 30.9 -> 27.8, 320 x 320 41.1 -> 40.9; beyond,
// 352 x 352 50.7 -> 55.5, 768 x 768 159 -> 170).  2D with all 14 moments: one on each CU (two would
// fit as well, but then one lane is faster: 64 x 64 36.6 -> 34.5, 192 x 192 37.2 -> 36.1, but 256 x
// 256 50.2 -> 54.1).  1D: two-wave workgroups, four waves per SIMD of the 1024 with seven moments or
// fewer, which is what the axial kernel's 128 registers allow (1000 cells of 5 moments 14.0 -> 12.9,
// 96000 21.0 -> 19.5, and in 20 first-order steps with load and read 140000 325 -> 319 but 160000 333
// -> 366; axial 18.4 -> 16.2, 27.8 -> 26.8, 20 steps of 112000 643 -> 640 but 140000 750 -> 793),
// two with 14 (1000 cells 20.5 -> 18.3, 48000 24.2 -> 22.8, but 64000 29.7 -> 35.7).
constexpr int two_lane_tiles(int nv, int dim) {
  if (dim == 1) return nv <= 7 ? 2048 : 1024;
  return nv <= 10 ? 512 : 256;
}

template <class SYS, int DIM, int ORDER, int PREC>
static hipError_t launch_stage_t(const StageParams& p, hipStream_t s) {
  if constexpr (PREC == 0) {
    if (p.nblk <= two_lane_tiles(SYS::NV, DIM)) return launch_stage_l<SYS, DIM, ORDER, PREC, 2>(p, s);
  }
  return launch_stage_l<SYS, DIM, ORDER, PREC, 1>(p, s);
}

template <int PREC>
static hipError_t launch_stage_p(int system, int dim, int order, bool reduced, const StageParams& p,
                                 hipStream_t s) {
  if (system == 5) {
    if (dim != 1) return hipErrorInvalidValue;
    return order == 2 ? launch_stage_t<Sys5, 1, 2, PREC>(p, s) : launch_stage_t<Sys5, 1, 1, PREC>(p, s);
  }
  if (dim == 1) {
    if (reduced)
      return order == 2 ? launch_stage_t<Sys14A, 1, 2, PREC>(p, s) : launch_stage_t<Sys14A, 1, 1, PREC>(p, s);
    return order == 2 ? launch_stage_t<Sys14, 1, 2, PREC>(p, s) : launch_stage_t<Sys14, 1, 1, PREC>(p, s);
  }
  if (reduced)
    return order == 2 ? launch_stage_t<Sys14P, 2, 2, PREC>(p, s) : launch_stage_t<Sys14P, 2, 1, PREC>(p, s);
  return order == 2 ? launch_stage_t<Sys14, 2, 2, PREC>(p, s) : launch_stage_t<Sys14, 2, 1, PREC>(p, s);
}

hipError_t launch_stage(int system, int dim, int order, int precision, bool reduced,
                        const StageParams& p, hipStream_t s) {
  if (precision == 1) return launch_stage_p<1>(system, dim, order, reduced, p, s);
  if (precision == 2) return launch_stage_p<2>(system, dim, order, reduced, p, s);
  return launch_stage_p<0>(system, dim, order, reduced, p, s);
}

hipError_t launch_cfl(int system, int dim, const CflParams& p, hipStream_t s) {
  const int grid = field_grid((long long)p.nx * p.ny);
  if (system == 5) hipLaunchKernelGGL((cfl_kernel<Sys5, 1>), dim3(grid), dim3(256), 0, s, p);
  else if (dim == 1) hipLaunchKernelGGL((cfl_kernel<Sys14, 1>), dim3(grid), dim3(256), 0, s, p);
  else hipLaunchKernelGGL((cfl_kernel<Sys14, 2>), dim3(grid), dim3(256), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_ctrl_reset(DevCtrl* c, RatePart* rates, double t0, hipStream_t s) {
  hipLaunchKernelGGL(ctrl_reset_kernel, dim3(1), dim3(RATE_PARTS), 0, s, c, rates, t0);
  return hipGetLastError();
}

hipError_t launch_zero_planes(double* U, long long plane, int nv, hipStream_t s) {
  if (nv != 14) return hipSuccess;
  long long n = 7 * plane;
  int grid = (int)((n + 255) / 256);
  if (grid > 8192) grid = 8192;
  hipLaunchKernelGGL(zero_planes_kernel, dim3(grid), dim3(256), 0, s, U, plane);
  return hipGetLastError();
}

hipError_t launch_ingest(int system, int dim, const IngestParams& p, hipStream_t s) {
  const int grid = field_grid((long long)p.nx * p.ny);
  if (p.inst) hipLaunchKernelGGL((ingest_kernel<Sys14, 1, true>), dim3(grid), dim3(256), 0, s, p);
  else if (system == 5) hipLaunchKernelGGL((ingest_kernel<Sys5, 1, false>), dim3(grid), dim3(256), 0, s, p);
  else if (dim == 1) hipLaunchKernelGGL((ingest_kernel<Sys14, 1, false>), dim3(grid), dim3(256), 0, s, p);
  else hipLaunchKernelGGL((ingest_kernel<Sys14, 2, false>), dim3(grid), dim3(256), 0, s, p);
  return hipGetLastError();
}

template <class SYS>
static hipError_t launch_egress_t(int repr, const double* U, double* dst, int nx, int ny, int pitch,
                                  double sigma_lim, hipStream_t s) {
  const dim3 grid(field_grid((long long)nx * ny)), wg(256);
  if (repr == 0) hipLaunchKernelGGL((egress_kernel<SYS, 0>), grid, wg, 0, s, U, dst, nx, ny, pitch, sigma_lim);
  else if (repr == 1) hipLaunchKernelGGL((egress_kernel<SYS, 1>), grid, wg, 0, s, U, dst, nx, ny, pitch, sigma_lim);
  else if (repr == 2) hipLaunchKernelGGL((egress_kernel<SYS, 2>), grid, wg, 0, s, U, dst, nx, ny, pitch, sigma_lim);
  else hipLaunchKernelGGL((egress_kernel<SYS, 3>), grid, wg, 0, s, U, dst, nx, ny, pitch, sigma_lim);
  return hipGetLastError();
}

hipError_t launch_egress(int system, int repr, const double* U, double* dst, int nx, int ny,
                         int pitch, double sigma_lim, hipStream_t s) {
  return system == 5 ? launch_egress_t<Sys5>(repr, U, dst, nx, ny, pitch, sigma_lim, s)
                     : launch_egress_t<Sys14>(repr, U, dst, nx, ny, pitch, sigma_lim, s);
}

hipError_t launch_count_sigma_limited(int system, const double* U, int nx, int ny, int pitch,
                                      double sigma_lim, DevCtrl* c, hipStream_t s) {
  const int grid = field_grid((long long)nx * ny);
  if (system == 5)
    hipLaunchKernelGGL((count_sigma_limited_kernel<Sys5>), dim3(grid), dim3(256), 0, s, U, nx, ny, pitch, sigma_lim, c);
  else
    hipLaunchKernelGGL((count_sigma_limited_kernel<Sys14>), dim3(grid), dim3(256), 0, s, U, nx, ny, pitch, sigma_lim, c);
  return hipGetLastError();
}

}  // namespace mx
