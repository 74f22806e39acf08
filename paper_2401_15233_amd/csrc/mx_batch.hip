// Batched independent 1D shock tubes in one launch per stage.
//
// Many 1D problems of uneven length, each with its own collision time, end time and CFL time
// step, are concatenated in one structure-of-arrays field.  The instances form a queue
// ordered by estimated work (cells x steps, from the initial CFL rate).  Each step, a
// one-workgroup finalize kernel gives every instance its time step and compacts the
// instances that still advance, in queue order, into a work list of tiles (tiles never
// straddle instances); the two stage launches of the step split that list into contiguous
// ranges, one per workgroup, so finished instances cost nothing.  A step is finalize + two
// stage launches, so a chunk of steps can be captured once in a hipGraph and replayed.  The
// per-cell arithmetic is the single-instance 1D kernel's (same device functions, same update
// formula), so a batched instance reproduces the same instance run alone bit for bit.
#include "mx_internal.hpp"
#include "mx_physics.hpp"
#include "mx_scheme.hpp"
#include "mx_axial.hpp"
#include "mx_batch.hpp"

namespace mx {

// a value that all lanes share, in scalar registers
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ long long uniform(long long x) {
  return ((long long)uniform((int)(x >> 32)) << 32) | (unsigned)uniform((int)x);
}
__device__ __forceinline__ double uniform(double x) { return __longlong_as_double(uniform(__double_as_longlong(x))); }

__device__ __forceinline__ int bmap(int g, int n, int lo, int hi, int& refl) {
  if (g < 0) {
    if (lo == 1) g = g + n * ((-g + n - 1) / n);
    else if (lo == 2) { g = -g - 1; refl = 1; }
    else g = 0;
  } else if (g >= n) {
    if (hi == 1) g = g % n;
    else if (hi == 2) { g = 2 * n - 1 - g; refl = 1; }
    else g = n - 1;
  }
  return g < 0 ? 0 : (g >= n ? n - 1 : g);
}

// One workgroup of 1024 threads walks the instance queue (instances ordered by estimated
// work): time step of each instance from its CFL rate, clipped to its t_end; then an ordered
// compaction of the instances that advance, with the exclusive prefix of their tile counts.
// The stage launches of the step split the resulting tile list into contiguous ranges.
__global__ __launch_bounds__(1024) void batch_finalize_kernel(BatchInst* in, const int* order, int n_inst,
                                                             double cfl, int tile_w, int* act_inst,
                                                             int* act_tile0, BatchCtrl* bc, int nb) {
  __shared__ int s_wave[16][2];   // per-wavefront totals of (active, tiles)
  __shared__ int s_carry[2];      // totals of the earlier chunks
  const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
  if (t == 0) { s_carry[0] = 0; s_carry[1] = 0; }
  __syncthreads();
  for (int base = 0; base < n_inst; base += 1024) {
    const int q = base + t;
    int a = 0, nt = 0, inst = 0;
    if (q < n_inst) {
      inst = order[q];
      BatchInst& c = in[inst];
      double dt = 0.0;
      if (c.status == 0) {
        double m = __longlong_as_double((long long)c.maxrate);
        dt = (m > 0.0) ? cfl * c.dx / m : 0.0;
        if (c.t >= c.t_end * (1.0 - 1e-14)) dt = 0.0;
        else dt = fmin(dt, c.t_end - c.t);
      }
      c.dt = dt;
      c.maxrate = 0ull;
      if (dt > 0.0) {
        c.t += dt;
        c.step += 1;
        c.dt_last = dt;
        a = 1;
        nt = (c.n + tile_w - 1) / tile_w;
      }
    }
    // inclusive scans within the wavefront
    int sa = a, sn = nt;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      int ya = __shfl_up(sa, o, 64), yn = __shfl_up(sn, o, 64);
      if (lane >= o) { sa += ya; sn += yn; }
    }
    if (lane == 63) { s_wave[wid][0] = sa; s_wave[wid][1] = sn; }
    __syncthreads();
    int oa = s_carry[0], on = s_carry[1];
    for (int w = 0; w < wid; ++w) { oa += s_wave[w][0]; on += s_wave[w][1]; }
    if (a) {
      act_inst[oa + sa - 1] = inst;
      act_tile0[oa + sa - 1] = on + sn - nt;
    }
    __syncthreads();  // every thread has read s_carry
    if (t == 1023) { s_carry[0] = oa + sa; s_carry[1] = on + sn; }
    __syncthreads();
  }
  if (t == 0) {
    const int n_tiles = s_carry[1];
    act_tile0[s_carry[0]] = n_tiles;
    bc->n_active = s_carry[0];
    bc->n_tiles = n_tiles;
    // split of the tile list over the nb workgroups of the stage launches: contiguous ranges
    // of `per` tiles.  Hardware deals consecutive workgroups round-robin to the 8 XCDs; each
    // XCD gets a band of neighbouring ranges, so that halos and instance records are shared
    // in its L2.  While the ranges in use fill more than half of the grid the bands are the
    // grid's eighths; once they fill half or less (the end of a batch) the bands divide the
    // ranges in use, which would otherwise all fall on the first XCDs (measured on one
    // 546-tile tube: 85 -> 37.5 us per step)
    const int per = (n_tiles + nb - 1) / nb;
    int band = 0;
    if (nb % 8 == 0 && per > 0) {
      const int used = (n_tiles + per - 1) / per;  // <= nb
      band = (2 * used <= nb) ? (used + 7) / 8 : nb / 8;
    }
    bc->per = per;
    bc->band = band;
  }
}

// Stage kernel: a workgroup of NT threads owns tiles of CPT * NT - 4 cells (CPT cells per
// thread), so the tile plus its two-cell halos is CPT whole rounds over the threads.  The
// step's tile list (active instances in queue order, each cut into tiles) is split into
// contiguous ranges, one per workgroup, with an XCD-aware order of the ranges; a workgroup
// finds its first tile by a binary search over the tile prefix and then walks forward.
//
// Bound by FP64 VALU work; a workgroup reduces status, counters and CFL rate once for the tiles of an
// instance in its range instead of for each tile.  512 tubes of 512 to 32768 cells (4.3 M cells, 256
// threads), 20 steps with load and read: 13.3 ms (a reduction per tile, and the CFL rate of the
// loaded field in a pass of its own: 18.2).  A variant that kept the thread's own cell, U^n and the
// next tile's cell in registers across the faces spilled 25 of 168 registers and took 15.4 ms.
template <class SYS, int PREC, int NT, int CPT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(SYS::NV <= 7 ? 3 : 2)))
void batch_stage_kernel(BatchParams p) {
  constexpr int NV = SYS::NV;
  constexpr int G = 2;
  constexpr int TX = tile_1d(CPT * NT);
  constexpr int LX = TX + 2 * G;
  constexpr int NFX = TX + 1;
  constexpr int NPX = TX + 2;
  static_assert(LX == CPT * NT, "tile and halo are whole rounds over the threads");
  __shared__ double sW[NV * LX];
  __shared__ double sFx[NV * NFX];
  __shared__ double sPx[NPX];
  const int t = threadIdx.x;
  const int lane = t & 63;

  const int n_tiles = uniform(p.bctrl->n_tiles);
  const int n_act = uniform(p.bctrl->n_active);
  // this workgroup's range of the tile list (split and XCD bands set by the finalize kernel)
  const int per = uniform(p.bctrl->per);
  const int band = uniform(p.bctrl->band);
  int slot = blockIdx.x;
  if (band > 0) {
    const int kx = blockIdx.x >> 3;
    slot = (kx < band) ? (blockIdx.x & 7) * band + kx : (int)gridDim.x;
  }
  const int k0 = slot * per;   // slot <= grid: at most n_tiles + grid
  const int k1 = min(k0 + per, n_tiles);
  if (k0 >= k1) return;  // uniform over the workgroup
  int j = 0;
  {
    int hi = n_act - 1;  // last active instance whose first tile is <= k0
    while (j < hi) {
      const int mid = (j + hi + 1) >> 1;
      if (uniform(p.act_tile0[mid]) <= k0) j = mid;
      else hi = mid - 1;
    }
  }
  // the tile in work: its instance and first cell (the record's constants of a step)
  struct Tile {
    BatchInst* c;
    int next;         // first tile of the next instance
    int n, i0;
    long long off;
    double dt, inv_dx, tau;   // tau: tau_ref of a tube's cells, inv_tau_constant of the others; 0: no source
  };
  auto open_instance = [&](int k) {   // every active instance has at least one tile
    Tile m;
    m.c = p.inst + uniform(p.act_inst[j]);
    m.next = uniform(p.act_tile0[j + 1]);
    m.n = uniform(m.c->n);
    m.i0 = (k - uniform(p.act_tile0[j])) * TX;
    m.off = uniform(m.c->off);
    m.dt = uniform(m.c->dt);
    m.inv_dx = uniform(m.c->inv_dx);
    m.tau = uniform(SYS::TUBE ? m.c->tau_ref : m.c->inv_tau_ref);
    return m;
  };
  // stage input of tile cell cc (interior or ghost source); refl: mirrored at a wall
  auto load_cell = [&](const Tile& m, int cc, double* U, int& refl) {
    refl = 0;
    const long long o = m.off + bmap(m.i0 + cc - G, m.n, p.bc_lo, p.bc_hi, refl);
#pragma unroll
    for (int v = 0; v < NV; ++v) U[v] = p.Ub[SYS::plane_of(v) * p.plane + o];
  };
  auto lds = [&](int ti, double* W) {
#pragma unroll
    for (int v = 0; v < NV; ++v) W[v] = sW[v * LX + ti + G];
  };

  Tile cur = open_instance(k0);
  double rate = 0.0;     // of the instance's tiles so far
  int n64 = 0, nfb = 0;
  for (int k = k0; k < k1; ++k) {
    const double dt = cur.dt;
    // (issue priority by phase as in the single kernel: 14.0 -> 13.3 ms, mixed 12.4 -> 11.4)
    __builtin_amdgcn_s_setprio(3);
    // 1. tile + halo -> primitives
#pragma unroll 1
    for (int r = 0; r < CPT; ++r) {
      const int cc = t + r * NT;
      double Uc[NV], W[NV];
      int refl;
      load_cell(cur, cc, Uc, refl);
      SYS::cons_to_prim(Uc, W);
      if (refl) {
#pragma unroll
        for (int v = 0; v < NV; ++v)
          if (SYS::odd(v, 0)) W[v] = -W[v];
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) sW[v * LX + cc] = W[v];
    }
    __syncthreads();

    // 2. common limiter factors (a spare thread repeats the last item)
#pragma unroll 1
    for (int r = 0; r < CPT; ++r) {
      const int cc = min(t + r * NT, NPX - 1);
      const int ti = cc - 1;
      double Wm[NV], Wc[NV], Wp[NV];
      lds(ti - 1, Wm); lds(ti, Wc); lds(ti + 1, Wp);
      double phi = cell_limiter<SYS>(Wm, Wc, Wp, p.limiter);
      if (p.fallback && phi > 0.0 && !faces_admissible<SYS>(Wm, Wc, Wp, phi)) {
        phi = 0.0;
        if (t + r * NT < NPX && ti >= 0 && ti < TX && cur.i0 + ti < cur.n) ++nfb;
      }
      sPx[cc] = phi;
    }
    __syncthreads();

    Tile nxt = cur;
    if (k + 1 < k1) {
      nxt.i0 += TX;
      if (k + 1 >= cur.next) {
        ++j;
        nxt = open_instance(k + 1);
      }
    }
    __builtin_amdgcn_s_setprio(0);
    // 3. faces: face fi lies between tile cells fi - 1 and fi.  (Mixed precision: the loop
    // stays a loop for CPT = 1 too, so that the compiler fuses products and sums there as it does
    // in the other kernels.)
    int rounds = CPT;
    if constexpr (PREC != 0) asm volatile("" : "+s"(rounds));
#pragma unroll 1
    for (int r = 0; r < rounds; ++r) {
      const int fi = min(t + r * NT, NFX - 1);
      double WL[NV], WR[NV], A[NV], B[NV], C[NV], D[NV];
      lds(fi - 2, A); lds(fi - 1, B); lds(fi, C); lds(fi + 1, D);
      face_state<SYS>(A, B, C, sPx[fi], 1.0, WL);
      face_state<SYS>(B, C, D, sPx[fi + 1], -1.0, WR);
      double Fh[NV];
      const int before = n64;
      if constexpr (PREC == 0) face_flux<SYS, 0>(WL, WR, p.sigma_lim, p.kws, p.flux, Fh);
      else face_flux_mixed<SYS, 0>(WL, WR, p.sigma_lim, p.kws, p.flux, Fh, n64);
      if (PREC != 0 && t + r * NT >= NFX) n64 = before;
#pragma unroll
      for (int v = 0; v < NV; ++v) sFx[v * NFX + fi] = Fh[v];
    }
    auto source = [&](int ci, double* Cs) {
      if (cur.tau > 0.0) {
        double W[NV];
        lds(ci, W);
        if constexpr (SYS::TUBE) SYS::source(W, 1.0 / tau_tube<SYS>(W, p.tau_mode, cur.tau, p.rho_ref, p.T_ref), Cs);
        else SYS::source(W, inv_tau<SYS>(W, p.tau_mode, cur.tau), Cs);
      } else {
#pragma unroll
        for (int v = 0; v < NV; ++v) Cs[v] = 0.0;
      }
    };
    __syncthreads();

    __builtin_amdgcn_s_setprio(1);
    // 4. update
    int flag = 0;
#pragma unroll 1
    for (int r = 0; r < CPT; ++r) {
      const int ci = min(t + r * NT, TX - 1);
      const bool own = t + r * NT < TX && cur.i0 + ci < cur.n;
      const long long g = cur.off + min(cur.i0 + ci, cur.n - 1);
      double Ub[NV], Ua[NV], Cs[NV], Un[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) Ub[v] = p.Ub[SYS::plane_of(v) * p.plane + g];
      if (p.mode != MODE_EULER) {
#pragma unroll
        for (int v = 0; v < NV; ++v) Ua[v] = p.Ua[SYS::plane_of(v) * p.plane + g];
      }
      source(ci, Cs);
      bool fin = true;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const double L = tfma(sFx[v * NFX + ci] - sFx[v * NFX + ci + 1], cur.inv_dx, Cs[v]);
        const double o = stage_update(p.mode, p.cdt, dt, L, Ub[v], Ua[v]);
        Un[v] = o;
        fin = fin && isfinite(o);
      }
      if (own) {
#pragma unroll
        for (int v = 0; v < NV; ++v) p.Uout[SYS::plane_of(v) * p.plane + g] = Un[v];
      }
      int bad = 0;
      double rc = 0.0;
      if (p.do_cfl) {
        double Wn[NV];
        if constexpr (SYS::TUBE) SYS::cons_to_prim(Un, Wn, false);
        else SYS::cons_to_prim(Un, Wn);
        if (!SYS::admissible(Wn)) bad = ST_UNREALIZABLE;
        rc = SYS::template cell_lambda<0>(Wn, p.sigma_lim, p.kws);
      } else if (!SYS::admissible_cons(Un)) {
        bad = ST_UNREALIZABLE;
      }
      if (!fin) bad = ST_NONFINITE;
      if (own) {
        flag |= bad;
        rate = fmax(rate, bad ? 0.0 : rc);
      }
    }
    if (__any(flag)) {   // a failed tube stops; rare
      flag = wave_or(flag);
      if (lane == 0) {
        atomicOr(&cur.c->status, flag);
        atomicMin(&cur.c->fail_step, (int)cur.c->step);
      }
    }
    // the instance's last tile of this range: its CFL rate
    if (p.do_cfl && (k + 1 == k1 || k + 1 >= cur.next)) {
      const double m = wave_max(rate);
      if (lane == 0) raise_max(&cur.c->maxrate, m);
      rate = 0.0;
    }
    __syncthreads();   // the update read the primitive tile
    cur = nxt;
  }
  // counters, once for the range
  nfb = wave_sum(nfb);
  if (lane == 0 && nfb) atomicAdd((unsigned long long*)&p.ctrl->n_fallback, (unsigned long long)nfb);
  if constexpr (PREC != 0) {
    n64 = wave_sum(n64);
    if (lane == 0 && n64) atomicAdd((unsigned long long*)&p.ctrl->n_fp64, (unsigned long long)n64);
    if (t == 0) atomicAdd((unsigned long long*)&p.ctrl->n_states, (unsigned long long)(k1 - k0) * (2 * NFX));
  }
}

// f(kernel) for the kernel of a launch shape
template <class SYS, int PREC, class F>
static hipError_t with_kernel_p(int nt, int cpt, F f) {
  if (nt == 64 && cpt == 1) return f(batch_stage_kernel<SYS, PREC, 64, 1>);
  if (nt == 64 && cpt == 2) return f(batch_stage_kernel<SYS, PREC, 64, 2>);
  if (nt == 64 && cpt == 4) return f(batch_stage_kernel<SYS, PREC, 64, 4>);
  if (nt == 128 && cpt == 1) return f(batch_stage_kernel<SYS, PREC, 128, 1>);
  if (nt == 128 && cpt == 2) return f(batch_stage_kernel<SYS, PREC, 128, 2>);
  if (nt == 256 && cpt == 1) return f(batch_stage_kernel<SYS, PREC, 256, 1>);
  return hipErrorInvalidValue;
}
template <class F>
static hipError_t with_kernel(int precision, bool reduced, int nt, int cpt, F f) {
  if (reduced)
    return precision == 0 ? with_kernel_p<Sys14A, 0>(nt, cpt, f) : with_kernel_p<Sys14A, 1>(nt, cpt, f);
  return precision == 0 ? with_kernel_p<Sys14, 0>(nt, cpt, f) : with_kernel_p<Sys14, 1>(nt, cpt, f);
}

bool batch_shape_supported(int nt, int cpt) {
  return (nt == 64 && (cpt == 1 || cpt == 2 || cpt == 4)) || (nt == 128 && (cpt == 1 || cpt == 2)) ||
         (nt == 256 && cpt == 1);
}

hipError_t launch_batch_stage(int precision, bool reduced, int nt, int cpt, const BatchParams& p, int grid,
                              hipStream_t s) {
  return with_kernel(precision, reduced, nt, cpt, [&](void (*kernel)(BatchParams)) {
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(nt), 0, s, p);
    return hipGetLastError();
  });
}

hipError_t batch_stage_residency(int precision, bool reduced, int nt, int cpt, int* workgroups) {
  return with_kernel(precision, reduced, nt, cpt, [&](void (*kernel)(BatchParams)) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(workgroups, (const void*)kernel, nt, 0);
  });
}

hipError_t launch_batch_finalize(BatchInst* in, const int* order, int n_inst, double cfl, int tile_w,
                                 int* act_inst, int* act_tile0, BatchCtrl* bc, int stage_grid,
                                 hipStream_t s) {
  if (stage_grid < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(batch_finalize_kernel, dim3(1), dim3(1024), 0, s, in, order, n_inst, cfl, tile_w,
                     act_inst, act_tile0, bc, stage_grid);
  return hipGetLastError();
}

}  // namespace mx
