// Per-cell and per-face pieces of the finite-volume scheme (Section 3 of the paper), on
// registers, templated on the system and the real type (host + device).
//   limiter_factor  one common, most stringent limiter factor for all primitives of a cell
//                   along one direction (Section 3.2), relative to the central slope
//   face_state      the cell's reconstructed state at its upper (sgn = +1) or lower face
//   face_flux       HLL or Rusanov combination of the two face states' physical fluxes with
//                   the approximate wave speeds (Section 3.1)
#pragma once
#include "mx_physics.hpp"
#if defined(__HIP_DEVICE_COMPILE__)
#include "mx_internal.hpp"
#endif

namespace mx {

// A variable whose two one-sided jumps are both below NEUTRAL_EPS times its natural scale
// does not take part in the common limiter: round-off is not a discontinuity.
constexpr double NEUTRAL_EPS = 1e-10;

// The variable that limits a cell: with one-sided jumps a, b, d = a + b and e = b - a, both
// limiters fall with the ratio |e| / |d| (minmod 2 min(|a|, |b|) / (|a| + |b|) = 1 - |e| / |d|, van
// Albada 2 a b / (a^2 + b^2) = (d^2 - e^2) / (d^2 + e^2), both zero from |e| = |d| on, where
// a b <= 0).  So the most stringent factor is that of the largest ratio, kept as a fraction
// num / den and compared by cross multiplication: no branch per variable or limiter, 248 VALU
// instructions for a cell and direction of the planar system where the two factors compared
// as they are written took 379 and a branch or two per variable.  vsel is the selected variable, or -1 (none: every variable neutral or e = 0).
template <class SYS, class T>
MX_HD void limiter_ratio(const T* Wm, const T* Wc, const T* Wp, T& num, T& den, int& vsel) {
  constexpr int NV = SYS::NV;
  T sc[NV];
  SYS::scales(Wc, sc);
  num = T(0); den = T(1);
  vsel = -1;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const T a = Wc[v] - Wm[v], b = Wp[v] - Wc[v];
    const T d = b + a, e = b - a;
    // num and den keep their signs until the end: a magnitude taken as an operand is free
    const bool take = !(tabs(a) + tabs(b) <= T(NEUTRAL_EPS) * sc[v]) && (tabs(e) * tabs(den) > tabs(num) * tabs(d));
    num = take ? e : num;
    den = take ? d : den;
    vsel = take ? v : vsel;
  }
  num = tabs(num);
  den = tabs(den);
}

// the factor of the ratio num / den (0 from num = den on)
template <class T> MX_HD T limiter_of_ratio(T num, T den, int kind) {
  if (!(num < den)) return T(0);
  if (kind == 0) return mdiv(den - num, den);
  const T n2 = num * num, d2 = den * den;
  return mdiv(d2 - n2, d2 + n2);
}

template <class SYS, class T>
MX_HD T limiter_factor(const T* Wm, const T* Wc, const T* Wp, int kind) {
  T num, den;
  int vsel;
  limiter_ratio<SYS>(Wm, Wc, Wp, num, den, vsel);
  return limiter_of_ratio(num, den, kind);
}

// A tube's factor (TUBE: the roundings are fixed): the formulas of both limiters as they stand, the
// running minimum kept as a fraction (den > 0) compared by cross multiplication; a jump that
// changes sign gives 0.
template <bool MINMOD, class SYS, class T>
MX_HD T limiter_tube(const T* Wm, const T* Wc, const T* Wp) {
#pragma clang fp contract(off)
  constexpr int NV = SYS::NV;
  T sc[NV];
  SYS::scales(Wc, sc);
  T num = T(1), den = T(1);
  bool turns = false;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const T a = Wc[v] - Wm[v], b = Wp[v] - Wc[v];
    const T aa = tabs(a), ab = tabs(b);
    const bool counts = !(aa + ab <= T(NEUTRAL_EPS) * sc[v]), turn = a * b <= T(0);
    const T fn = MINMOD ? T(2) * tmin(aa, ab) : T(2) * a * b, fd = MINMOD ? aa + ab : dfma(a, a, b * b);
    const bool take = counts && !turn && fn * den < num * fd;
    num = take ? fn : num;
    den = take ? fd : den;
    turns = turns || (counts && turn);
  }
  return turns ? T(0) : ((den == T(1)) ? num : mdiv2(num, den));
}

// what the stages take
template <class SYS, class T>
MX_HD T cell_limiter(const T* Wm, const T* Wc, const T* Wp, int kind) {
  if constexpr (SYS::TUBE) return kind == 0 ? limiter_tube<true, SYS>(Wm, Wc, Wp) : limiter_tube<false, SYS>(Wm, Wc, Wp);
  else return limiter_factor<SYS>(Wm, Wc, Wp, kind);
}

// The cell's state at its upper (sgn = +1) or lower (sgn = -1) face: Wc +- s/2 with the limited
// slope s = phi (a + b)/2 and a + b = Wp - Wm, i.e. Wc + sgn (phi/4)(Wp - Wm), one rounding per
// component.
template <class SYS, class T>
MX_HD void face_state(const T* Wm, const T* Wc, const T* Wp, T phi, T sgn, T* Wf) {
  const T q = sgn * T(0.25) * phi;
#pragma unroll
  for (int v = 0; v < SYS::NV; ++v) Wf[v] = tfma(q, Wp[v] - Wm[v], Wc[v]);
}

// Positivity check of both face states of a cell (rho > 0 and P positive definite): only the
// components the check reads are reconstructed, with face_state's expressions, so the check
// decides on exactly the face states the flux evaluation uses.
template <class SYS, class T>
MX_HD bool faces_admissible(const T* Wm, const T* Wc, const T* Wp, T phi) {
  constexpr int NV = SYS::NV;
  const T q = T(0.25) * phi;
  T Wu[NV], Wd[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    if (!SYS::admissibility_var(v)) { Wu[v] = Wd[v] = T(0); continue; }
    const T d = Wp[v] - Wm[v];
    Wu[v] = tfma(q, d, Wc[v]);
    Wd[v] = tfma(-q, d, Wc[v]);
  }
  return SYS::admissible(Wu) && SYS::admissible(Wd);
}

// 1 / tau of a cell.  Mode 0: tau = tau_ref (rho_ref / rho) sqrt(T_ref / T), T = p / rho, so
// 1 / tau = k rho sqrt(T) with k = 1 / (tau_ref rho_ref sqrt(T_ref)); mode 1: k = 1 / tau_ref.
// k comes from inv_tau_constant, once per run: a cell takes one reciprocal and one reciprocal
// square root (the quotients and the root as they stand took about 110 VALU instructions more).
template <class SYS, class T> MX_HD T inv_tau(const T* W, int mode, T k) {
  if (mode != 0) return k;
  const T temp = SYS::pressure(W) * mrcp(W[0]);
  return k * (W[0] * (temp * mrsqrt(temp)));
}
// tau of a tube's cell, in the quotients and the root as they stand (TUBE: the roundings are fixed)
template <class SYS, class T> MX_HD T tau_tube(const T* W, int mode, T tau_ref, T rho_ref, T T_ref) {
  const T temp = SYS::pressure(W) / W[0];
  return (mode == 0) ? tau_ref * (rho_ref / W[0]) * sqrt(T_ref / temp) : tau_ref;
}

// Interface flux of two face states: HLL (Davis speeds) or Rusanov, in one form, the left
// side's share and then the right side's
//   Fh = (cL FL - d UL) + (cR FR + d UR).
// HLL: S- = min(SL, 0), S+ = max(SR, 0), cL = S+ / (S+ - S-), cR = -S- / (S+ - S-),
// d = S- S+ / (S+ - S-): the upwind fluxes of the supersonic cases follow from S- = 0 or
// S+ = 0 without a branch or a select per component.  Rusanov: cL = cR = 1/2, d = -a*/2.  A NaN
// wave speed of either side reaches every component through d.  (d U is at most
// CFL dx U / (2 dt), so rounding d UL and d UR apart moves the update by no more than its own
// rounding.)
template <class T> struct FaceCoef { T cL, cR, d; };
template <class T>
MX_HD FaceCoef<T> face_coef(T lminL, T lmaxL, T lminR, T lmaxR, int flux_kind) {
  FaceCoef<T> k;
  if (flux_kind == 0) {
    const T Sm = cmin(tmin(lminL, lminR), T(0)), Sp = cmax(tmax(lmaxL, lmaxR), T(0));
    const T inv = mrcp(Sp - Sm);
    k.cL = Sp * inv;
    k.cR = -Sm * inv;
    k.d = Sm * k.cL + T(0) * (lminL + lminR);
  } else {
    const T am = tmax(tmax(tabs(lminL), tabs(lmaxL)), tmax(tabs(lminR), tabs(lmaxR)));
    k.cL = k.cR = T(0.5);
    k.d = T(-0.5) * am;
  }
  return k;
}
// a component: the left side's share, and the flux from that and the right side (the same
// roundings in one lane or two)
template <class T> MX_HD T share_left(const FaceCoef<T>& k, T F, T U) { return tfma(k.cL, F, -(k.d * U)); }
template <class T> MX_HD T add_right(const FaceCoef<T>& k, T F, T U, T left) { return tfma(k.cR, F, tfma(k.d, U, left)); }

// The same flux of a tube (TUBE: the roundings are fixed): the upwind flux as it is, and the jump of U
// before its product.
template <class T> struct FaceSpeeds { T SL, SR, SLR, inv, am; };
template <class T>
MX_HD FaceSpeeds<T> face_speeds(T lminL, T lmaxL, T lminR, T lmaxR, int flux_kind) {
  FaceSpeeds<T> k = {};
  if (flux_kind == 0) {
    k.SL = tmin(lminL, lminR);
    k.SR = tmax(lmaxL, lmaxR);
    k.inv = mrcp2(k.SR - k.SL);
    k.SLR = k.SL * k.SR;
  } else {
    k.am = tmax(tmax(tabs(lminL), tabs(lmaxL)), tmax(tabs(lminR), tabs(lmaxR)));
  }
  return k;
}
template <class T>
MX_HD T flux_tube(const FaceSpeeds<T>& k, int flux_kind, T FL, T UL, T FR, T UR) {
#pragma clang fp contract(off)
  if (flux_kind == 0) {
    const T mid = dfma(k.SLR, UR - UL, dfma(k.SR, FL, -(k.SL * FR))) * k.inv;
    return (k.SL >= T(0)) ? FL : ((k.SR <= T(0)) ? FR : mid);
  }
  return dfma(T(0.5), FL + FR, -(T(0.5) * k.am * (UR - UL)));
}

template <class SYS, int D, class T>
MX_HD void face_flux(const T* WL, const T* WR, T sigma_lim, T kws, int flux_kind, T* Fh) {
  constexpr int NV = SYS::NV;
  T UL[NV], FL[NV], UR[NV], FR[NV];
  T lminL, lmaxL, lminR, lmaxR;
  SYS::template face_terms<D>(WL, sigma_lim, kws, UL, FL, lminL, lmaxL);
  if constexpr (SYS::TUBE) {   // the left side's results alone are held while the right side's come
#pragma unroll
    for (int v = 0; v < NV; ++v) { opaque(UL[v]); opaque(FL[v]); }
    opaque(lminL); opaque(lmaxL);
  }
  SYS::template face_terms<D>(WR, sigma_lim, kws, UR, FR, lminR, lmaxR);
  if constexpr (SYS::TUBE) {
    const FaceSpeeds<T> k = face_speeds(lminL, lmaxL, lminR, lmaxR, flux_kind);
#pragma unroll
    for (int v = 0; v < NV; ++v) Fh[v] = flux_tube(k, flux_kind, FL[v], UL[v], FR[v], UR[v]);
    return;
  }
  opaque(lminL); opaque(lmaxL); opaque(lminR); opaque(lmaxR);
  const FaceCoef<T> k = face_coef(lminL, lmaxL, lminR, lmaxR, flux_kind);
#pragma unroll
  for (int v = 0; v < NV; ++v) Fh[v] = add_right(k, FR[v], UR[v], share_left(k, FL[v], UL[v]));
}

#if defined(__HIP_DEVICE_COMPILE__)
// a value of the neighbouring lane (lane ^ 1)
__device__ __forceinline__ double lane_xor1(double x) { return dpp_move<0xB1>(x); }
#else
__device__ inline double lane_xor1(double x) { return x; }
#endif

// The same flux by two neighbouring lanes, each with one face state W (right: the right one);
// the right one gets the flux.  A lane evaluates one closure and pair of wave speeds, not two,
// so a face takes half as long and needs about half the registers.
template <class SYS, int D>
__device__ __forceinline__ void face_flux_pair(const double* W, bool right, double sigma_lim, double kws,
                                               int flux_kind, double* Fh) {
  constexpr int NV = SYS::NV;
  double U[NV], F[NV], lmin, lmax;
  SYS::template face_terms<D>(W, sigma_lim, kws, U, F, lmin, lmax);
  opaque(lmin); opaque(lmax);
  const double omin = lane_xor1(lmin), omax = lane_xor1(lmax);
  if constexpr (SYS::TUBE) {   // (of the right lane; the left one's result is not used)
    const FaceSpeeds<double> k = face_speeds(omin, omax, lmin, lmax, flux_kind);
#pragma unroll
    for (int v = 0; v < NV; ++v) Fh[v] = flux_tube(k, flux_kind, lane_xor1(F[v]), lane_xor1(U[v]), F[v], U[v]);
    return;
  }
  const FaceCoef<double> k = face_coef(right ? omin : lmin, right ? omax : lmax, right ? lmin : omin,
                                       right ? lmax : omax, flux_kind);
#pragma unroll
  for (int v = 0; v < NV; ++v) Fh[v] = add_right(k, F[v], U[v], lane_xor1(share_left(k, F[v], U[v])));
}

// Mixed precision (Section 3.3: the dimensionless closure is robust in single precision).
// The face states arrive in FP64 (primitive recovery and reconstruction stay FP64).  The
// bracket A of the sigma mapping is formed in FP64 (it cancels near equilibrium); the rest of
// the closure, the wave speeds and the physical flux of each face state are in FP32,
// except near the Junk subspace (A < -MIX_DA and sigma < MIX_SIG_JUNK, where q^3/sigma^2 is
// large) and near the realizability boundary (sigma > 1 - MIX_D1, where 1 - sigma and
// sqrt(3 - 3 sigma) cancel): there the state is re-evaluated in FP64.  The HLL dissipation
// term S_L S_R (U_R - U_L) / (S_R - S_L) uses FP64 conserved states, so that the jump is not
// cancelled in FP32.  Returns the number of FP64 re-evaluations (0, 1 or 2).
constexpr float MIX_DA = 1e-3f;
constexpr float MIX_SIG_JUNK = 1e-2f;
constexpr float MIX_D1 = 1e-3f;

template <class SYS, int D>
MX_HD void face_side_mixed(const double* W64, double sigma_lim, double kws, float* F, float& lmin,
                           float& lmax, int& n64) {
  constexpr int NV = SYS::NV;
  float W[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) W[v] = (float)W64[v];
  typename SYS::template Core<float> k;
  SYS::core_mixed(W64, (float)sigma_lim, k);
  bool near_junk = (k.A < -MIX_DA) && (k.sig < MIX_SIG_JUNK);
  bool near_boundary = k.sig > 1.0f - MIX_D1;
  if (near_junk || near_boundary || !(k.sig == k.sig)) {
    double U[NV], F64[NV], a, b;
    SYS::template face_terms<D>(W64, sigma_lim, kws, U, F64, a, b);
#pragma unroll
    for (int v = 0; v < NV; ++v) F[v] = (float)F64[v];
    lmin = (float)a;
    lmax = (float)b;
    ++n64;
  } else {
    SYS::template flux_speeds<D>(k, W, (float)kws, F, lmin, lmax);
  }
}

template <class SYS, int D>
MX_HD void face_flux_mixed(const double* WL, const double* WR, double sigma_lim, double kws,
                           int flux_kind, double* Fh, int& n64) {
  constexpr int NV = SYS::NV;
  float FL[NV], FR[NV], lminL, lmaxL, lminR, lmaxR;
  face_side_mixed<SYS, D>(WL, sigma_lim, kws, FL, lminL, lmaxL, n64);
  face_side_mixed<SYS, D>(WR, sigma_lim, kws, FR, lminR, lmaxR, n64);
  double UL[NV], UR[NV];
  SYS::prim_to_cons(WL, UL);
  SYS::prim_to_cons(WR, UR);
  if (flux_kind == 0) {
    float SL = tmin(lminL, lminR), SR = tmax(lmaxL, lmaxR);
    if (SL >= 0.0f) {
#pragma unroll
      for (int v = 0; v < NV; ++v) Fh[v] = (double)FL[v];
    } else if (SR <= 0.0f) {
#pragma unroll
      for (int v = 0; v < NV; ++v) Fh[v] = (double)FR[v];
    } else {
      float inv = 1.0f / (SR - SL);
      double diss = (double)SL * (double)SR / ((double)SR - (double)SL);
#pragma unroll
      for (int v = 0; v < NV; ++v)
        Fh[v] = (double)((SR * FL[v] - SL * FR[v]) * inv) + diss * (UR[v] - UL[v]);
    }
  } else {
    float am = tmax(tmax(tabs(lminL), tabs(lmaxL)), tmax(tabs(lminR), tabs(lmaxR)));
#pragma unroll
    for (int v = 0; v < NV; ++v)
      Fh[v] = (double)(0.5f * (FL[v] + FR[v])) - 0.5 * (double)am * (UR[v] - UL[v]);
  }
}

// Single precision (the FP32 setting): the closure, wave speeds, physical fluxes and the HLL /
// Rusanov combination of both face states in FP32, with no FP64 re-evaluation; the face
// states arrive in FP64 and the interface flux leaves in FP64.  It keeps the sequence of
// operations it always had (Core, closure_dir, flux, prim_to_cons, wavespeeds): rearranged as
// the FP64 path is, its results would move by single-precision rounding.
template <class SYS, int D>
MX_HD void face_flux_fp32(const double* WL, const double* WR, double sigma_lim, double kws,
                          int flux_kind, double* Fh) {
  constexpr int NV = SYS::NV;
  float wl[NV], wr[NV], f[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) { wl[v] = (float)WL[v]; wr[v] = (float)WR[v]; }
  float UL[NV], FL[NV], UR[NV], FR[NV];
  float lminL, lmaxL, lminR, lmaxR;
  SYS::template face_terms_fp32<D>(wl, (float)sigma_lim, (float)kws, UL, FL, lminL, lmaxL);
  SYS::template face_terms_fp32<D>(wr, (float)sigma_lim, (float)kws, UR, FR, lminR, lmaxR);
  if (flux_kind == 0) {
    float SL = tmin(lminL, lminR), SR = tmax(lmaxL, lmaxR);
    if (SL >= 0.0f) {
#pragma unroll
      for (int v = 0; v < NV; ++v) f[v] = FL[v];
    } else if (SR <= 0.0f) {
#pragma unroll
      for (int v = 0; v < NV; ++v) f[v] = FR[v];
    } else {
      float inv = mrcp(SR - SL);
      float SLR = SL * SR;
#pragma unroll
      for (int v = 0; v < NV; ++v) f[v] = (SR * FL[v] - SL * FR[v] + SLR * (UR[v] - UL[v])) * inv;
    }
  } else {
    float am = tmax(tmax(tabs(lminL), tabs(lmaxL)), tmax(tabs(lminR), tabs(lmaxR)));
#pragma unroll
    for (int v = 0; v < NV; ++v) f[v] = 0.5f * (FL[v] + FR[v]) - 0.5f * am * (UR[v] - UL[v]);
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) Fh[v] = (double)f[v];
}

}  // namespace mx
