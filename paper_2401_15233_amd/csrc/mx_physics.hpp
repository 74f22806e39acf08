// Pointwise physics of the 5- and 14-moment maximum-entropy systems, for gfx950 kernels.
//
// Everything here acts on registers of one thread: primitive <-> conserved maps, the
// sigma-limited interpolative closure evaluated in dimensionless variables, approximate
// wave speeds, physical fluxes along one axis, the BGK source.  All functions are
// __host__ __device__ and templated on the real type so that the same code can run in a
// host-side operation counter.
//
// Paper passages (arXiv 2401.15233):
//   conserved / flux / source terms   Section 2.3 (5-moment system) and Section 2.4 (14-moment
//                                      equations and BGK sources)
//   dimensionless variables           eq. dimensionless-variables; closure evaluated
//                                      dimensionless as Section 3.3 recommends
//   parabolic mapping sigma            eqs. sigma-mapping-5mom, sigma-mapping-14mom
//   closing moments                    eqs. closure-1D1V-s-approx, closure-14mom-*-approx
//   sigma limiting                     Section 2.3 and Appendix A
//   wave speeds                        Section 5.1 (eq. 14mom-approx-ws-equations) and
//                                      Appendix B (Baradaran, eq. ws-max-baradaran-orig)
//
// The 14-moment closure is written in reduced form.  With P, q dimensionless (rho = 1) and
//   Cm = 2 tr(P^2) I + 4 P^2,  w = Cm^-1 q  (= P B^-1 q because B = P Cm and P, Cm commute),
//   z = P^-1 q,
// the closing tensors become
//   Q_ijk   = 2 [w_i (P^2)_jk + w_j (P^2)_ik + w_k (P^2)_ij]
//   Q_idl z_l = 2 [w_i (P^2 z)_d + w_d (P^2 z)_i + (w.z) (P^2)_id]
//   Q_dkl z_k z_l = 2 [w_d (z.P^2 z) + 2 (w.z) (P^2 z)_d]
//   (W q)_d = (2 t1^3 + 12 t3 - 2 t2 t1) w_d + (14 t2 - 6 t1^2)(P w)_d + 20 t1 (P^2 w)_d
//             + 20 (P^3 w)_d,
// t_k = tr(P^k), so only two symmetric 3x3 solves are needed (P^-1 q and Cm^-1 q, Cm is
// always well conditioned) and only the ten closing values a flux along axis d uses.
#pragma once
#include <hip/hip_runtime.h>
#include <cmath>
#include <type_traits>

namespace mx {

#define MX_HD __host__ __device__ __forceinline__

// Hides a value's origin from the device compiler; no instruction is emitted and host code
// is unchanged.  A reverse that reads the laundered copy recomputes the forward intermediates
// it needs where it needs them, instead of the compiler sharing them with an earlier forward
// evaluation (or hoisting them) and keeping them live across the whole reverse.  Compile-time
// constants (the z-odd zeros of a planar run) are left as they are, so that they still fold.
template <class T> MX_HD void opaque(T& x) {
#if defined(__HIP_DEVICE_COMPILE__)
  if (!__builtin_constant_p(x)) asm volatile("" : "+v"(x));
#else
  (void)x;
#endif
}

// storage index of symmetric (i, j): xx xy xz yy yz zz
MX_HD constexpr int sidx(int i, int j) {
  return (i == j) ? (i == 0 ? 0 : (i == 1 ? 3 : 5))
                  : ((i + j) == 1 ? 1 : ((i + j) == 2 ? 2 : 4));
}

template <class T> MX_HD T sq(T a) { return a * a; }
// a * b + c: one rounding for the real types (fused multiply-add), the plain expression for
// the host's counting and dual-number types
template <class T> MX_HD T tfma(T a, T b, T c) { return a * b + c; }
template <> MX_HD double tfma<double>(double a, double b, double c) { return __builtin_fma(a, b, c); }
template <> MX_HD float tfma<float>(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
// the same with one rounding on the device only: the plain expression on the host
template <class T> MX_HD T dfma(T a, T b, T c) { return a * b + c; }
#if defined(__HIP_DEVICE_COMPILE__)
template <> MX_HD double dfma<double>(double a, double b, double c) { return __builtin_fma(a, b, c); }
template <> MX_HD float dfma<float>(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
#endif
template <class T> MX_HD T tmax(T a, T b) { return a > b ? a : b; }
template <class T> MX_HD T tmin(T a, T b) { return a < b ? a : b; }
template <class T> MX_HD T tabs(T a) { return a < T(0) ? -a : a; }
#if defined(__HIP_DEVICE_COMPILE__)
// on the device: clearing the sign bit is one instruction where the compare and select take
// three; it also maps -0 to +0, so a magnitude (a CFL rate reduced as a positive bit pattern)
// is never negative zero
template <> MX_HD double tabs<double>(double a) { return __builtin_fabs(a); }
template <> MX_HD float tabs<float>(float a) { return __builtin_fabsf(a); }
#endif

// FP64 square root, reciprocal and quotient.  On the device: the hardware reciprocal /
// reciprocal-square-root seed (measured on 4M samples: 4.6e-8 and 5.2e-8 relative) refined to
// the last bit.  1/b: one third-order step r <- r + r (e + e^2), e = 1 - b r (error e^3).  The
// quotient: one second-order step of the reciprocal (1e-15), then a residual correction of
// a r, which squares that error.  The square root: one step of the coupled iteration on
// g ~ sqrt(a), h ~ 1/(2 sqrt(a)) (1e-15), then a residual correction of g.  Each gives the
// correctly rounded result on those samples (1.11e-16 relative at most), as the sequences with
// one more iteration do (mrcp2 and its kin), in one (1/b), two (a/b) and three (sqrt)
// instructions less.  The arguments of the step (densities, pressures, determinants, positive
// sums) are positive and far from the exponent range's ends; sqrt(0) = 0 is kept, and a
// negative, zero-divisor or non-finite argument still gives a non-finite result, which the
// step's state check reports.  On the host: the IEEE operations.
//   mrcp2, mdiv2, msqrt2   the same with one iteration more, for the tubes (below): near 1, where a
//               quotient or root comes within 1e-32 of a tie, the shorter ones may round otherwise
//   mrsqrt      1/sqrt(a), a > 0 (1.4e-16 relative)
//   msqrt_pos   sqrt(max(a, 1e-290)): an argument that may round to zero or below; no select
//   cmax, cmin  maximum / minimum with a value that is never NaN (a NaN first operand gives
//               it, as the compare and select of tmax and tmin do): one instruction for three
#if defined(__HIP_DEVICE_COMPILE__)
MX_HD double msqrt(double a) {
  const double y = __builtin_amdgcn_rsq(a);
  double g = a * y, h = 0.5 * y;
  const double r = __builtin_fma(-g, h, 0.5);
  g = __builtin_fma(g, r, g);
  h = __builtin_fma(h, r, h);
  const double d = __builtin_fma(-g, g, a);
  const double s = __builtin_fma(d, h, g);
  return a == 0.0 ? a : s;
}
MX_HD double mrcp(double b) {
  const double r = __builtin_amdgcn_rcp(b);
  double e = __builtin_fma(-b, r, 1.0);
  e = __builtin_fma(e, e, e);
  return __builtin_fma(r, e, r);
}
MX_HD double mrcp2(double b) {
  double r = __builtin_amdgcn_rcp(b);
  r = __builtin_fma(r, __builtin_fma(-b, r, 1.0), r);
  return __builtin_fma(r, __builtin_fma(-b, r, 1.0), r);
}
MX_HD double mdiv2(double a, double b) {
  const double r = mrcp2(b);
  const double q = a * r;
  return __builtin_fma(__builtin_fma(-b, q, a), r, q);
}
MX_HD double msqrt2(double a) {
  const double y = __builtin_amdgcn_rsq(a);
  double g = a * y, h = 0.5 * y;
  double r = __builtin_fma(-g, h, 0.5);
  g = __builtin_fma(g, r, g);
  h = __builtin_fma(h, r, h);
  r = __builtin_fma(-g, h, 0.5);
  g = __builtin_fma(g, r, g);
  h = __builtin_fma(h, r, h);
  const double s = __builtin_fma(__builtin_fma(-g, g, a), h, g);
  return a == 0.0 ? a : s;
}
MX_HD double mdiv(double a, double b) {
  double r = __builtin_amdgcn_rcp(b);
  r = __builtin_fma(r, __builtin_fma(-b, r, 1.0), r);
  const double q = a * r;
  return __builtin_fma(__builtin_fma(-b, q, a), r, q);
}
MX_HD double mrsqrt(double a) {
  const double y = __builtin_amdgcn_rsq(a);
  const double e = __builtin_fma(-(a * y), y, 1.0);
  return __builtin_fma(__builtin_fma(0.375, e, 0.5) * e, y, y);
}
MX_HD double cmax(double a, double b) { return __builtin_fmax(a, b); }
MX_HD double cmin(double a, double b) { return __builtin_fmin(a, b); }
MX_HD double msqrt_pos(double x) {
  const double a = cmax(x, 1e-290);
  const double y = __builtin_amdgcn_rsq(a);
  double g = a * y, h = 0.5 * y;
  const double r = __builtin_fma(-g, h, 0.5);
  g = __builtin_fma(g, r, g);
  h = __builtin_fma(h, r, h);
  return __builtin_fma(__builtin_fma(-g, g, a), h, g);
}
#else
MX_HD double msqrt(double a) { return sqrt(a); }
MX_HD double mrcp(double b) { return 1.0 / b; }
MX_HD double mrcp2(double b) { return 1.0 / b; }
MX_HD double mdiv2(double a, double b) { return a / b; }
MX_HD double msqrt2(double a) { return sqrt(a); }
MX_HD double mdiv(double a, double b) { return a / b; }
MX_HD double mrsqrt(double a) { return 1.0 / sqrt(a); }
#endif
template <class T> MX_HD T mrcp(T b) { return T(1) / b; }
template <class T> MX_HD T mrcp2(T b) { return T(1) / b; }
template <class T> MX_HD T mdiv2(T a, T b) { return a / b; }
template <class T> MX_HD T mdiv(T a, T b) { return a / b; }
template <class T> MX_HD T mrsqrt(T a) { return T(1) / msqrt(a); }
template <class T> MX_HD T cmax(T a, T b) { return tmax(a, b); }
template <class T> MX_HD T cmin(T a, T b) { return tmin(a, b); }
template <class T> MX_HD T msqrt_pos(T a) { return msqrt(tmax(a, T(1e-290))); }
MX_HD double mexp(double a) { return exp(a); }
MX_HD double mlog(double a) { return log(a); }
// single precision: the hardware square root / exponential / logarithm (about 1 ulp)
#if defined(__HIP_DEVICE_COMPILE__)
MX_HD float msqrt(float a) { return __builtin_amdgcn_sqrtf(a); }
MX_HD float mexp(float a) { return __expf(a); }
MX_HD float mlog(float a) { return __logf(a); }
#else
MX_HD float msqrt(float a) { return sqrtf(a); }
MX_HD float mexp(float a) { return expf(a); }
MX_HD float mlog(float a) { return logf(a); }
#endif

template <class T> MX_HD T msqrt2(T a) { return msqrt(a); }

// symmetric 3x3 (6 stored) times vector
template <class T> MX_HD void symv(const T* S, const T* x, T* y) {
  y[0] = S[0] * x[0] + S[1] * x[1] + S[2] * x[2];
  y[1] = S[1] * x[0] + S[3] * x[1] + S[4] * x[2];
  y[2] = S[2] * x[0] + S[4] * x[1] + S[5] * x[2];
}

// product of two commuting-symmetric matrices stored as 6 (result symmetric): A*A
template <class T> MX_HD void symsq(const T* A, T* B) {
  B[0] = A[0] * A[0] + A[1] * A[1] + A[2] * A[2];
  B[1] = A[0] * A[1] + A[1] * A[3] + A[2] * A[4];
  B[2] = A[0] * A[2] + A[1] * A[4] + A[2] * A[5];
  B[3] = A[1] * A[1] + A[3] * A[3] + A[4] * A[4];
  B[4] = A[1] * A[2] + A[3] * A[4] + A[4] * A[5];
  B[5] = A[2] * A[2] + A[4] * A[4] + A[5] * A[5];
}

// adjugate of a symmetric matrix and its determinant
template <class T> MX_HD T symadj(const T* A, T* C) {
  C[0] = A[3] * A[5] - A[4] * A[4];
  C[1] = A[2] * A[4] - A[1] * A[5];
  C[2] = A[1] * A[4] - A[2] * A[3];
  C[3] = A[0] * A[5] - A[2] * A[2];
  C[4] = A[1] * A[2] - A[0] * A[4];
  C[5] = A[0] * A[3] - A[1] * A[1];
  return A[0] * C[0] + A[1] * C[1] + A[2] * C[2];
}

// rho > 0 and the pressure tensor positive definite (leading principal minors)
template <class T> MX_HD bool spd_ok(T rho, const T* P) {
  T m2 = P[0] * P[3] - P[1] * P[1];
  T m3 = P[0] * (P[3] * P[5] - P[4] * P[4]) - P[1] * (P[1] * P[5] - P[4] * P[2]) +
         P[2] * (P[1] * P[4] - P[3] * P[2]);
  return (rho > T(0)) && (P[0] > T(0)) && (m2 > T(0)) && (m3 > T(0));
}

// positive root of the mapping quadratic, cancellation-free for A < 0
template <class T> MX_HD T sigma_root(T A, T X, T num_small, T denom_big) {
  T sX = msqrt2(X);
  return (A >= T(0)) ? mdiv2(A + sX, denom_big) : mdiv2(num_small, sX - A);
}

// zeta + sqrt(max(0, zeta^2 + rest)), cancellation-free for zeta < 0
template <class T> MX_HD T hyperbola(T zeta, T rest) {
  T X = zeta * zeta + rest;
  if (!(X > T(0))) return zeta;
  T sX = msqrt2(X);
  return (zeta >= T(0)) ? zeta + sX : mdiv2(rest, sX - zeta);
}

// Baradaran's B, Y, E, C at sigma_w and the normal pressure P*_dd
template <class T> struct BYEC { T B, Y, E, C; };
template <class T> MX_HD BYEC<T> byec(T sw, T Pdd) {
  BYEC<T> r;
  r.C = msqrt2(tmax((T(3) - T(3) * sw) * Pdd, T(0)));
  r.E = T(0.8) * r.C;
  T rs = msqrt2(sw);
  r.B = T(5) - T(4) * rs + msqrt2(tmax(T(10) - T(16) * rs + T(6) * sw, T(0)));
  r.Y = r.B + r.E * r.E - T(2) * r.E * msqrt2(r.B);
  return r;
}

// Tubes.  A system with TUBE (1D: Sys14A, Sys5) has every FP64 rounding of its stages fixed: the operations
// stand in the order of the formulas and the fused ones are written out, with contraction off (left to
// the compiler, it is chosen by what surrounds an expression, and kernels differ).  The front of a
// Riemann problem runs into uniform states, where the jumps fall, cell by cell, through the
// neutral threshold of the common limiter; a rounding that leaves one on the other side of it changes
// that cell's slopes.  Measured on Sod tubes of 200 cells from 2500 pairs of states, 20 steps: the
// face state in the algebra of Sys14::Norm gives results more than 1e-9 (2-norm) or 4e-8
// (largest value) from these for 16 of them (SSP-RK2, minmod), 26 (van Albada), 66 (midpoint,
// Rusanov) and 140 (point-implicit), by 5e-4 at most.  So a tube keeps one set of roundings, in
// one lane or two, alone or in a batch.  (Without a limiter the 5-moment system is no calmer:
// collisionless at sigma_lim = 1e-2, the CFL step follows near-Junk cells and collapses in 4 to 5
// of 100 roundings of the same formulas.)  That algebra would be faster: 20 steps of 20000 cells 372
// us against 449, 512 tubes 9.5 ms against 13.3, 40 steps of 1000 5-moment cells 302 us against 344.
//
// A tube's sigma_root and hyperbola(+-q), with the fused operations written out and the two
// cases of each picked by selects, so that lanes of both cases share one division:
//   zeta = +-q, rest = -0.8 zeta sigma_w C + 4 sigma_w^2 Y
template <class T> MX_HD T tube_sigma(T A, T X, T D2, T t4) {
#pragma clang fp contract(off)
  const T big = tabs(A) + msqrt2(X);
  const bool pos = A >= T(0);
  return mdiv2(pos ? big : D2, pos ? t4 : big);
}
template <class T> MX_HD void tube_roots(T q, T sw, T C, T Y, T& hmax, T& hmin) {
#pragma clang fp contract(off)
  const T s2 = T(4) * sw * sw;
  const T e = T(0.8) * q * sw * C;
  const T rmax = dfma(s2, Y, -e), rmin = e + s2 * Y;
  const T Xmax = dfma(q, q, rmax), Xmin = q * q + rmin;
  const T smax = msqrt2(Xmax), smin = msqrt2(Xmin);
  const T aq = tabs(q);
  const bool fwd = q >= T(0);
  const T sp = fwd ? smax : smin, sn = fwd ? smin : smax;   // of zeta >= 0, and of the other
  const T hp = aq + sp;
  const T hn = (aq == T(0)) ? sn : mdiv2(fwd ? rmin : rmax, aq + sn);
  hmax = (Xmax > T(0)) ? (fwd ? hp : hn) : q;
  hmin = (Xmin > T(0)) ? (fwd ? hn : hp) : -q;
}

// The two factors of the wave-speed fit that depend on the normal pressure alone,
// a = 1.4 P^1.1 exp(-P^2) and b = 0.9 P exp(-P^1.4 / 2), zero for P <= 0.
// P04 = P^0.4 (their derivatives need it).
template <class T> MX_HD void fit_ab(T P, T& a, T& b, T& P04) {
  a = T(0); b = T(0); P04 = T(0);
  if (P > T(0)) {
    T lP = mlog(P);
    P04 = mexp(T(0.4) * lP);
    a = T(1.4) * mexp(T(1.1) * lP - P * P);
    b = T(0.9) * P * mexp(T(-0.5) * (P * P04));
  }
}
#if defined(__HIP_DEVICE_COMPILE__)
// On the device, FP64: no logarithm and two exponentials instead of three.  u = P^-0.1 from
// the single-precision logarithm and exponential units; P u^10 = 1 + d with |d| < 1e-5, so
//   P^0.1 = P u^9 (1 + d)^-0.9,   P^0.4 = P u^6 (1 + d)^-0.6
// with both powers of 1 + d to second order (the next term is below 1e-16).  The
// exponentials: argument k ln 2 + r, |r| <= 0.347, a polynomial of degree 11 in r (interpolated
// at the Chebyshev points of (e^r - 1 - r) / r^2, 1.6e-17 relative).  For exp(-P^2) the
// reduction subtracts k ln 2 (its upper part of 38 bits, so that the product is exact) from
// the unrounded square.  Against 80-bit evaluation on 4M samples: a 6.8e-16 at most and
// 1.2e-16 on average, b 1.1e-15 and 1.0e-16 (the logarithm and exponentials of the math
// library in the formulas above: 4.2e-15, 4.0e-16 and 1.2e-15, 1.1e-16, part of it the rounding
// of the exponents 1.1 and 1.4).  P is at most 3 for a positive definite pressure tensor; above
// 32 a is zero and b below 1e-26, so the clamp changes nothing that reaches a wave speed.
MX_HD double exp_reduced(double k, double r) {
  double p = 2.5100472505694996e-08;
  p = __builtin_fma(p, r, 2.7620201591031547e-07);
  p = __builtin_fma(p, r, 2.7557268275905696e-06);
  p = __builtin_fma(p, r, 2.4801521057868204e-05);
  p = __builtin_fma(p, r, 0.00019841269863171557);
  p = __builtin_fma(p, r, 0.0013888888917367081);
  p = __builtin_fma(p, r, 0.008333333333330039);
  p = __builtin_fma(p, r, 0.041666666666623824);
  p = __builtin_fma(p, r, 0.16666666666666669);
  p = __builtin_fma(p, r, 0.5);
  return __builtin_ldexp(1.0 + __builtin_fma(r * r, p, r), (int)k);
}
MX_HD void fit_ab(double Pin, double& a, double& b, double& P04) {
  const double P = cmin(Pin, 32.0);
  const float pf = __builtin_fmaxf((float)P, 1e-30f);
  const double u = (double)__builtin_amdgcn_exp2f(-0.1f * __builtin_amdgcn_logf(pf));
  const double u2 = u * u, u4 = u2 * u2, u6 = u4 * u2, u8 = u4 * u4, u9 = u8 * u, u10 = u8 * u2;
  const double d = __builtin_fma(P, u10, -1.0);
  const double w9 = d * __builtin_fma(0.855, d, -0.9), w6 = d * __builtin_fma(0.48, d, -0.6);
  const double PP = P * P;
  const double v6 = __builtin_fma(u6, w6, u6);
  const double P11 = PP * __builtin_fma(u9, w9, u9), P14 = PP * v6;
  P04 = P * v6;
  const double ka = __builtin_rint(PP * -1.4426950408889634);
  double ra = __builtin_fma(-P, P, ka * -0x1.62e42fefa0000p-1);
  ra = __builtin_fma(ka, -1.6465949582897082e-12, ra);
  const double x = -0.5 * P14;
  const double kb = __builtin_rint(x * 1.4426950408889634);
  double rb = __builtin_fma(kb, -0.6931471805599453, x);
  rb = __builtin_fma(kb, -2.3190468138462996e-17, rb);
  a = 1.4 * P11 * exp_reduced(ka, ra);
  b = 0.9 * P * exp_reduced(kb, rb);
}
#endif

// The part of the wave-speed fit that depends on sigma_bar alone (rsb, isb: its square root and
// reciprocal): 1 - sigma_w, 1/sigma_w, 2 sigma_w and sqrt(B), sigma_w = min(sigma_bar, 1).
// 10 - 16 r + 6 r^2 = 2 (1 - r)(5 - 3 r) with r = sqrt(sigma_w).
template <class T> struct SigmaFit { T om, isw, sw2, sB; };
template <class T> MX_HD void sigma_fit(T sb, T rsb, T isb, SigmaFit<T>& f) {
  const T sw = cmin(sb, T(1)), r = cmin(rsb, T(1));
  f.om = T(1) - sw;
  f.isw = cmax(isb, T(1));
  f.sw2 = T(2) * sw;
  f.sB = msqrt_pos(T(5) - T(4) * r + msqrt_pos(T(2) * (T(1) - r) * (T(5) - T(3) * r)));
}

// Both approximate wave speeds along one direction (Section 5.1) from the dimensionless normal
// pressure P >= 0, normal and transverse heat flux; kc = k_ws c.  With Y = (sqrt(B) - E)^2 and
// zeta = +-q_d + |q_t| alpha the fit is
//   Lambda = pref (zeta + sqrt(zeta^2 - zeta sigma_w E + (2 sigma_w (sqrt(B) - E))^2 + q_t^2/10)) + E.
// alpha > 0, so of the two zeta only the smaller can be negative, and only it needs the
// cancellation-free form rest / (sqrt(X) - zeta): one division instead of two.
template <class T>
MX_HD void wave_roots(const SigmaFit<T>& f, T pref, T E, T qd, T qt, T alpha, T ud, T kc, T& lmin, T& lmax) {
  const T D = f.sw2 * (f.sB - E);
  const T g = T(0.5) * f.sw2 * E;
  const T aq = tabs(qd);
  const T w = qt * alpha;
  const T base = tfma(T(0.1), qt * qt, D * D);
  const T zp = w + aq, zn = w - aq;
  // (tfma: which products are fused must not depend on the kernel around)
  const T hp = zp + msqrt_pos(tfma(zp, zp - g, base));
  const T rest = tfma(-zn, g, base);
  const T sn = msqrt_pos(tfma(zn, zn, rest)) + tabs(zn);
  T hn = mdiv(rest, sn);
  hn = (zn >= T(0)) ? sn : hn;
  const T Lp = tfma(pref, hp, E), Ln = tfma(pref, hn, E);
  const bool fwd = qd >= T(0);
  const T Lmax = fwd ? Lp : Ln, Lmin = fwd ? Ln : Lp;
  lmax = tfma(kc, Lmax, ud);
  lmin = tfma(-kc, Lmin, ud);
}
template <class T>
MX_HD void wave_pair(const SigmaFit<T>& f, T P, T qd, T qt, T ud, T kc, T& lmin, T& lmax) {
  T a, b, P04;
  fit_ab(P, a, b, P04);
  wave_roots(f, T(0.5) * tfma(b, f.isw, a), T(0.8) * msqrt_pos(T(3) * f.om * P), qd, qt,
                         T(0.6) * P * P - T(0.38) * P + T(0.35), ud, kc, lmin, lmax);
}

// sigma (sigma_root's two forms, the magnitude |A| + sqrt(X) shared), sigma_bar, its reciprocal
// and square root
template <class T> struct SigmaBar { T sig, sb, isb, rsb; };
template <class T> MX_HD void sigma_bar(T A, T D, T t2, T sigma_lim, SigmaBar<T>& s) {
  const T big = tabs(A) + msqrt(tfma(A, A, T(8) * (t2 * D)));
  const bool pos = A >= T(0);
  s.sig = mdiv(pos ? big : T(2) * D, pos ? T(4) * t2 : big);
  s.sb = cmax(s.sig, sigma_lim);
  s.isb = mrcp(s.sb);
  s.rsb = msqrt_pos(s.sb);
}

// ===================================================================== 14 moments
struct Sys14 {
  static constexpr int NV = 14;
  static constexpr bool TUBE = false;
  static constexpr bool JETS = true;       // jet inflow boundaries apply
  MX_HD static constexpr int plane_of(int v) { return v; }   // storage plane of moment v
  template <class T> MX_HD static void from14(const T* W14, T* W) {
#pragma unroll
    for (int v = 0; v < 14; ++v) W[v] = W14[v];
  }

  template <class T> MX_HD static void cons_to_prim(const T* U, T* W) {
    T rho = U[0];
    T ir = mrcp2(rho);
    T u[3] = {U[1] * ir, U[2] * ir, U[3] * ir};
    T P[6];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = i; j < 3; ++j) P[sidx(i, j)] = U[4 + sidx(i, j)] - rho * (u[i] * u[j]);
    T uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    T trP = P[0] + P[3] + P[5];
    T Pu[3];
    symv(P, u, Pu);
    T q[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) q[i] = U[10 + i] - (rho * uu) * u[i] - trP * u[i] - T(2) * Pu[i];
    T uPu = u[0] * Pu[0] + u[1] * Pu[1] + u[2] * Pu[2];
    T uq = u[0] * q[0] + u[1] * q[1] + u[2] * q[2];
    W[0] = rho;
    W[1] = u[0]; W[2] = u[1]; W[3] = u[2];
#pragma unroll
    for (int k = 0; k < 6; ++k) W[4 + k] = P[k];
    W[10] = q[0]; W[11] = q[1]; W[12] = q[2];
    W[13] = U[13] - rho * uu * uu - T(2) * uu * trP - T(4) * uPu - T(4) * uq;
  }

  template <class T> MX_HD static void prim_to_cons(const T* W, T* U) {
    T rho = W[0];
    const T* u = W + 1;
    const T* P = W + 4;
    const T* q = W + 10;
    T uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    T trP = P[0] + P[3] + P[5];
    T Pu[3];
    symv(P, u, Pu);
    T uPu = u[0] * Pu[0] + u[1] * Pu[1] + u[2] * Pu[2];
    T uq = u[0] * q[0] + u[1] * q[1] + u[2] * q[2];
    U[0] = rho;
    U[1] = rho * u[0]; U[2] = rho * u[1]; U[3] = rho * u[2];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = i; j < 3; ++j) U[4 + sidx(i, j)] = rho * (u[i] * u[j]) + P[sidx(i, j)];
#pragma unroll
    for (int i = 0; i < 3; ++i) U[10 + i] = (rho * uu) * u[i] + trP * u[i] + T(2) * Pu[i] + q[i];
    U[13] = rho * uu * uu + T(2) * uu * trP + T(4) * uPu + T(4) * uq + W[13];
  }

  template <class T> MX_HD static T pressure(const T* W) { return (W[4] + W[7] + W[9]) * T(1.0 / 3.0); }

  template <class T> MX_HD static bool admissible(const T* W) { return spd_ok(W[0], W + 4); }
  // the primitives admissible() reads: rho and the pressure tensor
  MX_HD static constexpr bool admissibility_var(int v) { return v == 0 || (v >= 4 && v < 10); }
  // admissible(cons_to_prim(U)) without recovering q and R (the same expressions for rho, u, P)
  template <class T> MX_HD static bool admissible_cons(const T* U) {
    T rho = U[0];
    T ir = mrcp(rho);
    T u[3] = {U[1] * ir, U[2] * ir, U[3] * ir};
    T P[6];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = i; j < 3; ++j) P[sidx(i, j)] = U[4 + sidx(i, j)] - rho * (u[i] * u[j]);
    return spd_ok(rho, P);
  }

  // natural scale of each primitive (rho, c, p, rho c^3 = p c, rho c^4 = p^2 / rho) for the neutral-variable
  // test of the common limiter
  template <class T> MX_HD static void scales(const T* W, T* sc) {
    T rho = tabs(W[0]);
    T p = tabs(W[4] + W[7] + W[9]) * T(1.0 / 3.0);
    T T0 = p * mrcp(rho);
    T c = T0 * mrsqrt(T0);
    sc[0] = rho;
    sc[1] = sc[2] = sc[3] = c;
#pragma unroll
    for (int k = 4; k < 10; ++k) sc[k] = p;
    sc[10] = sc[11] = sc[12] = p * c;
    sc[13] = p * T0;
  }

  // components odd under reflection of axis d
  MX_HD static constexpr bool odd(int v, int d) {
    return (v == 1 + d) || (v == 10 + d) ||
           (v >= 4 && v < 10 && ((d == 0 && (v == 5 || v == 6)) || (d == 1 && (v == 5 || v == 8)) ||
                                 (d == 2 && (v == 6 || v == 8))));
  }

  // Dimensionless state, sigma and P^-1 q.
  template <class T> struct Core {
    T rho, c, Ph[6], qh[3], z[3], P2[6], t1, t2, A, sig, sb;
  };

  template <class T> MX_HD static void core(const T* W, T sigma_lim, Core<T>& k) {
    k.rho = W[0];
    T p = (W[4] + W[7] + W[9]) * T(1.0 / 3.0);
    T irho = mrcp2(k.rho);
    T ip = mrcp2(p);
    k.c = msqrt2(p * irho);
    T ic = msqrt2(k.rho * ip);          // 1 / c
#pragma unroll
    for (int m = 0; m < 6; ++m) k.Ph[m] = W[4 + m] * ip;
    T is3 = irho * (ic * ic * ic);     // 1 / (rho c^3)
#pragma unroll
    for (int i = 0; i < 3; ++i) k.qh[i] = W[10 + i] * is3;
    T Rh = W[13] * (is3 * ic);
    k.t1 = k.Ph[0] + k.Ph[3] + k.Ph[5];
    symsq(k.Ph, k.P2);
    k.t2 = k.P2[0] + k.P2[3] + k.P2[5];
    T C[6];
    T det = symadj(k.Ph, C);
    T idet = mrcp2(det);
    T y[3];
    symv(C, k.qh, y);
#pragma unroll
    for (int i = 0; i < 3; ++i) k.z[i] = y[i] * idet;
    T D = k.qh[0] * k.z[0] + k.qh[1] * k.z[1] + k.qh[2] * k.z[2];
    T A = T(2) * k.t2 + k.t1 * k.t1 - Rh;
    T X = A * A + T(8) * k.t2 * D;
    k.A = A;
    k.sig = sigma_root(A, X, T(2) * D, T(4) * k.t2);
    k.sb = tmax(k.sig, sigma_lim);
  }

  // Mixed precision core: the bracket A = 2 tr(P*^2) + tr(P*)^2 - R* of the sigma mapping
  // cancels near equilibrium (R* ~ 15 against A ~ 0), and the wave speeds scale like
  // 1/sigma, so A and the traces it needs are formed in FP64; the rest in FP32.
  MX_HD static void core_mixed(const double* W, float sigma_lim, Core<float>& k) {
    double p = (W[4] + W[7] + W[9]) * (1.0 / 3.0);
    double ip = mrcp(p);
    double Ph[6], P2[6];
#pragma unroll
    for (int m = 0; m < 6; ++m) Ph[m] = W[4 + m] * ip;
    symsq(Ph, P2);
    double t1 = Ph[0] + Ph[3] + Ph[5];
    double t2 = P2[0] + P2[3] + P2[5];
    double A = 2.0 * t2 + t1 * t1 - W[13] * W[0] * ip * ip;
    k.rho = (float)W[0];
    float irho = 1.0f / k.rho;
    float ipf = (float)ip;
    k.c = msqrt((float)p * irho);
    float ic = msqrt(k.rho * ipf);
#pragma unroll
    for (int m = 0; m < 6; ++m) { k.Ph[m] = (float)Ph[m]; k.P2[m] = (float)P2[m]; }
    k.t1 = (float)t1;
    k.t2 = (float)t2;
    k.A = (float)A;
    float is3 = irho * (ic * ic * ic);
#pragma unroll
    for (int i = 0; i < 3; ++i) k.qh[i] = (float)W[10 + i] * is3;
    float C[6];
    float det = symadj(k.Ph, C);
    float idet = 1.0f / det;
    float y[3];
    symv(C, k.qh, y);
#pragma unroll
    for (int i = 0; i < 3; ++i) k.z[i] = y[i] * idet;
    float D = k.qh[0] * k.z[0] + k.qh[1] * k.z[1] + k.qh[2] * k.z[2];
    float X = k.A * k.A + 8.0f * k.t2 * D;
    k.sig = sigma_root(k.A, X, 2.0f * D, 4.0f * k.t2);
    k.sb = tmax(k.sig, sigma_lim);
  }

  // Closing values used by a flux along axis d: Q_ijd (6), R_id(kk) (3), S_d(jjkk),
  // dimensional.
  template <int d, class T>
  MX_HD static void closure_dir(const Core<T>& k, T* Qd, T* Rd, T& Sd) {
    T Cm[6];
#pragma unroll
    for (int m = 0; m < 6; ++m) Cm[m] = T(4) * k.P2[m];
    Cm[0] += T(2) * k.t2; Cm[3] += T(2) * k.t2; Cm[5] += T(2) * k.t2;
    T Ca[6];
    T detc = symadj(Cm, Ca);
    T y[3];
    symv(Ca, k.qh, y);
    T idc = mrcp(detc);
    T w[3] = {y[0] * idc, y[1] * idc, y[2] * idc};
    T P2z[3];
    symv(k.P2, k.z, P2z);
    T zP2z = k.z[0] * P2z[0] + k.z[1] * P2z[1] + k.z[2] * P2z[2];
    T wz = w[0] * k.z[0] + w[1] * k.z[1] + w[2] * k.z[2];
    T s3 = k.rho * (k.c * k.c * k.c);
    T s4 = s3 * k.c;
    T s5 = s4 * k.c;
    // Q_ijd
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = i; j < 3; ++j)
        Qd[sidx(i, j)] = T(2) * (w[i] * k.P2[sidx(j, d)] + w[j] * k.P2[sidx(i, d)] +
                                 w[d] * k.P2[sidx(i, j)]) * s3;
    // R_id(kk)
    T isb = mrcp(k.sb);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      T Qz = T(2) * (w[i] * P2z[d] + w[d] * P2z[i] + wz * k.P2[sidx(i, d)]);
      Rd[i] = (Qz * isb + T(2) * (T(1) - k.sb) * k.P2[sidx(i, d)] + k.t1 * k.Ph[sidx(i, d)]) * s4;
    }
    // S_d
    T Pw[3], P2w[3], P3w_d;
    symv(k.Ph, w, Pw);
    symv(k.P2, w, P2w);
    T t3 = k.P2[0] * k.Ph[0] + k.P2[3] * k.Ph[3] + k.P2[5] * k.Ph[5] +
           T(2) * (k.P2[1] * k.Ph[1] + k.P2[2] * k.Ph[2] + k.P2[4] * k.Ph[4]);
    P3w_d = k.P2[sidx(d, 0)] * Pw[0] + k.P2[sidx(d, 1)] * Pw[1] + k.P2[sidx(d, 2)] * Pw[2];
    T t1 = k.t1, t2 = k.t2;
    T Wq = (T(2) * t1 * t1 * t1 + T(12) * t3 - T(2) * t2 * t1) * w[d] +
           (T(14) * t2 - T(6) * t1 * t1) * Pw[d] + T(20) * t1 * P2w[d] + T(20) * P3w_d;
    T Qzz = T(2) * (w[d] * zP2z + T(2) * wz * P2z[d]);
    T rsb = msqrt(k.sb);
    Sd = (Qzz * (isb * isb) + T(2) * rsb * t1 * k.qh[d] + (T(1) - rsb) * Wq) * s5;
  }

  // Physical flux along d (14 components) from primitives and closing values.
  template <int d, class T>
  MX_HD static void flux(const T* W, const T* Qd, const T* Rd, T Sd, T* F) {
    T rho = W[0];
    const T* u = W + 1;
    const T* P = W + 4;
    const T* q = W + 10;
    T ud = u[d];
    T uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    T trP = P[0] + P[3] + P[5];
    T Pd[3] = {P[sidx(0, d)], P[sidx(1, d)], P[sidx(2, d)]};
    T uPd = u[0] * Pd[0] + u[1] * Pd[1] + u[2] * Pd[2];
    T Pu[3];
    symv(P, u, Pu);
    T uPu = u[0] * Pu[0] + u[1] * Pu[1] + u[2] * Pu[2];
    T uq = u[0] * q[0] + u[1] * q[1] + u[2] * q[2];
    T Qu[3];
    symv(Qd, u, Qu);
    T uQu = u[0] * Qu[0] + u[1] * Qu[1] + u[2] * Qu[2];
    T uR = u[0] * Rd[0] + u[1] * Rd[1] + u[2] * Rd[2];
    T rud = rho * ud;
    F[0] = rud;
#pragma unroll
    for (int i = 0; i < 3; ++i) F[1 + i] = rud * u[i] + Pd[i];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = i; j < 3; ++j)
        F[4 + sidx(i, j)] = rud * (u[i] * u[j]) + u[i] * Pd[j] + u[j] * Pd[i] + ud * P[sidx(i, j)] +
                            Qd[sidx(i, j)];
#pragma unroll
    for (int i = 0; i < 3; ++i)
      F[10 + i] = (rud * uu) * u[i] + (ud * trP) * u[i] + T(2) * uPd * u[i] + T(2) * ud * Pu[i] +
                  uu * Pd[i] + u[i] * q[d] + ud * q[i] + T(2) * Qu[i] + Rd[i];
    F[13] = rud * uu * uu + T(2) * ud * uu * trP + T(4) * uu * uPd + T(4) * ud * uPu +
            T(2) * uu * q[d] + T(4) * ud * uq + T(4) * uQu + T(4) * uR + ud * W[13] + Sd;
  }

  // Approximate minimum / maximum wave speed along d (Section 5.1).
  template <int d, class T>
  MX_HD static void wavespeeds(const Core<T>& k, T ud, T kws, T& lmin, T& lmax) {
    constexpr int t1i = (d == 0) ? 1 : 0;
    constexpr int t2i = (d == 2) ? 1 : 2;
    if constexpr (!std::is_same<T, float>::value) {
      SigmaFit<T> f;
      sigma_fit(k.sb, msqrt_pos(k.sb), mrcp(k.sb), f);
      wave_pair(f, cmax(k.Ph[sidx(d, d)], T(0)), k.qh[d],
                      msqrt_pos(k.qh[t1i] * k.qh[t1i] + k.qh[t2i] * k.qh[t2i]), ud, kws * k.c, lmin, lmax);
    } else {
      wavespeeds_formula<d>(k, ud, kws, lmin, lmax);
    }
  }
  // the fit as the formulas stand (single precision, and the first CFL rate of a loaded 1D field)
  template <int d, class T>
  MX_HD static void wavespeeds_formula(const Core<T>& k, T ud, T kws, T& lmin, T& lmax) {
    constexpr int t1i = (d == 0) ? 1 : 0;
    constexpr int t2i = (d == 2) ? 1 : 2;
    T sw = tmin(k.sb, T(1));
    T Pdd = tmax(k.Ph[sidx(d, d)], T(0));
    T qd = k.qh[d];
    T qt = msqrt2(k.qh[t1i] * k.qh[t1i] + k.qh[t2i] * k.qh[t2i]);
    T alpha = T(0.6) * Pdd * Pdd - T(0.38) * Pdd + T(0.35);
    T a = T(0), b = T(0);
    if (Pdd > T(0)) {
      T lP = mlog(Pdd);
      a = T(1.4) * mexp(T(1.1) * lP - Pdd * Pdd);
      b = T(0.9) * Pdd * mexp(T(-0.5) * mexp(T(1.4) * lP));
    }
    BYEC<T> g = byec(sw, Pdd);
    T pref = mdiv2(a * sw + b, T(2) * sw);
    T base = T(4) * sw * sw * g.Y + qt * qt * T(0.1);
    T zmax = qd + qt * alpha;
    T zmin = -qd + qt * alpha;
    T Lmax = pref * hyperbola(zmax, T(-0.8) * zmax * sw * g.C + base) + g.E;
    T Lmin = pref * hyperbola(zmin, T(-0.8) * zmin * sw * g.C + base) + g.E;
    lmax = ud + kws * Lmax * k.c;
    lmin = ud - kws * Lmin * k.c;
  }

  // Dimensionless state of the flux and wave speeds in FP64: P* = P / p, P*^2, h = q / p = c q*,
  // z = P*^-1 h, T = p / rho, 1/c, sigma_bar.  Dimensional closing values follow from these
  // without powers of c: with v = (2 P*^2 + tr(P*^2) I)^-1 q (v = 2 rho c^3 w),
  //   Q_ijd = v_i (P*^2)_jd + v_j (P*^2)_id + v_d (P*^2)_ij,
  //   R_id  = (v_i (P* h)_d + v_d (P* h)_i + (v.z)(P*^2)_id) / sigma
  //           + 2 (1 - sigma) p T (P*^2)_id + 3 T P_id,
  //   S_d   = (v_d |P* z|^2 + 2 (v.z)(P* h)_d) / sigma^2
  //           + T (6 sqrt(sigma) q_d + (1 - sqrt(sigma)) Wq),
  // since P*^2 z = P* h, z.P*^2 z = h.h and tr P* = 3.  Wq is (2 t1^3 + 12 t3 - 2 t2 t1) w_d + ...
  // with P*^3 and t3 = tr(P*^3) eliminated by the Cayley-Hamilton theorem:
  //   Wq = (24 t2 - 54 + 28 det P*) v_d + (12 t2 - 72) (P* v)_d + 60 (P*^2 v)_d.
  template <class T> struct Norm {
    T trP, pT, T0, ic, kc, Ph[6], h[3], z[3], P2[6], t2, det;
    SigmaBar<T> s;
  };
  template <class T> MX_HD static void norm(const T* W, T sigma_lim, T kws, Norm<T>& n) {
    n.trP = W[4] + W[7] + W[9];
    const T p = n.trP * T(1.0 / 3.0);
    const T ip = mrcp(p);
    n.T0 = p * mrcp(W[0]);
    n.pT = p * n.T0;
    n.ic = mrsqrt(n.T0);
    const T ic2 = W[0] * ip;
    n.kc = kws * (n.T0 * n.ic);
#pragma unroll
    for (int m = 0; m < 6; ++m) n.Ph[m] = W[4 + m] * ip;
#pragma unroll
    for (int i = 0; i < 3; ++i) n.h[i] = W[10 + i] * ip;
    symsq(n.Ph, n.P2);
    const T t1 = n.Ph[0] + n.Ph[3] + n.Ph[5];
    n.t2 = n.P2[0] + n.P2[3] + n.P2[5];
    T C[6], y[3];
    n.det = symadj(n.Ph, C);
    const T idet = mrcp(n.det);
    symv(C, n.h, y);
#pragma unroll
    for (int i = 0; i < 3; ++i) n.z[i] = y[i] * idet;
    const T D = (n.h[0] * n.z[0] + n.h[1] * n.z[1] + n.h[2] * n.z[2]) * ic2;
    sigma_bar(tfma(t1, t1, T(2) * n.t2) - W[13] * (ic2 * ip), D, n.t2, sigma_lim, n.s);
  }
  template <int d, class T>
  MX_HD static void speeds(const Norm<T>& n, const SigmaFit<T>& f, T ud, T& lmin, T& lmax) {
    constexpr int t1i = (d == 0) ? 1 : 0;
    constexpr int t2i = (d == 2) ? 1 : 2;
    wave_pair(f, cmax(n.Ph[sidx(d, d)], T(0)), n.h[d] * n.ic,
                    msqrt_pos(n.h[t1i] * n.h[t1i] + n.h[t2i] * n.h[t2i]) * n.ic, ud, n.kc, lmin, lmax);
  }

  // U, F_d and the wave speeds of a face state.  F is written with U: each flux is u_d U plus
  // the terms in which d is a velocity's or a tensor's second index (u_j P_jd = (P u)_d).
  template <int d, class T>
  MX_HD static void face_terms(const T* W, T sigma_lim, T kws, T* U, T* F, T& lmin, T& lmax) {
    Norm<T> n;
    norm(W, sigma_lim, kws, n);
    const T rho = W[0];
    const T* u = W + 1;
    const T* P = W + 4;
    const T* q = W + 10;
    T M[6], Ma[6], v[3];
#pragma unroll
    for (int m = 0; m < 6; ++m) M[m] = T(2) * n.P2[m];
    M[0] = M[0] + n.t2; M[3] = M[3] + n.t2; M[5] = M[5] + n.t2;
    const T idm = mrcp(symadj(M, Ma));
    symv(Ma, q, v);
#pragma unroll
    for (int i = 0; i < 3; ++i) v[i] = v[i] * idm;
    const T vz = v[0] * n.z[0] + v[1] * n.z[1] + v[2] * n.z[2];
    const T hh = n.h[0] * n.h[0] + n.h[1] * n.h[1] + n.h[2] * n.h[2];
    T Phh[3];
    symv(n.Ph, n.h, Phh);
    const T isb = n.s.isb;
    T Q[6], R[3], vs[3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = i; j < 3; ++j)
        Q[sidx(i, j)] = v[i] * n.P2[sidx(j, d)] + v[j] * n.P2[sidx(i, d)] + v[d] * n.P2[sidx(i, j)];
#pragma unroll
    for (int i = 0; i < 3; ++i) vs[i] = v[i] * isb;
    const T k2 = vz * isb + T(2) * (T(1) - n.s.sb) * n.pT;
    const T T3 = T(3) * n.T0;
#pragma unroll
    for (int i = 0; i < 3; ++i)
      R[i] = vs[i] * Phh[d] + vs[d] * Phh[i] + k2 * n.P2[sidx(i, d)] + T3 * P[sidx(i, d)];
    const T n1 = n.Ph[sidx(d, 0)] * v[0] + n.Ph[sidx(d, 1)] * v[1] + n.Ph[sidx(d, 2)] * v[2];
    const T n2 = n.P2[sidx(d, 0)] * v[0] + n.P2[sidx(d, 1)] * v[1] + n.P2[sidx(d, 2)] * v[2];
    const T Wq = (T(24) * n.t2 - T(54) + T(28) * n.det) * v[d] + (T(12) * n.t2 - T(72)) * n1 + T(60) * n2;
    const T S = (v[d] * hh + T(2) * vz * Phh[d]) * (isb * isb) +
                n.T0 * (T(6) * n.s.rsb * q[d] + (T(1) - n.s.rsb) * Wq);

    const T ud = u[d];
    const T uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    const T e = rho * uu + n.trP;
    T Pu[3], s[3], Qu[3], Rq[3];
    symv(P, u, Pu);
#pragma unroll
    for (int i = 0; i < 3; ++i) s[i] = Pu[i] + q[i];
    U[0] = rho;
#pragma unroll
    for (int i = 0; i < 3; ++i) U[1 + i] = rho * u[i];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = i; j < 3; ++j) U[4 + sidx(i, j)] = U[1 + i] * u[j] + P[sidx(i, j)];
#pragma unroll
    for (int i = 0; i < 3; ++i) U[10 + i] = e * u[i] + (s[i] + Pu[i]);
    U[13] = uu * (e + n.trP) + T(4) * (u[0] * s[0] + u[1] * s[1] + u[2] * s[2]) + W[13];
    const T m = T(2) * Pu[d] + q[d];
    symv(Q, u, Qu);
#pragma unroll
    for (int i = 0; i < 3; ++i) Rq[i] = R[i] + Qu[i];
    F[0] = U[1 + d];
#pragma unroll
    for (int i = 0; i < 3; ++i) F[1 + i] = ud * U[1 + i] + P[sidx(i, d)];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = i; j < 3; ++j)
        F[4 + sidx(i, j)] = ud * U[4 + sidx(i, j)] + (u[i] * P[sidx(j, d)] + (u[j] * P[sidx(i, d)] + Q[sidx(i, j)]));
#pragma unroll
    for (int i = 0; i < 3; ++i) F[10 + i] = ud * U[10 + i] + (u[i] * m + (uu * P[sidx(i, d)] + (Rq[i] + Qu[i])));
    F[13] = ud * U[13] + (T(2) * uu * m + (T(4) * (u[0] * Rq[0] + u[1] * Rq[1] + u[2] * Rq[2]) + S));

    SigmaFit<T> f;
    sigma_fit(n.s.sb, n.s.rsb, isb, f);
    speeds<d>(n, f, ud, lmin, lmax);
  }

  // U, F_d and the wave speeds of a face state in single precision (the FP32 setting)
  template <int d>
  MX_HD static void face_terms_fp32(const float* W, float sigma_lim, float kws, float* U, float* F, float& lmin,
                                    float& lmax) {
    Core<float> k;
    core(W, sigma_lim, k);
    float Qd[6], Rd[3], Sd;
    closure_dir<d>(k, Qd, Rd, Sd);
    flux<d>(W, Qd, Rd, Sd, F);
    prim_to_cons(W, U);
    wavespeeds<d>(k, W[1 + d], kws, lmin, lmax);
  }

  // F_d and the wave speeds from a prepared core (mixed precision path)
  template <int d, class T>
  MX_HD static void flux_speeds(const Core<T>& k, const T* W, T kws, T* F, T& lmin, T& lmax) {
    T Qd[6], Rd[3], Sd;
    closure_dir<d>(k, Qd, Rd, Sd);
    flux<d>(W, Qd, Rd, Sd, F);
    wavespeeds<d>(k, W[1 + d], kws, lmin, lmax);
  }

  // max(|lambda_min|, |lambda_max|) along d at a cell state
  template <int d, class T> MX_HD static T cell_lambda(const T* W, T sigma_lim, T kws) {
    Norm<T> n;
    norm(W, sigma_lim, kws, n);
    SigmaFit<T> f;
    sigma_fit(n.s.sb, n.s.rsb, n.s.isb, f);
    T lmin, lmax;
    speeds<d>(n, f, W[1 + d], lmin, lmax);
    return tmax(tabs(lmin), tabs(lmax));
  }

  // cell_lambda<0> of a loaded 1D field, which may be a tube: its roundings are a tube's
  template <class T> MX_HD static T tube_lambda(const T* W, T sigma_lim, T kws) {
    Core<T> k;
    core(W, sigma_lim, k);
    T lmin, lmax;
    wavespeeds_formula<0>(k, W[1], kws, lmin, lmax);
    return tmax(tabs(lmin), tabs(lmax));
  }

  // 2D CFL rate Lambda_x / dx + Lambda_y / dy of a cell state (one dimensionless state and
  // sigma part for both directions)
  template <class T>
  MX_HD static T cell_rate2d(const T* W, T sigma_lim, T kws, T dx, T dy) {
    Norm<T> n;
    norm(W, sigma_lim, kws, n);
    SigmaFit<T> f;
    sigma_fit(n.s.sb, n.s.rsb, n.s.isb, f);
    T a, b, c, d;
    speeds<0>(n, f, W[1], a, b);
    speeds<1>(n, f, W[2], c, d);
    return mdiv(tmax(tabs(a), tabs(b)), dx) + mdiv(tmax(tabs(c), tabs(d)), dy);
  }

  template <class T> MX_HD static T sigma(const T* W) {
    Core<T> k;
    core(W, T(0), k);
    return k.sig;
  }

  // local Maxwellian of a state: same rho, u and p, P = p I, q = 0, R = 15 p^2 / rho (the
  // state the BGK source relaxes to; it has the same rho, rho u and energy)
  template <class T> MX_HD static void equilibrium(const T* W, T* We) {
    T p = (W[4] + W[7] + W[9]) * T(1.0 / 3.0);
    We[0] = W[0]; We[1] = W[1]; We[2] = W[2]; We[3] = W[3];
    We[4] = p; We[5] = T(0); We[6] = T(0); We[7] = p; We[8] = T(0); We[9] = p;
    We[10] = T(0); We[11] = T(0); We[12] = T(0);
    We[13] = mdiv(T(15) * p * p, W[0]);
  }

  // BGK source; inv_tau = 1/tau at the cell centre
  template <class T> MX_HD static void source(const T* W, T inv_tau, T* C) {
    T rho = W[0];
    const T* u = W + 1;
    const T* P = W + 4;
    const T* q = W + 10;
    T p = (P[0] + P[3] + P[5]) * T(1.0 / 3.0);
    T Pu[3];
    symv(P, u, Pu);
    T uPu = u[0] * Pu[0] + u[1] * Pu[1] + u[2] * Pu[2];
    T uq = u[0] * q[0] + u[1] * q[1] + u[2] * q[2];
    T uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    C[0] = C[1] = C[2] = C[3] = T(0);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = i; j < 3; ++j)
        C[4 + sidx(i, j)] = -(P[sidx(i, j)] - (i == j ? p : T(0))) * inv_tau;
#pragma unroll
    for (int i = 0; i < 3; ++i) C[10 + i] = -(T(2) * Pu[i] + q[i] - T(2) * u[i] * p) * inv_tau;
    C[13] = -((T(4) * uPu + T(4) * uq + W[13]) - (T(4) * uu * p + mdiv(T(15) * p * p, rho))) * inv_tau;
  }
};

// ===================================================================== 5 moments
struct Sys5 {
  static constexpr int NV = 5;
  static constexpr bool TUBE = true;
  static constexpr bool JETS = false;
  MX_HD static constexpr int plane_of(int v) { return v; }

  // (TUBE: the roundings are fixed, as in Sys14A)
  template <class T> MX_HD static void cons_to_prim(const T* U, T* W) { cons_to_prim(U, W, true); }
  template <class T> MX_HD static void cons_to_prim(const T* U, T* W, bool fused) {
#pragma clang fp contract(off)
    T rho = U[0];
    T u = mdiv2(U[1], rho);
    T ru = rho * u;
    T ruu = ru * u;
    T P = fused ? dfma(-u, ru, U[2]) : U[2] - ruu;
    T q = dfma(T(-3) * u, P, dfma(-u, ruu, U[3]));
    T r = dfma(T(-4) * u, q, dfma(T(-6) * u * u, P, dfma(-u, ruu * u, U[4])));
    W[0] = rho; W[1] = u; W[2] = P; W[3] = q; W[4] = r;
  }

  template <class T> MX_HD static void prim_to_cons(const T* W, T* U) {
    T rho = W[0], u = W[1], P = W[2], q = W[3], r = W[4];
    U[0] = rho;
    U[1] = rho * u;
    U[2] = rho * u * u + P;
    U[3] = rho * u * u * u + T(3) * u * P + q;
    U[4] = rho * u * u * u * u + T(6) * u * u * P + T(4) * u * q + r;
  }

  template <class T> MX_HD static T pressure(const T* W) { return W[2]; }
  template <class T> MX_HD static bool admissible(const T* W) { return W[0] > T(0) && W[2] > T(0); }
  MX_HD static constexpr bool admissibility_var(int v) { return v == 0 || v == 2; }
  template <class T> MX_HD static bool admissible_cons(const T* U) {
    T rho = U[0];
    T u = mdiv2(U[1], rho);
    T P = U[2] - rho * u * u;
    return rho > T(0) && P > T(0);
  }

  template <class T> MX_HD static void scales(const T* W, T* sc) {
    T rho = tabs(W[0]);
    T p = tabs(W[2]);
    T c = msqrt2(mdiv2(p, rho));
    sc[0] = rho; sc[1] = c; sc[2] = p; sc[3] = rho * c * c * c; sc[4] = sc[3] * c;
  }

  MX_HD static constexpr bool odd(int v, int) { return v == 1 || v == 3; }

  template <class T> struct Core { T rho, c, qh, A, sig, sb; };

  template <class T> MX_HD static void core(const T* W, T sigma_lim, Core<T>& k) {
    k.rho = W[0];
    T irho = mrcp2(k.rho);
    T ip = mrcp2(W[2]);
    k.c = msqrt2(W[2] * irho);
    T ic = msqrt2(k.rho * ip);
    T is3 = irho * (ic * ic * ic);
    k.qh = W[3] * is3;
    T rh = W[4] * (is3 * ic);
    T A = T(3) - rh;
    T X = A * A + T(8) * k.qh * k.qh;
    k.A = A;
    k.sig = sigma_root(A, X, T(2) * k.qh * k.qh, T(4));
    k.sb = tmax(k.sig, sigma_lim);
  }

  MX_HD static void core_mixed(const double* W, float sigma_lim, Core<float>& k) {
    double ip = mrcp2(W[2]);
    double A = 3.0 - W[4] * W[0] * ip * ip;
    k.rho = (float)W[0];
    float irho = 1.0f / k.rho;
    float ipf = (float)ip;
    k.c = msqrt2((float)W[2] * irho);
    float ic = msqrt2(k.rho * ipf);
    float is3 = irho * (ic * ic * ic);
    k.qh = (float)W[3] * is3;
    k.A = (float)A;
    float X = k.A * k.A + 8.0f * k.qh * k.qh;
    k.sig = sigma_root(k.A, X, 2.0f * k.qh * k.qh, 4.0f);
    k.sb = tmax(k.sig, sigma_lim);
  }

  template <class T> MX_HD static T closing_s(const Core<T>& k) {
    T ss = mdiv2(k.qh * k.qh * k.qh, k.sb * k.sb) + (T(10) - T(8) * msqrt2(k.sb)) * k.qh;
    T c2 = k.c * k.c;
    return ss * k.rho * (c2 * c2 * k.c);
  }

  template <class T> MX_HD static void flux(const T* W, T s, T* F) {
    T rho = W[0], u = W[1], P = W[2], q = W[3], r = W[4];
    T u2 = u * u;
    F[0] = rho * u;
    F[1] = rho * u2 + P;
    F[2] = rho * u2 * u + T(3) * u * P + q;
    F[3] = rho * u2 * u2 + T(6) * u2 * P + T(4) * u * q + r;
    F[4] = rho * u2 * u2 * u + T(10) * u2 * u * P + T(10) * u2 * q + T(5) * u * r + s;
  }

  template <class T> MX_HD static void wavespeeds(const Core<T>& k, T u, T kws, T& lmin, T& lmax) {
    T sw = tmin(k.sb, T(1));
    BYEC<T> g = byec(sw, T(1));
    T base = T(4) * sw * sw * g.Y;
    T i2s = mrcp2(T(2) * sw);
    T Lmax = hyperbola(k.qh, T(-0.8) * k.qh * sw * g.C + base) * i2s + g.E;
    T Lmin = hyperbola(-k.qh, T(0.8) * k.qh * sw * g.C + base) * i2s + g.E;
    lmax = u + kws * Lmax * k.c;
    lmin = u - kws * Lmin * k.c;
  }

  // ---- FP64 face state and CFL rate with their roundings fixed (single precision keeps the functions
  // above)
  template <class T> MX_HD static void tube_core(const T* W, T sigma_lim, Core<T>& k) {
#pragma clang fp contract(off)
    k.rho = W[0];
    T irho = mrcp2(k.rho);
    T ip = mrcp2(W[2]);
    k.c = msqrt2(W[2] * irho);
    T ic = msqrt2(k.rho * ip);
    T is3 = irho * (ic * ic * ic);
    k.qh = W[3] * is3;
    T A = dfma(-W[4], is3 * ic, T(3));
    T X = dfma(k.qh, T(8) * k.qh, A * A);
    k.A = A;
    k.sig = tube_sigma(A, X, T(2) * k.qh * k.qh, T(4));
    k.sb = tmax(k.sig, sigma_lim);
  }
  template <class T> MX_HD static void tube_speeds(const Core<T>& k, T u, T kws, T& lmin, T& lmax) {
#pragma clang fp contract(off)
    T sw = tmin(k.sb, T(1));
    BYEC<T> g = byec(sw, T(1));
    T hmax, hmin;
    tube_roots(k.qh, sw, g.C, g.Y, hmax, hmin);
    T i2s = mrcp2(T(2) * sw);
    lmax = dfma(kws * dfma(i2s, hmax, g.E), k.c, u);
    lmin = dfma(-(kws * dfma(i2s, hmin, g.E)), k.c, u);
  }
  template <int d, class T>
  MX_HD static void face_terms(const T* W, T sigma_lim, T kws, T* U, T* F, T& lmin, T& lmax) {
#pragma clang fp contract(off)
    Core<T> k;
    tube_core(W, sigma_lim, k);
    const T rho = W[0], u = W[1], P = W[2], q = W[3], r = W[4];
    // closing moment s = ss rho c^5
    const T ss = dfma(k.qh, dfma(T(-8), msqrt2(k.sb), T(10)), mdiv2(k.qh * k.qh * k.qh, k.sb * k.sb));
    const T c2 = k.c * k.c, c5 = c2 * c2 * k.c;
    const T u2 = u * u, ru = rho * u, ru2 = rho * u2, ru4 = ru2 * u2;
    F[0] = ru;
    F[1] = dfma(rho, u2, P);
    F[2] = dfma(T(3) * u, P, ru2 * u) + q;
    F[3] = dfma(T(4) * u, q, dfma(T(6) * u2, P, ru4)) + r;
    F[4] = dfma(c5, ss * rho, dfma(T(5) * u, r, dfma(T(10) * u2, q, dfma(ru4, u, T(10) * u2 * u * P))));
    const T ruuu = ru * u * u;
    U[0] = rho;
    U[1] = ru;
    U[2] = dfma(ru, u, P);
    U[3] = dfma(T(3) * u, P, ruuu) + q;
    U[4] = dfma(T(4) * u, q, dfma(T(6) * u * u, P, ruuu * u)) + r;
    tube_speeds(k, u, kws, lmin, lmax);
  }

  template <int d>
  MX_HD static void face_terms_fp32(const float* W, float sigma_lim, float kws, float* U, float* F, float& lmin,
                                    float& lmax) {
    Core<float> k;
    core(W, sigma_lim, k);
    flux(W, closing_s(k), F);
    prim_to_cons(W, U);
    wavespeeds(k, W[1], kws, lmin, lmax);
  }

  template <int d, class T>
  MX_HD static void flux_speeds(const Core<T>& k, const T* W, T kws, T* F, T& lmin, T& lmax) {
    flux(W, closing_s(k), F);
    wavespeeds(k, W[1], kws, lmin, lmax);
  }

  template <int d, class T> MX_HD static T cell_lambda(const T* W, T sigma_lim, T kws) {
    Core<T> k;
    tube_core(W, sigma_lim, k);
    T lmin, lmax;
    tube_speeds(k, W[1], kws, lmin, lmax);
    return tmax(tabs(lmin), tabs(lmax));
  }

  template <class T> MX_HD static T sigma(const T* W) {
    Core<T> k;
    core(W, T(0), k);
    return k.sig;
  }

  // 1D1V local Maxwellian: same rho, u, P; q = 0, r = 3 P^2 / rho
  template <class T> MX_HD static void equilibrium(const T* W, T* We) {
    We[0] = W[0]; We[1] = W[1]; We[2] = W[2]; We[3] = T(0);
    We[4] = mdiv2(T(3) * W[2] * W[2], W[0]);
  }

  // its conserved moments (the implicit source)
  template <class T> MX_HD static void equilibrium_cons(const T* W, T* U) {
#pragma clang fp contract(off)
    T We[NV];
    equilibrium(W, We);
    T rho = We[0], u = We[1], P = We[2];
    T ru = rho * u, ruu = ru * u, ruuu = ruu * u;
    U[0] = rho;
    U[1] = ru;
    U[2] = ruu + P;
    U[3] = dfma(T(3) * u, P, ruuu);
    U[4] = dfma(T(6) * u * u, P, ruuu * u) + We[4];
  }

  template <class T> MX_HD static void source(const T* W, T inv_tau, T* C) {
#pragma clang fp contract(off)
    T rho = W[0], u = W[1], P = W[2], q = W[3], r = W[4];
    C[0] = C[1] = C[2] = T(0);
    C[3] = -q * inv_tau;
    C[4] = -(dfma(T(4) * u, q, r) - mdiv2(T(3) * P * P, rho)) * inv_tau;
  }
};

}  // namespace mx
