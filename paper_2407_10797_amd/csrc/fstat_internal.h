// fstat_internal.h -- device-side building blocks shared by the libfstat kernels.
//
// Physics (Fu, Wang & Mohanty, arXiv:2407.10797):
//   * template phase Psi(f) of App. A (TaylorF2 up to alpha_6 plus the
//     leading eccentric term), evaluated in cycles with double-double
//     arithmetic for every term that reaches 10^2..10^7 cycles, so that the
//     fractional cycle is exact to ~1e-14;
//   * SPA time t_f = (1/2pi) dPsi/df (Sec. IV) from the analytic derivative;
//   * zeroth-order TDI-X response at t_f (Sec. IV, Eq. freDres with N = 0) on
//     a rigid-arm, first-order analytic orbit.
// The template-independent factor of the TDI-X transfer, the f^{-7/6}
// amplitude, 1/S_n and 4 df are folded into per-bin data at plan time, so a
// bin needs only the particle-dependent part T'_{+,x} (see prep kernel).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fstat {

// ---- physical constants (SI; light-seconds for lengths) -------------------
constexpr double kMsunS = 4.925490947641267e-6;  // G Msun / c^3
constexpr double kYear = 31557600.0;             // Julian year
constexpr double kC = 299792458.0;
constexpr double kAU = 1.495978707e11;
constexpr double kArm = 2.5e9;
constexpr double kF0Ecc = 0.01;                  // e0 reference GW frequency
constexpr double kPi = 3.141592653589793238462643383279502884;
constexpr double kLs = kArm / kC;                // arm light time [s]
constexpr double kRs = kAU / kC;                 // orbit radius [s]
constexpr double kSqrt3 = 1.7320508075688772935;
constexpr double kRankCut = 1e-12;               // singular-M eigenvalue ratio
constexpr int kSurMinNp = 16;                    // surrogate only in stages with Np >= 16

// ---- double-double helpers ---------------------------------------------------
// Error-free transformations must not be contracted: with fp-contract=fast the
// compiler may fuse an addition that consumes a rounded product into an FMA on
// the exact product, double-counting the product's error term.  Every function
// that builds or consumes double-double values switches contraction off.
#define FSTAT_NO_CONTRACT _Pragma("clang fp contract(off)")

struct dd {
  double hi, lo;
};

__host__ __device__ __forceinline__ dd two_prod(double a, double b) {
  FSTAT_NO_CONTRACT
  double p = a * b;
  return {p, __builtin_fma(a, b, -p)};
}
__host__ __device__ __forceinline__ dd two_sum(double a, double b) {
  FSTAT_NO_CONTRACT
  double s = a + b;
  double bb = s - a;
  return {s, (a - (s - bb)) + (b - bb)};
}
__host__ __device__ __forceinline__ dd quick_two_sum(double a, double b) {
  FSTAT_NO_CONTRACT
  double s = a + b;
  return {s, b - (s - a)};
}
__host__ __device__ __forceinline__ dd dd_add(dd a, dd b) {
  FSTAT_NO_CONTRACT
  dd s = two_sum(a.hi, b.hi);
  s.lo += a.lo + b.lo;
  return quick_two_sum(s.hi, s.lo);
}
__host__ __device__ __forceinline__ dd dd_mul(dd a, dd b) {
  FSTAT_NO_CONTRACT
  dd p = two_prod(a.hi, b.hi);
  p.lo += a.hi * b.lo + a.lo * b.hi;
  return quick_two_sum(p.hi, p.lo);
}
__host__ __device__ __forceinline__ dd dd_mul_d(dd a, double b) {
  FSTAT_NO_CONTRACT
  dd p = two_prod(a.hi, b);
  p.lo += a.lo * b;
  return quick_two_sum(p.hi, p.lo);
}
// The same without the closing renormalisation and with fused low-order terms,
// for chains of a few products and sums: lo stays within a few ulp of hi, so the
// products dropped (lo * lo) are ~1e-31 of the result, as in dd_mul; 4, 3 and 8
// operations for 9, 7 and 11.
__host__ __device__ __forceinline__ dd lz_mul(dd a, dd b) {
  const double p = a.hi * b.hi;
  return {p, __builtin_fma(a.lo, b.hi, __builtin_fma(a.hi, b.lo, __builtin_fma(a.hi, b.hi, -p)))};
}
__host__ __device__ __forceinline__ dd lz_mul_d(dd a, double b) {
  const double p = a.hi * b;
  return {p, __builtin_fma(a.lo, b, __builtin_fma(a.hi, b, -p))};
}
__host__ __device__ __forceinline__ dd lz_add(dd a, dd b) {
  FSTAT_NO_CONTRACT
  dd s = two_sum(a.hi, b.hi);
  s.lo += a.lo + b.lo;
  return s;
}
__host__ __device__ __forceinline__ dd dd_div(dd a, dd b) {
  FSTAT_NO_CONTRACT
  double q1 = a.hi / b.hi;
  dd r = dd_add(a, dd_mul_d(b, -q1));
  double q2 = r.hi / b.hi;
  return quick_two_sum(q1, q2);
}
// x^(1/n), x > 0, as double-double: a double estimate w0 and one Newton step
// on w^n = x (quadratic convergence from ~1 ulp).
__host__ __device__ __forceinline__ dd dd_root(dd x, int n, double w0) {
  FSTAT_NO_CONTRACT
  dd wn = dd{w0, 0.0};
  for (int i = 1; i < n; ++i) wn = dd_mul_d(wn, w0);
  double r = ((x.hi - wn.hi) + (x.lo - wn.lo)) / x.hi;   // 1 - w0^n / x
  return quick_two_sum(w0, w0 * r / (double)n);
}
__host__ __device__ __forceinline__ double dd_frac(dd a) {
  FSTAT_NO_CONTRACT
  return (a.hi - floor(a.hi)) + a.lo;
}

// ---- per-particle constants (filled by the setup kernel) -------------------
// Phase in cycles, with x = Mc f, y = x^{-1/3}, v = (pi M f)^{1/3} = vfac / y
// (App. A; (3/128)(pi Mc f)^{-5/3} v^k / (2 pi) = cN vfac^k y^{5-k}):
//   Psi/(2 pi) = f t_c + cN y^5 + c1 y^3 + c15 y^2 + ce y^{34/3}     (double-double)
//              + c2 y + c5 ln v + (c6 / y)(a6k + b6 ln v) + const    (double)
// cN = 3/(256 pi^{8/3}); c1 = cN alpha_2 vfac^2; c15 = cN alpha_3 vfac^3;
// ce = cN (-2355/1462) e0^2 (f0 Mc)^{19/9}; c2 = cN alpha_4 vfac^4;
// c5 = 3 cN c5' vfac^5 with alpha_5 = c5'(1 + 3 ln(v sqrt 6)); c6 = cN vfac^6;
// alpha_6 = a6k + b6 ln v.  The terms that reach 10^2..10^7 cycles are
// carried as double-double, so the fractional cycle is exact to ~1e-14.
// Numerical orbit: nseg segments of length dt from t0, each a degree-9
// Chebyshev series per spacecraft and coordinate (positions in seconds of
// light travel), coef [nseg][3][3][10]; coef == nullptr: analytic orbit.
// Read-only device memory addressed through the constant address space, so
// that wave-uniform reads become scalar loads.
typedef __attribute__((address_space(4))) double kconst_double;
struct OrbitTable {
  const double* coef = nullptr;
  int32_t nseg = 0;
  double t0 = 0.0;
  double dt = 1.0;
};

struct PartConst {
  double tc;
  double mc_hi, mc_lo;     // Mc [s]
  double cN_hi, cN_lo, c1_hi, c1_lo, c15_hi, c15_lo, ce_hi, ce_lo;
  double c2, c5, c6, a6k, b6, ln_vfac;
  double c5v5;             // cN c5' vfac^5 (enters t_f)
  double ecc_k;            // -(2355/1462) e0^2: Psi_e = ecc_k (f0/f)^{19/9} Psi_N
  double nn_mc, nn_e0;     // surrogate inputs for Mc and e0, mapped to [-1, 1]
  double k[3], u[3], v[3];
  double flo, fhi;
  int32_t j_lo, j_hi;      // support bins (inclusive); j_lo > j_hi when empty
  int32_t np;
  int32_t status;          // 0 ok, 1 empty support, 2 invalid parameters
  int32_t sur;             // 1: eccentric term from the surrogate knots
  int32_t pad_;
};

enum { kStatusOk = 0, kStatusEmpty = 1, kStatusInvalid = 2 };

// The template's constants of a particle at a wave-uniform address, by scalar
// loads (read-only memory, constant address space).
typedef __attribute__((address_space(4))) PartConst kconst_PartConst;
__device__ __forceinline__ PartConst load_particle(const kconst_PartConst* p) {
  PartConst P;
  P.tc = p->tc;
  P.mc_hi = p->mc_hi; P.mc_lo = p->mc_lo;
  P.cN_hi = p->cN_hi; P.cN_lo = p->cN_lo; P.c1_hi = p->c1_hi; P.c1_lo = p->c1_lo;
  P.c15_hi = p->c15_hi; P.c15_lo = p->c15_lo; P.ce_hi = p->ce_hi; P.ce_lo = p->ce_lo;
  P.c2 = p->c2; P.c5 = p->c5; P.c6 = p->c6; P.a6k = p->a6k; P.b6 = p->b6;
  P.ln_vfac = p->ln_vfac; P.c5v5 = p->c5v5;
  for (int i = 0; i < 3; ++i) { P.k[i] = p->k[i]; P.u[i] = p->u[i]; P.v[i] = p->v[i]; }
  P.sur = p->sur;
  return P;
}

// ---- phase and SPA time -------------------------------------------------------
// Fractional cycle of Psi(f)/(2 pi) (constant phase offsets dropped: the
// F-statistic absorbs them) and the SPA time t_f = (1/2 pi) dPsi/df.
// Cubic Lagrange interpolation through four knots x_a (ek[0..3]) with
// coefficients c_a = value_a / prod_{b != a}(x_a - x_b) (ek[4..7]):
// I(f) = sum_a c_a prod_{b != a} (f - x_b).
__host__ __device__ __forceinline__ double knot_interp(const double* ek, double f) {
  double d0 = f - ek[0], d1 = f - ek[1], d2 = f - ek[2], d3 = f - ek[3];
  double d01 = d0 * d1, d23 = d2 * d3;
  return ek[4] * (d1 * d23) + ek[5] * (d0 * d23) + ek[6] * (d01 * d3) + ek[7] * (d01 * d2);
}

// ek == nullptr: analytic eccentric term; otherwise the eccentric term (cycles)
// is interpolated from the surrogate's knot values of the current partition.
__host__ __device__ __forceinline__ void phase_and_tf(const PartConst& P, double f, double& frac,
                                             double& tf, const double* ek = nullptr) {
  FSTAT_NO_CONTRACT
  dd ft = two_prod(f, P.tc);
  double c_ft = (ft.hi - floor(ft.hi)) + ft.lo;
  dd x = dd_mul_d(dd{P.mc_hi, P.mc_lo}, f);
  double lx = log(x.hi);
  // y = x^{-1/3}: y0 within a few ulp (the cube of w0 = x^{-1/9}, which the
  // eccentric term needs anyway), then one Newton step on x y^3 = 1
  const double w0 = ek ? 0.0 : exp(lx * (-1.0 / 9.0));
  double y0 = ek ? exp(lx * (-1.0 / 3.0)) : w0 * w0 * w0;
  dd b = dd_mul(dd_mul_d(two_prod(y0, y0), y0), x);
  double r = (1.0 - b.hi) - b.lo;
  dd y = quick_two_sum(y0, y0 * r * (1.0 / 3.0));
  dd y2 = dd_mul(y, y);
  dd y3 = dd_mul(y2, y);
  dd y5 = dd_mul(y3, y2);
  double xy2 = x.hi * y2.hi;                         // x^{1/3} = 1 / y
  dd tN = dd_mul(dd{P.cN_hi, P.cN_lo}, y5);
  dd t1 = dd_mul(dd{P.c1_hi, P.c1_lo}, y3);
  dd t15 = dd_mul(dd{P.c15_hi, P.c15_lo}, y2);
  dd te;
  if (ek) {
    te = dd{knot_interp(ek, f), 0.0};
  } else {
    // w = y^{1/3}: estimate w0, then one Newton step on w^3 = y
    dd w3 = dd_mul_d(two_prod(w0, w0), w0);
    double rw = ((y.hi - w3.hi) + (y.lo - w3.lo)) * xy2;
    dd w = quick_two_sum(w0, w0 * rw * (1.0 / 3.0));
    te = dd_mul(dd_mul(dd{P.ce_hi, P.ce_lo}, dd_mul(dd_mul(y5, y5), y)), w);
  }
  double lnv = P.ln_vfac + lx * (1.0 / 3.0);
  double t2 = P.c2 * y.hi;
  double t6 = P.c6 * xy2;
  double small = t2 + P.c5 * lnv + t6 * (P.a6k + P.b6 * lnv);
  double ph = c_ft + dd_frac(tN) + dd_frac(t1) + dd_frac(t15) + dd_frac(te) + small;
  frac = ph - floor(ph);
  // t_f: a term c y^m = c x^{-m/3} contributes -(m/3) c y^m / f to dPsi/df/(2 pi);
  // 1/f = Mc / x = Mc y^3
  double D = (-5.0 / 3.0) * tN.hi - t1.hi - (2.0 / 3.0) * t15.hi - (1.0 / 3.0) * t2 + P.c5v5 +
             t6 * (P.a6k + P.b6 + P.b6 * lnv) * (1.0 / 3.0) - (34.0 / 9.0) * te.hi;
  tf = P.tc + D * (P.mc_hi * y3.hi);
}

// The same phase unreduced (whole cycles kept, double-double) and t_f, at a
// frequency given as double-double: the interpolating bin loop takes phase
// differences across a work item from it, at node positions between bins,
// where rounding f to a double would move the phase by t_f * 1e-16 f
// (~1e-9 cycles at t_f ~ 1e8 s).
//
// log x of a normal positive x from a table of kLogTab {1 / c, log c}: the top
// mantissa bits pick c, log(m / c) by six terms in r = m / c - 1, |r| <= 2^-8
// (remainder 2e-18).  log c has 40 fractional bits and ln 2 is split, so that
// their sum is exact, and each c is one whose reciprocal rounds to less than
// 2e-18: what is left is the last rounding and ~1e-17, 0.5 ulp as the library's log
// where |log x| is of order one and more (x = Mc f is 5e-7 to 3e-5 in the searches; near
// x = 1 the terms cancel and only the absolute error stays), in 17 operations for its ~70.
constexpr int kLogTab = 128;
__device__ __forceinline__ double log_tab(double x, const double2* lt) {
  const int hi = __double2hiint(x);
  const double m = __hiloint2double((hi & 0xfffff) | 0x3ff00000, __double2loint(x));
  const double e = (double)((hi >> 20) - 1023);
  const double2 t = lt[(hi >> 13) & (kLogTab - 1)];
  const double r = fma(m, t.x, -1.0);
  const double q = fma(r, fma(r, fma(r, fma(r, -1.0 / 6.0, 1.0 / 5.0), -0.25), 1.0 / 3.0), -0.5);
  return fma(e, 0x1.62e42fefa38p-1, t.y) + fma(e, 0x1.ef35793c7673p-45, fma(r * r, q, r));
}
// x^{-1/9} within a few ulp: an FP32 estimate (2e-7) and one third-order step
// on x w^9 = 1 (its remainder, ~20 e^3, is below 1e-18); outside FP32's range the
// result is not finite and the item is left to the exact loop.
__device__ __forceinline__ double ninth_root_inv(double x) {
  const double w = (double)__builtin_amdgcn_exp2f(__builtin_amdgcn_logf((float)x) * (-1.0f / 9.0f));
  const double w2 = w * w, w4 = w2 * w2;
  const double e = fma(-(w4 * w4), w * x, 1.0);
  return fma(w * e, fma(e, 5.0 / 81.0, 1.0 / 9.0), w);
}
__device__ __forceinline__ dd phase_full(const PartConst& P, dd f, dd& tf, const double* ek,
                                         const double2* lt) {
  FSTAT_NO_CONTRACT
  const dd ft = lz_mul_d(f, P.tc);
  const dd x = lz_mul(dd{P.mc_hi, P.mc_lo}, f);
  const double lx = log_tab(x.hi, lt);
  const double w0 = ninth_root_inv(x.hi);
  const double y0 = w0 * w0 * w0;
  const dd b = lz_mul(lz_mul_d(two_prod(y0, y0), y0), x);
  const double r = (1.0 - b.hi) - b.lo;
  const dd y = quick_two_sum(y0, y0 * r * (1.0 / 3.0));
  const dd y2 = lz_mul(y, y);
  const dd y3 = lz_mul(y2, y);
  const dd y5 = lz_mul(y3, y2);
  const double xy2 = x.hi * y2.hi;
  const dd tN = lz_mul(dd{P.cN_hi, P.cN_lo}, y5);
  const dd t1 = lz_mul(dd{P.c1_hi, P.c1_lo}, y3);
  const dd t15 = lz_mul(dd{P.c15_hi, P.c15_lo}, y2);
  dd te;
  if (ek) {
    te = dd{knot_interp(ek, f.hi), 0.0};
  } else {
    const dd w3 = lz_mul_d(two_prod(w0, w0), w0);
    const double rw = ((y.hi - w3.hi) + (y.lo - w3.lo)) * xy2;
    const dd w = quick_two_sum(w0, w0 * rw * (1.0 / 3.0));
    te = lz_mul(lz_mul(dd{P.ce_hi, P.ce_lo}, lz_mul(lz_mul(y5, y5), y)), w);
  }
  const double lnv = P.ln_vfac + lx * (1.0 / 3.0);
  // the alpha_4 term reaches ~1e2 cycles: double-double too, so that its
  // rounding does not add ~1e-14-cycle noise between interpolation nodes
  const dd t2d = lz_mul_d(y, P.c2);
  const double t2 = t2d.hi;
  const double t6 = P.c6 * xy2;
  const double small = P.c5 * lnv + t6 * (P.a6k + P.b6 * lnv);
  const dd ph = lz_add(lz_add(lz_add(ft, tN), lz_add(t1, t15)),
                       lz_add(te, lz_add(t2d, dd{small, 0.0})));
  // t_f in double-double as well: its rounding (1e-8 s at 1e8 s) would turn
  // the orbit angle and the 1000-s Doppler term into ~1e-13-cycle noise
  dd D = lz_add(lz_add(lz_mul_d(tN, -5.0 / 3.0), dd{-t1.hi, -t1.lo}),
                lz_add(lz_mul_d(t15, -2.0 / 3.0), lz_mul_d(te, -34.0 / 9.0)));
  D = lz_add(D, dd{-(1.0 / 3.0) * t2 + P.c5v5 + t6 * (P.a6k + P.b6 + P.b6 * lnv) * (1.0 / 3.0), 0.0});
  tf = lz_add(dd{P.tc, 0.0}, lz_mul(D, lz_mul(dd{P.mc_hi, P.mc_lo}, y3)));
  tf = quick_two_sum(tf.hi, tf.lo);
  return quick_two_sum(ph.hi, ph.lo);
}

// The same phase and t_f in plain FP64 (whole cycles kept): at ~1e7 cycles
// the phase rounds to ~2e-9 cycles, enough where the sine is taken in FP32
// (~6e-8 turns).  y = x^{-1/3} from w0^3 with one Newton step, as above.
__device__ __forceinline__ double phase_full_fp64(const PartConst& P, double f,
                                                  double& tf, const double* ek,
                                                  const double2* lt) {
  const double x = P.mc_hi * f;
  const double lx = log_tab(x, lt);
  const double w0 = ninth_root_inv(x);
  const double y0 = w0 * w0 * w0;
  const double r = fma(-(y0 * y0) * y0, x, 1.0);
  const double y = fma(y0 * r, 1.0 / 3.0, y0);
  const double y2 = y * y, y3 = y2 * y, y5 = y3 * y2;
  const double xy2 = x * y2;
  const double tN = P.cN_hi * y5, t1 = P.c1_hi * y3, t15 = P.c15_hi * y2;
  const double te = ek ? knot_interp(ek, f) : P.ce_hi * (y5 * y5 * y) * w0;
  const double lnv = P.ln_vfac + lx * (1.0 / 3.0);
  const double t2 = P.c2 * y;
  const double t6 = P.c6 * xy2;
  const double small = P.c5 * lnv + t6 * (P.a6k + P.b6 * lnv);
  const double D = (-5.0 / 3.0) * tN - t1 - (2.0 / 3.0) * t15 - (1.0 / 3.0) * t2 + P.c5v5 +
                   t6 * (P.a6k + P.b6 + P.b6 * lnv) * (1.0 / 3.0) - (34.0 / 9.0) * te;
  tf = P.tc + D * (P.mc_hi * y3);
  return f * P.tc + (tN + ((t1 + t15) + (te + (t2 + small))));
}

// Per-particle phase coefficients (see PartConst), double-double where the
// term they multiply reaches 10^2..10^7 cycles.
__host__ __device__ inline void fill_constants(PartConst& P, const double* th) {
  FSTAT_NO_CONTRACT
  double tc = th[0], mc = th[1], dmu = th[2], theta = th[3], phi = th[4], e0 = th[5];
  P.tc = tc;
  dd m = two_prod(mc, kMsunS);                       // Mc [s], exact
  P.mc_hi = m.hi; P.mc_lo = m.lo;
  dd d2 = two_prod(dmu, dmu);
  dd one_m = dd_add(dd{1.0, 0.0}, dd{-d2.hi, -d2.lo});
  dd eta = dd{one_m.hi * 0.25, one_m.lo * 0.25};      // (1 - dmu^2)/4
  // constants of the series as double-double
  const dd pi = {3.141592653589793116e+00, 1.2246467991473532e-16};
  const dd pi13 = {1.46459188756152336e+00, -1.01504731086581778e-16};       // pi^{1/3}
  const dd cN = {5.53539090143848902e-04, -4.81692159938612682e-20};         // 3 / (256 pi^{8/3})
  const dd r2a = {4.91402116402116373e+00, 2.86660759797394900e-16};         // 3715 / 756
  const dd r2b = {6.11111111111111072e+00, 3.94745964311166748e-16};         // 55 / 9
  const dd rec = {-1.61080711354309170e+00, 4.00956058140959402e-17};        // -2355 / 1462
  dd ie5 = dd_root(dd_div(dd{1.0, 0.0}, eta), 5, pow(eta.hi, -0.2));   // eta^{-1/5}
  dd vfac = dd_mul(pi13, ie5);                        // v = vfac (Mc f)^{1/3}
  dd vf2 = dd_mul(vfac, vfac), vf3 = dd_mul(vf2, vfac);
  dd a2 = dd_add(r2a, dd_mul(r2b, eta));
  dd c1 = dd_mul(dd_mul(cN, a2), vf2);
  dd c15 = dd_mul(dd_mul(cN, dd_mul_d(pi, -16.0)), vf3);
  dd z = dd_mul_d(m, kF0Ecc);                         // f0 Mc
  dd z19 = dd_mul(dd_mul(z, z), dd_root(z, 9, pow(z.hi, 1.0 / 9.0)));   // (f0 Mc)^{19/9}
  dd ce = dd_mul(dd_mul(cN, rec), dd_mul(two_prod(e0, e0), z19));
  P.cN_hi = cN.hi; P.cN_lo = cN.lo;
  P.c1_hi = c1.hi; P.c1_lo = c1.lo;
  P.c15_hi = c15.hi; P.c15_lo = c15.lo;
  P.ce_hi = ce.hi; P.ce_lo = ce.lo;
  double et = eta.hi, vf = vfac.hi, K = cN.hi;
  const double pisq = kPi * kPi;
  double a4 = 15293365.0 / 508032.0 + 27145.0 * et / 504.0 + 3085.0 * et * et / 72.0;
  double c5p = kPi * (38645.0 / 756.0 - 65.0 * et / 9.0);
  const double euler = 0.57721566490153286061;
  double a6c = 11583231236531.0 / 4694215680.0 - 640.0 * pisq / 3.0 - 6848.0 * euler / 21.0 +
               (-15737765635.0 / 3048192.0 + 2255.0 * pisq / 12.0) * et +
               76055.0 * et * et / 1728.0 - 127825.0 * et * et * et / 1296.0;
  double vf4 = vf * vf * vf * vf, vf5 = vf4 * vf, vf6 = vf5 * vf;
  P.c2 = K * a4 * vf4;
  P.c5v5 = K * c5p * vf5;
  P.c5 = 3.0 * P.c5v5;
  P.c6 = K * vf6;
  P.b6 = -6848.0 / 21.0;
  P.a6k = a6c + P.b6 * 1.38629436111989061883;   // ln 4
  P.ln_vfac = log(vf);
  P.ecc_k = -(2355.0 / 1462.0) * e0 * e0;
  P.nn_mc = (mc - 30.0) / 20.0;
  P.nn_e0 = e0 / 0.075 - 1.0;
  P.sur = 0;
  P.pad_ = 0;
  double st, ct, sp, cp;
  sincos(theta, &st, &ct);
  sincos(phi, &sp, &cp);
  P.k[0] = -st * cp; P.k[1] = -st * sp; P.k[2] = -ct;
  P.u[0] = ct * cp;  P.u[1] = ct * sp;  P.u[2] = -st;
  P.v[0] = sp;       P.v[1] = -cp;      P.v[2] = 0.0;
}

// Newtonian and eccentric phase terms (cycles) of the plain template at f:
// tN = cN y^5 and te = ce y^{34/3} (App. A), in double precision; used to
// build the surrogate's training targets and to check its knot values.
__host__ __device__ __forceinline__ void newton_and_ecc(const PartConst& P, double f, double& tN,
                                                       double& te) {
  FSTAT_NO_CONTRACT
  dd x = dd_mul_d(dd{P.mc_hi, P.mc_lo}, f);
  double lx = log(x.hi);
  double y = exp(lx * (-1.0 / 3.0));
  double y5 = y * y * y * y * y;
  tN = (P.cN_hi + P.cN_lo) * y5;
  te = (P.ce_hi + P.ce_lo) * y5 * y5 * y * exp(lx * (-1.0 / 9.0));
}

// ---- per-bin template (particle-dependent part) -------------------------------
// Full basis template (Sec. II.A, Eq. response; Sec. IV, Eq. freDres, N = 0):
//   A^1 = C(f) f^{-7/6} e^{-i Phi} T''_+,  Phi = Psi + 2 pi f k.p_1,
// with C(f) = (1 - z^2)(-i pi f L) e^{-i pi f L} folded into the per-bin data,
// and for a rigid constellation (arms of length L along the orbit's arm
// directions n_a = 1->2, n_b = 1->3) the link propagation phase
// e^{-i pi f k.(p_s + p_r)} = e^{-2 pi i f k.p_1} e^{-i pi f L k.n}: the common
// factor joins the template phase, the arm factor reuses the sincos of the
// link sinc argument.  Per arm
//   S = e^{-i x0 kn} [sinc(x0 (1 + kn)) + z sinc(x0 (1 - kn))],  x0 = pi f L,
//   T''_P = F^P_b S_b - F^P_a S_a,  F^+ = (u.n)^2 - (v.n)^2,  F^x = 2 (u.n)(v.n).
__host__ __device__ __forceinline__ double sinc_from(double num, double den) {
  // num = sin(den) computed by angle addition; series near den = 0
  return (fabs(den) < 1e-6) ? 1.0 - den * den * (1.0 / 6.0) : num / den;
}

// a * b + c as one three-operand FMA into a fresh register, a wave-uniform
// (a scalar register: constants cost scalar moves, not vector ones)
__device__ __forceinline__ double fma3(double a, double b, double c) {
  double d;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "s"(a), "v"(b), "v"(c));
  return d;
}

// sin(2 pi r), cos(2 pi r) for |r| < 2^22 turns: r = n / kSinTab + x with x
// exact and |x| <= 1 / (2 kSinTab); the coarse factor from the LDS table, the
// fine one from short Taylor series (sin to theta^5, cos to theta^6:
// remainders below 1e-19 for |theta| <= pi / kSinTab), combined by the
// angle-addition formulas.  In the bin loop |r| stays below ~1e4 turns (the
// item's start phase is below one turn, the linear term below half a turn
// per bin, the residual a few hundred turns at most).
constexpr int kSinTab = 512;
__device__ __forceinline__ void sincos_tab(double r, const double2* tab, double& s, double& c) {
  const double n = rint(r * (double)kSinTab);
  const double x = fma(-1.0 / (double)kSinTab, n, r);
  const double2 e = tab[(int)n & (kSinTab - 1)];
  const double th = x * 6.283185307179586477;
  const double z = th * th;
  const double ps = fma3(1.0 / 120.0, z, -1.0 / 6.0);
  const double pc = fma(fma3(-1.0 / 720.0, z, 1.0 / 24.0), z, -0.5);
  const double sl = fma(th * z, ps, th);
  const double cl = fma(z, pc, 1.0);
  s = fma(e.x, cl, e.y * sl);
  c = fma(e.y, cl, -(e.x * sl));
}

// sin(pi x), cos(pi x): from the table when one is given, else the library.  TAB:
// one is always given; without the test the library's code and registers drop
// out (the node kernel).  The exact loop keeps the test: its removal merges code
// in which the compiler then fuses other products, and F of ill-conditioned
// partitions moves by eps cond(M) with each such choice.
template <bool TAB>
__device__ __forceinline__ void sincospi_t(double x, const double2* tab, double* s, double* c) {
  if (TAB || tab) sincos_tab(0.5 * x, tab, *s, *c);
  else sincospi(x, s, c);
}

// hardware reciprocal / reciprocal square root seeds refined by two Newton
// steps (accurate to about one ulp)
__device__ __forceinline__ double rcp_nr(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = __builtin_fma(-x, r, 1.0);
  r = __builtin_fma(r, e, r);
  e = __builtin_fma(-x, r, 1.0);
  return __builtin_fma(r, e, r);
}
__device__ __forceinline__ double rsq_nr(double x) {
  double r = __builtin_amdgcn_rsq(x);
  double h = 0.5 * x;
  r = r * __builtin_fma(-h * r, r, 1.5);
  return r * __builtin_fma(-h * r, r, 1.5);
}

// spacecraft offsets from the guiding centre R (cos a, sin a, 0) for the
// first-order analytic orbit: beta_i = 2 pi i / 3, e R / 2 = L / (4 sqrt 3),
// sqrt(3) e R = L / 2
template <typename T>
__device__ __forceinline__ void orbit_offsets(T ca, T sa, T d[3][3]) {
  const T q = (T)(kLs / (4.0 * kSqrt3));
  const T hz = (T)(0.5 * kLs);
  const T cb[3] = {(T)1.0, (T)-0.5, (T)-0.5};
  const T sb[3] = {(T)0.0, (T)(0.5 * kSqrt3), (T)(-0.5 * kSqrt3)};
  T c2a = ca * ca - sa * sa, s2a = (T)2.0 * sa * ca;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    d[i][0] = q * (c2a * cb[i] + s2a * sb[i] - (T)3.0 * cb[i]);
    d[i][1] = q * (s2a * cb[i] - c2a * sb[i] - (T)3.0 * sb[i]);
    d[i][2] = -hz * (ca * cb[i] + sa * sb[i]);
  }
}

// Channel codes (Grid::chan): weights of M_0 = X, M_1 = Y, M_2 = Z in a channel
__device__ __forceinline__ void channel_weights(int code, double w[3]) {
  const double r2 = 0.70710678118654752440, r6 = 0.40824829046386301637,
               r3 = 0.57735026918962576451;
  w[0] = w[1] = w[2] = 0.0;
  if (code <= 2) w[code] = 1.0;
  else if (code == 3) { w[0] = -r2; w[2] = r2; }
  else if (code == 4) { w[0] = r6; w[1] = -2.0 * r6; w[2] = r6; }
  else { w[0] = w[1] = w[2] = r3; }
}

// TDI transfer (T''_+, T''_x) at f of the Michelson combination at spacecraft
// a (a = 0: X) relative to the phase reference p_1: arms from p_a to p_{a+1},
// p_{a+2}, and the factor exp(-2 pi i f k.(p_a - p_1)) of the vertex's offset.
// d are the spacecraft offsets, s0, c0 = sin, cos(pi f L).  Delays and sinc
// arguments take the nominal arm length L.  The link phase pi f k.(p_s + p_r)
// takes L n for the arm vector on the analytic (rigid) constellation, the arm
// vector itself when `table` (a numerical orbit, whose arms need not have
// length L).
template <bool TAB>
__device__ __forceinline__ void michelson_fp64(const PartConst& P, double f, double s0, double c0,
                                               const double d[3][3], int a, double& tpr,
                                               double& tpi, double& txr, double& txi,
                                               bool table = false, const double2* tab = nullptr) {
  const double kx = P.k[0], ky = P.k[1], kz = P.k[2];
  const double x0 = kPi * kLs * f;
  const double zr = c0 * c0 - s0 * s0, zi = -2.0 * s0 * c0;   // z = e^{-2 i x0}
  double out[2][4];
#pragma unroll
  for (int arm = 0; arm < 2; ++arm) {
    const int w = (a + 1 + arm) % 3;
    double ax = d[w][0] - d[a][0], ay = d[w][1] - d[a][1], az = d[w][2] - d[a][2];
    const double r2 = ax * ax + ay * ay + az * az;
    double inv = rsq_nr(r2);
    ax *= inv; ay *= inv; az *= inv;
    double kn = kx * ax + ky * ay + kz * az;
    double un = P.u[0] * ax + P.u[1] * ay + P.u[2] * az;
    double vn = P.v[0] * ax + P.v[1] * ay + P.v[2] * az;
    double sq, cq;
    sincospi_t<TAB>(kLs * f * kn, tab, &sq, &cq);
    double np_ = s0 * cq + c0 * sq, nm = s0 * cq - c0 * sq;   // sin(x0 (1 +- kn))
    double dp = x0 * (1.0 + kn), dm = x0 * (1.0 - kn);
    double sp, sm;
    if (fabs(dp) > 1e-6 && fabs(dm) > 1e-6) {
      double r = rcp_nr(dp * dm);
      sp = np_ * dm * r;
      sm = nm * dp * r;
    } else {
      sp = sinc_from(np_, dp);
      sm = sinc_from(nm, dm);
    }
    double Sr = sp + zr * sm, Si = zi * sm;
    if (table) {   // link phase from the arm vector: rotate by exp(-i pi f kn (|d| - L))
      double se, ce;
      sincospi_t<TAB>(f * kn * (r2 * inv - kLs), tab, &se, &ce);
      const double tr = sq * ce + cq * se, tc = cq * ce - sq * se;
      sq = tr;
      cq = tc;
    }
    out[arm][0] = cq * Sr + sq * Si;      // e^{-i x0 kn} S
    out[arm][1] = cq * Si - sq * Sr;
    out[arm][2] = un * un - vn * vn;
    out[arm][3] = 2.0 * un * vn;
  }
  double pr = out[1][2] * out[1][0] - out[0][2] * out[0][0];
  double pi = out[1][2] * out[1][1] - out[0][2] * out[0][1];
  double xr = out[1][3] * out[1][0] - out[0][3] * out[0][0];
  double xi = out[1][3] * out[1][1] - out[0][3] * out[0][1];
  if (a != 0) {
    const double kd = kx * (d[a][0] - d[0][0]) + ky * (d[a][1] - d[0][1]) + kz * (d[a][2] - d[0][2]);
    double sv, cv;
    sincospi_t<TAB>(2.0 * f * kd, tab, &sv, &cv);   // e^{-i 2 pi f kd} = cv - i sv
    const double r0 = pr * cv + pi * sv, i0 = pi * cv - pr * sv;
    const double r1 = xr * cv + xi * sv, i1 = xi * cv - xr * sv;
    pr = r0; pi = i0; xr = r1; xi = i1;
  }
  tpr = pr; tpi = pi; txr = xr; txi = xi;
}

// Transfer of channel `code` (relative to the phase reference p_1).
template <bool TAB>
__device__ __forceinline__ void response_ch_fp64(const PartConst& P, double f, double s0, double c0,
                                                 const double d[3][3], int code, double& tpr,
                                                 double& tpi, double& txr, double& txi,
                                                 bool table = false, const double2* tab = nullptr) {
  // all lanes at X (the node kernel): one copy with its spacecraft known
  if (TAB && __builtin_amdgcn_ballot_w64(code != 0) == 0) {
    michelson_fp64<TAB>(P, f, s0, c0, d, 0, tpr, tpi, txr, txi, table, tab);
    return;
  }
  double w[3];
  channel_weights(code, w);
  tpr = tpi = txr = txi = 0.0;
  // one copy of the Michelson code in a rolled loop: unrolled, the three
  // copies raise the kernels' register use above the occupancy limit
#pragma unroll 1
  for (int a = 0; a < 3; ++a) {
    if (w[a] == 0.0) continue;
    double pr, pi, xr, xi;
    michelson_fp64<TAB>(P, f, s0, c0, d, a, pr, pi, xr, xi, table, tab);
    tpr = fma(w[a], pr, tpr); tpi = fma(w[a], pi, tpi);
    txr = fma(w[a], xr, txr); txi = fma(w[a], xi, txi);
  }
}

// The nine degree-9 Chebyshev series of one table segment at x in [-1, 1]
// (Clenshaw's recurrence), coefficients c[9][10].
template <typename C>
__device__ __forceinline__ void clenshaw_positions(const C* c, double x, double p[3][3]) {
#pragma unroll
  for (int q = 0; q < 9; ++q) {
    const C* cq = c + 10 * q;
    double b1 = 0.0, b2 = 0.0;
#pragma unroll
    for (int k = 9; k >= 1; --k) {
      const double b0 = fma(2.0 * x, b1, cq[k] - b2);
      b2 = b1;
      b1 = b0;
    }
    p[q / 3][q % 3] = fma(x, b1, cq[0] - b2);
  }
}

// Spacecraft positions [s] at time t = th + tl (tl = 0 for a plain double)
// from an orbit table: Clenshaw on the segment that holds t (the first or last
// segment outside the table).  The offset from the segment's start is formed
// without rounding t itself (whose ulp at 1e8 s, 1.5e-8 s, would move the
// positions by ~1e-12 s and the Doppler phase by ~1e-13 cycles).
__device__ __forceinline__ void table_positions(const OrbitTable& o, double th, double tl,
                                                double p[3][3]) {
  int seg;
  double x;
  {
    FSTAT_NO_CONTRACT
    const dd a = two_sum(th, -o.t0);                      // t - t0
    seg = (int)floor(a.hi / o.dt);
    seg = min(max(seg, 0), o.nseg - 1);
    const dd s0 = two_prod(o.dt, (double)seg);            // segment start - t0
    // a.hi - s0.hi is exact inside the table (the two are within a factor 2)
    const double loc = (a.hi - s0.hi) + ((a.lo - s0.lo) + tl);
    x = 2.0 * loc / o.dt - 1.0;
  }
  // All active lanes in one segment (the usual case): its coefficients are
  // read through the scalar cache (wave-uniform address, read only);
  // otherwise each lane reads its own segment's.
  const int s = __builtin_amdgcn_readfirstlane(seg);
  if (__builtin_amdgcn_ballot_w64(seg != s) == 0)
    clenshaw_positions((const kconst_double*)(o.coef + (int64_t)s * 90), x, p);
  else
    clenshaw_positions(o.coef + (int64_t)seg * 90, x, p);
}

// k . p_1 from the table, with d[i] = p_i - p_1 (the response uses only
// differences of the d and k . (d_a - d_0)).
__device__ __forceinline__ double k_dot_p1_table(const PartConst& P, const OrbitTable& o, double th,
                                                 double tl, double d[3][3]) {
  double p[3][3];
  table_positions(o, th, tl, p);
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int c = 0; c < 3; ++c) d[i][c] = p[i][c] - p[0][c];
  return P.k[0] * p[0][0] + P.k[1] * p[0][1] + P.k[2] * p[0][2];
}

// k . p_1 [s] of spacecraft 1 at orbit angle (ca, sa); fills the offsets d
__device__ __forceinline__ double k_dot_p1(const PartConst& P, double ca, double sa, double d[3][3]) {
  orbit_offsets<double>(ca, sa, d);
  const double kx = P.k[0], ky = P.k[1], kz = P.k[2];
  return kRs * (kx * ca + ky * sa) + (kx * d[0][0] + ky * d[0][1] + kz * d[0][2]);
}

__device__ __forceinline__ void template_fp64(const PartConst& P, double f, double s0, double c0,
                                              double& cph, double& sph, double& tpr,
                                              double& tpi, double& txr, double& txi,
                                              const double* ek = nullptr, int code = 0,
                                              const OrbitTable* orb = nullptr,
                                              const double2* tab = nullptr) {
  double fr, tf;
  phase_and_tf(P, f, fr, tf, ek);
  double d[3][3];
  double kp1;
  if (orb && orb->coef) {
    kp1 = k_dot_p1_table(P, *orb, tf, 0.0, d);
  } else {
    double sa, ca;
    sincospi_t<false>(2.0 * tf * (1.0 / kYear), tab, &sa, &ca);
    kp1 = k_dot_p1(P, ca, sa, d);
  }
  double ph = fr + f * kp1;               // Phi / (2 pi) in cycles
  ph -= rint(ph);
  sincospi_t<false>(2.0 * ph, tab, &sph, &cph);
  response_ch_fp64<false>(P, f, s0, c0, d, code, tpr, tpi, txr, txi, orb && orb->coef, tab);
}

// The template at an arbitrary frequency fd (double-double; an interpolation
// node): the whole phase Phi / (2 pi) = Psi / (2 pi) + f k.p_1 in cycles
// (double-double, not reduced) and the transfer without the Doppler factor.
__device__ __forceinline__ dd template_node(const PartConst& P, dd fd, const double* ek,
                                            double& tpr, double& tpi, double& txr, double& txi,
                                            int code, const OrbitTable* orb, const double2* tab,
                                            const double2* lt) {
  dd tf;
  dd ph = phase_full(P, fd, tf, ek, lt);
  const double f = fd.hi;
  double d[3][3];
  double kp1;
  if (orb && orb->coef) {
    kp1 = k_dot_p1_table(P, *orb, tf.hi, tf.lo, d);
  } else {
    double sa, ca;
    {
      FSTAT_NO_CONTRACT
      const dd turns = dd_mul_d(tf, 1.0 / kYear);     // orbit angle in turns, reduced exactly
      sincospi_t<true>(2.0 * ((turns.hi - floor(turns.hi)) + turns.lo), tab, &sa, &ca);
    }
    kp1 = k_dot_p1(P, ca, sa, d);
  }
  double s0, c0;
  sincospi_t<true>(kLs * f, tab, &s0, &c0);
  response_ch_fp64<true>(P, f, s0, c0, d, code, tpr, tpi, txr, txi, orb && orb->coef, tab);
  return dd_add(ph, dd_mul_d(fd, kp1));
}

// The same node template in plain FP64 (the mixed path's interpolation nodes).
__device__ __forceinline__ double template_node_fp64(const PartConst& P, double f, const double* ek,
                                                     double& tpr, double& tpi, double& txr,
                                                     double& txi, int code,
                                                     const OrbitTable* orb, const double2* tab,
                                                     const double2* lt) {
  double tf;
  const double ph = phase_full_fp64(P, f, tf, ek, lt);
  double d[3][3];
  double kp1;
  if (orb && orb->coef) {
    kp1 = k_dot_p1_table(P, *orb, tf, 0.0, d);
  } else {
    double sa, ca;
    sincospi_t<true>(2.0 * tf * (1.0 / kYear), tab, &sa, &ca);
    kp1 = k_dot_p1(P, ca, sa, d);
  }
  double s0, c0;
  sincospi_t<true>(kLs * f, tab, &s0, &c0);
  response_ch_fp64<true>(P, f, s0, c0, d, code, tpr, tpi, txr, txi, orb && orb->coef, tab);
  return fma(f, kp1, ph);
}

// ---- per-partition solve (2x2 Hermitian closed form) --------------------------
// acc = {Re Z+, Im Z+, Re Zx, Im Zx, P, Q, Re R, Im R};  F = 1/2 z^H H^{-1} z,
// H = [[P, conj R], [R, Q]] is the complex form of the real 4x4 M of
// Eq. coherent_F_stat; rank-deficient H uses the pseudo-inverse.
// The fused operations are written out: left to the compiler, their choice
// (above all in det = PQ - |R|^2) changes with the surrounding code, and F with
// it by eps cond(M).
struct Herm {
  double lp, det;        // larger eigenvalue, determinant
};
__host__ __device__ __forceinline__ Herm herm_of(double P, double Q, double rr, double ri) {
  FSTAT_NO_CONTRACT
  const double hd = 0.5 * (P - Q), rr2 = rr * rr;
  const double rad = sqrt(__builtin_fma(ri, ri, __builtin_fma(hd, hd, rr2)));
  return {__builtin_fma(0.5, P + Q, rad), __builtin_fma(P, Q, -(rr2 + ri * ri))};
}
__host__ __device__ __forceinline__ double solve_partition(const double* a) {
  FSTAT_NO_CONTRACT
  const double zpr = a[0], zpi = a[1], zxr = a[2], zxi = a[3];
  const double P = a[4], Q = a[5], rr = a[6], ri = a[7];
  const Herm h = herm_of(P, Q, rr, ri);
  const double lp = h.lp, det = h.det;
  if (!(lp > 0.0)) return 0.0;
  const double lm = det / lp;
  if (lm > kRankCut * lp) {
    const double zp2 = __builtin_fma(zpr, zpr, zpi * zpi), zx2 = __builtin_fma(zxr, zxr, zxi * zxi);
    const double cr = __builtin_fma(zpr, rr, -(zpi * ri));        // Re, Im of R z_+
    const double ci = __builtin_fma(zpi, rr, zpr * ri);
    const double cross = __builtin_fma(zxr, cr, zxi * ci);
    return __builtin_fma(-2.0, cross, __builtin_fma(Q, zp2, P * zx2)) / (det + det);
  }
  // rank one: eigenvector of lambda_+ ; pick the better-conditioned form
  double v1r, v1i, v2r, v2i;
  if (P >= Q) { v1r = lp - Q; v1i = 0.0; v2r = rr; v2i = ri; }      // (lp - Q, R)
  else        { v1r = rr; v1i = -ri; v2r = lp - P; v2i = 0.0; }     // (conj R, lp - P)
  const double n2 =
      __builtin_fma(v2i, v2i, v2r * v2r + __builtin_fma(v1i, v1i, v1r * v1r));
  if (!(n2 > 0.0)) return 0.0;
  // v^H z
  const double pr = __builtin_fma(v2i, zxi, __builtin_fma(v2r, zxr, __builtin_fma(v1i, zpi, v1r * zpr)));
  const double pi = __builtin_fma(-v2i, zxr, __builtin_fma(v2r, zxi, __builtin_fma(v1r, zpi, -(v1i * zpr))));
  return 0.5 * __builtin_fma(pr, pr, pi * pi) / (lp * n2);
}

// ---- maximum-likelihood amplitudes of a partition (Eq. aandMN3) -------------
// The log-likelihood over the complex pair beta = (beta_+, beta_x) of the
// templates (T+ g, Tx g) is Re(beta^H z) - 1/2 beta^H H beta (up to the bin
// weighting), maximised by beta = H^{-1} z; when H is rank deficient the
// pseudo-inverse keeps the lambda_+ eigendirection only (the minimum-norm
// maximiser).  acc as for solve_partition; out {Re, Im} beta_+, {Re, Im} beta_x.
__host__ __device__ __forceinline__ void solve_beta(const double* a, double* out) {
  FSTAT_NO_CONTRACT
  const double zpr = a[0], zpi = a[1], zxr = a[2], zxi = a[3];
  const double P = a[4], Q = a[5], rr = a[6], ri = a[7];
  for (int k = 0; k < 4; ++k) out[k] = 0.0;
  const Herm h = herm_of(P, Q, rr, ri);
  const double lp = h.lp, det = h.det;
  if (!(lp > 0.0)) return;
  const double lm = det / lp;
  if (lm > kRankCut * lp) {
    // H^{-1} = [[Q, -conj R], [-R, P]] / det
    const double cxr = __builtin_fma(zxr, rr, zxi * ri);      // conj(R) z_x
    const double cxi = __builtin_fma(zxi, rr, -(zxr * ri));
    const double rpr = __builtin_fma(zpr, rr, -(zpi * ri));   // R z_+
    const double rpi = __builtin_fma(zpi, rr, zpr * ri);
    out[0] = __builtin_fma(zpr, Q, -cxr) / det;
    out[1] = __builtin_fma(zpi, Q, -cxi) / det;
    out[2] = __builtin_fma(zxr, P, -rpr) / det;
    out[3] = __builtin_fma(zxi, P, -rpi) / det;
    return;
  }
  double v1r, v1i, v2r, v2i;
  if (P >= Q) { v1r = lp - Q; v1i = 0.0; v2r = rr; v2i = ri; }
  else        { v1r = rr; v1i = -ri; v2r = lp - P; v2i = 0.0; }
  const double n2 =
      __builtin_fma(v2i, v2i, v2r * v2r + __builtin_fma(v1i, v1i, v1r * v1r));
  if (!(n2 > 0.0)) return;
  // v^H z
  const double pr = __builtin_fma(v2i, zxi, __builtin_fma(v2r, zxr, __builtin_fma(v1i, zpi, v1r * zpr)));
  const double pi = __builtin_fma(-v2i, zxr, __builtin_fma(v2r, zxi, __builtin_fma(v1r, zpi, -(v1i * zpr))));
  const double den = lp * n2;
  const double sr = pr / den, si = pi / den;
  out[0] = __builtin_fma(v1r, sr, -(v1i * si));
  out[1] = __builtin_fma(v1r, si, v1i * sr);
  out[2] = __builtin_fma(v2r, sr, -(v2i * si));
  out[3] = __builtin_fma(v2r, si, v2i * sr);
}

}  // namespace fstat
