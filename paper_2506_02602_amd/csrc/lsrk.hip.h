// Device side of the per-cell LSRK chemistry integrator (gfx950, FP64 VALU).
//
// One cell per lane.  The cell's state vector u = (T, Y_1..Y_N) lives in
// registers as a fully unrolled array; the right-hand side is the
// mechanism's generated straight-line function M::rhs.
//
// Step (paper Eq. 21, two registers plus the error register): with
// F_i = f(U), for stages i = 1..5
//     E <- E + (b_i - bhat_i) h F_i
//     U <- X + a_{i+1,i} h F_i ;  X <- U + (b_i - a_{i+1,i}) h F_i      (i < 5)
//     X <- X + b_5 h F_5                                               (i = 5)
// Control (Eq. 22): err = WRMS(E) with weights rtol |u_n| + atol over all
// N+1 components; accept iff err <= 1; factor 0.9 err^(-1/4) clamped to
// [0.2, 5] (NaN error: 0.2; zero error: 5); the last step is clipped to end
// on dt.  Coefficients: Kennedy-Carpenter-Lewis RK4(3)5[2R+]C, the scheme
// the paper cites as its ref. [37].
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace chemgpu {

// Exact rationals of the published tableau; each quotient is a compile-time
// IEEE division of two exactly representable integers (correctly rounded).
constexpr double LS_A[4] = {970286171893.0 / 4311952581923.0,
                            6584761158862.0 / 12103376702013.0,
                            2251764453980.0 / 15575788980749.0,
                            26877169314380.0 / 34165994151039.0};
constexpr double LS_B[5] = {1153189308089.0 / 22510343858157.0,
                            1772645290293.0 / 4653164025191.0,
                            -1672844663538.0 / 4480602732383.0,
                            2114624349019.0 / 3568978502595.0,
                            5198255086312.0 / 14908931495163.0};
constexpr double LS_BH[5] = {1016888040809.0 / 7410784769900.0,
                             11231460423587.0 / 58533540763752.0,
                             -1563879915014.0 / 6823010717585.0,
                             606302364029.0 / 971179775848.0,
                             1097981568119.0 / 3980877426909.0};

// The stages' b, a (0 in the last) and b - b^, read by scalar loads.
struct Stage { double b, a, e; };
static __constant__ Stage kStage[5] = {{LS_B[0], LS_A[0], LS_B[0] - LS_BH[0]},
                                       {LS_B[1], LS_A[1], LS_B[1] - LS_BH[1]},
                                       {LS_B[2], LS_A[2], LS_B[2] - LS_BH[2]},
                                       {LS_B[3], LS_A[3], LS_B[3] - LS_BH[3]},
                                       {LS_B[4], 0.0, LS_B[4] - LS_BH[4]}};

enum : int { CELL_RUNNING = -1, CELL_OK = 0, CELL_MAXSTEPS = 1, CELL_NONFINITE = 2,
             CELL_H_UNDERFLOW = 3 };

struct Control {
  double rtol, atol;
  int max_steps;
};

// e^x (the implicit comparator's rates and their derivatives, and the wide
// mechanisms' rates): Cody-Waite reduction x = n ln2 + r, |r| <= ln2/2, with
// ln 2 split into its correctly rounded double and the remainder (both
// products applied with FMAs), then p(r) ~ e^r of degree 11 in Horner form,
// scaled by 2^n with ldexp.  p is the Chebyshev
// approximation of e^r on [-ln2/2, ln2/2] (interpolation at the Chebyshev
// nodes, within a few per cent of the minimax polynomial), coefficients
// rounded to doubles: relative error below 1.7e-17 in exact arithmetic,
// 0.77 ulp with the Horner roundings (a CPU test re-evaluates these
// coefficients in extended precision).  n is clamped so that its conversion
// to int is defined; past the double range ldexp gives inf or 0 (or a
// subnormal); NaN propagates through r.  Within 1 ulp of a correctly
// rounded exponential on [-708, 709]; fewer instructions than the library
// exponential, which also tests for the out-of-range cases.  (Converting
// with an inline v_cvt_i32_f64, which saturates by itself, would save the
// clamp's two instructions, but the opaque statement costs the per-lane
// kernels their register allocation: mech9 went from 235 VGPRs to spills.)
template <bool RANGED = false>
__device__ __forceinline__ double exp_cw(double x) {
  constexpr double LOG2E = 1.4426950408889634;
  constexpr double LN2_HI = 0.6931471805599453;
  constexpr double LN2_LO = 2.3190468138462996e-17;
  constexpr double MAGIC = 6755399441055744.0;  // 1.5 2^52
  double n = x * LOG2E;
  int ni;
  if constexpr (RANGED) {
    const double t = n + MAGIC;  // (an own statement: not contracted)
    n = t - MAGIC;
    ni = __double2loint(t);
  } else {
    n = rint(n);
    n = fmax(fmin(n, 2100.0), -2100.0);
    ni = (int)n;
  }
  double r = fma(-n, LN2_HI, x);
  r = fma(-n, LN2_LO, r);
  double p = 0x1.af631d0059becp-26;
  p = fma(p, r, 0x1.28b4057f44145p-22);
  p = fma(p, r, 0x1.71ddf5749d126p-19);
  p = fma(p, r, 0x1.a01991ac8730ap-16);
  p = fma(p, r, 0x1.a01a01b14378fp-13);
  p = fma(p, r, 0x1.6c16c187fbe02p-10);
  p = fma(p, r, 0x1.111111110f225p-7);
  p = fma(p, r, 0x1.555555554f0cfp-5);
  p = fma(p, r, 0x1.555555555555ap-3);
  p = fma(p, r, 0x1.0000000000011p-1);
  p = fma(p, r, 1.0);
  p = fma(p, r, 1.0);
  return ldexp(p, ni);
}

// The same to the bit for |x| < 2^30, two instructions fewer (n by adding and
// taking off 1.5 2^52, which leaves it in the sum's low word), for the wide
// mechanisms' rates, whose ln T is checked: 64^3 cells of 32 species 30.3 ->
// 29.6 ms.
__device__ __forceinline__ double exp_ranged(double x) { return exp_cw<true>(x); }

// log2(e) in two parts.  The exponentials below reduce x to an integer m and f,
// |f| <= 1/2, with e^x = 2^((m + f)/S): m = S x log2(e) rounded to the nearest
// integer by adding and taking off 1.5 2^52 (m then also sits in the sum's low
// word), f = S x log2(e) - m by two FMAs, whose first is all but exact.  The
// exponents stay in base e, where the fits' coefficients are exact: with the
// coefficients rounded to base 2, which spares these two FMAs one, rates were off
// by 1.25 times as much.  For |m| < 2^31; NaN propagates through f.
constexpr double LOG2E_HI = 0x1.71547652b82fep+0, LOG2E_LO = 0x1.777d0ffda0d24p-56;

// 2^(m + f) by a degree-11 polynomial in Horner form (interpolation of (2^f -
// 1)/f at the Chebyshev nodes of |f| <= 1/2, coefficients rounded to doubles:
// relative error below 2e-17 in exact arithmetic, 0.8 ulp with the Horner
// roundings).
__device__ __forceinline__ double exp2_poly(double f, int m) {
  double p = 0x1.e9d3fe3952179p-32;
  p = fma(p, f, 0x1.e6063f7217bc6p-28);
  p = fma(p, f, 0x1.b524fae627834p-24);
  p = fma(p, f, 0x1.62bfd47773353p-20);
  p = fma(p, f, 0x1.ffcbfc670dcd4p-17);
  p = fma(p, f, 0x1.430913096fd9fp-13);
  p = fma(p, f, 0x1.5d87fe78a5276p-10);
  p = fma(p, f, 0x1.3b2ab6fba1ddap-7);
  p = fma(p, f, 0x1.c6b08d704a0c2p-5);
  p = fma(p, f, 0x1.ebfbdff82c598p-3);
  p = fma(p, f, 0x1.62e42fefa39efp-1);
  p = fma(p, f, 1.0);
  return ldexp(p, m);
}

// Exponentials of the activity form.  ExpPoly: the polynomial above (S = 1),
// for kernels without the table.
struct ExpPoly {
  __device__ __forceinline__ double operator()(double x) const {
    constexpr double MAGIC = 6755399441055744.0;  // 1.5 2^52
    const double t = fma(x, LOG2E_HI, MAGIC);
    const double n = t - MAGIC;
    const double f = fma(x, LOG2E_LO, fma(x, LOG2E_HI, -n));
    return exp2_poly(f, __double2loint(t));
  }
};

typedef const __attribute__((address_space(3))) double lds_cdouble;

// ExpTable (S = 4096): 2^((m + f)/4096) = 2^(m >> 12) e (1 + p(f)) with e =
// 2^((m & 4095)/4096) from LDS (correctly rounded) and p the degree-3 Taylor
// polynomial of 2^(f/4096) - 1 (truncation below 3e-18), e + e p rounded once:
// within 1.03 ulp.  The per-lane kernels are bound by VALU issue, and this takes
// 12 of those instructions and an LDS read where the polynomial takes 17; 29
// exponentials are in a stage of 9 species.  A smaller table needs a term more
// (2,048 entries) or two, a larger one does not fit the LDS beside the packing
// slots.  Against the polynomial (both on exponents in base 2, one FMA less): 4.2
// M stiff cells 22.2 -> 20.8 ms, 96-box hierarchy 8.2 -> 7.6, 65,536 cells x 100
// calls 8.1 -> 7.5.
struct ExpTable {
  lds_cdouble* E;
  __device__ __forceinline__ double operator()(double x) const {
    constexpr double MAGIC = 6755399441055744.0;  // 1.5 2^52
    constexpr double C1 = 0x1.62e42fefa39efp-1, C2 = 0x1.ebfbdff82c58fp-3, C3 = 0x1.c6b08d704a0c0p-5;
    const double t = fma(x, LOG2E_HI * 4096.0, MAGIC);
    const double n = t - MAGIC;
    const double f = fma(x, LOG2E_LO * 4096.0, fma(x, LOG2E_HI * 4096.0, -n));
    const int m = __double2loint(t);
    const double e = E[m & 4095];
    const double p = fma(f, fma(f, C3 * 0x1p-36, C2 * 0x1p-24), C1 * 0x1p-12);
    return ldexp(fma(e, f * p, e), m >> 12);
  }
};

// 2^(j/64), j = 0..63: each the double nearest the exact value (hexadecimal
// literals, so the table is bit-exact).  The kernels that use exp_tab stage it
// in LDS.
static __constant__ double kExp2Frac[64] = {
    0x1.0000000000000p+0, 0x1.02c9a3e778061p+0, 0x1.059b0d3158574p+0, 0x1.0874518759bc8p+0,
    0x1.0b5586cf9890fp+0, 0x1.0e3ec32d3d1a2p+0, 0x1.11301d0125b51p+0, 0x1.1429aaea92de0p+0,
    0x1.172b83c7d517bp+0, 0x1.1a35beb6fcb75p+0, 0x1.1d4873168b9aap+0, 0x1.2063b88628cd6p+0,
    0x1.2387a6e756238p+0, 0x1.26b4565e27cddp+0, 0x1.29e9df51fdee1p+0, 0x1.2d285a6e4030bp+0,
    0x1.306fe0a31b715p+0, 0x1.33c08b26416ffp+0, 0x1.371a7373aa9cbp+0, 0x1.3a7db34e59ff7p+0,
    0x1.3dea64c123422p+0, 0x1.4160a21f72e2ap+0, 0x1.44e086061892dp+0, 0x1.486a2b5c13cd0p+0,
    0x1.4bfdad5362a27p+0, 0x1.4f9b2769d2ca7p+0, 0x1.5342b569d4f82p+0, 0x1.56f4736b527dap+0,
    0x1.5ab07dd485429p+0, 0x1.5e76f15ad2148p+0, 0x1.6247eb03a5585p+0, 0x1.6623882552225p+0,
    0x1.6a09e667f3bcdp+0, 0x1.6dfb23c651a2fp+0, 0x1.71f75e8ec5f74p+0, 0x1.75feb564267c9p+0,
    0x1.7a11473eb0187p+0, 0x1.7e2f336cf4e62p+0, 0x1.82589994cce13p+0, 0x1.868d99b4492edp+0,
    0x1.8ace5422aa0dbp+0, 0x1.8f1ae99157736p+0, 0x1.93737b0cdc5e5p+0, 0x1.97d829fde4e50p+0,
    0x1.9c49182a3f090p+0, 0x1.a0c667b5de565p+0, 0x1.a5503b23e255dp+0, 0x1.a9e6b5579fdbfp+0,
    0x1.ae89f995ad3adp+0, 0x1.b33a2b84f15fbp+0, 0x1.b7f76f2fb5e47p+0, 0x1.bcc1e904bc1d2p+0,
    0x1.c199bdd85529cp+0, 0x1.c67f12e57d14bp+0, 0x1.cb720dcef9069p+0, 0x1.d072d4a07897cp+0,
    0x1.d5818dcfba487p+0, 0x1.da9e603db3285p+0, 0x1.dfc97337b9b5fp+0, 0x1.e502ee78b3ff6p+0,
    0x1.ea4afa2a490dap+0, 0x1.efa1bee615a27p+0, 0x1.f50765b6e4540p+0, 0x1.fa7c1819e90d8p+0,
};

// e^x from the 2^(j/64) table and a short polynomial (chem_eval_math; the
// cooperative kernel takes exp_coop below): m = 64 k + j is the integer nearest 64 x / ln 2 (clamped so the
// conversion is defined), r = x - m ln2/64 by two FMAs with ln2/64 split in
// two parts (|r| <= ln2/128), and e^x = 2^k 2^(j/64) (1 + p(r)) with p the
// degree-6 Taylor polynomial of e^r - 1 (truncation below 3e-20 relative) by
// Estrin's scheme; t + t p is rounded once.  E points at kExp2Frac's values
// (in LDS).  Error: the table entry's rounding (at most 2^-53 relative) plus
// the final rounding, about 1 ulp at most on [-745, 709]; inf above, 0 or a
// subnormal below, NaN through, like exp_cw.  18 VALU instructions and one
// LDS read.
__device__ __forceinline__ double exp_tab(double x, const double* E) {
  constexpr double K = 92.33248261689366;            // 64 / ln 2
  constexpr double L_HI = 0.010830424696249145;        // ln2 / 64, nearest double
  constexpr double L_LO = 3.623510646634843e-19;   // ln2 / 64 - L_HI
  double m = rint(x * K);
  m = fmax(fmin(m, 134400.0), -134400.0);
  double r = fma(-m, L_HI, x);
  r = fma(-m, L_LO, r);
  const int mi = (int)m;
  const double t = E[mi & 63];
  const double r2 = r * r;
  const double a = fma(r, 1.0 / 6.0, 0.5);
  const double b = fma(r, 1.0 / 120.0, 1.0 / 24.0);
  const double q = fma(r2, fma(r2, 1.0 / 720.0, b), a);
  const double p = fma(r2, q, r);
  return ldexp(fma(t, p, t), mi >> 6);
}

// The literals of exp_coop and log_near.  A wave alone on its SIMD spends 8
// cycles on each scalar move of a literal's half, so the cooperative kernel
// loads them once (pin): into scalar registers, or vector registers where an
// FMA has two of them.  (c_k: ln2^k/k! in units of 1/64 octave.)
struct NearConsts {
  double magic = 6755399441055744.0;  // 1.5 2^52
  double c1 = 0x1.62e42fefa39efp-1 / 64, c2 = 0x1.ebfbdff82c58fp-3 / 4096;
  double c3 = 0x1.c6b08d704a0c0p-5 / 262144, c4 = 0x1.3b2ab6fba4e77p-7 / 16777216;
  double c5 = 0x1.5d87fe78a6731p-10 / 1073741824, c6 = 0x1.430912f86c787p-13 / 68719476736;
  double l3 = 1.0 / 3.0, l4 = -0.25, l5 = 1.0 / 5.0, l6 = -1.0 / 6.0, l7 = 1.0 / 7.0, l8 = -0.125;
  double khi = LOG2E_HI * 64.0, klo = LOG2E_LO * 64.0;
  __device__ __forceinline__ void pin() {
    asm volatile("" : "+s"(magic), "+s"(c1), "+s"(c3), "+s"(c5), "+s"(c6), "+s"(klo));
    asm volatile("" : "+s"(l3), "+s"(l5), "+s"(l7), "+s"(l8));
    asm volatile("" : "+v"(khi), "+v"(c2), "+v"(c4), "+v"(l4), "+v"(l6));
  }
};

// e^x for the cooperative kernel (S = 64, see LOG2E_HI): 2^((m + f)/64) = 2^(m
// >> 6) 2^((m & 63)/64) (1 + p(f)) with p the degree-6 Taylor polynomial of
// 2^(f/64) - 1 (truncation below 4e-20 relative), t + t p rounded once.  E
// points at kExp2Frac's values (in LDS).  Error as exp_tab's, two steps of the
// dependent chain shorter.
__device__ __forceinline__ double exp_coop(double x, const double* E, const NearConsts& k) {
  const double t = fma(x, k.khi, k.magic);
  const double n = t - k.magic;
  const double f = fma(x, k.klo, fma(x, k.khi, -n));
  const int m = __double2loint(t);
  const double e = E[m & 63];
  const double f2 = f * f;
  const double a = fma(f, k.c3, k.c2);
  const double b = fma(f, k.c5, k.c4);
  const double q = fma(f2, fma(f2, k.c6, b), a);
  const double p = fma(f2, q, f * k.c1);
  return ldexp(fma(e, p, e), m >> 6);
}

// 1/x from the hardware reciprocal refined by two Newton steps: within an
// ulp of the quotient for normal x (T and the heat-capacity sum of the
// temperature equation, both positive), half the instructions of the IEEE
// division sequence.
__device__ __forceinline__ double rcp_nr(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  r = fma(fma(-x, r, 1.0), r, r);
  return r;
}

// ln x for finite x > 0 (NaN otherwise) with a short dependency chain: x =
// 2^e m with m in [sqrt(1/2), sqrt(2)), f = m - 1 (exact), s = f / (2 + f)
// (hardware reciprocal refined by two Newton steps), and
// ln m = 2 atanh s = f - (f^2/2 - s (f^2/2 + R(s^2))) with R the series
// sum_k>=1 2 z^k / (2k + 1) in z = s^2 (|z| < 0.0295, ten terms, Estrin's
// scheme); e ln 2 is added with ln 2 split so that e times its leading part is
// exact, in the order that keeps the cancellation for x near 1/sqrt(2)
// harmless.  Within 1 ulp of the correctly rounded logarithm; about a third of
// the library logarithm's instructions and dependency depth, which carries
// double-double intermediates for correct rounding.
struct LogParts { double hi, lo; };  // a logarithm and what its last rounding left off

__device__ __forceinline__ LogParts log_atanh_parts(double x) {
  constexpr double LN2_HI = 0.6931471803691238;     // ln 2, low 21 mantissa bits cleared
  constexpr double LN2_LO = 1.9082149292705877e-10;  // ln 2 - LN2_HI
  constexpr double SQRT_HALF = 0.70710678118654752;
  double m = __builtin_amdgcn_frexp_mant(x);         // [0.5, 1)
  int e = __builtin_amdgcn_frexp_exp(x);
  const bool lo_half = m < SQRT_HALF;
  m = lo_half ? m + m : m;
  e = lo_half ? e - 1 : e;
  const double f = m - 1.0;
  const double d = 2.0 + f;
  double r = __builtin_amdgcn_rcp(d);
  r = fma(fma(-d, r, 1.0), r, r);
  r = fma(fma(-d, r, 1.0), r, r);
  const double s = f * r;
  const double z = s * s;
  const double z2 = z * z, z4 = z2 * z2, z8 = z4 * z4;
  const double a0 = fma(2.0 / 5.0, z, 2.0 / 3.0), a1 = fma(2.0 / 9.0, z, 2.0 / 7.0);
  const double a2 = fma(2.0 / 13.0, z, 2.0 / 11.0), a3 = fma(2.0 / 17.0, z, 2.0 / 15.0);
  const double a4 = fma(2.0 / 21.0, z, 2.0 / 19.0);
  const double q = fma(a4, z8, fma(fma(a3, z2, a2), z4, fma(a1, z2, a0)));
  const double hfsq = 0.5 * f * f;
  const double de = (double)e;
  // (|b| <= 0.36, so next to |a| or a = 0: lo is the sum's exact remainder)
  const double a = de * LN2_HI;
  const double b = (hfsq - fma(s, fma(z, q, hfsq), de * LN2_LO)) - f;
  const double y = a - b;
  return {x > 0.0 ? y : __builtin_nan(""), (a - y) - b};
}

__device__ __forceinline__ double log_atanh(double x) { return log_atanh_parts(x).hi; }

// ln T, NaN outside (T_MIN, T_MAX): there (far outside the fits) a rate
// exponent could leave the range ExpTable and exp_coop take, and a NaN
// right-hand side is a rejected step.
template <class M>
__device__ __forceinline__ LogParts log_checked_parts(double T, double margin) {
  LogParts y = log_atanh_parts(T);
  if (!(T > M::T_MIN * margin && T * margin < M::T_MAX)) y.hi = __builtin_nan("");
  return y;
}

template <class M>
__device__ __forceinline__ double log_checked(double T, double margin) {
  return log_checked_parts<M>(T, margin).hi;
}

// ln T of a stage from that of the step's start, ln0 = log_checked_parts(T0,
// 1.02): ln T = ln T0 + ln(1 + d), d = (T - T0)/T0, by the Taylor series to d^8
// for |d| <= 2^-6 (truncation below 2^-57, absolute); ln T0's remainder goes
// into d, so the sum is rounded once like ln T itself.  A lane further off gets
// log_checked, whatever the other lanes of its wave hold; one that is not
// stays within 1.6 % of T0, so within the range T0 was checked for.
template <class M>
__device__ __forceinline__ double log_near(double T, double T0, const LogParts& ln0, double r0,
                                           const NearConsts& k) {
  const double d = fma(T - T0, r0, ln0.lo);
  const double d2 = d * d, d4 = d2 * d2;
  const double a = fma(d, k.l3, -0.5), b = fma(d, k.l5, k.l4);
  const double c = fma(d, k.l7, k.l6);
  const double q = fma(fma(d2, k.l8, c), d4, fma(b, d2, a));
  double y = ln0.hi + fma(d2, q, d);
  const bool far = !(fabs(d) <= 0x1p-6);
  if (__builtin_expect(__any(far), 0)) {
    const double full = log_checked<M>(T, 1.0);
    y = far ? full : y;
  }
  return y;
}

__device__ __forceinline__ double step_factor(double err) {
  if (err != err) return 0.2;
  if (err == 0.0) return 5.0;
  // err^(-1/4) as 1/sqrt(sqrt(err)): correctly rounded square roots and a
  // division, a few ulp from pow() at a tenth of its cost
  double fac = 0.9 / sqrt(sqrt(err));
  fac = fac < 0.2 ? 0.2 : fac;
  fac = fac > 5.0 ? 5.0 : fac;
  return fac;
}

// The same factor from the squared norm s = err^2, 0.9 s^(-1/8): three
// hardware reciprocal square roots, 1/sqrt(1/sqrt(1/sqrt(s))), whose relative
// error (some 2^-22) one step of third order, y (1 + r/8 + 9/128 r^2) with r = 1
// - s y^8, takes below 2^-60: 0.49 ulp rms, 2.1 at most (square roots and a
// division: 0.62, 2.4), in a third of their dependent chain.
__device__ __forceinline__ double step_factor_sq(double s) {
  if (!(s < 1e7)) return 0.2;        // also NaN and infinity
  if (s < 1e-7) return 5.0;
  double y = __builtin_amdgcn_rsq(__builtin_amdgcn_rsq(__builtin_amdgcn_rsq(s)));
  const double y2 = y * y, y4 = y2 * y2;
  const double r = fma(-s, y4 * y4, 1.0);
  y = fma(y * r, fma(9.0 / 128.0, r, 0.125), y);
  const double fac = 0.9 * y;
  return fac < 0.2 ? 0.2 : fac > 5.0 ? 5.0 : fac;
}

// One LSRK step of size h from u; X receives the new state, returns the WRMS
// error (its square where M::CONC, see step_factor_sq).  The per-lane kernels
// are bound by instruction issue, so small mechanisms (M::CONC) step
// concentrations in place of mass fractions (rho is constant: no conversion in
// the five right-hand sides), continue ln T of a stage from the step's start,
// and take the norm with reciprocals in place of divisions (with the rates of
// progress in activity form: 4.2 M stiff cells 27.6 -> 26.4 ms, 96-box hierarchy
// 10.4 -> 9.8, 65,536 cells x 100 calls 9.9 -> 9.1); ex is the exponential their
// rates use.  The stage loop stays rolled so that the generated RHS is inlined
// once; the stage coefficients are wave-uniform scalars.
template <class M, class Exp = ExpPoly>
__device__ __forceinline__ double lsrk_step(const double (&u)[M::NS + 1], double rho,
                                            double inv_rho, double h, double (&X)[M::NS + 1],
                                            const Control& c, const Exp& ex = Exp{}) {
  constexpr int N1 = M::NS + 1;
  double U[N1], E[N1], F[N1];
#pragma unroll
  for (int i = 0; i < N1; ++i) { X[i] = u[i]; E[i] = 0.0; }
  [[maybe_unused]] LogParts ln0;
  [[maybe_unused]] double r0;
  if constexpr (M::CONC) {
    // (hide rho's invariance: its products would be kept in registers over
    // all steps, and from here to the norm)
    asm volatile("" : "+v"(rho), "+v"(inv_rho));
#pragma unroll
    for (int i = 1; i < N1; ++i) X[i] = u[i] * (rho * M::INVW[i - 1]);
    ln0 = log_checked_parts<M>(u[0], 1.02);
    r0 = rcp_nr(u[0]);
  }
#pragma unroll
  for (int i = 0; i < N1; ++i) U[i] = X[i];
#pragma unroll 1
  for (int s = 0; s < 5; ++s) {
    if constexpr (M::CONC) M::rhs_c(U, log_near<M>(U[0], u[0], ln0, r0, NearConsts{}), F, ex);
    else M::rhs(U, rho, inv_rho, F);
    const double bs = kStage[s].b, as = kStage[s].a, eh = kStage[s].e * h;
    // (the last stage has a = 0: its U is X; a branch of its own would cost
    // every stage register moves where the two paths join)
    const double ah = as * h;
    const double bah = (bs - as) * h;
#pragma unroll
    for (int i = 0; i < N1; ++i) {
      E[i] += eh * F[i];
      U[i] = X[i] + ah * F[i];
      X[i] = U[i] + bah * F[i];
    }
  }
  if constexpr (M::CONC) asm volatile("" : "+v"(rho), "+v"(inv_rho));
  double sum = 0.0;
#pragma unroll
  for (int i = 0; i < N1; ++i) {
    const double sc = c.rtol * fabs(u[i]) + c.atol;
    double w;
    if constexpr (M::CONC) {
      double to_y = 1.0;
      if (i > 0) {
        to_y = M::W[i - 1] * inv_rho;
        // the increment from the same rounded start (its own statement: not
        // contracted), so that an unchanged concentration leaves Y as it was
        const double c0 = u[i] * (rho * M::INVW[i - 1]);
        X[i] = u[i] + (X[i] - c0) * to_y;
      }
      w = E[i] * to_y * rcp_nr(sc);
    } else {
      w = E[i] / sc;
    }
    sum += w * w;
  }
  return M::CONC ? sum * (1.0 / N1) : sqrt(sum * (1.0 / N1));
}

template <int N1>
__device__ __forceinline__ bool all_finite(const double (&u)[N1], double rho) {
  bool ok = isfinite(rho);
#pragma unroll
  for (int i = 0; i < N1; ++i) ok = ok && isfinite(u[i]);
  return ok;
}

}  // namespace chemgpu
