// Correctly rounded exp, log, sin and cos for the FP64 kernels.
//
// Each function evaluates its result in double-double arithmetic (Dekker's exact
// two-sum / two-product splits, relative error ~2^-100) and rounds once to double.  The
// rounded value is then the correctly rounded one except when the exact result lies
// within ~2^-100 of a rounding midpoint (probability ~2^-47 per call).  Correct rounding
// makes the FP64 step independent of the math library's last-bit choices, so two correct
// implementations of the method agree bit for bit.
//
//   exp: x = k ln2 + r, |r| <= ln2/2 (ln2 in three parts, the first with 42 bits so k*L1
//        is exact), e^r by a degree-25 Taylor polynomial in Horner form, times 2^k.
//   log: x = m 2^e, m in [1/sqrt2, sqrt2); one Newton step y1 = y0 + m e^{-y0} - 1 from the
//        library value y0 = log(m), with e^{-y0} in double-double; plus e ln2.  Next to x = 1 the
//        series of log(1 + r).
//   sin/cos: x = k pi/2 + r, |r| <= pi/4 (pi/2 in three parts, the first with 33 bits),
//        Taylor polynomials in r^2 to degree 29, quadrant from k mod 4.
// These full double-double evaluations (*_dd) are the slow paths.  The entry points cr_exp,
// cr_log, cr_sin, cr_cos and cr_sincos first evaluate a short series from a table of nodes, and
// return its rounding when an interval of 2^-66 of it on either side rounds to a single double
// (Ziv's test), which is then the correctly rounded result; about one call in 5000 falls through
// to the slow path.  The short forms' unrounded error is below 2^-67 of the result (sine and cosine:
// 2^-67.9 the largest of 3e6 arguments; exponential and logarithm: derived where they stand).
#pragma once

#include <hip/hip_runtime.h>

namespace qedk {

struct dd {
  double hi, lo;
};

__device__ __forceinline__ dd dd_two_sum(double a, double b) {
  const double s = a + b;
  const double bb = s - a;
  return {s, (a - (s - bb)) + (b - bb)};
}

__device__ __forceinline__ dd dd_fast_two_sum(double a, double b) {  // |a| >= |b|
  const double s = a + b;
  return {s, b - (s - a)};
}

__device__ __forceinline__ dd dd_two_prod(double a, double b) {
  const double p = a * b;
  return {p, fma(a, b, -p)};
}

__device__ __forceinline__ dd dd_add(dd a, dd b) {
  dd s = dd_two_sum(a.hi, b.hi);
  s.lo += a.lo + b.lo;
  return dd_fast_two_sum(s.hi, s.lo);
}

__device__ __forceinline__ dd dd_mul(dd a, dd b) {
  dd p = dd_two_prod(a.hi, b.hi);
  p.lo += a.hi * b.lo + a.lo * b.hi;
  return dd_fast_two_sum(p.hi, p.lo);
}

__device__ __forceinline__ dd dd_mul_d(dd a, double b) {
  dd p = dd_two_prod(a.hi, b);
  p.lo += a.lo * b;
  return dd_fast_two_sum(p.hi, p.lo);
}

// 1/n!, n = 0..29, as double-double; filled by the host (qed_crinit.h) in every source file whose
// kernels use it, as is the sine table below
static __constant__ dd c_inv_fact[30];

constexpr double kLn2A = 0x1.62e42fefa3800p-1;   // ln 2 = A + B + C, A with 42 significant bits
constexpr double kLn2B = 0x1.ef35793c76730p-45;
constexpr double kLn2C = 0x1.f97b57a079a19p-103;
constexpr double kLn2Hi = 0x1.62e42fefa39efp-1;  // ln 2 as a double-double
constexpr double kLn2Lo = 0x1.abc9e3b39803fp-56;
constexpr double kInvLn2 = 0x1.71547652b82fep+0;
constexpr double kPio2A = 0x1.921fb54400000p+0;  // pi/2 = A + B + C, A with 33 significant bits
constexpr double kPio2B = 0x1.0b4611a626331p-34;
constexpr double kPio2C = 0x1.1701b839a2520p-88;
constexpr double kTwoOverPi = 0x1.45f306dc9c883p-1;

// e^x as a double-double, for -740 < x < 709
__device__ inline dd exp_dd(double x) {
  const double k = rint(x * kInvLn2);
  // r = x - k ln2: k*A and x - k*A are exact (Sterbenz), k*B is split exactly, k*C is below
  // the working precision's last bit
  dd r = dd_add(dd{x - k * kLn2A, 0.0}, dd_two_prod(-k, kLn2B));
  r = dd_fast_two_sum(r.hi, r.lo - k * kLn2C);
  dd p = c_inv_fact[25];
#pragma unroll
  for (int n = 24; n >= 0; --n) p = dd_add(dd_mul(p, r), c_inv_fact[n]);
  const int ki = (int)k;
  return {ldexp(p.hi, ki), ldexp(p.lo, ki)};
}

__device__ __noinline__ double cr_exp_dd(double x) {
  if (!(x < 709.0)) return x != x ? x : (x > 709.782712893384 ? INFINITY : exp(x));
  if (!(x > -700.0)) return exp(x);  // results near the subnormal range are left to the library
  const dd e = exp_dd(x);
  return e.hi + e.lo;
}

__device__ __noinline__ double cr_log_dd(double x) {
  if (!(x > 0.0) || !(x < INFINITY)) return log(x);
  int e;
  double m = frexp(x, &e);
  if (m < 0.70710678118654752) {
    m *= 2.0;
    e -= 1;
  }
  if (e == 0 && fabs(m - 1.0) < 0x1p-7) {
    // next to 1 the Newton step's error, 2^-100 of 1, is large against the logarithm: its series
    // r (1 - r/2 + r^2/3 - ...) to r^15, 1/n = (n - 1)! / n!
    const double r = m - 1.0;  // exact
    double f = 87178291200.0;  // 14!
    dd p = dd_mul_d(c_inv_fact[15], f);
    for (int n = 14; n >= 1; --n) {
      f /= n;  // (n - 1)!, exact
      p = dd_add(dd_mul_d(c_inv_fact[n], f), dd_mul_d(p, -r));
    }
    p = dd_mul_d(p, r);
    return p.hi + p.lo;
  }
  const double y0 = log(m);
  // Newton step on e^y = m: y1 = y0 + m e^{-y0} - 1
  const dd t = dd_add(dd_mul_d(exp_dd(-y0), m), dd{-1.0, 0.0});
  const dd y = dd_add(dd{y0, 0.0}, t);
  const double ed = (double)e;
  dd l = dd_two_prod(ed, kLn2Hi);
  l.lo += ed * kLn2Lo;
  l = dd_fast_two_sum(l.hi, l.lo);
  const dd s = dd_add(l, y);
  return s.hi + s.lo;
}

// sin and cos of x (|x| < 2^20) in one reduction.  The entry points are out of line so that
// the double-double temporaries do not raise the register budget of the calling kernels.
__device__ __noinline__ void cr_sincos_dd(double x, double* sn, double* cs) {
  if (!(fabs(x) < 1048576.0)) {
    *sn = sin(x);
    *cs = cos(x);
    return;
  }
  const double k = rint(x * kTwoOverPi);
  dd r = dd_add(dd{x - k * kPio2A, 0.0}, dd_two_prod(-k, kPio2B));
  r = dd_fast_two_sum(r.hi, r.lo - k * kPio2C);
  const dd r2 = dd_mul(r, r);
  const dd mr2 = {-r2.hi, -r2.lo};
  // cos r = sum (-1)^n r^2n / (2n)!, sin r = r sum (-1)^n r^2n / (2n+1)!
  dd pc = c_inv_fact[28], ps = c_inv_fact[29];
#pragma unroll
  for (int n = 13; n >= 0; --n) {
    pc = dd_add(dd_mul(pc, mr2), c_inv_fact[2 * n]);
    ps = dd_add(dd_mul(ps, mr2), c_inv_fact[2 * n + 1]);
  }
  const dd s = dd_mul(ps, r);
  const double sv = s.hi + s.lo, cv = pc.hi + pc.lo;
  const int q = ((int)fmod(k, 4.0) + 4) & 3;
  *sn = q == 0 ? sv : q == 1 ? cv : q == 2 ? -sv : -cv;
  *cs = q == 0 ? cv : q == 1 ? -sv : q == 2 ? -cv : sv;
}

// sin(x + qs pi/2) alone: the same reduction and the same double-double polynomial as the
// matching output of cr_sincos (so the same bits), with only the polynomial the quadrant needs
// evaluated.  qs = 0: sin, qs = 1: cos.
__device__ __noinline__ double cr_sinq_dd(double x, int qs) {
  if (!(fabs(x) < 1048576.0)) return qs ? cos(x) : sin(x);
  const double k = rint(x * kTwoOverPi);
  dd r = dd_add(dd{x - k * kPio2A, 0.0}, dd_two_prod(-k, kPio2B));
  r = dd_fast_two_sum(r.hi, r.lo - k * kPio2C);
  const dd r2 = dd_mul(r, r);
  const dd mr2 = {-r2.hi, -r2.lo};
  const int q = (((int)fmod(k, 4.0) + 4) + qs) & 3;
  const bool odd = (q & 1) == 0;  // true: sin r series (odd factorials), false: cos r series
  dd p = odd ? c_inv_fact[29] : c_inv_fact[28];
#pragma unroll
  for (int n = 13; n >= 0; --n) p = dd_add(dd_mul(p, mr2), odd ? c_inv_fact[2 * n + 1] : c_inv_fact[2 * n]);
  if (odd) p = dd_mul(p, r);
  const double v = p.hi + p.lo;
  return (q & 2) ? -v : v;
}

// ---------------------------------------------------------------------------
// Fast path of the same correctly rounded sin and cos (Ziv's rounding test): an unrounded result
// well within kZivEps of the exact value (relative) is returned when every value within kZivEps of it
// rounds to the same double, i.e. when that double is the correctly rounded result; otherwise
// (probability ~2^-12 per call) the full double-double series above decides.
// ---------------------------------------------------------------------------
constexpr double kZivEps = 0x1p-66;

// the double nearest to v when every value within kZivEps |v| of it rounds to it
__device__ __forceinline__ bool ziv_round(dd v, double* out) {
  const double e = kZivEps * fabs(v.hi);
  const double a = v.hi + (v.lo + e), b = v.hi + (v.lo - e);
  *out = a;
  return a == b;
}

// The unrounded result comes from a table of the circle: k = rint(x 256/pi) (from the low bits of
// x 256/pi + 1.5 2^52), x = k pi/256 + r with r a double-double, |r| <= pi/512 (pi/256 in three parts:
// x - k A is exact, k B is split exactly),
//   sin x = S cos r + C sin r,  cos x = C cos r - S sin r,
// S = sin(k pi/256) and C its cosine as double-doubles.  cos r - 1 = -z/2 + z^2/24 - ... (z = r^2 a
// double-double in its first term) is below 2^-15.7 and sin r - r below 2^-17.3 of r, so their
// double parts err by less than 2^-69 of the result; the products with S and C are exact in
// their leading terms.  The error stays below 2^-67 of the result (where S or C is not zero, it is at
// most twice the result; the largest of 3e6 arguments, against 113 bits: 2^-67.9), so the rounding
// test decides.  The whole circle is in the table, so that no lane selects by quadrant or sign:
// about 75 instructions instead of the 110 of a table of [0, pi/4] and the 300 of the two series.
constexpr int kCircle = 512;             // angles j pi/256
constexpr int kSinTab = kCircle + kCircle / 4;  // a quarter more: the cosine is 128 entries ahead
constexpr int kSinTabWords = 2 * kSinTab;
constexpr double k256OverPi = 0x1.45f306dc9c883p+6;
constexpr double kRintBig = 0x1.8p52;    // x + this rounds x to an integer, in the low bits of the sum
static __constant__ __attribute__((aligned(16))) double c_sctab[kSinTabWords];  // sine, high and low word
// LDS copy of the table for a block (every thread calls this, then a barrier follows)
__device__ __forceinline__ void stage_sctab(double* dst) {
  for (int i = threadIdx.x; i < kSinTab; i += blockDim.x) ((double2*)dst)[i] = ((const double2*)c_sctab)[i];
}

struct ScArg {
  dd S, C, r;   // table sine and cosine, r
  double s3;    // sin r - r
  dd c1;        // cos r - 1
};
__device__ __forceinline__ ScArg sc_arg(double x, const double* tab) {
  ScArg a;
  const double b = fma(x, k256OverPi, kRintBig), k = b - kRintBig;
  const double2* T = (const double2*)tab + (__double2loint(b) & (kCircle - 1));
  const double2 s = T[0], c = T[kCircle / 4];
  a.S = {s.x, s.y};
  a.C = {c.x, c.y};
  const dd kb = dd_two_prod(-k, kPio2B * 0x1p-7);
  const dd t = dd_two_sum(fma(-k, kPio2A * 0x1p-7, x), kb.hi);
  a.r = dd_fast_two_sum(t.hi, t.lo + fma(-k, kPio2C * 0x1p-7, kb.lo));
  const double rh = a.r.hi;
  const dd z = dd_two_prod(rh, rh);
  const double zl = fma(2.0 * rh, a.r.lo, z.lo);
  const double p = fma(z.hi, fma(z.hi, -1.0 / 5040.0, 1.0 / 120.0), -1.0 / 6.0);
  const double q = fma(z.hi, fma(z.hi, 1.0 / 40320.0, -1.0 / 720.0), 1.0 / 24.0);
  a.s3 = rh * (z.hi * p);
  a.c1 = {-0.5 * z.hi, fma(z.hi * z.hi, q, -0.5 * zl)};
  return a;
}
// P (1 + c1) + Q (r + s3) as an unevaluated sum
__device__ __forceinline__ dd sc_combine(dd P, dd Q, const ScArg& a) {
  const dd u = dd_two_prod(P.hi, a.c1.hi), v = dd_two_prod(Q.hi, a.r.hi);
  double lo = fma(P.hi, a.c1.lo, fma(Q.hi, a.s3, fma(Q.hi, a.r.lo, fma(Q.lo, a.r.hi, fma(P.lo, a.c1.hi, P.lo)))));
  lo += u.lo + v.lo;
  const dd w = dd_two_sum(u.hi, v.hi), s = dd_two_sum(P.hi, w.hi);
  return dd_fast_two_sum(s.hi, s.lo + (w.lo + lo));
}
__device__ __forceinline__ dd sc_sin(const ScArg& a) { return sc_combine(a.S, a.C, a); }
__device__ __forceinline__ dd sc_cos(const ScArg& a) { return sc_combine(a.C, dd{-a.S.hi, -a.S.lo}, a); }

__device__ inline void cr_sincos(double x, double* sn, double* cs, const double* tab = c_sctab) {
  if (fabs(x) < 1048576.0) {
    const ScArg a = sc_arg(x, tab);
    double s, c;
    if (ziv_round(sc_sin(a), &s) && ziv_round(sc_cos(a), &c)) {
      *sn = s;
      *cs = c;
      return;
    }
  }
  cr_sincos_dd(x, sn, cs);
}

__device__ inline double cr_sin(double x, const double* tab = c_sctab) {
  double out;
  if (fabs(x) < 1048576.0 && ziv_round(sc_sin(sc_arg(x, tab)), &out)) return out;
  return cr_sinq_dd(x, 0);
}
__device__ inline double cr_cos(double x, const double* tab = c_sctab) {
  double out;
  if (fabs(x) < 1048576.0 && ziv_round(sc_cos(sc_arg(x, tab)), &out)) return out;
  return cr_sinq_dd(x, 1);
}

// A quotient and a square root of doubles, rounded as the operators round them, taken apart so that
// quotients with one divisor share its reciprocal and a root shares it with the quotients by it.
//   recip(b): 1/b by two Newton steps from the hardware's estimate (23 bits); quot(a, R): a r with
//   one exact remainder added back (Markstein), which is the rounded quotient, as in the operator's
//   own sequence; left out is its scaling of operands with exponents beyond +-1000.  Zero,
//   infinite and NaN operands are put right by div_fixup.  4 instructions for each further quotient by the same
//   divisor instead of 11.
//   root1(a): for a >= 1; s ~ sqrt a and h ~ 1/(2 sqrt a) by Goldschmidt's iteration from the
//   estimate of 1/sqrt a, then two exact remainders added back; 1/s from 2h in one Newton step.
// Bit for bit the operators' results on 1e9 random operands each (divisors 1 to 2^40).  A push has
// eight quotients and two roots of this kind; with the table of the circle above, the lepton kernel
// of a collision of 1e6 electrons went from 3.75 to 3.29 ms for 100 steps.
struct Recip {
  double b, r;
};
__device__ __forceinline__ Recip recip(double b) {
  double r = __builtin_amdgcn_rcp(b);
  r = fma(fma(-b, r, 1.0), r, r);
  r = fma(fma(-b, r, 1.0), r, r);
  return {b, r};
}
__device__ __forceinline__ double quot(double a, const Recip& R) {
  const double q = a * R.r;
  return __builtin_amdgcn_div_fixup(fma(fma(-R.b, q, a), R.r, q), R.b, a);
}
__device__ __forceinline__ Recip root1(double a) {
  const double y = __builtin_amdgcn_rsq(a);
  double s = a * y, h = 0.5 * y;
  const double e = fma(-h, s, 0.5);
  s = fma(s, e, s);
  h = fma(h, e, h);
  s = fma(fma(-s, s, a), h, s);
  s = fma(fma(-s, s, a), h, s);
  if (a == INFINITY) s = a;
  const double r = 2.0 * h;
  return {s, fma(fma(-s, r, 1.0), r, r)};
}

// The same in FP32 (one Newton step from estimates of 23 bits; exponents beyond +-100 left out)
struct Recipf {
  float b, r;
};
__device__ __forceinline__ Recipf recip(float b) {
  const float r = __builtin_amdgcn_rcpf(b);
  return {b, fmaf(fmaf(-b, r, 1.0f), r, r)};
}
__device__ __forceinline__ float quot(float a, const Recipf& R) {
  const float q = a * R.r;
  return __builtin_amdgcn_div_fixupf(fmaf(fmaf(-R.b, q, a), R.r, q), R.b, a);
}
__device__ __forceinline__ Recipf root1(float a) {
  const float y = __builtin_amdgcn_rsqf(a);
  float s = a * y, h = 0.5f * y;
  const float e = fmaf(-h, s, 0.5f);
  s = fmaf(s, e, s);
  h = fmaf(h, e, h);
  s = fmaf(fmaf(-s, s, a), h, s);
  if (a == INFINITY) s = a;
  const float r = 2.0f * h;
  return {s, fmaf(fmaf(-s, r, 1.0f), r, r)};
}

// Fast paths of the correctly rounded exp and log (the same rounding test), both from tables:
//   exp: x = k ln2/64 + r (double-double, |r| <= 0.00542), e^x = 2^(k/64) (1 + r + r^2/2 + ...).
//        T_j = 2^(j/64) is a double-double; r^2/2 and the terms up to r^7/7! are below 2^-16 of the
//        result, so their double sum errs by less than 2^-69 of it.
//   log: x = m 2^e, m in [3/4, 3/2); c_j ~ 1/m with 9 bits, picked by the 7 leading bits of the
//        mantissa, so that m c_j = 1 + r exactly as a double-double, |r| <= 2^-7; log x =
//        e ln2 + L_j + r - r^2/2 + (r^3/3 - ... - r^10/10), L_j = -log c_j a double-double, the
//        first two terms in double-double and the rest (below 2^-15 of log1p r) in double.
//        c_j = 1 next to m = 1 on both sides, so log x keeps its relative accuracy there.
// About 45 and 60 instructions where the series without tables took 165 and 170.
constexpr int kLogCrTab = 128, kExpTab = 64;
constexpr int kMathTab = 3 * kLogCrTab + 2 * kExpTab;  // c_j, L_j (high, low) each; then T_j (high, low)
static __constant__ __attribute__((aligned(16))) double c_mathtab[kMathTab];
__device__ __forceinline__ void stage_mathtab(double* dst) {
  for (int i = threadIdx.x; i < kMathTab; i += blockDim.x) dst[i] = c_mathtab[i];
}
constexpr double k64OverLn2 = 0x1.71547652b82fep+6;
constexpr double kLn2o64A = 0x1.62e42fefa0000p-7;  // ln2 / 64 = A + B + C, A with 36 significant bits
constexpr double kLn2o64B = 0x1.cf79abc9e3b3ap-46;
constexpr double kLn2o64C = -0x1.ff0342542fc33p-100;

__device__ inline double cr_exp(double x, const double* tab = c_mathtab) {
  if (x > -700.0 && x < 709.0) {
    const double k = rint(x * k64OverLn2);
    const int ki = (int)k;
    const double* T = tab + 3 * kLogCrTab + 2 * (ki & (kExpTab - 1));
    const double th = T[0], tl = T[1];
    const dd kb = dd_two_prod(-k, kLn2o64B);
    dd r = dd_two_sum(fma(-k, kLn2o64A, x), kb.hi);  // x - k A is exact
    r = dd_fast_two_sum(r.hi, r.lo + (kb.lo - k * kLn2o64C));
    const double rh = r.hi;
    double q = fma(rh, 1.0 / 5040.0, 1.0 / 720.0);
    q = fma(rh, q, 1.0 / 120.0);
    q = fma(rh, q, 1.0 / 24.0);
    q = fma(rh, q, 1.0 / 6.0);
    q = fma(rh, q, 0.5);
    const double lo = fma(rh * rh, q, fma(rh, r.lo, r.lo));  // e^r - 1 = rh + lo
    const dd p = dd_two_prod(th, rh);
    const dd s = dd_fast_two_sum(th, p.hi);
    double out;
    if (ziv_round(dd_fast_two_sum(s.hi, s.lo + (p.lo + fma(th, lo, fma(tl, rh, tl)))), &out))
      return ldexp(out, ki >> 6);
  }
  return cr_exp_dd(x);
}

__device__ inline double cr_log(double x, const double* tab = c_mathtab) {
  if (x >= 0x1p-1021 && x < INFINITY) {
    int e;
    double m = frexp(x, &e);  // [1/2, 1)
    const double* T = tab + 3 * (int)((uint32_t)(__double_as_longlong(m) >> 45) & (kLogCrTab - 1));
    const double c = T[0], lh = T[1], ll = T[2];
    if (m < 0.75) {
      m *= 2.0;
      e -= 1;
    }
    const dd p = dd_two_prod(m, c);
    const dd r = dd_two_sum(p.hi - 1.0, p.lo);  // m c - 1 (p.hi - 1 is exact)
    const double rh = r.hi;
    const dd z = dd_two_prod(rh, rh);
    double q = fma(rh, -1.0 / 10.0, 1.0 / 9.0);
    q = fma(rh, q, -1.0 / 8.0);
    q = fma(rh, q, 1.0 / 7.0);
    q = fma(rh, q, -1.0 / 6.0);
    q = fma(rh, q, 1.0 / 5.0);
    q = fma(rh, q, -1.0 / 4.0);
    q = fma(rh, q, 1.0 / 3.0);
    // -r^2/2 = -z/2 - rh r.lo; here the low words and the terms from r^3 on
    double lo = fma(z.hi * rh, q, fma(-rh, r.lo, fma(-0.5, z.lo, r.lo)));
    const dd a = dd_two_sum(rh, -0.5 * z.hi);
    const double ed = (double)e;
    const dd l = dd_two_prod(ed, kLn2Hi);
    lo += fma(ed, kLn2Lo, ll + l.lo) + a.lo;
    const dd b = dd_two_sum(l.hi, lh), s = dd_two_sum(b.hi, a.hi);
    double out;
    if (ziv_round(dd_fast_two_sum(s.hi, s.lo + (b.lo + lo)), &out)) return out;
  }
  return cr_log_dd(x);
}

}  // namespace qedk
