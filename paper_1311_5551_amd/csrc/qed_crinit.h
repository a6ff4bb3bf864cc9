// Upload of the correctly rounded math's constants: each source file whose kernels use them holds
// its own copy, filled once per device.
#pragma once

#include <cmath>

#include "qed_device.h"

namespace qedk {

// Reciprocal factorials 1/n! as double-doubles (Dekker splits; dd / integer division with one
// exact remainder), uploaded once per device (a bit of *done each) for the correctly rounded device math.
static hipError_t upload_crmath(unsigned long long* done) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 64 && (*done >> dev) & 1ull) return hipSuccess;
  dd f[30];
  f[0] = {1.0, 0.0};
  for (int n = 1; n < 30; ++n) {
    const double q1 = f[n - 1].hi / n;
    const double p = q1 * n, pe = std::fma(q1, (double)n, -p);
    const double rem = ((f[n - 1].hi - p) - pe) + f[n - 1].lo;
    const double q2 = rem / n;
    const double s = q1 + q2;
    f[n] = {s, q2 - (s - q1)};
  }
  e = hipMemcpyToSymbol(HIP_SYMBOL(c_inv_fact), f, sizeof(f));
  // log table of fast_log: c_j = 1 / (centre of the j-th sub-interval of [1/2, 1)), L_j = -log c_j
  double lt[2 * kLogTab];
  for (int j = 0; j < kLogTab; ++j) {
    const double c = 1.0 / (0.5 + (j + 0.5) / (2.0 * kLogTab));
    lt[2 * j] = c;
    lt[2 * j + 1] = -std::log(c);
  }
  if (e == hipSuccess) e = hipMemcpyToSymbol(HIP_SYMBOL(c_logtab), lt, sizeof(lt));
  // sine table of the correctly rounded sin and cos: sin(j pi/256) as double-doubles
  // (relative error below 2^-100) by Taylor series in the same arithmetic
  auto two_sum = [](double a, double b) -> dd {
    const double s = a + b, bb = s - a;
    return {s, (a - (s - bb)) + (b - bb)};
  };
  auto fast = [](double a, double b) -> dd { return {a + b, b - ((a + b) - a)}; };
  auto add = [&](dd a, dd b) {
    const dd s = two_sum(a.hi, b.hi), t = two_sum(a.lo, b.lo);
    const dd u = fast(s.hi, s.lo + t.hi);
    return fast(u.hi, u.lo + t.lo);
  };
  auto mul = [&](dd a, dd b) {
    const double p = a.hi * b.hi;
    return fast(p, std::fma(a.hi, b.hi, -p) + (a.hi * b.lo + a.lo * b.hi));
  };
  dd sn[kSinTab];
  double ph[2 * kPhTab];
  const dd unit = {0x1.921fb54442d18p-7, 0x1.1a62633145c07p-61};  // pi / 256
  for (int j = 0; j <= kCircle / 8; ++j) {
    const dd x = mul(unit, dd{(double)j, 0.0}), z = mul(x, x), m = {-z.hi, -z.lo};
    dd ps = f[29], pc = f[28];
    for (int n = 13; n >= 0; --n) {
      ps = add(mul(ps, m), f[2 * n + 1]);
      pc = add(mul(pc, m), f[2 * n]);
    }
    ps = mul(ps, x);
    // the whole circle by symmetry: angles o pi/2 + x and o pi/2 - x
    const dd s4[4] = {ps, pc, {-ps.hi, -ps.lo}, {-pc.hi, -pc.lo}};
    for (int o = 0; o < 4; ++o) {
      sn[kCircle / 4 * o + j] = s4[o];
      sn[(kCircle / 4 * o - j) & (kCircle - 1)] = s4[o & 1 ? o : 2 - o];
    }
  }
  for (int j = kCircle; j < kSinTab; ++j) sn[j] = sn[j - kCircle];
  for (int j = 0; j < kPhTab; ++j) {
    ph[2 * j] = sn[j].hi;
    ph[2 * j + 1] = sn[j + kCircle / 4].hi;
  }
  if (e == hipSuccess) e = hipMemcpyToSymbol(HIP_SYMBOL(c_sctab), sn, sizeof(sn));
  if (e == hipSuccess) e = hipMemcpyToSymbol(HIP_SYMBOL(c_phtab), ph, sizeof(ph));
  // tables of the correctly rounded log and exp: c_j and -log c_j for the 128 sub-intervals of the
  // mantissa (log c = 2 atanh t, t = (c - 1)/(c + 1), in double-double), and 2^(j/64) by the
  // exponential's Taylor series
  auto div = [&](dd a, dd b) {  // long division, three digits
    const double q1 = a.hi / b.hi;
    dd r = add(a, mul(b, dd{-q1, 0.0}));
    const double q2 = r.hi / b.hi;
    r = add(r, mul(b, dd{-q2, 0.0}));
    return add(fast(q1, q2), dd{r.hi / b.hi, 0.0});
  };
  double mt[kMathTab];
  for (int j = 0; j < kLogCrTab; ++j) {
    const double mid = 0.5 + j / 256.0 + 1.0 / 512.0;                         // of [1/2 + j/256, + 1/256)
    double cj = std::rint((mid < 0.75 ? 0.5 : 1.0) / mid * 512.0) / 512.0;  // 1/m, m in [3/4, 3/2)
    if (j == 0 || j == kLogCrTab - 1) cj = 1.0;
    const dd t = div(dd{cj - 1.0, 0.0}, dd{cj + 1.0, 0.0}), t2 = mul(t, t);
    dd p = {0.0, 0.0};
    for (int n = 61; n >= 1; n -= 2) p = add(mul(p, t2), div(dd{1.0, 0.0}, dd{(double)n, 0.0}));
    const dd l = mul(mul(p, t), dd{-2.0, 0.0});
    mt[3 * j] = cj;
    mt[3 * j + 1] = l.hi;
    mt[3 * j + 2] = l.lo;
  }
  for (int j = 0; j < kExpTab; ++j) {
    const dd x = mul(dd{kLn2Hi, kLn2Lo}, dd{j / 64.0, 0.0});
    dd p = f[29];
    for (int n = 28; n >= 0; --n) p = add(mul(p, x), f[n]);
    mt[3 * kLogCrTab + 2 * j] = p.hi;
    mt[3 * kLogCrTab + 2 * j + 1] = p.lo;
  }
  if (e == hipSuccess) e = hipMemcpyToSymbol(HIP_SYMBOL(c_mathtab), mt, sizeof(mt));
  if (e == hipSuccess && dev < 64) *done |= 1ull << dev;
  return e;
}

}  // namespace qedk
