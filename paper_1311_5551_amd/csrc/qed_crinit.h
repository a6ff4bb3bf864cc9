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
  if (e == hipSuccess && dev < 64) *done |= 1ull << dev;
  return e;
}

}  // namespace qedk
