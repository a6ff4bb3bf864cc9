// The device math of the kernels, one function over arrays, for the tests.
#include <hip/hip_runtime.h>

#include "../paper_1311_5551_amd/csrc/qed_crinit.h"

using namespace qedk;

enum { SIN, COS, SIN_OF_BOTH, COS_OF_BOTH, EXP, LOG, QUOT, ROOT, QUOT_BY_ROOT, FAST_SIN, FAST_COS, DD_SIN, DD_COS };

__global__ void k_f64(int fn, const double* a, const double* b, double* out, double* out2, long n) {
  const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double x = a[i], y = b[i];
  double r = 0.0, r2 = 0.0;
  switch (fn) {
    case SIN: r = cr_sin(x); break;
    case COS: r = cr_cos(x); break;
    case SIN_OF_BOTH: cr_sincos(x, &r, &r2); break;
    case COS_OF_BOTH: cr_sincos(x, &r2, &r); break;
    case EXP: r = cr_exp(x); break;
    case LOG: r = cr_log(x); break;
    case QUOT: r = quot(x, recip(y)); break;
    case ROOT: r = root1(x).b; break;
    case QUOT_BY_ROOT: r = quot(x, root1(y)); break;
    case FAST_SIN: r = fast_sin(x, c_phtab); break;
    case FAST_COS: r = fast_cos(x, c_phtab); break;
    case DD_SIN:
    case DD_COS: {
      const dd v = fn == DD_SIN ? sc_sin(sc_arg(x, c_sctab)) : sc_cos(sc_arg(x, c_sctab));
      r = v.hi;
      r2 = v.lo;
    }
  }
  out[i] = r;
  out2[i] = r2;
}
__global__ void k_f32(int fn, const float* a, const float* b, float* out, long n) {
  const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
  if (i >= n) return;
  out[i] = fn == QUOT ? quot(a[i], recip(b[i])) : fn == ROOT ? root1(a[i]).b : quot(a[i], root1(b[i]));
}

static hipError_t ready() {
  static unsigned long long done = 0;
  return upload_crmath(&done);
}
static dim3 blocks(long n) { return dim3((unsigned)((n + 255) / 256)); }

// arrays of n elements in device memory; synchronous; a HIP error code
extern "C" int probe_f64(int fn, const double* a, const double* b, double* out, double* out2, long n) {
  if (fn < SIN || fn > DD_COS || n < 1 || n > 1l << 30) return -1;
  const hipError_t e = ready();
  if (e != hipSuccess) return (int)e;
  hipLaunchKernelGGL(k_f64, blocks(n), dim3(256), 0, nullptr, fn, a, b, out, out2, n);
  return (int)hipDeviceSynchronize();
}
extern "C" int probe_f32(int fn, const float* a, const float* b, float* out, long n) {
  if ((fn != QUOT && fn != ROOT && fn != QUOT_BY_ROOT) || n < 1 || n > 1l << 30) return -1;
  hipLaunchKernelGGL(k_f32, blocks(n), dim3(256), 0, nullptr, fn, a, b, out, n);
  return (int)hipDeviceSynchronize();
}
