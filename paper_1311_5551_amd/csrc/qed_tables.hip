// Look-up table construction on the device (FP64), Sec. 3 of the paper with the
// functions of Appendix A (quantum synchrotron spectrum F, h) and Appendix B (T_pm, p_f).
//
// Quadrature design (independent of any CPU reference):
//  * for y >= 1, K_nu(y) and int_y^inf K_nu(t) dt from the integral representation
//      e^{-y} int_0^inf exp(-2 y sinh^2(t/2)) cosh(nu t) [/ cosh t] dt
//    by the trapezoid rule in t, which converges geometrically for this entire,
//    doubly-exponentially decaying integrand.  Steps 0.2, 0.1, 0.05 and 0.025 (at most
//    0.7/sqrt(y)) are strides of one node table per block, so a term costs one exponential.
//  * for y < 1, their ascending series (K_nu from I_{-nu} - I_nu; int_y^inf K_{5/3} =
//    2 K_{2/3}(y) - pi/sqrt(3) + int_0^y K_{1/3}, the last term by term): 11 terms in y^2/4, where
//    the trapezoid needs up to 375 for the small y that most of the spectrum's range has.
//  * synchrotron integrals in v = ln y, y = 2 xi / (3 eta (1 - xi)), xi = 2 chi/eta:
//      xi = a y / (1 + a y), 1 - xi = 1 / (1 + a y), a = 3 eta / 2,
//      dchi/chi = (1 - xi) dv,
//    so both ends of the spectrum are resolved without cancellation.  Composite
//    16-point Gauss-Legendre panels no wider than 0.25 in v; below v0 = -70 the
//    spectrum follows its chi^{1/3} power law and the tail is added in closed form.
//  * pair splits in theta with f = sin^2 theta (the table's own f grid is uniform
//    in theta), f (1 - f) = sin^2 theta cos^2 theta.
// One workgroup of 1024 threads per table row.  All nodes of a row are evaluated side by side: 16
// lanes take a 16-point panel and add it in a fixed order, panel sums go to LDS, and sums over
// panels run in panel order (deterministic).  Before, one thread searched the energy cut (80 serial
// integrands), Newton re-integrated the whole range at each step, and a thread summed each
// segment alone, the longest some 200 nodes of up to 375 terms each: 49 ms for the 256 x 256 rows
// against 0.1 ms now (the whole call with its copies: 51 -> 0.82 ms).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>

#include "qed_device.h"

namespace qedk {

struct GL16 {
  double x[16], w[16];
};

constexpr double kV0 = -70.0;       // lower end of the v = ln y integrals
constexpr double kPanel = 0.25;     // widest panel in v
constexpr int kRowThreads = 1024;
constexpr int kMaxRow = 1024;       // columns of a table row, at most
constexpr int kMaxPanels = 320;     // panels of [kV0, ln 745]
constexpr int kSer = 11;            // terms of the ascending series (y < 1)
constexpr int kNodes = 224;         // trapezoid nodes t = k kStep, y >= 1
constexpr double kStep = 0.025;
constexpr double kPiOverSqrt3 = 1.8137993642342178506;

// series coefficients in q = y^2/4, made on the host:
//   K_{2/3} = pi/sqrt3 ((y/2)^{-2/3} sum a q^k - (y/2)^{2/3} sum b q^k),  a = 1/(k! Gamma(k+1/3)), b = 1/(k! Gamma(k+5/3))
//   int_0^y K_{1/3} = pi/sqrt3 ((y/2)^{2/3} sum c q^k - (y/2)^{4/3} sum d q^k),
//     c = 1/(k! Gamma(k+2/3) (k+1/3)),  d = 1/(k! Gamma(k+4/3) (k+2/3))
struct BesselSeries {
  double a[kSer], b[kSer], c[kSer], d[kSer];
};

// trapezoid nodes: 2 sinh^2(t/2), cosh(2t/3), cosh(5t/3)/cosh t
struct BesselNodes {
  double s2[kNodes], c23[kNodes], j53[kNodes];
};
__device__ void fill_nodes(BesselNodes& n) {
  for (int k = threadIdx.x; k < kNodes; k += blockDim.x) {
    const double t = k * kStep, sh = sinh(0.5 * t);
    n.s2[k] = 2.0 * sh * sh;
    n.c23[k] = cosh(2.0 / 3.0 * t);
    n.j53[k] = cosh(5.0 / 3.0 * t) / cosh(t);
  }
  __syncthreads();
}

__device__ __forceinline__ double horner(const double* c, double q) {
  double s = c[kSer - 1];
#pragma unroll
  for (int k = kSer - 2; k >= 0; --k) s = fma(s, q, c[k]);
  return s;
}

// K_{2/3}(y) and, with J, int_y^inf K_{5/3}; y = e^v, 0 above 745 (below the FP64 range)
template <bool WANT_J>
__device__ __forceinline__ void bessel(const BesselSeries& S, const BesselNodes& N, double y, double v, double* K,
                                       double* J) {
  *K = 0.0;
  if (WANT_J) *J = 0.0;
  if (!(y < 745.0)) return;
  if (y < 1.0) {
    const double q = 0.25 * y * y;
    const double p = exp(2.0 / 3.0 * (v - 0.69314718055994530942));  // (y/2)^{2/3}
    const double k = kPiOverSqrt3 * (horner(S.a, q) / p - p * horner(S.b, q));
    *K = k;
    if (WANT_J) *J = 2.0 * k - kPiOverSqrt3 + kPiOverSqrt3 * p * (horner(S.c, q) - p * horner(S.d, q));
    return;
  }
  const int st = y <= 12.25 ? 8 : y <= 49.0 ? 4 : y <= 196.0 ? 2 : 1;
  double sk = 0.5, sj = 0.5;  // node t = 0: cosh = 1
  for (int k = st; k < kNodes; k += st) {
    const double a = y * N.s2[k];
    if (a > 52.0) break;  // e^-52 cosh(5t/3) is below 1e-19 of the sum
    const double e = exp(-a);
    sk = fma(e, N.c23[k], sk);
    if (WANT_J) sj = fma(e, N.j53[k], sj);
  }
  const double he = st * kStep * exp(-y);
  *K = he * sk;
  if (WANT_J) *J = he * sj;
}

// K_{1/3}(y): the same two forms
__device__ double bessel13(double y) {
  if (!(y < 745.0)) return 0.0;
  const double h = y > 12.25 ? 0.7 / sqrt(y) : 0.2;
  if (y < 1.0) {  // pi/sqrt3 ((y/2)^{-1/3} sum q^k/(k! Gamma(k+2/3)) - (y/2)^{1/3} sum q^k/(k! Gamma(k+4/3)))
    const double q = 0.25 * y * y, p = cbrt(0.5 * y);
    double ta = 1.0 / tgamma(2.0 / 3.0), tb = 1.0 / tgamma(4.0 / 3.0), sa = 0.0, sb = 0.0;
    for (int k = 0; k < kSer; ++k) {
      sa += ta;
      sb += tb;
      ta *= q / ((k + 1) * (k + 2.0 / 3.0));
      tb *= q / ((k + 1) * (k + 4.0 / 3.0));
    }
    return kPiOverSqrt3 * (sa / p - p * sb);
  }
  double s = 0.5;
  for (int k = 1; k < 64; ++k) {
    const double t = k * h, sh = sinh(0.5 * t), a = 2.0 * y * sh * sh;
    if (a > 52.0) break;
    s += exp(-a) * cosh(t / 3.0);
  }
  return h * s * exp(-y);
}

// number density F (1 - xi) and energy density (in units of eta/2) F xi (1 - xi) in v = ln y, for
// an eta row with a = 3 eta / 2: F / chi dchi = F (1 - xi) dv
__device__ __forceinline__ void densities(const BesselSeries& S, const BesselNodes& N, double a, double v, double* num,
                                          double* en) {
  const double y = exp(v), ay = a * y;
  const double om = 1.0 / (1.0 + ay), xi = ay * om;
  double k23, j53;
  bessel<true>(S, N, y, v, &k23, &j53);
  const double f = xi * xi * y * k23 + om * y * j53;
  *num = f * om;
  *en = f * xi * om;
}

// sum over the 16 lanes of a panel, in a fixed order
__device__ __forceinline__ double panel_sum(double v) {
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// Row i of h, g and P_chi.  Energy and number of every panel of [kV0, ln 745]; total energy of the
// spectrum (and g from it); v_c of the energy cut by Newton inside the panel that holds it;
// log-spaced chi grid from chi_min to eta/2; number integral of each segment; prefix sums
// normalised by h = the total number integral.
__global__ __launch_bounds__(kRowThreads) void k_build_eta_rows(qed_table_params p, GL16 gl, BesselSeries S, double* h,
                                                                  double* lnchi_min, double* dlnchi, double* P,
                                                                  double* g) {
  __shared__ BesselNodes N;
  __shared__ double gx[16], gw[16];
  __shared__ double sE[kMaxPanels], sN[kMaxPanels];
  __shared__ double sv[kMaxRow];              // v of the chi grid
  __shared__ int off[kMaxRow + 1];            // first panel of each segment
  __shared__ double sP[kMaxRow + kMaxPanels];  // panel sums of the segments
  __shared__ double seg[kMaxRow];
  __shared__ double sh_vc, sh_below;
  const int i = blockIdx.x, tid = threadIdx.x, q = tid & 15, grp = tid >> 4;
  constexpr int kGroups = kRowThreads / 16;
  if (tid < 16) {
    gx[tid] = gl.x[tid];
    gw[tid] = gl.w[tid];
  }
  fill_nodes(N);
  const double le0 = log(p.eta_min), le1 = log(p.eta_max);
  const double eta = exp(le0 + i * ((le1 - le0) / (p.n_eta - 1)));
  const double a = 1.5 * eta;
  const double stop = log(0.5 * eta);
  const double vmax = log(745.0);

  // panels of the whole range
  const int np = (int)ceil((vmax - kV0) / kPanel);  // 307
  const double w = (vmax - kV0) / np, hw = 0.5 * w;
  for (int k = grp; k < np; k += kGroups) {
    double dn, de;
    densities(S, N, a, kV0 + (k + 0.5) * w + hw * gx[q], &dn, &de);
    const double n = panel_sum(gw[q] * hw * dn), e = panel_sum(gw[q] * hw * de);
    if (q == 0) {
      sN[k] = n;
      sE[k] = e;
    }
  }
  __syncthreads();
  if (tid < 64) {  // one wave: the cut
    // tails below kV0: the spectrum ~ y^{1/3} in number and y^{4/3} in energy
    double n0, e0;
    densities(S, N, a, kV0, &n0, &e0);
    const double e_tail = 0.75 * e0;
    double e_tot = e_tail;
    for (int k = 0; k < np; ++k) e_tot += sE[k];
    const double target = p.cutoff_energy_frac * e_tot;
    // g = 3 sqrt3 / (2 pi eta^2) int_0^{eta/2} F dchi, and the energy density is in units of eta/2
    if (tid == 0) g[i] = 3.0 * sqrt(3.0) / (4.0 * kPi * eta) * e_tot;
    double Ec = e_tail, below = 3.0 * n0;
    int pc = 0;
    while (pc < np - 1 && Ec + sE[pc] < target) {
      Ec += sE[pc];
      below += sN[pc];
      ++pc;
    }
    const double va = kV0 + pc * w;
    double lo = va, hi = va + w, vc = va + 0.5 * w, part = 0.0;
    for (int it = 0; it < 80; ++it) {
      // lanes 0..15: the panel's part up to vc; the others: the density there
      const double half = 0.5 * (vc - va);
      double dn, de;
      densities(S, N, a, tid < 16 ? va + half + half * gx[q] : vc, &dn, &de);
      const double E = __shfl(panel_sum(gw[q] * half * de), 0);
      part = __shfl(panel_sum(gw[q] * half * dn), 0);
      const double rho = __shfl(de, 16);
      const double r = Ec + E - target;
      if (r > 0.0) hi = vc;
      else lo = vc;
      double nv = vc - r / rho;
      if (!(nv > lo && nv < hi)) nv = 0.5 * (lo + hi);  // stay inside the bracket
      const double d = nv - vc;
      vc = nv;
      if (!(fabs(d) >= 1e-15 * fabs(vc))) break;
    }
    {  // the number up to the cut
      const double half = 0.5 * (vc - va);
      double dn, de;
      densities(S, N, a, va + half + half * gx[q], &dn, &de);
      part = __shfl(panel_sum(gw[q] * half * dn), 0);
    }
    if (tid == 0) {
      sh_vc = vc;
      sh_below = below + part;
    }
  }
  __syncthreads();
  const double vc = sh_vc;
  // ln chi_min = ln(eta/2) + ln xi_c, xi_c = a y_c / (1 + a y_c)
  const double smin = stop + vc + log(a) - log1p(a * exp(vc));
  const int n = p.n_chi;
  const double ds = (stop - smin) / (n - 1);

  // segment j covers [s_{j-1}, s_j]; in v: v = d - ln a - ln(-expm1(d)), d = s - ln(eta/2)
  for (int j = tid; j < n; j += kRowThreads) {
    double v;
    if (j == 0) {
      v = vc;
    } else if (j >= n - 1) {
      v = vmax;
    } else {
      const double d = (smin + j * ds) - stop;
      v = d - log(a) - log(-expm1(d));
      v = v < vmax ? v : vmax;
    }
    sv[j] = v;
  }
  __syncthreads();
  if (tid == 0) {  // panels no wider than kPanel; none for an empty segment
    int o = 0;
    off[0] = 0;
    for (int j = 1; j < n; ++j) {
      off[j] = o;
      const double d = sv[j] - sv[j - 1];
      if (d > 0.0) o += max(1, (int)ceil(d / kPanel));
    }
    off[n] = o;
  }
  __syncthreads();
  const int total = min(off[n], kMaxRow + kMaxPanels);
  for (int k = grp; k < total; k += kGroups) {
    int lo = 1, hi = n - 1;  // the last segment that starts at or before panel k
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (off[mid] <= k) lo = mid;
      else hi = mid - 1;
    }
    const int cnt = off[lo + 1] - off[lo];
    const double pw = (sv[lo] - sv[lo - 1]) / cnt, ph = 0.5 * pw;
    double dn, de;
    densities(S, N, a, sv[lo - 1] + (k - off[lo] + 0.5) * pw + ph * gx[q], &dn, &de);
    const double s = panel_sum(gw[q] * dn) * ph;
    if (q == 0) sP[k] = s;
  }
  __syncthreads();
  for (int j = 1 + tid; j < n; j += kRowThreads) {
    double s = 0.0;
    for (int k = off[j]; k < min(off[j + 1], total); ++k) s += sP[k];
    seg[j] = s;
  }
  __syncthreads();
  if (tid == 0) {
    double cum = sh_below;
    seg[0] = cum;
    for (int j = 1; j < n; ++j) {
      cum += seg[j];
      seg[j] = cum;
    }
    h[i] = cum;
    lnchi_min[i] = smin;
    dlnchi[i] = ds;
  }
  __syncthreads();
  const double hv = seg[n - 1];
  for (int j = tid; j < n; j += kRowThreads) P[(size_t)i * n + j] = (j == n - 1) ? 1.0 : seg[j] / hv;
}

// unnormalised pair split density times df/dtheta, at f = sin^2 theta:
// (2 + g)/g K_{2/3}(1/(3 chi g)) sin(2 theta), g = f(1 - f) = sin^2 theta cos^2 theta
__device__ __forceinline__ double pair_integrand(const BesselSeries& S, const BesselNodes& N, double chi, double theta) {
  double s, c;
  sincos(theta, &s, &c);
  const double g = s * s * c * c;
  if (!(g > 0.0)) return 0.0;
  const double y = 1.0 / (3.0 * chi * g);
  double k23;
  bessel<false>(S, N, y, y < 1.0 ? log(y) : 0.0, &k23, nullptr);
  return (2.0 + g) / g * k23 * (2.0 * s * c);
}

// Row k of T and P_f: T = 0.16 K_{1/3}^2(2/(3 chi)) / chi; f_l = sin^2(pi l / 2(n_f - 1));
// each segment by two 16-point Gauss-Legendre panels in theta (32 lanes a segment); prefix sums
// normalised by k(chi)
__global__ __launch_bounds__(kRowThreads) void k_build_pair_rows(qed_table_params p, GL16 gl, BesselSeries S, double* T,
                                                                   double* fgrid, double* Pf, double* knorm) {
  __shared__ BesselNodes N;
  __shared__ double gx[16], gw[16];
  __shared__ double seg[kMaxRow];
  const int k = blockIdx.x, tid = threadIdx.x, q = tid & 15;
  if (tid < 16) {
    gx[tid] = gl.x[tid];
    gw[tid] = gl.w[tid];
  }
  fill_nodes(N);
  const double lc0 = log(p.chi_pair_min), lc1 = log(p.chi_pair_max);
  const double chi = exp(lc0 + k * ((lc1 - lc0) / (p.n_chi_pair - 1)));
  const int n = p.n_f;
  const double dth = 0.5 * kPi / (n - 1);
  if (tid == kRowThreads - 1) {
    const double k13 = bessel13(2.0 / (3.0 * chi));
    T[k] = 0.16 * k13 * k13 / chi;
  }
  for (int l0 = 1; l0 < n; l0 += kRowThreads / 32) {  // block-uniform trip count
    const int l = l0 + (tid >> 5);
    const double c = (l - 1) * dth + (((tid >> 4) & 1) + 0.5) * 0.5 * dth, hw = 0.25 * dth;
    const double v = l < n ? gw[q] * pair_integrand(S, N, chi, c + hw * gx[q]) : 0.0;
    const double half = panel_sum(v) * hw;
    const double s = half + __shfl_xor(half, 16);
    if ((tid & 31) == 0 && l < n) seg[l] = s;
  }
  __syncthreads();
  if (tid == 0) {
    double cum = 0.0;
    seg[0] = 0.0;
    for (int l = 1; l < n; ++l) {
      cum += seg[l];
      seg[l] = cum;
    }
    knorm[k] = cum;
  }
  __syncthreads();
  const double kn = seg[n - 1];
  for (int l = tid; l < n; l += kRowThreads) {
    Pf[(size_t)k * n + l] = (l == 0) ? 0.0 : (l == n - 1 ? 1.0 : seg[l] / kn);
    if (k == 0) {
      const double s = sin(l * dth);
      fgrid[l] = (l == 0) ? 0.0 : (l == n - 1 ? 1.0 : s * s);
    }
  }
}

}  // namespace qedk

// host-side launchers (called from qed_capi.hip)
namespace qedk {

// 16-point Gauss-Legendre nodes and weights on [-1, 1]: Newton iteration on P_16 from the
// Chebyshev-like starting guesses cos(pi (i - 1/4) / (n + 1/2)).
static GL16 gauss_legendre16() {
  GL16 g;
  const int n = 16;
  for (int i = 0; i < n / 2; ++i) {
    double z = cos(kPi * (i + 0.75) / (n + 0.5)), dp = 1.0;
    for (int it = 0; it < 100; ++it) {
      double pk = 1.0, pkm1 = 0.0;
      for (int k = 1; k <= n; ++k) {
        const double pkm2 = pkm1;
        pkm1 = pk;
        pk = ((2 * k - 1) * z * pkm1 - (k - 1) * pkm2) / k;
      }
      dp = n * (z * pk - pkm1) / (z * z - 1.0);
      const double dz = pk / dp;
      z -= dz;
      if (fabs(dz) < 1e-16) {
        // refresh the derivative at the final node
        pk = 1.0;
        pkm1 = 0.0;
        for (int k = 1; k <= n; ++k) {
          const double pkm2 = pkm1;
          pkm1 = pk;
          pk = ((2 * k - 1) * z * pkm1 - (k - 1) * pkm2) / k;
        }
        dp = n * (z * pk - pkm1) / (z * z - 1.0);
        break;
      }
    }
    g.x[i] = -z;
    g.x[n - 1 - i] = z;
    g.w[i] = g.w[n - 1 - i] = 2.0 / ((1.0 - z * z) * dp * dp);
  }
  return g;
}

static BesselSeries bessel_series() {
  BesselSeries S;
  long double f = 1.0L;  // k!
  for (int k = 0; k < kSer; ++k) {
    if (k) f *= k;
    S.a[k] = (double)(1.0L / (f * tgammal(k + 1.0L / 3.0L)));
    S.b[k] = (double)(1.0L / (f * tgammal(k + 5.0L / 3.0L)));
    S.c[k] = (double)(1.0L / (f * tgammal(k + 2.0L / 3.0L) * (k + 1.0L / 3.0L)));
    S.d[k] = (double)(1.0L / (f * tgammal(k + 4.0L / 3.0L) * (k + 2.0L / 3.0L)));
  }
  return S;
}

hipError_t launch_build_tables(const qed_table_params& p, double* h, double* lnchi_min, double* dlnchi, double* P,
                               double* T, double* fgrid, double* Pf, double* knorm, double* g, hipStream_t s) {
  const GL16 gl = gauss_legendre16();
  const BesselSeries ser = bessel_series();
  hipLaunchKernelGGL(k_build_eta_rows, dim3(p.n_eta), dim3(kRowThreads), 0, s, p, gl, ser, h, lnchi_min, dlnchi, P, g);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_build_pair_rows, dim3(p.n_chi_pair), dim3(kRowThreads), 0, s, p, gl, ser, T, fgrid, Pf, knorm);
  return hipGetLastError();
}

}  // namespace qedk
