// The step of one particle, shared by the kernels that advance all particles by one step
// (qed_step.hip) and those that advance each particle by many (qed_multi.hip): the lepton push
// with its optical depth, the field-free drift, the emission event, the appended photon, and the
// photon's pair rate.  Both sets of kernels so give the same bits for the same particle and step.
#pragma once

#include "qed_device.h"
#include "qed_kernels.h"
#include "qed_mixed.h"

namespace qedk {

// position, momentum and optical depth of one lepton; FP32-mixed: (hi, lo) pairs
template <bool MIXED>
struct LepState {
  using Real = typename std::conditional<MIXED, float, double>::type;
  Real x, y, z, ux, uy, uz;
  float xl, yl, zl, uxl, uyl, uzl;  // FP32-mixed low words
  double tau;
  double g;  // gamma = sqrt(1 + u^2) of the momentum held (FP32-mixed: of hi + lo)
};
template <bool MIXED>
__device__ __forceinline__ void lepton_gamma(LepState<MIXED>& st) {
  double ux = st.ux, uy = st.uy, uz = st.uz;
  if (MIXED) {
    ux += st.uxl;
    uy += st.uyl;
    uz += st.uzl;
  }
  st.g = sqrt(1.0 + (ux * ux + uy * uy + uz * uz));
}

// Field components that are zero everywhere for a field kind.  The push leaves their terms out
// (a product with zero added to a finite value is that value), which in the linearly polarised
// pulse is half of its arithmetic.
template <int FK>
struct ZeroField {
  static constexpr bool pw = FK == QED_FIELD_LP_PULSE || FK == QED_FIELD_CP_WAVE || FK == QED_FIELD_CP_STANDING;
  static constexpr bool ex = pw || FK == QED_FIELD_GRID_CP_STANDING, bx = ex, ey = false, bz = false;
  static constexpr bool ez = FK == QED_FIELD_LP_PULSE, by = FK == QED_FIELD_LP_PULSE;
};
// c + (p q - r s), p q or r s left out where known to be zero
template <bool ZP, bool ZR, class T>
__device__ __forceinline__ T add_cross(T c, T p, T q, T r, T s) {
  if constexpr (ZP && ZR) return c;
  else if constexpr (ZP) return c - r * s;
  else if constexpr (ZR) return c + p * q;
  else return c + (p * q - r * s);
}
template <bool ZP, bool ZR, class T>
__device__ __forceinline__ T cross2(T p, T q, T r, T s) {
  if constexpr (ZP && ZR) return T(0);
  else if constexpr (ZP) return -(r * s);
  else if constexpr (ZR) return p * q;
  else return p * q - r * s;
}
template <bool Z, class T>
__device__ __forceinline__ T add_mul(T c, T p, T q) {
  if constexpr (Z) return c;
  else return c + p * q;
}
// g e + c, with e known to be zero: c
template <bool Z, class T>
__device__ __forceinline__ T mul_add(T g, T e, T c) {
  if constexpr (Z) return c;
  else return g * e + c;
}
// p0 q0 + p1 q1 + p2 q2 in this order
template <bool Z0, bool Z1, bool Z2, class T>
__device__ __forceinline__ T dot3(T p0, T q0, T p1, T q1, T p2, T q2) {
  if constexpr (Z0 && Z1) return Z2 ? T(0) : p2 * q2;
  else if constexpr (Z0) return add_mul<Z2>(p1 * q1, p2, q2);
  else return add_mul<Z2>(add_mul<Z1>(p0 * q0, p1, q1), p2, q2);
}
// eta = |gamma E + u x B|^2 - (u . E)^2, as a square root
template <int FK, class T>
__device__ __forceinline__ T eta_of(T g, T ux, T uy, T uz, const T E[3], const T B[3]) {
  using Z = ZeroField<FK>;
  const T ax = mul_add<Z::ex>(g, E[0], cross2<Z::bz, Z::by>(uy, B[2], uz, B[1]));
  const T ay = mul_add<Z::ey>(g, E[1], cross2<Z::bx, Z::bz>(uz, B[0], ux, B[2]));
  const T az = mul_add<Z::ez>(g, E[2], cross2<Z::by, Z::bx>(ux, B[1], uy, B[0]));
  const T ue = dot3<Z::ex, Z::ey, Z::ez>(ux, E[0], uy, E[1], uz, E[2]);
  const T r2 = dot3<Z::ex && Z::by && Z::bz, false, Z::ez && Z::bx && Z::by>(ax, ax, ay, ay, az, az) - ue * ue;
  return sqrt(r2 > T(0) ? r2 : T(0));
}

// what a lepton's step needs besides its state, uniform over a wave
struct LepEnv {
  double dt, hq;      // hq: half-step charge factor of the species
  float dtf;
  bool emit, rr, rr_q, d3;
  const double* sh;   // LDS: h (FP64), g with QED_RR_QUANTUM; the FP32 copy of h in sh32
  const float* sh32;
  const double* slog; // LDS: log table
  const double* sct;  // LDS: sine table of the correctly rounded sin and cos
};

// One full step of a lepton: field at the start-of-step position, Boris push, deterministic
// reaction or emission depth.  True (and the eta in *eta_out) when the optical depth reached
// zero.  *wk: field work; *rd: energy radiated deterministically.  after_push is called with the
// position before the push and v_z of the move, st holding the position after it (FP64 form).
template <int FK, bool MIXED, class AfterPush>
__device__ __forceinline__ bool lepton_full(LepState<MIXED>& st, const qed_field& sF, const FieldK& fK, double t,
                                            const StepConst& sc, const Tabs& tb, const LepEnv& e, double* eta_out,
                                            double* wk, double* rd, unsigned& n_range, unsigned& n_bad,
                                            AfterPush after_push) {
  using Z = ZeroField<FK>;
  bool pend = false;
  const double dt = e.dt, hq = e.hq;
  if constexpr (!MIXED) {
    double x = st.x, y = st.y, z = st.z;
    const double ux = st.ux, uy = st.uy, uz = st.uz;
    double tau = st.tau;
    double E[3], Bf[3];
    field_at<FK>(sF, x, y, t, E, Bf, &fK, e.sct);
    const double umx = add_mul<Z::ex>(ux, hq, E[0]), umy = add_mul<Z::ey>(uy, hq, E[1]),
                 umz = add_mul<Z::ez>(uz, hq, E[2]);
    const double hg = quot(hq, root1(1.0 + (umx * umx + umy * umy + umz * umz)));
    const double tx = hg * Bf[0], ty = hg * Bf[1], tz = hg * Bf[2];
    const double sf = quot(2.0, recip(1.0 + dot3<Z::bx, Z::by, Z::bz>(tx, tx, ty, ty, tz, tz)));
    const double sx = sf * tx, sy = sf * ty, sz = sf * tz;
    const double upx = add_cross<Z::bz, Z::by>(umx, umy, tz, umz, ty),
                 upy = add_cross<Z::bx, Z::bz>(umy, umz, tx, umx, tz),
                 upz = add_cross<Z::by, Z::bx>(umz, umx, ty, umy, tx);
    const double ulx = add_cross<Z::bz, Z::by>(umx, upy, sz, upz, sy),
                 uly = add_cross<Z::bx, Z::bz>(umy, upz, sx, upx, sz),
                 ulz = add_cross<Z::by, Z::bx>(umz, upx, sy, upy, sx);
    const double u1x = add_mul<Z::ex>(ulx, hq, E[0]), u1y = add_mul<Z::ey>(uly, hq, E[1]),
                 u1z = add_mul<Z::ez>(ulz, hq, E[2]);
    const Recip G1 = root1(1.0 + (u1x * u1x + u1y * u1y + u1z * u1z));
    const double g1 = G1.b;
    *wk = quot(2.0 * hq * dot3<Z::ex, Z::ey, Z::ez>(E[0], ulx + umx, E[1], uly + umy, E[2], ulz + umz), recip(g1 + st.g));
    x += quot(dt * u1x, G1);
    y += quot(dt * u1y, G1);
    if (e.d3) z += quot(dt * u1z, G1);
    after_push(st.x, st.y, x, y, quot(u1z, G1));
    double wx = u1x, wy = u1y, wz = u1z;  // stored momentum
    st.g = g1;
    if (e.rr) {
      // continuous reaction (eqs. 8, 9): gamma -> max(gamma - (2/3) alpha kappa eta^2 g dt, 1)
      // along u; the energy removed is what the stored momentum lost
      const double eta = eta_of<FK>(g1, u1x, u1y, u1z, E, Bf);
      if (eta > 0.0) {
        const double gq = e.rr_q ? lookup_g(e.sh, tb, eta, n_range) : 1.0;
        const double gn = fmax(g1 - sc.a_rr * eta * eta * gq * dt, 1.0);
        const double um = sqrt(u1x * u1x + u1y * u1y + u1z * u1z);
        const double s = um > 0.0 ? sqrt((gn - 1.0) * (gn + 1.0)) / um : 0.0;
        wx = s * u1x;
        wy = s * u1y;
        wz = s * u1z;
        st.g = sqrt(1.0 + (wx * wx + wy * wy + wz * wz));
        *rd = g1 - st.g;
      }
    }
    if (e.emit) {
      const double eta = eta_of<FK>(g1, u1x, u1y, u1z, E, Bf);
      if (eta > 0.0) {
        const double h = lookup_h(e.sh, e.slog, tb, eta, n_range);
        tau -= sc.a_gamma * quot(eta, G1) * h * dt;
        if (tau <= 0.0) {
          pend = true;
          *eta_out = eta;
        }
      }
    }
    if (!isfinite(tau) || !isfinite(wx) || !isfinite(wy) || !isfinite(wz)) ++n_bad;
    st.x = x;
    st.y = y;
    st.z = z;
    st.ux = wx;
    st.uy = wy;
    st.uz = wz;
    st.tau = tau;
  } else {
    float xh = st.x, xl = st.xl, yh = st.y, yl = st.yl, zh = st.z, zl = st.zl;
    float uxh = st.ux, uxl = st.uxl, uyh = st.uy, uyl = st.uyl, uzh = st.uz, uzl = st.uzl;
    double tau = st.tau;
    const float dtf = e.dtf;
    const double g0d = st.g;
    float E[3], Bf[3];
    field_at32<FK>(sF, fK, (double)xh + xl, (double)yh + yl, t, E, Bf);
    const float hqf = (float)hq;
    const float umx = add_mul<Z::ex>(uxh, hqf, E[0]), umy = add_mul<Z::ey>(uyh, hqf, E[1]),
                umz = add_mul<Z::ez>(uzh, hqf, E[2]);
    const float hg = quot(hqf, root1(1.0f + (umx * umx + umy * umy + umz * umz)));
    const float tx = hg * Bf[0], ty = hg * Bf[1], tz = hg * Bf[2];
    const float sf = quot(2.0f, recip(1.0f + dot3<Z::bx, Z::by, Z::bz>(tx, tx, ty, ty, tz, tz)));
    const float sx = sf * tx, sy = sf * ty, sz = sf * tz;
    const float upx = add_cross<Z::bz, Z::by>(umx, umy, tz, umz, ty),
                upy = add_cross<Z::bx, Z::bz>(umy, umz, tx, umx, tz),
                upz = add_cross<Z::by, Z::bx>(umz, umx, ty, umy, tx);
    // rotation increment (u+ - u-) formed directly, without cancellation
    const float rx = cross2<Z::bz, Z::by>(upy, sz, upz, sy), ry = cross2<Z::bx, Z::bz>(upz, sx, upx, sz),
                rz = cross2<Z::by, Z::bx>(upx, sy, upy, sx);
    comp_add(uxh, uxl, mul_add<Z::ex>(2.0f * hqf, E[0], rx));
    comp_add(uyh, uyl, mul_add<Z::ey>(2.0f * hqf, E[1], ry));
    comp_add(uzh, uzl, mul_add<Z::ez>(2.0f * hqf, E[2], rz));
    const Recipf G1 = root1(1.0f + (uxh * uxh + uyh * uyh + uzh * uzh));
    const float g1 = G1.b;
    comp_add(xh, xl, quot(dtf * uxh, G1));
    comp_add(yh, yl, quot(dtf * uyh, G1));
    if (e.d3) comp_add(zh, zl, quot(dtf * uzh, G1));
    // field work from the stored states (FP64), so the ledger closes on what is stored
    const double ux1 = (double)uxh + uxl, uy1 = (double)uyh + uyl, uz1 = (double)uzh + uzl;
    const double g1d = root1(1.0 + (ux1 * ux1 + uy1 * uy1 + uz1 * uz1)).b;
    *wk = g1d - g0d;
    st.g = g1d;
    if (e.rr) {
      // continuous reaction with eta in FP32 (as for emission) and the energy update in
      // FP64 on the stored momentum; the energy removed is what the stored pairs lost
      const double eta = (double)eta_of<FK>(g1, uxh, uyh, uzh, E, Bf);
      if (eta > 0.0) {
        const double gq = e.rr_q ? lookup_g(e.sh, tb, eta, n_range) : 1.0;
        const double gn = fmax(g1d - sc.a_rr * eta * eta * gq * dt, 1.0);
        const double um = sqrt(ux1 * ux1 + uy1 * uy1 + uz1 * uz1);
        const double s = um > 0.0 ? sqrt((gn - 1.0) * (gn + 1.0)) / um : 0.0;
        split_double(s * ux1, uxh, uxl);
        split_double(s * uy1, uyh, uyl);
        split_double(s * uz1, uzh, uzl);
        const double vx = (double)uxh + uxl, vy = (double)uyh + uyl, vz = (double)uzh + uzl;
        st.g = sqrt(1.0 + (vx * vx + vy * vy + vz * vz));
        *rd = g1d - st.g;
      }
    }
    if (e.emit) {
      const float eta = eta_of<FK>(g1, uxh, uyh, uzh, E, Bf);
      if (eta > 0.0f) {
        const float h = lookup32(e.sh32, tb.n_eta, tb.le0, tb.idle, eta, n_range, false);
        tau -= sc.a_gamma * dt * ((double)eta / (double)g1) * (double)h;  // FP32 look-up, FP64 decrement
        if (tau <= 0.0) {
          pend = true;
          *eta_out = (double)eta;
        }
      }
    }
    if (!isfinite(tau) || !isfinite(uxh) || !isfinite(uyh) || !isfinite(uzh)) ++n_bad;
    st.x = xh;
    st.xl = xl;
    st.y = yh;
    st.yl = yl;
    st.z = zh;
    st.zl = zl;
    st.ux = uxh;
    st.uxl = uxl;
    st.uy = uyh;
    st.uyl = uyl;
    st.uz = uzh;
    st.uzl = uzl;
    st.tau = tau;
  }
  return pend;
}

// The move of a field-free drift (outside the plane-wave pulse the Boris step reduces exactly to
// x += dt u / gamma, with u and tau unchanged).
template <bool MIXED>
struct DriftMove {
  typename LepState<MIXED>::Real dx, dy, dz;
  bool bad;  // non-finite gamma
};
template <bool MIXED>
__device__ __forceinline__ DriftMove<MIXED> drift_move(const LepState<MIXED>& st, const LepEnv& e) {
  DriftMove<MIXED> m;
  if constexpr (!MIXED) {
    const Recip g1 = recip(st.g);
    m.dx = quot(e.dt * st.ux, g1);
    m.dy = quot(e.dt * st.uy, g1);
    m.dz = quot(e.dt * st.uz, g1);
    m.bad = !isfinite(st.g);
  } else {
    const Recipf g1 = root1(1.0f + (st.ux * st.ux + st.uy * st.uy + st.uz * st.uz));
    m.dx = quot(e.dtf * st.ux, g1);
    m.dy = quot(e.dtf * st.uy, g1);
    m.dz = quot(e.dtf * st.uz, g1);
    m.bad = !isfinite(g1.b);
  }
  return m;
}
template <bool MIXED>
__device__ __forceinline__ void drift_apply(LepState<MIXED>& st, const DriftMove<MIXED>& m, bool d3) {
  if constexpr (!MIXED) {
    st.x = st.x + m.dx;
    st.y = st.y + m.dy;
    if (d3) st.z = st.z + m.dz;
  } else {
    comp_add(st.x, st.xl, m.dx);
    comp_add(st.y, st.yl, m.dy);
    if (d3) comp_add(st.z, st.zl, m.dz);
  }
}

// Whether a lepton at (high word of) x can be inside the plane-wave pulse at time t: an FP32 test
// of the phase with a margin far above its rounding error.
__device__ __forceinline__ bool near_pulse(double t, float tpf0, float psif_max, float xf) {
  const float psif = ((float)t - tpf0) - xf;
  const float m = 1e-5f * ((fabsf((float)t) + fabsf(tpf0)) + fabsf(xf)) + 1e-30f;
  return psif >= -m && psif <= psif_max + m;
}

// One emission (Sec. 3, Appendix A): chi from the 2-D inverse CDF at the emitter's eta, photon
// momentum (2 chi / eta) u, recoil, fresh optical depths.  The momentum of `st` (the high and low
// words in the FP32-mixed form) and its depth are updated; without a photon (a draw below the
// energy cut) only the depth is.
struct Emission {
  bool child;
  double kx, ky, kz, tau, defect;
  uint64_t uid;
};
template <bool MIXED>
__device__ __forceinline__ Emission emit_photon(const Tabs& tb, LepState<MIXED>& st, double eta, uint64_t uid,
                                                uint64_t step, uint64_t seed, uint64_t key,
                                                const double* mtab = c_mathtab) {
  Emission m;
  m.child = false;
  m.kx = m.ky = m.kz = m.tau = m.defect = 0.0;
  m.uid = 0;
  uint64_t r[4];
  philox4x64_10(uid, step, KIND_EMIT, 0, seed, key, r);
  double ux1 = st.ux, uy1 = st.uy, uz1 = st.uz;
  if constexpr (MIXED) {
    ux1 = (double)st.ux + st.uxl;
    uy1 = (double)st.uy + st.uyl;
    uz1 = (double)st.uz + st.uzl;
  }
  const double g1 = st.g;
  double chi;
  if (sample_chi(tb, eta, unit_open(r[0]), &chi, mtab)) {
    const double xi = 2.0 * chi / eta;
    double ux, uy, uz;
    if constexpr (MIXED) {
      // the emitter loses exactly the stored (FP32) photon momentum
      m.kx = (float)(xi * ux1);
      m.ky = (float)(xi * uy1);
      m.kz = (float)(xi * uz1);
      split_double(ux1 - m.kx, st.ux, st.uxl);
      ux = (double)st.ux + st.uxl;
      split_double(uy1 - m.ky, st.uy, st.uyl);
      uy = (double)st.uy + st.uyl;
      split_double(uz1 - m.kz, st.uz, st.uzl);
      uz = (double)st.uz + st.uzl;
    } else {
      m.kx = xi * ux1;
      m.ky = xi * uy1;
      m.kz = xi * uz1;
      ux = ux1 - m.kx;
      uy = uy1 - m.ky;
      uz = uz1 - m.kz;
      st.ux = ux;
      st.uy = uy;
      st.uz = uz;
    }
    const double g2 = sqrt(1.0 + (ux * ux + uy * uy + uz * uz));
    const double eps = sqrt(m.kx * m.kx + m.ky * m.ky + m.kz * m.kz);
    m.defect = g2 + eps - g1;
    st.g = g2;
    m.child = true;
    m.tau = optical_depth(r[3], mtab);
    m.uid = r[2];
  }
  st.tau = optical_depth(r[1], mtab);
  return m;
}

// A new photon's arrays, pair window and record; returns the packed window.  `pk`: its place in
// the workspace's per-photon arrays.
template <int FK, bool MIXED>
__device__ __forceinline__ uint32_t store_photon(const qed_species& G, long long slot, int64_t pk, bool d3, double cx,
                                                 double cy, double cz, const Emission& m, int32_t birth,
                                                 const qed_field& F, double eps_min, double cp_min,
                                                 const StepConst& sc,
                                                 uint32_t* win, void* rec) {
  using Real = typename std::conditional<MIXED, float, double>::type;
  as_global((Real*)G.x_dev)[slot] = (Real)cx;
  as_global((Real*)G.y_dev)[slot] = (Real)cy;
  if (d3) as_global((Real*)G.z_dev)[slot] = (Real)cz;
  as_global((Real*)G.ux_dev)[slot] = (Real)m.kx;
  as_global((Real*)G.uy_dev)[slot] = (Real)m.ky;
  as_global((Real*)G.uz_dev)[slot] = (Real)m.kz;
  as_global(G.tau_dev)[slot] = m.tau;
  as_global(G.uid_dev)[slot] = m.uid;
  as_global(G.birth_step_dev)[slot] = birth;
  // the steps in which the new photon can create a pair, from its stored state
  const double sx = (double)(Real)cx, sy = (double)(Real)cy;
  const double skx = (double)(Real)m.kx, sky = (double)(Real)m.ky, skz = (double)(Real)m.kz;
  const uint32_t wn = pack_window(photon_window(F, eps_min, cp_min, sc.t0, sc.dt, skx, sky, skz, sx,
                                                birth));
  win[pk] = wn;
  make_photon_rec<MIXED, FK>(((PhotonRecT<MIXED, FK>*)rec)[pk], F, sc.t0, sc.dt, skx, sky, skz, sx, sy, birth);
  return wn;
}

// Pair rate of a photon in one step: T(chi) and the decrement of its optical depth (eq. 3).
struct PairRate {
  double T, dtau;
};

// From the photon's direction, energy and birth (general fields)
template <int FK, bool MIXED>
__device__ __forceinline__ PairRate pair_rate(const qed_field& sF, const FieldK& fK, const Tabs& tb, const double* sT,
                                              const float* sT32, const double* sLog, const double* sPh, double rate,
                                              int64_t step, double t,
                                              double dt, typename LepState<MIXED>::Real kx,
                                              typename LepState<MIXED>::Real ky, typename LepState<MIXED>::Real kz,
                                              typename LepState<MIXED>::Real xb, typename LepState<MIXED>::Real yb,
                                              int32_t bs, unsigned& n_range) {
  using Real = typename LepState<MIXED>::Real;
  constexpr bool NEED_X = FK != QED_FIELD_UNIFORM;
  constexpr bool NEED_Y = FK == QED_FIELD_GRID_CP_STANDING || FK == QED_FIELD_GRID_FDTD;
  const Real eps = sqrt(kx * kx + ky * ky + kz * kz);
  const Real inv = (Real)1 / eps;
  const Real nx = kx * inv, ny = ky * inv, nz = kz * inv;
  double x = 0.0, y = 0.0;
  if (NEED_X) {
    const double age = (double)(step - (int64_t)bs) * dt;
    x = (double)xb + age * nx;
    if (NEED_Y) y = (double)yb + age * ny;
  }
  double chi, T;
  if (MIXED) {
    float E[3], Bf[3];
    field_at32<FK>(sF, fK, x, y, t, E, Bf);
    const float ax = E[0] + (ny * Bf[2] - nz * Bf[1]);
    const float ay = E[1] + (nz * Bf[0] - nx * Bf[2]);
    const float az = E[2] + (nx * Bf[1] - ny * Bf[0]);
    const float ne = nx * E[0] + ny * E[1] + nz * E[2];
    const float r2 = (ax * ax + ay * ay + az * az) - ne * ne;
    const float chif = 0.5f * (float)eps * sqrtf(r2 > 0.0f ? r2 : 0.0f);
    chi = chif;
    T = lookup32(sT32, tb.n_cp, tb.lc0, tb.idlc, chif, n_range, true);
  } else {
    double E[3], Bf[3];
    field_at<FK, false>(sF, x, y, t, E, Bf, &fK, sPh);
    const double ax = E[0] + (ny * Bf[2] - nz * Bf[1]);
    const double ay = E[1] + (nz * Bf[0] - nx * Bf[2]);
    const double az = E[2] + (nx * Bf[1] - ny * Bf[0]);
    const double ne = nx * E[0] + ny * E[1] + nz * E[2];
    const double r2 = (ax * ax + ay * ay + az * az) - ne * ne;
    chi = 0.5 * (double)eps * sqrt(r2 > 0.0 ? r2 : 0.0);
    T = lookup_T(sT, sLog, tb, chi, n_range);
  }
  return {T, rate * chi * T * (double)inv};  // FP64 (chi, T, 1/eps FP32 if mixed)
}

// In the plane-wave pulse, from the photon's record: psi(n) = A + n S, chi = c |e(psi)|, and the
// decrement a_pair |e| T(chi) S / 2 (PhotonRecPW)
template <bool MIXED>
__device__ __forceinline__ PairRate pair_rate_pw(const qed_field& sF, const FieldK& fK, const Tabs& tb,
                                                 const double* sT, const float* sT32, const double* sLog,
                                                 const double* sPh, double a_pair, double step, double A, double S,
                                                 double cr, unsigned& n_range) {
  const double psi = MIXED ? A + step * S : fma(step, S, A);
  double T = 0.0, ae = 0.0;
  if (psi >= 0.0 && psi <= sF.p[1]) {
    if (MIXED) {
      float sn, cs, d;
      fast_sincosf((float)(psi * fK.pi_over_len), &sn, &d);
      fast_sincosf(reduce_phase(psi + sF.p[3]), &d, &cs);
      const float e = fabsf((float)sF.p[0] * sn * sn * cs);
      ae = e;
      T = lookup32(sT32, tb.n_cp, tb.lc0, tb.idlc, (float)cr * e, n_range, true);
    } else {
      const double sn = fast_sin(psi * fK.pi_over_len, sPh), cs = fast_cos(psi + sF.p[3], sPh);
      ae = fabs(sF.p[0] * sn * sn * cs);
      T = lookup_T(sT, sLog, tb, cr * ae, n_range);
    }
  }
  return {T, 0.5 * a_pair * ae * T * S};
}

template <bool MIXED>
__device__ __forceinline__ void write_lepton(const qed_species& S, long long slot, double x, double y, double z,
                                             double ux, double uy, double uz, double tau, uint64_t uid, bool d3) {
  if (MIXED) {
    float h, l;
    split_double(x, h, l); ((float*)S.x_dev)[slot] = h; S.x_lo_dev[slot] = l;
    split_double(y, h, l); ((float*)S.y_dev)[slot] = h; S.y_lo_dev[slot] = l;
    if (d3) { split_double(z, h, l); ((float*)S.z_dev)[slot] = h; S.z_lo_dev[slot] = l; }
    split_double(ux, h, l); ((float*)S.ux_dev)[slot] = h; S.ux_lo_dev[slot] = l;
    split_double(uy, h, l); ((float*)S.uy_dev)[slot] = h; S.uy_lo_dev[slot] = l;
    split_double(uz, h, l); ((float*)S.uz_dev)[slot] = h; S.uz_lo_dev[slot] = l;
  } else {
    ((double*)S.x_dev)[slot] = x;
    ((double*)S.y_dev)[slot] = y;
    if (d3) ((double*)S.z_dev)[slot] = z;
    ((double*)S.ux_dev)[slot] = ux;
    ((double*)S.uy_dev)[slot] = uy;
    ((double*)S.uz_dev)[slot] = uz;
  }
  S.tau_dev[slot] = tau;
  S.uid_dev[slot] = uid;
}

// Pair creation by photon k of instance ii (when `want`): chi at the photon's position (FP64
// form: correctly rounded field), energy split f from the P_f table, electron with (1 - f) k
// and positron with f k at the position after the step, fresh optical depths, photon removed.
// Every lane of the wave calls this (the appends are wave-aggregated); lanes may be at different
// steps.  lep_born, if given, takes the step at which each new lepton is first stepped (per
// lepton slot, at acc.lep_off).
template <int FK, bool MIXED>
__device__ __forceinline__ void pair_event(const StepArgs& a, int ii, int64_t k, bool want, int64_t step, double t,
                                           int32_t* lep_born = nullptr) {
  using Real = typename std::conditional<MIXED, float, double>::type;
  const double dt = a.sc.dt;
  const qed_instance& I = a.inst[ii];
  const qed_species& S = I.s[2];
  const bool d3 = I.dims == 3;
  // the children's species and the photon's record offset, read before the first store (which the
  // compiler cannot tell apart from them), so that the loads share a memory round trip
  const qed_species Se = I.s[0], Sp = I.s[1];
  const int64_t moff = a.acc[ii].mover_off;
  double px = 0, py = 0, pz = 0, etau = 0, ptau = 0, ex = 0, ey = 0, ez = 0, pkx = 0, pky = 0, pkz = 0;
  double defect = 0.0, dropped_e = 0.0;
  unsigned n_drop = 0;
  uint64_t euid = 0, puid = 0;
  if (want) {
    const Real kxr = ((const Real*)S.ux_dev)[k], kyr = ((const Real*)S.uy_dev)[k], kzr = ((const Real*)S.uz_dev)[k];
    const Real xbr = ((const Real*)S.x_dev)[k], ybr = ((const Real*)S.y_dev)[k];
    const int32_t bs = S.birth_step_dev[k];
    const uint64_t uid = S.uid_dev[k];
    const Real eps = sqrt(kxr * kxr + kyr * kyr + kzr * kzr);
    const Real nx = kxr / eps, ny = kyr / eps, nz = kzr / eps;
    const double age = (double)(step - (int64_t)bs) * dt;
    const double x = (double)xbr + age * nx;
    const double y = (double)ybr + age * ny;
    double chi;
    if (MIXED) {
      float E[3], Bf[3];
      field_at32<FK>(I.field, field_k(I.field), x, y, t, E, Bf);
      const float ax = E[0] + (ny * Bf[2] - nz * Bf[1]);
      const float ay = E[1] + (nz * Bf[0] - nx * Bf[2]);
      const float az = E[2] + (nx * Bf[1] - ny * Bf[0]);
      const float ne = nx * E[0] + ny * E[1] + nz * E[2];
      const float r2 = (ax * ax + ay * ay + az * az) - ne * ne;
      chi = 0.5f * (float)eps * sqrtf(r2 > 0.0f ? r2 : 0.0f);
    } else {
      double E[3], Bf[3];
      field_at<FK, true>(I.field, x, y, t, E, Bf);
      const double ax = E[0] + (ny * Bf[2] - nz * Bf[1]);
      const double ay = E[1] + (nz * Bf[0] - nx * Bf[2]);
      const double az = E[2] + (nx * Bf[1] - ny * Bf[0]);
      const double ne = nx * E[0] + ny * E[1] + nz * E[2];
      const double r2 = (ax * ax + ay * ay + az * az) - ne * ne;
      chi = 0.5 * (double)eps * sqrt(r2 > 0.0 ? r2 : 0.0);
    }
    uint64_t r0[4], r1[4];
    philox4x64_10(uid, (uint64_t)step, KIND_PAIR, 0, I.seed, I.key_instance, r0);
    philox4x64_10(uid, (uint64_t)step, KIND_PAIR, 1, I.seed, I.key_instance, r1);
    const double f = sample_f(a.tb, chi, unit_open(r0[0]));
    const double kxd = kxr, kyd = kyr, kzd = kzr;
    pkx = f * kxd;
    pky = f * kyd;
    pkz = f * kzd;
    if (MIXED) {
      ex = kxd - pkx;
      ey = kyd - pky;
      ez = kzd - pkz;
    } else {
      ex = (1.0 - f) * kxd;
      ey = (1.0 - f) * kyd;
      ez = (1.0 - f) * kzd;
    }
    const double gp = sqrt(1.0 + (pkx * pkx + pky * pky + pkz * pkz));
    const double ge = sqrt(1.0 + (ex * ex + ey * ey + ez * ez));
    const double epsd = MIXED ? sqrt(kxd * kxd + kyd * kyd + kzd * kzd) : (double)eps;
    const double age1 = age + dt;
    px = (double)xbr + age1 * nx;
    py = (double)ybr + age1 * ny;
    pz = d3 ? (double)((const Real*)S.z_dev)[k] + age1 * nz : 0.0;
    euid = r0[1];
    puid = r0[2];
    etau = optical_depth(r0[3]);
    ptau = optical_depth(r1[0]);
    S.tau_dev[k] = kTauGone;
    a.win[moff + k] = kWinEmpty;
    defect = gp + ge - epsd;
  }
  // append electron and positron, one atomic per wave, instance and species
  long long se, spo;
  wave_reserve2_grouped(want, ii, Se.count_dev, Sp.count_dev, &se, &spo);
  if (want) {
    if (se < Se.capacity) {
      write_lepton<MIXED>(Se, se, px, py, pz, ex, ey, ez, etau, euid, d3);
      if (lep_born) lep_born[a.acc[ii].lep_off[0] + se] = (int32_t)(step + 1);
    } else {
      ++n_drop;
      dropped_e += sqrt(1.0 + (ex * ex + ey * ey + ez * ez));
    }
    if (spo < Sp.capacity) {
      write_lepton<MIXED>(Sp, spo, px, py, pz, pkx, pky, pkz, ptau, puid, d3);
      if (lep_born) lep_born[a.acc[ii].lep_off[1] + spo] = (int32_t)(step + 1);
    } else {
      ++n_drop;
      dropped_e += sqrt(1.0 + (pkx * pkx + pky * pky + pkz * pkz));
    }
  }
  add_event_stats(1, want, ii, a.acc, defect, dropped_e, want ? 1u : 0u, 0u, n_drop);
}

}  // namespace qedk
