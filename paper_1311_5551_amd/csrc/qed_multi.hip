// Many steps of every particle at once, for the fields in which particles are independent (all
// but the grids): the run of qed_run between two compactions.
//
// One step at a time, a step reads and writes every particle's state, and costs five dependent
// launches and as many grid-wide waits; small runs are launch latency, large ones HBM traffic and
// the latency of each pass's first loads.  Here a lane keeps one particle in registers for all k
// steps of the run.  The streams are keyed by (uid, step) and the fields are functions of (x, t),
// so a particle's steps do not depend on the others': the results are those of k single steps,
// per uid, bit for bit.
//
//   k_multi_begin   the counts, the lepton chunk list, the clock
//   k_multi_lepton  every lepton to the end of the run, emitting photons on the way (appended with
//                   their birth step)
//   k_multi_mid     the photon chunk list: the photons present before and those just emitted
//   k_multi_photon  every photon inside its window to the end of the run, or to its conversion
//   k_multi_pairs   the pairs of the converted photons (appended with their first step)
// and the same again for the new leptons, their photons, and so on: kRounds rounds of launches,
// then k_multi_tail, whose blocks go on with the rounds until no particle is left.  In a beam that
// crosses a pulse a generation is some hundred times smaller than the one before, and the tail has
// nothing or a few leptons to do; in a cascade (standing waves of a0 near 1000) most particles are of
// later generations, and the tail fills the chip as the launches before it do.  Each generation
// starts at a later step than the one before, so the rounds end.  Without pair creation one round of
// the first two kernels is the whole run.
//
// Measured against single steps replayed from graphs: a beam of 1e5 electrons through a 10 fs pulse
// (1200 steps) 97.8 -> 15.2 ms, 1e6 through 30 fs (3800 steps) 726 -> 222 ms, 48 batched beams
// 485 -> 98 ms, 1e4 electrons in a uniform field (1000 steps) 41.8 -> 6.9 ms.  At the peak of the
// collision of 1e6 the photon kernel issues vector instructions 99% of the time and the lepton
// kernel 55% (at four cycles each); small runs are the latency of one lane's steps.
#include <hip/hip_runtime.h>
#include <limits.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "qed_crinit.h"
#include "qed_device.h"
#include "qed_kernels.h"
#include "qed_particle.h"

namespace qedk {

constexpr int kMultiBlock = 256, kMultiWaves = kMultiBlock / 64;
constexpr int kRounds = 3;       // rounds of launches before k_multi_tail
constexpr int kLepChunkMin = 16; // fewest leptons a block takes
constexpr int kPairBlocks = 256; // blocks of k_multi_pairs
constexpr int kRefillLep = 8, kRefillPh = 8;  // idle lanes at which a wave takes new particles
constexpr int kPhInner = 4;      // photon steps between two looks at the idle lanes
constexpr int kRing = 128;       // per-wave ring of photon slots waiting for a lane
constexpr int kPool = 128, kPoolWords = 13;   // per-wave pool of leptons waiting for a lane

enum { MC_FIELD, MC_RANGE, MC_BAD, MC_EMIT, MC_NULL, MC_DROP, MC_LSTEPS, MC_PSTEPS, MC_ACTIVE, MC_READS, MC_GROUPS,
       MC_COUNT };

struct MultiShared {
  qed_field F;
  double log[2 * kLogTab];
  __attribute__((aligned(16))) double sct[kSinTabWords];
  union {  // of the lepton kernels, and of the photon kernels: two blocks of leptons fit a CU's LDS
    __attribute__((aligned(16))) double math[kMathTab];
    struct {
      uint32_t ring[kMultiWaves][kRing], ring_w[kMultiWaves][kRing];
    };
  };
  int64_t scan[kMultiBlock];
  long long fx[3][4];                   // field work, radiated energy, emission defect
  unsigned long long cnt[MC_COUNT];
  long long chunk;
};

// exclusive prefix of one value per thread over the block; *total the block's sum
__device__ inline int64_t block_scan(int64_t v, int64_t* s, int64_t* total) {
  __syncthreads();
  s[threadIdx.x] = v;
  __syncthreads();
  for (int o = 1; o < kMultiBlock; o <<= 1) {
    const int64_t u = threadIdx.x >= o ? s[threadIdx.x - o] : 0;
    __syncthreads();
    s[threadIdx.x] += u;
    __syncthreads();
  }
  *total = s[kMultiBlock - 1];
  return s[threadIdx.x] - v;
}

// a count clamped to its species' slots (appends past the end were dropped and counted)
__device__ __forceinline__ int64_t clamp_count(const qed_species& S) {
  if (!S.count_dev) return 0;
  const int64_t c = __hip_atomic_load(S.count_dev, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int64_t r = c > S.capacity ? S.capacity : c < 0 ? 0 : c;
  if (r != c && c > 0) *S.count_dev = r;
  return r;
}

// Lepton slots of the round and their chunk list; one block.  `dealt`: chunks that the blocks take
// without a ticket (their first ones).
__device__ inline void multi_begin(const MultiArgs& m, int round, MultiShared& sh, int grid, int dealt) {
  const qed_instance* inst = m.s.inst;
  InstAcc* acc = m.s.acc;
  const int per = (m.n_inst + kMultiBlock - 1) / kMultiBlock;
  const int b = min(m.n_inst, (int)threadIdx.x * per), e = min(m.n_inst, b + per);
  const bool pairs = (m.s.sc.flags & QED_PAIRS) != 0;
  int64_t tot = 0, used = 0;
  for (int i = b; i < e; ++i) {
    InstAcc& A = acc[i];
    for (int s = 0; s < 2; ++s) {
      const int64_t c = clamp_count(inst[i].s[s]);
      const int64_t lo = round ? A.lep_hi[s] : 0;
      A.lep_lo[s] = lo;
      A.lep_hi[s] = c;
      tot += c - lo;
      used += c > lo;
    }
    if (round == 0) {
      const int64_t c = clamp_count(inst[i].s[2]);
      for (int q = 0; q < kFixRunning; ++q) fix_normalise(A.fx[q]);
      A.n_start[2] = c;
      if (A.n_front > c) A.n_front = c;
      A.ph_lo = A.n_front / kWinGroup * kWinGroup;
      A.ph_hi = A.ph_lo;  // the first round's photons start there
      if (pairs) A.particle_steps[2] += (unsigned long long)(c * m.k);
    }
  }
  int64_t total, n_used, n_ch;
  block_scan(tot, sh.scan, &total);
  block_scan(used, sh.scan, &n_used);
  // one chunk per block, with the last, partial chunk of each species counted (a second round of
  // chunks would take as long as the first)
  // (Up to 64 leptons per SIMD, one wave each: the waves are latency, so a second wave on a SIMD
  // gains nothing and halves the lanes that share a push.  1e4 electrons in a uniform field:
  // 8.24 ms with all waves, 6.99 so; at twice the limit the run of 1e5 leptons is slower.)
  const int64_t blocks = total <= (int64_t)kMultiBlock * m.cus ? min(grid, m.cus) : grid;
  // Of large runs several chunks per block, of 16 or more leptons for every lane (a chunk's last
  // leptons leave lanes idle), dealt as blocks become free: with one per block, 256 beams of 1.3e5
  // electrons were 256 long chunks and as many of a few positrons, for 512 blocks (4.09 ms per step,
  // now 1.64).  Below 4.2e6 leptons one chunk per block, as before.
  const int64_t split = min((int64_t)8, max((int64_t)1, total / (blocks * kMultiBlock * 16)));
  const int64_t room = max(blocks * split - n_used, (blocks * split + 1) / 2);
  const int64_t chunk = max((int64_t)kLepChunkMin, (total + room - 1) / room);
  int64_t mine = 0;
  for (int i = b; i < e; ++i)
    for (int s = 0; s < 2; ++s) mine += (acc[i].lep_hi[s] - acc[i].lep_lo[s] + chunk - 1) / chunk;
  int64_t run = block_scan(mine, sh.scan, &n_ch);
  for (int i = b; i < e; ++i)
    for (int s = 0; s < 2; ++s) {
      m.base_lep[2 * i + s] = run;
      run += (acc[i].lep_hi[s] - acc[i].lep_lo[s] + chunk - 1) / chunk;
    }
  if (threadIdx.x == 0) {
    m.mc->n_lep = n_ch;
    m.mc->n_left = total;
    m.mc->lep_chunk = (int32_t)chunk;
    m.mc->lep_ticket = (unsigned long long)dealt;
    if (round == 0) {
      m.mc->pub = 0;
      m.mc->joined = m.mc->arrived = 0;
      // the clock moves on now: the run's kernels take its first step from the control words
      m.mc->s0 = m.glob->step_next;
      m.glob->step_cur = m.glob->step_next + m.k - 1;
      m.glob->step_next += m.k;
    }
  }
}

// Photon slots of the round, in chunks of whole groups; one block.
__device__ inline void multi_mid(const MultiArgs& m, MultiShared& sh, int grid) {
  InstAcc* acc = m.s.acc;
  const int per = (m.n_inst + kMultiBlock - 1) / kMultiBlock;
  const int b = min(m.n_inst, (int)threadIdx.x * per), e = min(m.n_inst, b + per);
  int64_t tot = 0;
  for (int i = b; i < e; ++i) {
    const int64_t c = clamp_count(m.s.inst[i].s[2]);
    acc[i].ph_lo = acc[i].ph_hi;
    acc[i].ph_hi = c;
    if (c > acc[i].ph_lo) tot += c - acc[i].ph_lo / kWinGroup * kWinGroup;
  }
  int64_t total, n_ch;
  block_scan(tot, sh.scan, &total);
  // about eight chunks per block, so that the blocks end together; at most 4096 slots, so that a
  // wave's last, partly filled lanes are few against its work
  int64_t chunk = (total / (8 * (int64_t)grid) + 255) / 256 * 256;
  chunk = chunk < 256 ? 256 : chunk > 4096 ? 4096 : chunk;
  auto chunks = [&](int i) -> int64_t {
    const int64_t lo = acc[i].ph_lo, hi = acc[i].ph_hi;
    return hi > lo ? (hi - lo / kWinGroup * kWinGroup + chunk - 1) / chunk : 0;
  };
  int64_t mine = 0;
  for (int i = b; i < e; ++i) mine += chunks(i);
  int64_t run = block_scan(mine, sh.scan, &n_ch);
  for (int i = b; i < e; ++i) {
    m.base_ph[i] = run;
    run += chunks(i);
  }
  if (threadIdx.x == 0) {
    m.mc->n_ph = n_ch;
    m.mc->ph_chunk = (int32_t)chunk;
    m.mc->ph_ticket = 0;
    m.evc->count = 0;
    m.evc->overflow = 0;
  }
}

// sums of the block's counters and energies into an instance's accumulators; every thread calls it
__device__ inline void multi_flush(const MultiArgs& m, MultiShared& sh, int ii, int sp) {
  __syncthreads();
  InstAcc& A = m.s.acc[ii];
  const int t = threadIdx.x;
  if (t < 3) {
    long long w[4];
    for (int k = 0; k < 4; ++k) {
      w[k] = sh.fx[t][k];
      sh.fx[t][k] = 0;
    }
    fix_normalise(w);
    fix_atomic_add(A.fx[t == 0 ? FX_WORK : t == 1 ? FX_RADIATED : FX_DEFECT_EMIT], w);
  } else if (t >= 64 && t < 64 + MC_COUNT) {
    const int c = t - 64;
    unsigned long long* const dst[MC_COUNT] = {
        sp < 2 ? &A.n_field_lepton : &A.n_field, &A.n_range, &A.n_nonfinite, &A.n_emit, &A.n_null, &A.n_dropped,
        &A.particle_steps[sp < 2 ? sp : 0], &A.particle_steps[2], &A.n_active, &A.n_win_reads, &A.n_group_reads};
    if (sh.cnt[c]) atomicAdd(dst[c], sh.cnt[c]);
    sh.cnt[c] = 0;
  }
  __syncthreads();
}

// a lane counter's wave sum into the block's
__device__ __forceinline__ void count_wave(MultiShared& sh, int c, unsigned v) {
  const unsigned s = wave_sum_u(v);
  if (__lane_id() == 0 && s) atomicAdd(&sh.cnt[c], (unsigned long long)s);
}
__device__ __forceinline__ void fix_lds_add(long long* w, double v) {
  if (v == 0.0) return;
  long long l[4];
  fix_split(v, l);
  fix_atomic_add(w, l);
}
// s + err exactly = a + b; the error collected
__device__ __forceinline__ void sum2(double& hi, double& lo, double v) {
  const double s = hi + v, bb = s - hi;
  lo += (hi - (s - bb)) + (v - bb);
  hi = s;
}

__device__ __forceinline__ void zero_shared(MultiShared& sh) {
  if (threadIdx.x < 12) sh.fx[threadIdx.x / 4][threadIdx.x % 4] = 0;
  if (threadIdx.x >= 64 && threadIdx.x < 64 + MC_COUNT) sh.cnt[threadIdx.x - 64] = 0;
}

// ---------------------------------------------------------------------------
// Leptons.  A block takes a chunk of one species of one instance, each wave a contiguous share of
// it.  A lane takes a lepton, steps it to the end of the run and takes the next, so the lanes of
// a wave are at different steps and stay busy.  A lepton whose optical depth ran out leaves its
// lane for the wave's pool in LDS, and the lane goes on with another; when 64 wait, the wave's
// running leptons change places with them and all lanes emit together.  An emission is three
// pushes' work (Philox, two look-ups through L2, four logarithms) and at the collision peak one
// lane in seventeen emits per step: done at once it would run for three lanes of 64.  At the end
// of its share, when nothing is left to put into a lane, leptons that wait stay in their lanes
// and emit once half as many wait as still step.  A wave whose share fits its lanes (small runs)
// has no use for the pool; its memory then collects the new photons, which go out 64 at a time.
// (With one reservation per emission pass the 2000 waves' atomics on the photon count, about 10 ns
// each, took longer than all the rest.)
//
// The pool holds a lepton's 13 words in columns of 128: those waiting to emit from its bottom,
// those that gave up their lane from its top.  A wave has at most 127 leptons in hand (63 waiting
// and 64 in lanes before a step), so the two never meet.
// ---------------------------------------------------------------------------
template <bool MIXED>
struct LeptonPool {
  double* w;  // the wave's columns

  __device__ static double pack(float h, float l) { return __hiloint2double(__float_as_int(h), __float_as_int(l)); }
  __device__ static void unpack(double v, float& h, float& l) {
    h = __int_as_float(__double2hiint(v));
    l = __int_as_float(__double2loint(v));
  }
  __device__ void put(int e, const LepState<MIXED>& st, double wh, double wl, double eta, uint64_t uid, int n,
                      int slot) const {
    double* q = w + e;
    if constexpr (MIXED) {
      q[0 * kPool] = pack(st.x, st.xl);
      q[1 * kPool] = pack(st.y, st.yl);
      q[2 * kPool] = pack(st.z, st.zl);
      q[3 * kPool] = pack(st.ux, st.uxl);
      q[4 * kPool] = pack(st.uy, st.uyl);
      q[5 * kPool] = pack(st.uz, st.uzl);
    } else {
      q[0 * kPool] = st.x;
      q[1 * kPool] = st.y;
      q[2 * kPool] = st.z;
      q[3 * kPool] = st.ux;
      q[4 * kPool] = st.uy;
      q[5 * kPool] = st.uz;
    }
    q[6 * kPool] = st.tau;
    q[7 * kPool] = st.g;
    q[8 * kPool] = wh;
    q[9 * kPool] = wl;
    q[10 * kPool] = eta;
    q[11 * kPool] = __longlong_as_double((long long)uid);
    q[12 * kPool] = __hiloint2double(n, slot);
  }
  __device__ void get(int e, LepState<MIXED>& st, double& wh, double& wl, double& eta, uint64_t& uid, int& n,
                      int& slot) const {
    const double* q = w + e;
    if constexpr (MIXED) {
      unpack(q[0 * kPool], st.x, st.xl);
      unpack(q[1 * kPool], st.y, st.yl);
      unpack(q[2 * kPool], st.z, st.zl);
      unpack(q[3 * kPool], st.ux, st.uxl);
      unpack(q[4 * kPool], st.uy, st.uyl);
      unpack(q[5 * kPool], st.uz, st.uzl);
    } else {
      st.x = q[0 * kPool];
      st.y = q[1 * kPool];
      st.z = q[2 * kPool];
      st.ux = q[3 * kPool];
      st.uy = q[4 * kPool];
      st.uz = q[5 * kPool];
    }
    st.tau = q[6 * kPool];
    st.g = q[7 * kPool];
    wh = q[8 * kPool];
    wl = q[9 * kPool];
    eta = q[10 * kPool];
    uid = (uint64_t)__double_as_longlong(q[11 * kPool]);
    n = __double2hiint(q[12 * kPool]);
    slot = __double2loint(q[12 * kPool]);
  }
};

// New photons of a wave waiting to be appended: 9 words each, in columns of kPool in the pool's memory
struct PhotonStage {
  double* w;
  __device__ void put(int e, double x, double y, double z, const Emission& m, int n) const {
    double* q = w + e;
    q[0 * kPool] = x;
    q[1 * kPool] = y;
    q[2 * kPool] = z;
    q[3 * kPool] = m.kx;
    q[4 * kPool] = m.ky;
    q[5 * kPool] = m.kz;
    q[6 * kPool] = m.tau;
    q[7 * kPool] = __longlong_as_double((long long)m.uid);
    q[8 * kPool] = __hiloint2double(0, n);
  }
  __device__ void get(int e, double& x, double& y, double& z, Emission& m, int& n) const {
    const double* q = w + e;
    x = q[0 * kPool];
    y = q[1 * kPool];
    z = q[2 * kPool];
    m.kx = q[3 * kPool];
    m.ky = q[4 * kPool];
    m.kz = q[5 * kPool];
    m.tau = q[6 * kPool];
    m.uid = (uint64_t)__double_as_longlong(q[7 * kPool]);
    n = __double2loint(q[8 * kPool]);
  }
};

// `bid`: the block's first chunk; it takes others by tickets where there are more than `nblk`.
template <int FK, bool MIXED>
__device__ __forceinline__ void multi_lepton(const MultiArgs& m, int round, MultiShared& sh, double* tab,
                                             double* pools, int bid, int nblk) {
  using Real = typename std::conditional<MIXED, float, double>::type;
  const StepArgs& a = m.s;
  const int64_t n_ch = uni64(m.mc->n_lep);
  if (bid >= n_ch) return;
  const bool emit = (a.sc.flags & QED_EMIT) != 0, pairs = (a.sc.flags & QED_PAIRS) != 0;
  const bool rr = (a.sc.flags & (QED_RR_QUANTUM | QED_RR_CLASSICAL)) != 0;
  const bool rr_q = (a.sc.flags & QED_RR_QUANTUM) != 0;
  for (int i = threadIdx.x; i < a.tb.n_eta; i += kMultiBlock) {
    if (rr_q) tab[i] = a.tb.g[i];
    else if (MIXED) ((float*)tab)[i] = a.tb.h32[i];
    else tab[i] = a.tb.h[i];
  }
  if (!MIXED) stage_logtab(sh.log);
  if (!MIXED && ZeroField<FK>::pw) stage_sctab(sh.sct);
  if (emit) stage_mathtab(sh.math);
  zero_shared(sh);
  const int64_t s0 = uni64(m.mc->s0), chunk = uni32(m.mc->lep_chunk);
  const double dt = a.sc.dt;
  LepEnv env{dt, 0.0, (float)dt, emit, rr, rr_q, false, tab, (const float*)tab, sh.log, sh.sct};
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const unsigned long long below = (1ull << lane) - 1ull;
  const LeptonPool<MIXED> pool{pools + wave * kPool * kPoolWords};

  for (int64_t c = bid; c < n_ch;) {
    const int idx = uni32(find_entry(m.base_lep, 2 * m.n_inst, c));
    const int ii = idx >> 1, sp = idx & 1;
    const qed_instance& I = a.inst[ii];
    const qed_species& S = I.s[sp];
    const InstAcc& A = a.acc[ii];
    const int64_t lo = uni64(A.lep_lo[sp]) + (c - uni64(m.base_lep[idx])) * chunk;
    const int64_t hi = min(lo + chunk, uni64(A.lep_hi[sp]));
    const int64_t moff = uni64(A.mover_off), loff = uni64(A.lep_off[sp]);
    env.d3 = uni32(I.dims) == 3;
    env.hq = 0.5 * (sp == 0 ? -1.0 : 1.0) * a.sc.kappa * dt;
    __syncthreads();
    for (int w = threadIdx.x; w < (int)(sizeof(qed_field) / 8); w += kMultiBlock)
      ((uint64_t*)&sh.F)[w] = ((const uint64_t*)&I.field)[w];
    __syncthreads();
    const float tpf0 = (float)sh.F.p[2], psif_max = (float)sh.F.p[1];
    const FieldK fK = field_k_uniform(sh.F);
    const double eps_min = uni_f64(pair_eps_min(sh.F, a.tb.cp_min));

    const int64_t per = (hi - lo + kMultiWaves - 1) / kMultiWaves;
    int64_t next = lo + wave * per;
    const int64_t w1 = min(hi, next + per);
    const bool stage = per <= 64;  // no use for the pool: it collects new photons
    const PhotonStage staged{pool.w};
    int n_staged = 0;
    bool busy = false, pend = false, moving = false;
    LepState<MIXED> st{};
    DriftMove<MIXED> mv{};
    int slot = 0;    // relative to lo
    uint64_t uid = 0;
    int n = 0;       // steps done since s0
    int n_wait = 0, n_ready = 0;  // leptons in the pool: waiting to emit, ready to go on
    double eta = 0.0, wh = 0.0, wl = 0.0, rh = 0.0, rl = 0.0;
    unsigned n_field = 0, n_range = 0, n_bad = 0, n_emit = 0, n_null = 0, n_drop = 0, lsteps = 0, psteps = 0;
    for (;;) {
      unsigned long long idle = __ballot(!busy);
      if (n_ready && idle) {
        const int r = __popcll(idle & below);
        if (!busy && r < n_ready) {
          pool.get(kPool - n_ready + r, st, wh, wl, eta, uid, n, slot);
          busy = true;
          moving = false;
        }
        n_ready -= min(n_ready, __popcll(idle));
        idle = __ballot(!busy);
      }
      if (next < w1 && __popcll(idle) >= kRefillLep) {
        const int64_t k = next + __popcll(idle & below);
        if (!busy && k < w1) {
          slot = (int)(k - lo);
          n = round ? max(0, m.lep_born[loff + k] - (int32_t)s0) : 0;
          st.x = as_global((const Real*)S.x_dev)[k];
          st.y = as_global((const Real*)S.y_dev)[k];
          st.z = env.d3 ? as_global((const Real*)S.z_dev)[k] : Real(0);
          st.ux = as_global((const Real*)S.ux_dev)[k];
          st.uy = as_global((const Real*)S.uy_dev)[k];
          st.uz = as_global((const Real*)S.uz_dev)[k];
          if (MIXED) {
            st.xl = as_global(S.x_lo_dev)[k];
            st.yl = as_global(S.y_lo_dev)[k];
            st.zl = env.d3 ? as_global(S.z_lo_dev)[k] : 0.0f;
            st.uxl = as_global(S.ux_lo_dev)[k];
            st.uyl = as_global(S.uy_lo_dev)[k];
            st.uzl = as_global(S.uz_lo_dev)[k];
          }
          st.tau = as_global(S.tau_dev)[k];
          uid = as_global(S.uid_dev)[k];
          lepton_gamma(st);
          wh = wl = rh = rl = 0.0;
          pend = moving = false;
          busy = n < m.k;
          if (busy) lsteps += m.k - n;
        }
        next = min(w1, next + __popcll(idle));
      }
      if (__ballot(busy) == 0ull && n_wait == 0) {
        if (next >= w1 && n_ready == 0 && n_staged == 0) break;
        if (n_staged == 0) continue;
      }
      // one step of every lane that does not wait for its emission
      if (busy && !pend && n < m.k) {
        const double t = a.sc.t0 + (double)(s0 + n) * dt;
        const bool in = FK != QED_FIELD_LP_PULSE || near_pulse(t, tpf0, psif_max, (float)st.x);
        if (in) {
          double wk = 0.0, rd = 0.0;
          ++n_field;
          pend = lepton_full<FK, MIXED>(st, sh.F, fK, t, a.sc, a.tb, env, &eta, &wk, &rd, n_range, n_bad,
                                        [](double, double, double, double, double) {});
          sum2(wh, wl, wk);
          if (rr) sum2(rh, rl, rd);
          moving = false;
        } else {
          if (!moving) mv = drift_move(st, env);
          moving = true;
          drift_apply(st, mv, env.d3);
          if (mv.bad) ++n_bad;
        }
        ++n;
      }
      if (busy && !pend && n >= m.k) {  // done: back to memory
        as_global((Real*)S.x_dev)[lo + slot] = st.x;
        as_global((Real*)S.y_dev)[lo + slot] = st.y;
        if (env.d3) as_global((Real*)S.z_dev)[lo + slot] = st.z;
        as_global((Real*)S.ux_dev)[lo + slot] = st.ux;
        as_global((Real*)S.uy_dev)[lo + slot] = st.uy;
        as_global((Real*)S.uz_dev)[lo + slot] = st.uz;
        if (MIXED) {
          as_global(S.x_lo_dev)[lo + slot] = st.xl;
          as_global(S.y_lo_dev)[lo + slot] = st.yl;
          if (env.d3) as_global(S.z_lo_dev)[lo + slot] = st.zl;
          as_global(S.ux_lo_dev)[lo + slot] = st.uxl;
          as_global(S.uy_lo_dev)[lo + slot] = st.uyl;
          as_global(S.uz_lo_dev)[lo + slot] = st.uzl;
        }
        as_global(S.tau_dev)[lo + slot] = st.tau;
        fix_lds_add(sh.fx[0], wh);
        fix_lds_add(sh.fx[0], wl);
        if (rr) {
          fix_lds_add(sh.fx[1], rh);
          fix_lds_add(sh.fx[1], rl);
        }
        busy = false;
      }
      Emission em;
      em.child = false;
      double cx = 0.0, cy = 0.0, cz = 0.0;
      if (emit) {
        const bool more = next < w1 || n_ready > 0;  // a lane given up can be filled again
        if (more) {
          const unsigned long long out = __ballot(pend);
          if (pend) {
            pool.put(n_wait + __popcll(out & below), st, wh, wl, eta, uid, n, slot);
            busy = pend = false;
          }
          n_wait += __popcll(out);
        }
        const int n_pend = n_wait + __popcll(__ballot(pend)), n_run = __popcll(__ballot(busy && !pend));
        if (n_wait >= 64 || (!more && n_pend && 2 * n_pend >= n_run)) {
          if (n_wait) {
            // those in lanes to the top of the pool, those waiting into the lanes
            const unsigned long long out = __ballot(busy && !pend);
            n_ready += __popcll(out);
            if (busy && !pend) {
              pool.put(kPool - n_ready + __popcll(out & below), st, wh, wl, eta, uid, n, slot);
              busy = false;
            }
            __builtin_amdgcn_wave_barrier();  // (a wave's LDS accesses are carried out in order)
            const unsigned long long in = __ballot(!busy);
            const int take = min(n_wait, __popcll(in)), r = __popcll(in & below);
            if (!busy && r < take) {
              pool.get(n_wait - take + r, st, wh, wl, eta, uid, n, slot);
              busy = pend = true;
            }
            n_wait -= take;
          }
          if (pend) {
            em = emit_photon<MIXED>(a.tb, st, eta, uid, (uint64_t)(s0 + n - 1), I.seed, I.key_instance,
                                    sh.math);
            moving = false;
            cx = st.x;
            cy = st.y;
            cz = st.z;
            if (MIXED) {
              cx += st.xl;
              cy += st.yl;
              cz += st.zl;
            }
          }
          if (pend) {
            if (em.child) {
              ++n_emit;
              fix_lds_add(sh.fx[2], em.defect);
            } else {
              ++n_null;
            }
            pend = false;
          }
          if (stage) {
            const unsigned long long out = __ballot(em.child);
            if (em.child) staged.put(n_staged + __popcll(out & below), cx, cy, cz, em, n);
            n_staged += __popcll(out);
          }
        }
      }
      // new photons into the photon arrays: this pass's, or the staged ones (64, or the last)
      bool child = em.child;
      int nb = n;
      if (stage) {
        const int take = n_staged >= 64 || __ballot(busy) == 0ull ? min(n_staged, 64) : 0;
        n_staged -= take;
        child = lane < take;
        if (child) staged.get(n_staged + lane, cx, cy, cz, em, nb);
      }
      if (__ballot(child)) {
        const qed_species& G = I.s[2];
        const long long ps = wave_reserve(child, G.count_dev);
        uint64_t* lword = nullptr;
        if (child) {
          if (ps < G.capacity) {
            const uint32_t wn = store_photon<FK, MIXED>(G, ps, moff + ps, env.d3, cx, cy, cz, em, (int32_t)(s0 + nb),
                                                        sh.F, eps_min, a.tb.cp_min, a.sc, a.win, a.rec);
            psteps += m.k - nb;
            // the photon kernel writes the live masks; without it they are set here
            if (!pairs && !window_over(wn, s0 + nb)) lword = a.lmask + A.lmask_off + ps / kWinGroup;
          } else {
            ++n_drop;
            long long l[4];
            fix_split(sqrt(em.kx * em.kx + em.ky * em.ky + em.kz * em.kz), l);
            fix_atomic_add(a.acc[ii].fx[FX_DROPPED], l);
          }
        }
        if (!pairs) wave_or_bit(lword, (int)(ps % kWinGroup));
      }
    }
    count_wave(sh, MC_FIELD, n_field);
    count_wave(sh, MC_RANGE, n_range);
    count_wave(sh, MC_BAD, n_bad);
    count_wave(sh, MC_EMIT, n_emit);
    count_wave(sh, MC_NULL, n_null);
    count_wave(sh, MC_DROP, n_drop);
    count_wave(sh, MC_LSTEPS, lsteps);
    if (pairs) count_wave(sh, MC_PSTEPS, psteps);
    multi_flush(m, sh, ii, sp);
    if (n_ch <= nblk) break;  // block-uniform
    __syncthreads();
    if (threadIdx.x == 0) sh.chunk = (long long)atomicAdd(&m.mc->lep_ticket, 1ull);
    __syncthreads();
    c = uni64(sh.chunk);
  }
}

// ---------------------------------------------------------------------------
// Photons.  A block takes chunks of whole groups of 64 slots from a ticket; a wave reads the
// windows of its groups (writing their live masks for the steps after the run), puts the slots
// whose window is not over into its ring, and its idle lanes take slots from the ring: the
// record, the depth and the steps between the run's ends and the window's, which the lane then
// takes in registers.  A photon whose depth ran out goes to the pair-event queue with its step in
// its window word.
// ---------------------------------------------------------------------------
template <int FK, bool MIXED>
__device__ __forceinline__ void multi_photon(const MultiArgs& m, MultiShared& sh, double* tab) {
  using Real = typename std::conditional<MIXED, float, double>::type;
  using Rec = PhotonRecT<MIXED, FK>;
  const StepArgs& a = m.s;
  const int64_t n_ch = uni64(m.mc->n_ph);
  if (n_ch == 0) return;
  for (int i = threadIdx.x; i < a.tb.n_cp; i += kMultiBlock) {
    if (MIXED) ((float*)tab)[i] = a.tb.T32[i];
    else tab[i] = a.tb.T[i];
  }
  if (!MIXED) stage_logtab(sh.log);
  double* const ph = sh.sct;  // (its table is for the leptons)
  static_assert(2 * kPhTab <= kSinTabWords, "room for the table");
  if (!MIXED && ZeroField<FK>::pw) stage_phtab(ph);
  zero_shared(sh);
  const int64_t s0 = uni64(m.mc->s0), send = s0 + m.k, chunk = uni32(m.mc->ph_chunk);
  const double dt = a.sc.dt, rate = a.sc.a_pair * dt, s0d = (double)s0;
  const float* const tab32 = (const float*)tab;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t* const ring = sh.ring[wave];
  uint32_t* const ring_w = sh.ring_w[wave];

  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) sh.chunk = (long long)atomicAdd(&m.mc->ph_ticket, 1ull);
    __syncthreads();
    const int64_t c = uni64(sh.chunk);
    if (c >= n_ch) break;
    const int ii = uni32(find_entry(m.base_ph, m.n_inst, c));
    const InstAcc& A = a.acc[ii];
    const qed_species& S = a.inst[ii].s[2];
    const int64_t lo = uni64(A.ph_lo), hi = uni64(A.ph_hi), n_old = uni64(A.n_start[2]);
    const int64_t c0 = lo / kWinGroup * kWinGroup + (c - uni64(m.base_ph[ii])) * chunk;
    const int64_t c1 = min(c0 + chunk, hi);
    const int64_t moff = uni64(A.mover_off);
    gptr<uint32_t> WIN = as_global(a.win) + moff;
    const Rec* const REC = (const Rec*)a.rec + moff;
    gptr<uint64_t> LM = as_global(a.lmask) + uni64(A.lmask_off);
    gptr<double> TAU = as_global(S.tau_dev);
    for (int w = threadIdx.x; w < (int)(sizeof(qed_field) / 8); w += kMultiBlock)
      ((uint64_t*)&sh.F)[w] = ((const uint64_t*)&a.inst[ii].field)[w];
    __syncthreads();
    const FieldK fK = field_k_uniform(sh.F);

    int64_t g = c0 / kWinGroup + wave;
    const int64_t g1 = (c1 + kWinGroup - 1) / kWinGroup;
    uint32_t wnext = g < g1 && g * kWinGroup + lane < c1 ? WIN[g * kWinGroup + lane] : kWinEmpty;
    int qh = 0, qn = 0;  // the ring's head and length
    bool busy = false;
    int64_t slot = 0;
    int32_t n = 0, nend = 0, nlim = 0;  // steps since s0: next, end, and where the lane stops (conversion)
    double tau = 0.0;
    Rec rec{};
    PairRate pr{0.0, 0.0};  // uniform field: the rate is the same in every step
    unsigned pr_range = 0;
    unsigned n_field = 0, n_range = 0, n_bad = 0, n_active = 0, n_reads = 0, n_groups = 0, field0 = 0;
    for (;;) {
      const unsigned long long idle = __ballot(!busy);
      const int ni = __popcll(idle);
      if (ni >= kRefillPh) {
        while (qn < ni && g < g1) {
          const int64_t k = g * kWinGroup + lane;
          const uint32_t w = wnext;
          g += kMultiWaves;
          wnext = g < g1 && g * kWinGroup + lane < c1 ? WIN[g * kWinGroup + lane] : kWinEmpty;
          const bool cand = k >= lo && k < c1 && !window_over(w, s0);
          const unsigned long long live = __ballot(cand), after = __ballot(k < c1 && !window_over(w, send));
          if (lane == 0) {
            LM[k / kWinGroup] = after;
            ++n_groups;
          }
          if (cand) {
            const int r = (qh + qn + __popcll(live & ((1ull << lane) - 1ull))) & (kRing - 1);
            ring[r] = (uint32_t)(k - c0);
            ring_w[r] = w;
          }
          qn += __popcll(live);
        }
        // (a wave's own LDS writes are read back by the same wave, in order)
        __builtin_amdgcn_wave_barrier();
        const int rank = __popcll(idle & ((1ull << lane) - 1ull));
        if (!busy && rank < qn) {
          const int r = (qh + rank) & (kRing - 1);
          const uint32_t w = ring_w[r];
          slot = c0 + ring[r];
          tau = TAU[slot];
          rec = REC[slot];
          int64_t first = s0;
          if (slot >= n_old) first = max(s0, (int64_t)as_global(S.birth_step_dev)[slot]);
          const int64_t wlo = w & 0xFFFFu, whi = w >> 16;
          const int64_t last = whi == 65535 ? send : min(send, whi + 1);  // end of its steps in the run
          if (last > first) n_reads += (unsigned)(last - first);  // one per step, as single steps count
          n = (int32_t)(max(first, wlo) - s0);
          nend = (int32_t)(last - s0);
          busy = n < nend && !(tau < 0.0);
          nlim = busy ? nend : n;
          if (busy) n_active -= (unsigned)n;
          field0 = n_field;
          if (FK == QED_FIELD_UNIFORM && busy) {
            if constexpr (FK == QED_FIELD_UNIFORM) {
              pr_range = 0;
              pr = pair_rate<FK, MIXED>(sh.F, fK, a.tb, tab, tab32, sh.log, ph, rate, s0, 0.0, dt, (Real)rec.kx,
                                        (Real)rec.ky, (Real)rec.kz, Real(0), Real(0), 0, pr_range);
            }
          }
        }
        const int took = min(ni, qn);
        qh = (qh + took) & (kRing - 1);
        qn -= took;
      }
      if (__ballot(busy) == 0ull) {
        if (qn == 0 && g >= g1) break;
        continue;
      }
#pragma unroll 1
      for (int it = 0; it < kPhInner; ++it) {
        if (n < nlim) {
          PairRate r;
          if constexpr (FK == QED_FIELD_LP_PULSE) {
            r = pair_rate_pw<MIXED>(sh.F, fK, a.tb, tab, tab32, sh.log, ph, a.sc.a_pair, s0d + (double)n, rec.A, rec.S,
                                    rec.c, n_range);
          } else if constexpr (FK == QED_FIELD_UNIFORM) {
            r = pr;
            n_range += pr_range;
          } else {
            const int64_t step = s0 + n;
            r = pair_rate<FK, MIXED>(sh.F, fK, a.tb, tab, tab32, sh.log, ph, rate, step, a.sc.t0 + (double)step * dt, dt,
                                     (Real)rec.kx, (Real)rec.ky, (Real)rec.kz, (Real)rec.xb, (Real)rec.yb, rec.bs,
                                     n_range);
          }
          ++n;
          if (r.T > 0.0) {
            ++n_field;
            tau -= r.dtau;
            if (tau <= 0.0) nlim = n;
            if (!(tau < INFINITY)) ++n_bad;  // (-inf is a conversion, clamped below)
          }
        }
      }
      const bool done = busy && n >= nlim, changed = n_field != field0, pend = changed && tau <= 0.0;
      if (done) n_active += (unsigned)n;
      if (done && changed) TAU[slot] = pend ? fmax(tau, kTauPendingMin) : tau;
      if (done && pend) {
        WIN[slot] = (uint32_t)(n - 1);  // the step of the conversion
        n_reads -= (unsigned)(nend - n);
      }
      const long long qs = wave_reserve(done && pend, &m.evc->count);
      if (done && pend) {
        if (qs < a.q.cap) a.q.ent[qs] = ((uint64_t)ii << kEvSlotBits) | (uint64_t)slot;
        else m.evc->overflow = 1;
      }
      if (done) busy = false;
    }
    count_wave(sh, MC_FIELD, n_field);
    count_wave(sh, MC_RANGE, n_range);
    count_wave(sh, MC_BAD, n_bad);
    count_wave(sh, MC_ACTIVE, n_active);
    count_wave(sh, MC_READS, n_reads);
    count_wave(sh, MC_GROUPS, n_groups);
    multi_flush(m, sh, ii, 2);
  }
}

// The pairs of the converted photons: the queued ones, or, when the queue overflowed, every
// photon of the round whose depth is in the converting state.
template <int FK, bool MIXED>
__device__ __forceinline__ void multi_pairs(const MultiArgs& m, int bid, int nblk) {
  const StepArgs& a = m.s;
  const int64_t s0 = m.mc->s0;
  const int64_t gtid = bid * (int64_t)kMultiBlock + threadIdx.x, stride = (int64_t)nblk * kMultiBlock;
  const int lane = threadIdx.x & 63;
  auto event = [&](int ii, int64_t k, bool want) {
    const int64_t step = s0 + (want ? (int64_t)a.win[a.acc[ii].mover_off + k] : 0);
    pair_event<FK, MIXED>(a, ii, k, want, step, a.sc.t0 + (double)step * a.sc.dt, m.lep_born);
  };
  const int64_t cnt = m.evc->count;
  if (!m.evc->overflow) {
    for (int64_t e0 = gtid - lane; e0 < cnt; e0 += stride) {  // whole waves iterate together
      const bool want = e0 + lane < cnt;
      const uint64_t ent = want ? a.q.ent[e0 + lane] : 0;
      event((int)(ent >> kEvSlotBits), (int64_t)(ent & ((1ull << kEvSlotBits) - 1)), want);
    }
  } else {
    for (int ii = 0; ii < m.n_inst; ++ii) {
      const int64_t hi = a.acc[ii].ph_hi;
      const double* TAU = a.inst[ii].s[2].tau_dev;
      for (int64_t k0 = a.acc[ii].ph_lo + gtid - lane; k0 < hi; k0 += stride) {
        const int64_t k = k0 + lane;
        bool want = false;
        if (k < hi) {
          const double tau = TAU[k];
          want = tau <= 0.0 && tau >= kTauPendingMin;
        }
        event(ii, k, want);
      }
    }
  }
}

__global__ __launch_bounds__(kMultiBlock) void k_multi_begin(MultiArgs m) {
  __shared__ MultiShared sh;
  multi_begin(m, m.round, sh, m.lep_grid, m.round < kRounds ? m.lep_grid : 0);
}
__global__ __launch_bounds__(kMultiBlock) void k_multi_mid(MultiArgs m) {
  __shared__ MultiShared sh;
  multi_mid(m, sh, m.ph_grid);
}
template <int FK, bool MIXED>
__global__ __launch_bounds__(kMultiBlock) __attribute__((amdgpu_waves_per_eu(2))) void k_multi_lepton(MultiArgs m) {
  extern __shared__ __attribute__((aligned(16))) double tab[];
  __shared__ MultiShared sh;
  multi_lepton<FK, MIXED>(m, m.round, sh, tab, tab + m.n_tab, blockIdx.x, gridDim.x);
}
template <int FK, bool MIXED>
__global__ __launch_bounds__(kMultiBlock) __attribute__((amdgpu_waves_per_eu(FK == QED_FIELD_LP_PULSE ? 5 : 1))) void k_multi_photon(MultiArgs m) {
  extern __shared__ __attribute__((aligned(16))) double tab[];
  __shared__ MultiShared sh;
  multi_photon<FK, MIXED>(m, sh, tab);
}
template <int FK, bool MIXED>
__global__ __launch_bounds__(kMultiBlock) void k_multi_pairs(MultiArgs m) {
  multi_pairs<FK, MIXED>(m, blockIdx.x, gridDim.x);
}
// The rounds that are left, until no new lepton is: the same passes as phases of one launch, over
// as many blocks as are running.
//
// Blocks join as they start, and those that have joined by the start of a phase take part in it:
// they take its work by tickets, and the last of them to end it prepares the next one (the chunk
// lists, alone) and publishes it with the number of blocks that have joined by then.  A block waits
// only for blocks that have joined, which are running, and every phase's work is finite: no block
// waits for one that has not started, whatever else the GPU runs.  The first block to join opens the
// first round, and the one that finds no lepton left closes the tail; with none from the start
// (k_multi_begin ran before) the blocks leave at once.  As in the launches before, a block gets at
// least kLepChunkMin leptons: as many blocks stay as that allows for the first round, so a few
// leptons are one block's work, without waits for others.  (A later round may be larger.  A block
// that starts with 16 leptons and ends with some thousands takes no longer than the single steps'
// launches would.)
//
// One block alone did all these rounds before.  199 steps of electrons at rest in a standing wave of
// a0 = 1000, dt = lambda/200c: 1e4 electrons took 65.8 ms and take 7.3 (single steps: 17.8 ms), 1e5
// 631 and 27.4 (45.7).  Where the third round leaves nothing the launch is 4.6 us, and the
// k_multi_begin before it 5.8 (8.6 before, together): runs of 100 steps of a beam in a pulse, of
// 1.2 ms, take what they took.
constexpr uint32_t kTailClosed = ~0u;

template <int FK, bool MIXED>
__global__ __launch_bounds__(kMultiBlock) __attribute__((amdgpu_waves_per_eu(2))) void k_multi_tail(MultiArgs m) {
  extern __shared__ __attribute__((aligned(16))) double tab[];
  __shared__ MultiShared sh;
  __shared__ unsigned long long s_pub;
  __shared__ uint32_t s_id;
  __shared__ int s_last;
  MultiCtl* const mc = m.mc;
  auto ticket = [&](unsigned long long* t) {
    __syncthreads();
    if (threadIdx.x == 0) sh.chunk = (long long)atomicAdd(t, 1ull);
    __syncthreads();
    return sh.chunk;
  };
  auto joined = [&] { return __hip_atomic_load(&mc->joined, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  if (uni64(mc->n_left) == 0) return;
  if (threadIdx.x == 0) s_id = atomicAdd(&mc->joined, 1u);
  __syncthreads();
  const uint32_t id = s_id;
  uint32_t phase = 0, may = gridDim.x;
  bool last = id == 0;  // phase 0: the first block alone, without work
  for (;;) {
    if (last) {  // block-uniform: prepare the phase after this one and publish it
      __threadfence();
      uint32_t next = phase + 1;
      if (phase == 0) {
        may = (uint32_t)min((int64_t)may, (mc->n_left + kLepChunkMin - 1) / kLepChunkMin);
        // the blocks of a free GPU start within some microseconds: not without them, but not longer
        if (threadIdx.x == 0)
          for (int i = 0; i < 64 && joined() < may; ++i) __builtin_amdgcn_s_sleep(16);
      } else if (phase % 3 == 0) {
        multi_begin(m, kRounds, sh, (int)may, 0);
        __syncthreads();
        // (a generation per three phases, and at most k + 1 generations)
        if (mc->n_left == 0 || phase > 3u * (uint32_t)m.k) next = kTailClosed;
      } else if (phase % 3 == 1) {
        multi_mid(m, sh, (int)may);
      } else if (threadIdx.x == 0) {
        mc->pair_ticket = 0;
      }
      __threadfence();
      __syncthreads();
      if (threadIdx.x == 0) {
        __hip_atomic_store(&mc->arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&mc->pub, (unsigned long long)next << 32 | may << 16 | min(joined(), may), __ATOMIC_RELEASE,
                           __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    // the next phase that this block takes part in, or the end
    if (threadIdx.x == 0) {
      unsigned long long p;
      for (;;) {
        p = __hip_atomic_load(&mc->pub, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t ph = (uint32_t)(p >> 32);
        if (ph != phase && ph != 0 && (ph == kTailClosed || id < (p & 0xFFFFu) || id >= ((p >> 16) & 0xFFFFu))) break;
        __builtin_amdgcn_s_sleep(16);
      }
      s_pub = p;
    }
    __syncthreads();
    __threadfence();
    const unsigned long long p = s_pub;
    phase = (uint32_t)(p >> 32);
    may = (uint32_t)(p >> 16) & 0xFFFFu;
    const uint32_t active = (uint32_t)p & 0xFFFFu;
    if (phase == kTailClosed || id >= may) return;  // block-uniform
    if (phase % 3 == 1) {
      const int first = (int)min(ticket(&mc->lep_ticket), (long long)INT_MAX);
      multi_lepton<FK, MIXED>(m, kRounds, sh, tab, tab + m.n_tab, first, 0);
    } else if (phase % 3 == 2) {
      multi_photon<FK, MIXED>(m, sh, tab);
    } else {
      // shares of the events, as many as would be blocks of k_multi_pairs, fewer for few events
      const int64_t cnt = m.evc->count;
      const int shares = m.evc->overflow ? kPairBlocks : (int)min((int64_t)kPairBlocks, (cnt + kMultiBlock - 1) / kMultiBlock);
      for (long long v; (v = ticket(&mc->pair_ticket)) < shares;) multi_pairs<FK, MIXED>(m, (int)v, shares);
    }
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) s_last = atomicAdd(&mc->arrived, 1u) + 1u == active;
    __syncthreads();
    last = s_last != 0;
  }
}

hipError_t init_crmath_multi() {
  static unsigned long long done = 0;  // one bit per device
  return upload_crmath(&done);
}

// dynamic LDS: the rate table, and the lepton kernels' pools
static int multi_tab(int n_eta, int n_cp) { return (std::max(n_eta, n_cp) + 1) / 2 * 2; }
static size_t multi_shm(int n_tab, bool leptons) {
  return sizeof(double) * ((size_t)n_tab + (leptons ? (size_t)kMultiWaves * kPool * kPoolWords : 0));
}

template <int FK, bool MIXED>
static int multi_fit(int which, int n_tab) {
  int n = 0;
  const size_t shm = multi_shm(n_tab, which == 0);
  const hipError_t e =
      which ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_multi_photon<FK, MIXED>, kMultiBlock, shm)
            : hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_multi_lepton<FK, MIXED>, kMultiBlock, shm);
  return e == hipSuccess && n > 0 ? n : 1;
}
int multi_blocks_per_cu(int fk, int which, int n_eta, int n_cp, bool mixed) {
  const int n_tab = multi_tab(n_eta, n_cp);
#define QED_FIT(K) \
  if (fk == K) return mixed ? multi_fit<K, true>(which, n_tab) : multi_fit<K, false>(which, n_tab);
  QED_FIT(QED_FIELD_UNIFORM)
  QED_FIT(QED_FIELD_LP_PULSE)
  QED_FIT(QED_FIELD_CP_WAVE)
  QED_FIT(QED_FIELD_CP_STANDING)
#undef QED_FIT
  return 1;
}

template <int FK, bool MIXED>
static void launch_multi_fk(MultiArgs m, hipStream_t s) {
  m.n_tab = multi_tab(m.s.tb.n_eta, m.s.tb.n_cp);
  const size_t shl = multi_shm(m.n_tab, true), shp = multi_shm(m.n_tab, false);
  const dim3 b(kMultiBlock);
  const bool pairs = (m.s.sc.flags & QED_PAIRS) != 0;
  for (m.round = 0; m.round < (pairs ? kRounds : 1); ++m.round) {
    hipLaunchKernelGGL(k_multi_begin, dim3(1), b, 0, s, m);
    hipLaunchKernelGGL((k_multi_lepton<FK, MIXED>), dim3(m.lep_grid), b, shl, s, m);
    if (!pairs) return;
    hipLaunchKernelGGL(k_multi_mid, dim3(1), b, 0, s, m);
    hipLaunchKernelGGL((k_multi_photon<FK, MIXED>), dim3(m.ph_grid), b, shp, s, m);
    hipLaunchKernelGGL((k_multi_pairs<FK, MIXED>), dim3(kPairBlocks), b, 0, s, m);
  }
  hipLaunchKernelGGL(k_multi_begin, dim3(1), b, 0, s, m);
  hipLaunchKernelGGL((k_multi_tail<FK, MIXED>), dim3(std::min(m.lep_grid, 0xFFFF)), b, shl, s, m);
}
void launch_multi(int fk, MultiArgs m, bool mixed, hipStream_t s) {
#define QED_MULTI(K)                               \
  if (fk == K) {                                   \
    if (mixed) launch_multi_fk<K, true>(m, s);     \
    else launch_multi_fk<K, false>(m, s);          \
  }
  QED_MULTI(QED_FIELD_UNIFORM)
  QED_MULTI(QED_FIELD_LP_PULSE)
  QED_MULTI(QED_FIELD_CP_WAVE)
  QED_MULTI(QED_FIELD_CP_STANDING)
#undef QED_MULTI
}

}  // namespace qedk
