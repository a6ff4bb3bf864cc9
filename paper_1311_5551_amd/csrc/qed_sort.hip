// Photons whose pair window is over (in the refreshed grid those below the energy that can reach
// chi_min: half of them in the cascade) go to the front of the array, where the photon sweep does
// not start and later sorts do not touch them; the others are sorted behind it.
//
// Spatial reordering of the particles of an instance with a grid field, by 8 x 8-cell tile of
// their position: a counting sort (histogram of tile keys with each particle's rank in its tile,
// exclusive scan, destination slots) followed by a permutation of every array of the species.  Particles that
// share a tile then sit next to each other, so the lanes of a wave gather from the same grid
// cache lines.  The order within a tile follows the atomics; per-particle results of later steps
// do not depend on the order (random streams are keyed by uid).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "qed_device.h"
#include "qed_kernels.h"

namespace qedk {

constexpr int kTile = 8;

// Bucket of every particle (1 + its tile; 0 for a photon that goes to the front), the bucket counts, and the particle's rank among those of its bucket.
// Particles mostly lie in the order of the sort before, so the 64 of a wave share a few tiles: one
// atomic per run of equal keys among its lanes adds the run and ranks its particles.  (One atomic
// per particle serialised on a tile's counter, and a second pass of them made the destinations:
// 1.6 ms per species and sort of 1.6e7 particles, 3.3 + 2.9 ms for the first, unsorted, one.)
template <bool MIXED>
__global__ __launch_bounds__(256) void k_sort_key(const qed_instance* __restrict__ inst, int ii, int s,
                                                  const Glob* __restrict__ glob, double dt, int32_t* __restrict__ key,
                                                  uint32_t* __restrict__ rank, uint32_t* __restrict__ hist,
                                                  int tiles_x, const InstAcc* __restrict__ acc,
                                                  const uint32_t* __restrict__ win) {
  using Real = typename std::conditional<MIXED, float, double>::type;
  const qed_instance& I = inst[ii];
  const qed_species& S = I.s[s];
  const qed_field& F = I.field;
  int64_t n = *S.count_dev;
  if (n > S.capacity) n = S.capacity;
  const int64_t step = glob->step_next;
  const int64_t n0 = s == 2 ? acc->n_front : 0;
  const uint32_t* W = win ? win + acc->mover_off : nullptr;
  const int lane = threadIdx.x & 63;
  const unsigned long long below = (1ull << lane) - 1ull;
  // a contiguous range of slots per block
  int64_t b0, b1;
  block_range(n0, n, blockIdx.x, gridDim.x, &b0, &b1);
  if (b0 >= b1) return;  // the whole block
  // (a converted photon waits for its compaction behind the front)
  auto to_front = [&](int64_t k) { return window_over(W[k], step) && !(S.tau_dev[k] < 0.0); };
  // the front's new photons are counted first: one atomic per block reserves their places (they are
  // many, and in one bucket)
  __shared__ unsigned sredu[16];
  __shared__ uint32_t s_base;
  if (W) {
    unsigned u[1] = {0};
    for (int64_t k = b0 + threadIdx.x; k < b1; k += blockDim.x)
      if (to_front(k)) ++u[0];
    block_sum_u(u, sredu);
    if (threadIdx.x == 0) s_base = u[0] ? atomicAdd(&hist[0], u[0]) : 0u;
    __syncthreads();
  }
  uint32_t run = W ? s_base : 0u;
  for (int64_t k0 = b0 + threadIdx.x - lane; k0 < b1 + threadIdx.x - lane; k0 += blockDim.x) {  // block-uniform
    const int64_t k = min(k0 + lane, b1 - 1);
    const bool valid = k0 + lane < b1;
    double x, y;
    if (s < 2) {
      x = ((const Real*)S.x_dev)[k];
      y = ((const Real*)S.y_dev)[k];
      if (MIXED) {
        x += S.x_lo_dev[k];
        y += S.y_lo_dev[k];
      }
    } else {  // photon position at the start of the next step
      const double kx = ((const Real*)S.ux_dev)[k], ky = ((const Real*)S.uy_dev)[k], kz = ((const Real*)S.uz_dev)[k];
      const double e = sqrt(kx * kx + ky * ky + kz * kz);
      const double age = (double)(step - (int64_t)S.birth_step_dev[k]) * dt;
      x = (double)((const Real*)S.x_dev)[k] + (e > 0.0 ? age * kx / e : 0.0);
      y = (double)((const Real*)S.y_dev)[k] + (e > 0.0 ? age * ky / e : 0.0);
    }
    double gx = floor((x - F.x0) / F.dx), gy = floor((y - F.y0) / F.dy);
    if (!(fabs(gx) < 1e15)) gx = 0.0;  // non-finite positions go to tile 0
    if (!(fabs(gy) < 1e15)) gy = 0.0;
    const int64_t i = wrap_index((int64_t)gx, F.nx), j = wrap_index((int64_t)gy, F.ny);
    const bool front = W && valid && to_front(k);
    uint32_t at_front = 0;
    if (W) {
      unsigned tot;
      at_front = run + block_rank(front, sredu, &tot);
      run += tot;
    }
    const int32_t kk = front ? 0 : 1 + (int32_t)((j / kTile) * tiles_x + i / kTile);
    // runs of equal keys among the wave's lanes that go to a tile
    const unsigned long long in = __ballot(valid && !front);
    const bool mine = (in >> lane) & 1ull;
    const int prev = 63 - __clzll((long long)(in & below));  // the lane before among them (-1: none)
    const int32_t pk = __shfl(kk, prev < 0 ? lane : prev);
    const unsigned long long heads = __ballot(mine && (prev < 0 || kk != pk));
    const unsigned long long upto = heads & (below | (1ull << lane));
    const int head = upto ? 63 - __clzll((long long)upto) : 0;
    const unsigned long long after = lane == 63 ? 0ull : heads & (~0ull << (lane + 1));
    const unsigned long long same = after ? in & ((1ull << (__ffsll((long long)after) - 1)) - 1ull) : in;
    uint32_t base = 0;
    if (mine && head == lane) base = atomicAdd(&hist[kk], (uint32_t)__popcll(same & ~below));
    base = __shfl(base, head);
    if (valid) {
      key[k] = kk;
      rank[k] = front ? at_front : base + (uint32_t)__popcll(in & below & (~0ull << head));
    }
  }
}

__global__ __launch_bounds__(256) void k_fill_zero(uint32_t* __restrict__ a, int m) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < m; i += gridDim.x * blockDim.x) a[i] = 0u;
}

// exclusive scan of hist[0, m) in place, one block of 1024 threads that walks it in runs of 16384:
// 16 consecutive entries per thread, wave scans by shuffles, the waves' totals in LDS.  (One run of
// m / 1024 entries per thread read a line per entry: 219 us for 131072 tiles.)
__global__ __launch_bounds__(1024) void k_sort_scan(uint32_t* __restrict__ hist, int m) {
  constexpr int kPer = 16;
  __shared__ uint32_t part[16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t carry = 0;
  for (int64_t r0 = 0; r0 < m; r0 += 1024 * kPer) {
    const int64_t b = r0 + (int64_t)threadIdx.x * kPer;
    uint32_t v[kPer], sum = 0;
    if (b + kPer <= m) {
      const uint4* q = (const uint4*)(hist + b);
#pragma unroll
      for (int i = 0; i < kPer / 4; ++i) {
        const uint4 t = q[i];
        v[4 * i] = t.x;
        v[4 * i + 1] = t.y;
        v[4 * i + 2] = t.z;
        v[4 * i + 3] = t.w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < kPer; ++i) v[i] = b + i < m ? hist[b + i] : 0u;
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) sum += v[i];
    uint32_t inc = sum;  // inclusive scan over the wave
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t u = __shfl_up(inc, o);
      if (lane >= o) inc += u;
    }
    __syncthreads();  // part is free
    if (lane == 63) part[wave] = inc;
    __syncthreads();
    uint32_t before = carry, total = 0;
    for (int w = 0; w < 16; ++w) {
      if (w < wave) before += part[w];
      total += part[w];
    }
    uint32_t run = before + inc - sum;
    if (b + kPer <= m) {
      uint4* q = (uint4*)(hist + b);
#pragma unroll
      for (int i = 0; i < kPer / 4; ++i) {
        uint4 t;
        t.x = run;
        t.y = t.x + v[4 * i];
        t.z = t.y + v[4 * i + 1];
        t.w = t.z + v[4 * i + 2];
        run = t.w + v[4 * i + 3];
        q[i] = t;
      }
    } else {
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        if (b + i < m) hist[b + i] = run;
        run += v[i];
      }
    }
    carry += total;
  }
}

// destination slot: behind the front (*first slots, or none), the bucket's first slot plus the rank
__global__ __launch_bounds__(256) void k_sort_dst(const qed_species* __restrict__ sp, const int32_t* __restrict__ key,
                                                  const uint32_t* __restrict__ offs, uint32_t* __restrict__ dst,
                                                  const int64_t* __restrict__ first) {
  int64_t n = *sp->count_dev;
  if (n > sp->capacity) n = sp->capacity;
  const int64_t F = first ? *first : 0;
  for (int64_t k = F + blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x)
    dst[k] += (uint32_t)F + offs[key[k]];
}

// stage[dst[k]] = a[k], then a[k] = stage[k] (two kernels)
template <class T>
__global__ __launch_bounds__(256) void k_scatter(const qed_species* __restrict__ sp, const T* __restrict__ a,
                                                 T* __restrict__ stage, const uint32_t* __restrict__ dst,
                                                 const int64_t* __restrict__ first) {
  int64_t n = *sp->count_dev;
  if (n > sp->capacity) n = sp->capacity;
  const int64_t F = first ? *first : 0;
  for (int64_t k = F + blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x)
    stage[dst[k]] = a[k];
}
template <class T>
__global__ __launch_bounds__(256) void k_copy_back(const qed_species* __restrict__ sp, T* __restrict__ a,
                                                   const T* __restrict__ stage, const int64_t* __restrict__ first) {
  int64_t n = *sp->count_dev;
  if (n > sp->capacity) n = sp->capacity;
  const int64_t F = first ? *first : 0;
  for (int64_t k = F + blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x)
    a[k] = stage[k];
}

// the photons of bucket 0 have joined the front
__global__ void k_sort_front(InstAcc* acc, const uint32_t* __restrict__ offs) { acc->n_front += offs[1]; }

template <class T>
static void permute(const qed_species* sp_dev, void* a, void* stage, const uint32_t* dst, const int64_t* first,
                    int grid, hipStream_t s) {
  if (!a) return;
  hipLaunchKernelGGL(k_scatter<T>, dim3(grid), dim3(256), 0, s, sp_dev, (const T*)a, (T*)stage, dst, first);
  hipLaunchKernelGGL(k_copy_back<T>, dim3(grid), dim3(256), 0, s, sp_dev, (T*)a, (const T*)stage, first);
}

hipError_t launch_sort_species(const qed_instance* inst_dev, const qed_instance& inst_host, int ii, int s,
                               InstAcc* acc_dev, const uint32_t* win, const Glob* glob, double dt, bool mixed,
                               const SortScratch& w, int grid, hipStream_t st) {
  const qed_field& F = inst_host.field;
  const int tiles_x = (F.nx + kTile - 1) / kTile, tiles_y = (F.ny + kTile - 1) / kTile;
  const int n_tiles = tiles_x * tiles_y + 1;  // and the front's bucket
  InstAcc* const acc = acc_dev + ii;
  const int64_t* const first = s == 2 ? &acc->n_front : nullptr;
  if (n_tiles > w.hist_len) return hipErrorInvalidValue;
  const qed_species* sp_dev = &inst_dev[ii].s[s];
  const qed_species& S = inst_host.s[s];
  hipLaunchKernelGGL(k_fill_zero, dim3(256), dim3(256), 0, st, w.hist, n_tiles);
  if (mixed)
    hipLaunchKernelGGL(k_sort_key<true>, dim3(grid), dim3(256), 0, st, inst_dev, ii, s, glob, dt, w.key, w.dst,
                       w.hist, tiles_x, (const InstAcc*)acc, s == 2 ? win : nullptr);
  else
    hipLaunchKernelGGL(k_sort_key<false>, dim3(grid), dim3(256), 0, st, inst_dev, ii, s, glob, dt, w.key, w.dst,
                       w.hist, tiles_x, (const InstAcc*)acc, s == 2 ? win : nullptr);
  hipLaunchKernelGGL(k_sort_scan, dim3(1), dim3(1024), 0, st, w.hist, n_tiles);
  hipLaunchKernelGGL(k_sort_dst, dim3(grid), dim3(256), 0, st, sp_dev, w.key, w.hist, w.dst, first);
  const bool d3 = inst_host.dims == 3;
  if (mixed) {
    permute<float>(sp_dev, S.x_dev, w.stage, w.dst, first, grid, st);
    permute<float>(sp_dev, S.y_dev, w.stage, w.dst, first, grid, st);
    if (d3) permute<float>(sp_dev, S.z_dev, w.stage, w.dst, first, grid, st);
    permute<float>(sp_dev, S.ux_dev, w.stage, w.dst, first, grid, st);
    permute<float>(sp_dev, S.uy_dev, w.stage, w.dst, first, grid, st);
    permute<float>(sp_dev, S.uz_dev, w.stage, w.dst, first, grid, st);
    if (s < 2) {
      permute<float>(sp_dev, S.x_lo_dev, w.stage, w.dst, first, grid, st);
      permute<float>(sp_dev, S.y_lo_dev, w.stage, w.dst, first, grid, st);
      if (d3) permute<float>(sp_dev, S.z_lo_dev, w.stage, w.dst, first, grid, st);
      permute<float>(sp_dev, S.ux_lo_dev, w.stage, w.dst, first, grid, st);
      permute<float>(sp_dev, S.uy_lo_dev, w.stage, w.dst, first, grid, st);
      permute<float>(sp_dev, S.uz_lo_dev, w.stage, w.dst, first, grid, st);
    }
  } else {
    permute<double>(sp_dev, S.x_dev, w.stage, w.dst, first, grid, st);
    permute<double>(sp_dev, S.y_dev, w.stage, w.dst, first, grid, st);
    if (d3) permute<double>(sp_dev, S.z_dev, w.stage, w.dst, first, grid, st);
    permute<double>(sp_dev, S.ux_dev, w.stage, w.dst, first, grid, st);
    permute<double>(sp_dev, S.uy_dev, w.stage, w.dst, first, grid, st);
    permute<double>(sp_dev, S.uz_dev, w.stage, w.dst, first, grid, st);
  }
  permute<double>(sp_dev, S.tau_dev, w.stage, w.dst, first, grid, st);
  permute<uint64_t>(sp_dev, S.uid_dev, w.stage, w.dst, first, grid, st);
  if (s == 2) {
    permute<int32_t>(sp_dev, S.birth_step_dev, w.stage, w.dst, first, grid, st);
    hipLaunchKernelGGL(k_sort_front, dim3(1), dim3(1), 0, st, acc, w.hist);
  }
  return hipGetLastError();
}

// Scratch of qed_sort_static: a fixed array in device memory (each GPU holds its own copy from
// the load of the library to the end of the process), laid out as the staging words (8 B per
// slot), the tile keys and destination slots (4 B per slot each), then the tile histogram.  In
// host code its name is not a device address: the address comes from hipGetSymbolAddress, taken
// once per device with that device current, and only that address is handed to kernels.
static __device__ __align__(256) unsigned char scratch[kStaticSortBytes];

hipError_t static_sort_scratch(SortScratch* out) {
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  {
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
      void* p = nullptr;
      e = hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch));
      if (e != hipSuccess) return e;
      addr[dev] = p;
    }
  }
  char* base = (char*)addr[dev];
  out->stage = base;
  out->key = (int32_t*)(base + kStaticSortSlots * 8);
  out->dst = (uint32_t*)(base + kStaticSortSlots * 12);
  out->hist = (uint32_t*)(base + kStaticSortSlots * 16);
  out->hist_len = kStaticSortTiles + 1;
  return hipSuccess;
}

}  // namespace qedk
