// Sums over all workgroups of a running kernel.
//
// A kernel whose whole state fits the chip's registers (the coarsest
// multigrid level's CG, a CG on a small mesh) can stay resident over its
// iterations instead of ending at each reduction.  Every reduction is then
// one exchange between the workgroups: each publishes its partial sums in a
// slot of its own, and every workgroup reads all slots and adds them in the
// same fixed order, so all obtain bit-identical totals.
//
// A slot word is (tag << 32 | 32 bits of a double): a reader that finds the
// tag of the exchange it waits for has the data with it, so one store and
// one load make the round trip (no counter, no release flag).  Tags increase
// by one per exchange over all launches; the running value is kept in device
// memory (`epoch`: read by every workgroup at its start, advanced by
// workgroup 0 at its end, which lies behind an exchange of all), so a
// captured launch can be replayed.  Two sets of slots alternate: a workgroup
// can be at most one exchange ahead of another.
//
// Every wait is bounded: after kGridSpinLimit polls a workgroup gives up and
// the kernel ends (its callers then write NaN results).  All workgroups must
// be resident together; the launchers keep their grids at most a quarter of
// what the chip holds, so that four such kernels on four streams also fit.
#pragma once

#include "common.hpp"

namespace sem {

constexpr int kGridSpinLimit = 1 << 21;  // polls of about a microsecond each
constexpr int kGridWords = 4;            // slot words: two doubles in two halves each

__device__ __forceinline__ uint64_t grid_load(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void grid_store(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sums of a and b over the workgroup (NW wavefronts), on every thread, in a
// fixed order.  `red` holds 2 * NW doubles; a barrier separates two uses.
template <int NW>
__device__ __forceinline__ void group_sum2(double& a, double& b, double* red) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const double sa = wave_sum_d(a), sb = wave_sum_d(b);
  __syncthreads();
  if (lane == 0) {
    red[2 * wv] = sa;
    red[2 * wv + 1] = sb;
  }
  __syncthreads();
  a = 0.0;
  b = 0.0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    a += red[2 * w];
    b += red[2 * w + 1];
  }
}

// First half of an exchange: a, b <- their sums over the workgroup, published
// in its slot.  `slots`: 2 x nblk x kGridWords words.
template <int NW>
__device__ __forceinline__ void grid_put2(double& a, double& b, uint32_t tag, int nblk,
                                          uint64_t* __restrict__ slots, double* red) {
  group_sum2<NW>(a, b, red);
  if (nblk == 1) return;
  uint64_t* set = slots + (size_t)(tag & 1) * nblk * kGridWords;
  if (threadIdx.x < kGridWords) {
    const double v = threadIdx.x < 2 ? a : b;
    const uint32_t half =
        (uint32_t)((threadIdx.x & 1) ? __double2hiint(v) : __double2loint(v));
    grid_store(set + (size_t)blockIdx.x * kGridWords + threadIdx.x, (uint64_t)tag << 32 | half);
  }
}

// Second half: a, b <- the sums over all workgroups.  False when a wait gave
// up, here or before (`gave_up`, on any thread): the same on every thread of
// the workgroup.
template <int NW>
__device__ __forceinline__ bool grid_get2(double& a, double& b, uint32_t tag, int nblk,
                                          const uint64_t* __restrict__ slots, double* red,
                                          int gave_up) {
  if (nblk == 1) return !__syncthreads_or(gave_up);
  const uint64_t* set = slots + (size_t)(tag & 1) * nblk * kGridWords;
  double ta = 0.0, tb = 0.0;
  for (int s = threadIdx.x; s < nblk; s += NW * 64) {
    const uint64_t* q = set + (size_t)s * kGridWords;
    uint64_t w0, w1, w2, w3;
    int spin = 0;
    for (;;) {
      w0 = grid_load(q);
      w1 = grid_load(q + 1);
      w2 = grid_load(q + 2);
      w3 = grid_load(q + 3);
      if ((uint32_t)(w0 >> 32) == tag && (uint32_t)(w1 >> 32) == tag &&
          (uint32_t)(w2 >> 32) == tag && (uint32_t)(w3 >> 32) == tag)
        break;
      if (++spin >= kGridSpinLimit) {
        gave_up = 1;
        break;
      }
    }
    ta += __hiloint2double((int)(uint32_t)w1, (int)(uint32_t)w0);
    tb += __hiloint2double((int)(uint32_t)w3, (int)(uint32_t)w2);
  }
  if (__syncthreads_or(gave_up)) return false;
  a = ta;
  b = tb;
  group_sum2<NW>(a, b, red);
  return true;
}

// a, b <- their sums over all workgroups
template <int NW>
__device__ __forceinline__ bool grid_sum2(double& a, double& b, uint32_t tag, int nblk,
                                          uint64_t* __restrict__ slots, double* red) {
  grid_put2<NW>(a, b, tag, nblk, slots, red);
  return grid_get2<NW>(a, b, tag, nblk, slots, red, 0);
}

// Single values handed from workgroup to workgroup without an exchange: the
// words carry the tag, as the slots do, so a reader waits for the value
// itself.  A place may be written again once an exchange lies between the
// reads of its old value and the new write.
template <typename T>
constexpr int kTagWords = sizeof(T) / 4;

template <typename T>
__device__ __forceinline__ void put_tagged(uint64_t* __restrict__ at, T v, uint32_t tag) {
  const uint64_t hi = (uint64_t)tag << 32;
  if constexpr (sizeof(T) == 8) {
    grid_store(at, hi | (uint32_t)__double2loint(v));
    grid_store(at + 1, hi | (uint32_t)__double2hiint(v));
  } else {
    grid_store(at, hi | (uint32_t)__float_as_int(v));
  }
}

template <typename T>
struct Tagged {
  uint64_t w[kTagWords<T>];
  __device__ __forceinline__ void load(const uint64_t* __restrict__ at) {
#pragma unroll
    for (int i = 0; i < kTagWords<T>; ++i) w[i] = grid_load(at + i);
  }
  __device__ __forceinline__ bool has(uint32_t tag) const {
    bool ok = true;
#pragma unroll
    for (int i = 0; i < kTagWords<T>; ++i) ok = ok && (uint32_t)(w[i] >> 32) == tag;
    return ok;
  }
  // waits for the value (the first load may have been issued before)
  __device__ __forceinline__ T get(const uint64_t* __restrict__ at, uint32_t tag, int& gave_up) {
    for (int spin = 0; !has(tag); load(at))
      if (++spin >= kGridSpinLimit) {
        gave_up = 1;
        break;
      }
    if constexpr (sizeof(T) == 8) return __hiloint2double((int)(uint32_t)w[1], (int)(uint32_t)w[0]);
    else return __int_as_float((int)(uint32_t)w[0]);
  }
};

}  // namespace sem
