// Device-side helpers shared by the kernel files of the stage-level partition search (value
// limits, address-space casts, the atomic fold, wave broadcasts, input limits).
#pragma once

#include "rannc_dp_internal.h"

#include "../../include/rannc_dp.h"

namespace rannc {

template <typename VT> struct Lim;
template <> struct Lim<uint32_t> { static constexpr uint32_t inf = 0xFFFFFFFFu; };
// 64-bit tables: "no plan" is the bit pattern of +infinity in double precision, above every value
// a search can form (they stay below 2^62).  Bit patterns below it, read as doubles, are
// non-negative finite numbers (normal or denormal, never NaN) whose order is the order of the
// integers, so the maximum and minimum of two 64-bit values are ONE double-precision instruction
// each instead of a 64-bit compare and four selects.  The boundary still reports INT64_MAX.
template <> struct Lim<uint64_t> { static constexpr uint64_t inf = 0x7FF0000000000000ull; };

template <typename VT> __device__ __forceinline__ VT vmax(VT a, VT b) { return a > b ? a : b; }
template <typename VT> __device__ __forceinline__ VT vmin(VT a, VT b) { return a < b ? a : b; }
// (inline assembly: the compiler's own double-precision maximum first rewrites each operand to
// quiet signalling NaNs, which cannot occur here, at three instructions instead of one; double
// precision denormals are always enabled on this target)
template <> __device__ __forceinline__ uint64_t vmax<uint64_t>(uint64_t a, uint64_t b) {
  uint64_t r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
template <> __device__ __forceinline__ uint64_t vmin<uint64_t>(uint64_t a, uint64_t b) {
  uint64_t r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
// maximum with a wave-uniform first operand that lives in scalar registers
template <typename VT> __device__ __forceinline__ VT vmax_su(VT a_uniform, VT b) { return vmax(a_uniform, b); }
template <> __device__ __forceinline__ uint64_t vmax_su<uint64_t>(uint64_t a_uniform, uint64_t b) {
  uint64_t r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "s"(a_uniform), "v"(b));
  return r;
}

// Pointers that are read out of a descriptor in memory are generic to the compiler, and generic
// (FLAT) loads count against the 4-bit LDS/scalar counter: at most 15 of them can be in flight per
// wave.  Everything the library addresses is device memory, so the hot kernels say so and get
// GLOBAL loads, which have 63 in flight.
#define RANNC_GLOBAL __attribute__((address_space(1)))
template <typename T> __device__ __forceinline__ T RANNC_GLOBAL *gptr(T *p) { return (T RANNC_GLOBAL *)p; }

template <typename VT> __device__ __forceinline__ void global_min(VT RANNC_GLOBAL *p, VT v) {
  (void)__hip_atomic_fetch_min(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Workgroup barrier that orders LDS accesses only.  __syncthreads() also waits for every global load
// and store the wave has in flight (its fence covers global memory); where the waves exchange data
// through LDS alone, that wait puts a memory round trip in front of every barrier.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ __forceinline__ uint32_t lane_bcast(uint32_t v, int q) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, q);
}
__device__ __forceinline__ uint64_t lane_bcast(uint64_t v, int q) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, q);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), q);
  return ((uint64_t)hi << 32) | lo;
}

// Smallest value of the wave (all lanes active), the same in every lane.  Four steps inside the rows of
// sixteen lanes without the LDS crossbar, then the four rows through scalar registers.
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xB1, 0xF, 0xF, false));   // quad_perm 1 0 3 2
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x4E, 0xF, 0xF, false));   // quad_perm 2 3 0 1
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x141, 0xF, 0xF, false));  // row_half_mirror
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x140, 0xF, 0xF, false));  // row_mirror
  return min(min(lane_bcast(v, 0), lane_bcast(v, 16)), min(lane_bcast(v, 32), lane_bcast(v, 48)));
}
__device__ __forceinline__ uint64_t wave_min(uint64_t v) {
  const uint32_t hi = wave_min((uint32_t)(v >> 32));
  const uint32_t lo = wave_min((uint32_t)(v >> 32) == hi ? (uint32_t)v : ~0u);
  return (uint64_t)hi << 32 | lo;
}

// x <= v r for v < 2^62, r < 2^32
__device__ __forceinline__ bool at_most_times(uint64_t x, uint64_t v, uint32_t r) {
  return __umul64hi(v, (uint64_t)r) != 0 || x <= v * (uint64_t)r;
}
__device__ __forceinline__ bool at_most_times(uint64_t x, uint32_t v, uint32_t r) { return x <= (uint64_t)v * r; }

// ceil(x / v) where that is at most 64 (at least 1), else something above 64; v >= 1, inv_v: about 1 / v.  Below
// 2^7 the quotient is off by far less than one, so that its whole part is too small by at most two (n - 1 for a
// quotient just above n) and never too large by more than one.  (A 64-bit division is 150 instructions.)
template <typename VT> __device__ __forceinline__ int ceil_ratio(uint64_t x, VT v, float inv_v) {
  int r = max((int)min((float)x * inv_v, 100.0f), 1);
  if (r > 1 && at_most_times(x, v, (uint32_t)r - 1u)) --r;
  if (!at_most_times(x, v, (uint32_t)r)) ++r;
  if (!at_most_times(x, v, (uint32_t)r)) ++r;
  return r;
}

// ceil(x / r) for any 1 <= r <= 64 from the correctly rounded reciprocal 1/r, in double precision:
//     t = x + (r/2 - 1 + r o)     y = t (1/r) + 1.5 2^52     (one fused multiply-add)
// t / r = (x + r - 1)/r - 1/2 + o, and the fraction of (x + r - 1)/r is at most 63/64, so t (1/r) lies
// between k - 1/2 + o and k + 1/2 - (1/64 - o) for k = ceil(x / r); the addition rounds it to k, which
// is then the low part of the sum, as long as t is exact and the product is off by less than o.
// 32-bit x: o = 2^-18 (t a multiple of 2^-18 below 2^33; product off by less than 2^-20).  64-bit x up to
// 2^44: o = 2^-8 (t a multiple of 2^-8 below 2^45: 53 bits; off by less than 2^-9).
template <typename VT> struct CeilDiv;
template <> struct CeilDiv<uint32_t> {
  static constexpr double kOffset = 0x1p-18;
  static __device__ __forceinline__ uint32_t at(double t, double inv) {
    return (uint32_t)__double_as_longlong(__builtin_fma(t, inv, 0x1.8p52));
  }
};
template <> struct CeilDiv<uint64_t> {
  static constexpr double kOffset = 0x1p-8;
  static __device__ __forceinline__ uint64_t at(double t, double inv) {
    return (uint64_t)__double_as_longlong(__builtin_fma(t, inv, 0x1.8p52)) & ((1ull << 51) - 1ull);
  }
};
template <typename VT> __device__ __forceinline__ double ceil_div_offset(int r) {
  return 0.5 * (double)r - 1.0 + (double)r * CeilDiv<VT>::kOffset;
}
template <typename VT> __device__ __forceinline__ VT ceil_div(VT x, int r, double inv) {
  return CeilDiv<VT>::at((double)x + ceil_div_offset<VT>(r), inv);
}
constexpr int64_t kCeilDivMax = (int64_t)1 << 44;

static constexpr uint64_t kSumLimit = 1ull << 62;
static constexpr uint64_t kCutLimit = (kSumLimit - 1) / 1000;  // largest bytes of a cut: 1000 * bytes < 2^62

// Time in ns to send `bytes` at `bw` bytes per microsecond from one replica (the communication term
// of a stage's execution time, Sec. III-C); flags as in the prefix sums.  With r replicas each
// sends 1/r of it: ceil(1000*bytes / (r*bw)) = ceil(ceil(1000*bytes / bw) / r), so the per-cut
// value is all the table builder needs.
__device__ __forceinline__ uint64_t cut_time(int64_t bytes, int64_t bw, int &flags) {
  if (bytes < 0) { flags |= 1; bytes = 0; }
  uint64_t u = (uint64_t)bytes;
  if (u > kCutLimit) { flags |= 2; u = kCutLimit; }
  return (u * 1000ull + (uint64_t)bw - 1) / (uint64_t)bw;
}
static constexpr int kNoRow = 0x7fffffff;

// Split-objective level kernel: waves per workgroup (each takes every eighth device total; sixteen
// measured slower).
constexpr int kSplitWaves = 8;

}  // namespace rannc
