// Prefix sums held as doubles in LDS, and what is computed with them: shared by the kernels that answer searches without
// their tables (rannc_dp_reach.hip, rannc_dp_form.hip).
#pragma once

#include "rannc_dp_device.h"

namespace rannc {

// All sums are held as doubles.  Up to these bounds every product and sum below (replicas times a difference of
// sums, at most 2^6 * 2^47) is a whole number below 2^53 and exact, and so is ceil_div on the times.
constexpr double kReachMaxTime = (double)kCeilDivMax, kReachMaxBytes = 0x1p46;
// (the compiler's own maximum first makes quiet the signalling NaNs that cannot occur here)
__device__ __forceinline__ double dmax(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double dmin(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
constexpr int kReachPad = 4;  // entries in front of the sums

// Prefix sums of one array by one wave, PER consecutive entries per lane and turn, into s[1 .. N]; the inputs are
// copied to `save` (or null).  flags, high: as in prepare_sums.  Returns the total (modulo 2^64).
template <int PER>
__device__ __forceinline__ uint64_t reach_sums(const int64_t RANNC_GLOBAL *in, int64_t RANNC_GLOBAL *save, double *s, int N, int &flags,
                                               uint32_t &high) {
  const int lane = threadIdx.x & 63;
  uint64_t carry = 0;
  if (lane == 0) s[0] = 0.0;
#pragma unroll 1
  for (int base = 0; base < N; base += 64 * PER) {
    const int i0 = base + lane * PER;
    uint64_t v[PER], sum = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) v[k] = (uint64_t)in[min(i0 + k, N - 1)];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      uint64_t x = i0 + k < N ? v[k] : 0;
      if (save && i0 + k < N) save[i0 + k] = (int64_t)x;
      if ((int64_t)x < 0) { flags |= 1; x = 0; }
      if (x >= kSumLimit) { flags |= 2; x = 0; }
      sum += x;
      v[k] = sum;
      high |= (uint32_t)(sum >> 32);
    }
    uint64_t run = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint64_t x = __shfl_up(run, o);
      if (lane >= o) run += x;
      high |= (uint32_t)(run >> 32);
    }
    const uint64_t before = carry + run - sum;
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (i0 + k < N) {
        s[i0 + k + 1] = (double)(before + v[k]);
        high |= (uint32_t)((before + v[k]) >> 32);
      }
    carry += lane_bcast(run, 63);
  }
  return carry;
}

// lanes where b holds (of a comparison: one scalar pair, no value in between)
__device__ __forceinline__ uint64_t lanes(bool b) { return __builtin_amdgcn_ballot_w64(b); }
__device__ __forceinline__ double lane_double(double x, int q) {
  return __longlong_as_double((long long)lane_bcast((uint64_t)__double_as_longlong(x), q));
}

}  // namespace rannc
