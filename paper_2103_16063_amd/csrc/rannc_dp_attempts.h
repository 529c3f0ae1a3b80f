// The bounds that rannc_dp_bound.hip runs Algorithm 1's levels at, one after the other, until one gives the last cell a value.
#pragma once

#include <hip/hip_runtime.h>

namespace rannc {

enum LevelState { kLevelsNone, kLevelsFound, kLevelsOpen };  // of a bound: no value; a value; more cells than there is room for

// least: no value is smaller.  asked: it is a bound at which many cells were left, so that no plan has been priced; else the
// first bound is a plan's price.  With one objective that price is a value, and tables take 40 to 80 us: two attempts, the first one
// behind `least` itself, which has no value where something is sent.  With the maxima apart they take 30 us to milliseconds.
// (600 searches of either form, one objective: 42 took a tenth longer than with tables, up to 2.8 times, where four attempts
// began at `least`; 37, and 2.6 % less over all.)
struct Attempts {
  double least;
  bool asked, apart;  // apart: forward and backward maxima
  bool small;         // of few blocks and devices
  __host__ __device__ int most() const { return !apart ? 2 : small ? 4 : 6; }
  __host__ __device__ double first(double price) const {
    return !asked ? price : apart ? least : least + floor(least * 0.015625) + 1.0;
  }
  // the bound behind U, which gave `state` as attempt number k (from 0); negative: no further one
  __host__ __device__ double next(int k, double U, LevelState state) const {
    if (state == kLevelsFound || k + 1 >= most()) return -1.0;
    // (too many cells are too many at larger bounds; at a smaller one they may do)
    if (state == kLevelsOpen) return k == 0 && U > least ? least + floor((U - least) * 0.25) : -1.0;
    return apart && asked && k == 0 ? U + floor(U * 0.015625) + 1.0 : least + (U - least + 1.0) * (apart ? 2.0 : 4.0);
  }
};

}  // namespace rannc
