// gfx950 kernel that answers a min-max search without its value tables: optimum, fewest stages and the canonical
// plan, for callers that want nothing else (rannc_dp_solve_to_host).  The tables themselves are made by the kernels in
// rannc_dp_kernels.hip, when they are asked for.
//
// Without send times the stage time h(i, j, r) of Sec. III-C and its bytes grow with the stage and fall with r, so
// for a given bound X the largest j for which the stage (i, j) on r replicas takes at most X and fits memory never
// falls as i grows.  Let R_s(d) be the last block that at most s stages on at most d devices reach, no stage above X:
//     R_s(d) = max over d' < d of (the end of the longest stage behind R_{s-1}(d') on d - d' replicas)
// D (D + 1) / 2 stages per level instead of N (N + 1) / 2 merges of D values, and the optimum is the smallest X with
// R_S(D) = N.  The stage counts of a plan are found the same way: the fewest s with R_s(D) = N at the optimum.
//
// Exactly s stages (the cells V[s][j][d] of the tables) against at most s: let s* be the fewest stages of a plan of
// value v = V[s*][N][D].  A cell (s, i, d) from which s* - s further stages reach N within v has no plan of fewer
// than s stages within v, or the whole would have fewer than s*.  For these LIVE cells "at most s stages" and
// "exactly s stages" are the same, their i are the interval from the first row that completes the plan to R_s(d), and
// every candidate of a live cell of value at most v lies in a live cell.  The walk of Algorithm 1's argmin (smallest
// i, then smallest d', of the candidates that attain the cell's value) therefore stays among them, and so does the
// recurrence for their values.  There are few: at the optimum the devices just suffice.
//
// Bound by latency: the devices are taken one after the other, some 350 ns each (sums of a row from lanes to scalars,
// a dozen dependent double-precision instructions, the next rows from LDS).  Per call, tables / this kernel: 96 blocks at 16
// devices 57 / 24 us, 1024 at 64 274 / 71 where memory binds and 453 / 17 where one stage holds everything, 701 at 48
// with 64-bit values 249 / 28, 2048 searches of 128 blocks 1666 / 143.
#include "rannc_dp_once.h"
#include "rannc_dp_sums.h"

#include <algorithm>
#include <type_traits>

namespace rannc {

// One bound X, by one wave; lane l holds the reach of d = l + 1 devices.
// A reach is of use only if the D - d devices that are left could take the rest within X, memory aside: T[reach] >=
// T[N] - (D - d) X.  Just above the optimum few blocks lie between that floor and the block that d devices reach
// without any waste, T <= d X, and a source that extends no lane beyond its floor costs one comparison.
struct Reach {
  const double *T, *P, *A;  // sums; T[N + 1] is infinite
  int N, D;
  double M, X;
  int most, next, reach;             // block reached without waste; the next one to be reached; the one reached
  double Tn, Pn, An, Tr, Pr, Ar;     // sums at the two

  __device__ __forceinline__ void start(double x) {
    X = x;
    const int lane = threadIdx.x & 63;
    const double d = (double)(lane + 1), cap = d * X, least = T[N] - ((double)D - d) * X;
    int lo = 0, below = 0;
    for (int bit = 1 << (31 - __clz(N)); bit; bit >>= 1) {  // (two independent chains of reads)
      const int j = min(lo + bit, N + 1), k = min(below + bit, N + 1);
      const double tj = T[j], tk = T[k];
      lo = tj <= cap ? j : lo;
      below = tk < least ? k : below;
    }
    most = lo;
    next = lane < D ? below + 1 : N + 1;  // (row 0 is no reach; least <= T[N], so that below < N)
    reach = 0;
    Tn = T[next]; Pn = P[next]; An = A[next];
    Tr = Pr = Ar = 0.0;
  }
  // the stage behind the block with sums Ti, Pi, Ai that d' devices reach: the lanes whose reach it extends
  __device__ __forceinline__ uint64_t push(int devices, double Ti, double Pi, double Ai) {
    const int lane = threadIdx.x & 63;
    const double r = (double)(lane + 1 - devices), until = __builtin_fma(r, X, Ti), room = M + Pi;
    // bytes P + ceil(A / r) <= M  <=>  r (M - P) - A >= 0
    auto fits = [&](double t, double p, double a) { return t <= until && __builtin_fma(r, room - p, Ai - a) >= 0.0; };
    const bool ok = lane >= devices && fits(Tn, Pn, An);
    const uint64_t m = lanes(ok);
    if (m == 0ull) return m;
    int lo = next, hi = ok ? most : next;
    while (lanes(lo < hi) != 0ull) {
      const int mid = (lo + hi + 1) >> 1;
      if (fits(T[mid], P[mid], A[mid])) lo = mid;
      else hi = mid - 1;
    }
    if (ok) {
      reach = lo;
      next = lo + 1;
      Tr = T[lo]; Pr = P[lo]; Ar = A[lo];
      Tn = T[next]; Pn = P[next]; An = A[next];
    }
    return m;
  }
  // the fewest stages, at most S, in which D devices reach N, or 0; table: R_s(d) of the levels below, 0 where no
  // reach is of use, at table[(s - 1) * stride + d - 1] (or null)
  __device__ __forceinline__ int stages(double x, int S, uint16_t *table, int stride) {
    const int lane = threadIdx.x & 63;
    start(x);
    uint64_t changed = push(0, 0.0, 0.0, 0.0);
    for (int s = 1;; ++s) {
      if (lanes(reach == N) != 0ull) return s;
      if (s == S || changed == 0ull) return 0;
      if (table && lane < D) table[(s - 1) * stride + lane] = (uint16_t)reach;
      const int reach0 = reach;
      const double T0 = Tr, P0 = Pr, A0 = Ar;
      uint64_t todo = changed;
      changed = 0ull;
      for (int row = 0; todo; todo &= todo - 1ull) {
        const int from = __ffsll((long long)todo) - 1;
        const int i = (int)lane_bcast((uint32_t)reach0, from);
        if (i == row) continue;
        row = i;
        changed |= push(from + 1, lane_double(T0, from), lane_double(P0, from), lane_double(A0, from));
      }
    }
  }
};

struct ReachPlan {
  int32_t end[RANNC_DP_MAX_DEVICES], replicas[RANNC_DP_MAX_DEVICES];
};

// The canonical plan of s stages and value v over all blocks and devices, by one wave.  reach: R_1 .. R_{s-1} at v;
// first, base: the same shape; value: `cells` entries.  False: more live cells than that.
__device__ __forceinline__ bool reach_plan(const Reach &w, int s_all, double v, const uint16_t *reach, uint16_t *first, uint16_t *base,
                                           int stride, double *value, int cells, ReachPlan &plan) {
  const int lane = threadIdx.x & 63, N = w.N, D = w.D;
  const double *const T = w.T, *const P = w.P, *const A = w.A;
  const double M = w.M;
  auto stage = [&](int i, int j, int r, double x) {  // takes at most x and fits
    return T[j] - T[i] <= (double)r * x && __builtin_fma((double)r, M + P[i] - P[j], A[i] - A[j]) >= 0.0;
  };
  auto lds_order = [] {  // what this wave has written to LDS is what it reads
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  // live cells, from the top: (s, i, lane + 1) for first[s][lane] <= i <= reach[s][lane]
  int total = 0;
  for (int s = s_all - 1; s >= 1; --s) {
    const int last = lane < D ? (int)reach[(s - 1) * stride + lane] : 0;
    int least = 0xFFFF;
    auto into = [&](int j, int d) {  // the candidates of the live cell (s + 1, j, d)
      const int r = d - (lane + 1);
      const bool ok = r >= 1 && last >= 1 && last < j && stage(last, j, max(r, 1), v);
      if (lanes(ok) == 0ull) return;
      int lo = 1, hi = ok ? last : 1;
      while (lanes(lo < hi) != 0ull) {
        const int mid = (lo + hi) >> 1;
        if (stage(mid, j, max(r, 1), v)) hi = mid;
        else lo = mid + 1;
        lo = min(lo, hi);
      }
      if (ok) least = min(least, lo);
    };
    if (s == s_all - 1) {
      into(N, D);
    } else {
      const int above_first = lane < D ? (int)first[s * stride + lane] : 0xFFFF, above_last = lane < D ? (int)reach[s * stride + lane] : 0;
      for (uint64_t m = lanes(above_first <= above_last); m; m &= m - 1ull) {
        const int d = __ffsll((long long)m) - 1;
        const int j0 = (int)lane_bcast((uint32_t)above_first, d), j1 = (int)lane_bcast((uint32_t)above_last, d);
        for (int j = j0; j <= j1; ++j) into(j, d + 1);
      }
    }
    const int mine = least <= last ? last - least + 1 : 0;
    int run = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int x = __shfl_up(run, o);
      if (lane >= o) run += x;
    }
    const int count = (int)lane_bcast((uint32_t)run, 63);
    if (total + count > cells) return false;
    if (lane < D) {
      first[(s - 1) * stride + lane] = (uint16_t)least;
      base[(s - 1) * stride + lane] = (uint16_t)(total + run - mine);
    }
    total += count;
    lds_order();
  }
  // their values, from the bottom.  (One cell to a level: nothing is left to choose.)
  const bool choose = total > s_all - 1;
  for (int s = 1; s < s_all; ++s) {
    const int from = lane < D ? (int)first[(s - 1) * stride + lane] : 0xFFFF, last = lane < D ? (int)reach[(s - 1) * stride + lane] : 0;
    const int at = lane < D ? (int)base[(s - 1) * stride + lane] : 0;
    if (!choose || s == 1) {
      for (int i = from; i <= last; ++i) value[at + i - from] = choose ? ceil(T[i] / (double)(lane + 1)) : 0.0;
    } else {
      const int below_first = lane < D ? (int)first[(s - 2) * stride + lane] : 0xFFFF, below_last = lane < D ? (int)reach[(s - 2) * stride + lane] : 0;
      const int below_at = lane < D ? (int)base[(s - 2) * stride + lane] : 0;
      for (uint64_t m = lanes(from <= last); m; m &= m - 1ull) {
        const int d = __ffsll((long long)m) - 1;
        const int j0 = (int)lane_bcast((uint32_t)from, d), j1 = (int)lane_bcast((uint32_t)last, d), to = (int)lane_bcast((uint32_t)at, d);
        const int r = d - lane;
        for (int j = j0; j <= j1; ++j) {
          double best = __builtin_inf();
          if (r >= 1)
            for (int i = below_first; i <= min(below_last, j - 1); ++i)
              if (stage(i, j, r, v)) best = fmin(best, fmax(value[below_at + i - below_first], ceil((T[j] - T[i]) / (double)r)));
          const uint64_t least = wave_min((uint64_t)__double_as_longlong(best));  // (no value is negative)
          if (lane == 0) value[to + j - j0] = __longlong_as_double((long long)least);
        }
      }
    }
    lds_order();
  }
  // the walk
  int j = N, d = D;
  double x = v;
  for (int s = s_all; s >= 2; --s) {
    const int from = lane < D ? (int)first[(s - 2) * stride + lane] : 0xFFFF, last = lane < D ? (int)reach[(s - 2) * stride + lane] : 0;
    const int at = lane < D ? (int)base[(s - 2) * stride + lane] : 0;
    uint32_t key = ~0u;
    double mine = 0.0;
    if (lane + 1 < d)
      for (int i = from; i <= min(last, j - 1); ++i) {
        mine = value[at + i - from];
        if (mine <= x && stage(i, j, d - lane - 1, x)) { key = (uint32_t)i << 8 | (uint32_t)(lane + 1); break; }
      }
    const uint32_t best = wave_min(key);
    if (best == ~0u) return false;  // (there is one; left to the tables)
    const int before = (int)(best & 255u);
    if (lane == 0) { plan.end[s - 1] = j; plan.replicas[s - 1] = d - before; }
    if (choose) x = lane_double(mine, before - 1);
    j = (int)(best >> 8);
    d = before;
  }
  if (lane == 0) { plan.end[0] = j; plan.replicas[0] = d; }
  lds_order();
  return true;
}

// The same from the chain's end: lane l holds the first block behind which e = l + 1 devices can take the rest, in any
// number of stages.  (Rows count from the front: blocks i + 1 .. N.)  Of use are the rows that the D - e devices in
// front could reach without waste, T[row] <= (D - e) X: the window, from there down to T[row] >= T[N] - e X.  A lane holds
// the sums of the four rows that are next, which is what most pushes extend a row by at most.
typedef __attribute__((address_space(3))) uint32_t LdsWord;
struct Completion {
  const double *T, *P, *A;  // sums; T[-4 .. -1] is minus infinity
  int N, D;
  double M;
  int top, least;  // the window
  int row;         // the smallest so far (N: none)
  uint64_t held;   // lanes with one

  // Whether all devices take all blocks within x; then bit `wave` of *mask is set, as soon as that is known.  Given up
  // where a wave below, with a smaller bound, has found so: a larger bound takes longer.
  __device__ __forceinline__ void run(double x, uint32_t *mask, int wave) {
    constexpr int K = kReachPad;
    const int lane = threadIdx.x & 63;
    const double e = (double)(lane + 1), until = T[N] - e * x, cap = ((double)D - e) * x;
    int lo = 0, below = -1;
    for (int bit = 1 << (31 - __clz(N)); bit; bit >>= 1) {  // (two independent chains of reads)
      const int j = min(lo + bit, N), k = min(below + bit, N);
      const double tj = T[j], tk = T[k];
      lo = tj <= cap ? j : lo;
      below = tk < until ? k : below;
    }
    top = lane < D ? min(lo, N - 1) : -1;  // (a stage is not empty)
    least = below + 1;
    row = N;
    int next = top;
    double t[K], p[K], a[K], Tr = 0.0, Pr = 0.0, Ar = 0.0;
    auto fetch = [&]() {
#pragma unroll
      for (int k = 0; k < K; ++k) { t[k] = T[next - k]; p[k] = P[next - k]; a[k] = A[next - k]; }
    };
    next = max(next, -1);
    fetch();
    held = 0ull;
    uint64_t whole = 0ull;  // lanes that take all blocks
    // the stages in front of the last source, the row with sums Tj, Pj, Aj that `devices` complete
    int devices = 0;
    double Tj = T[N], Pj = P[N], Aj = A[N];
    uint64_t later = ~0ull;  // lanes behind it
#pragma unroll 1
    for (;;) {
      const double r = (double)(lane + 1 - devices), from = __builtin_fma(-r, x, Tj), room = M - Pj;
      auto fits = [&](double ti, double pi, double ai) { return (ti >= from) & (__builtin_fma(r, room + pi, ai - Aj) >= 0.0); };
      const uint64_t m = lanes(lane >= devices) & lanes(t[0] >= from) & lanes(__builtin_fma(r, room + p[0], a[0] - Aj) >= 0.0);
      const bool ok = (m >> lane & 1ull) != 0ull;
      const uint32_t found = __hip_atomic_load((LdsWord *)mask, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (m != 0ull) {
        held |= m;
        // (the rows that fit are the first ones)
        const bool f1 = fits(t[1], p[1], a[1]), f2 = fits(t[2], p[2], a[2]), f3 = fits(t[3], p[3], a[3]);
        int to = next - (f3 ? 3 : f2 ? 2 : f1 ? 1 : 0);
        if (lanes(ok & f3 & (to > least)) != 0ull) {
          int l = (ok & f3) ? min(least, to) : to, h = to;
          while (lanes(l < h) != 0ull) {
            const int mid = (l + h) >> 1;
            const bool f = fits(T[mid], P[mid], A[mid]);
            h = f ? mid : h;
            l = f ? l : min(mid + 1, h);
          }
          to = h;
        }
        if (ok) {
          row = to;
          next = to - 1;
          if (to == 0 && !whole) atomicOr(mask, 1u << wave);
          Tr = T[to]; Pr = P[to]; Ar = A[to];
          fetch();
        }
        whole |= lanes(ok & (to == 0));
      }
      if (((uint32_t)__builtin_amdgcn_readfirstlane((int)found) & ((1u << wave) - 1u)) != 0u) break;
      const uint64_t rest = held & later;
      if (rest == 0ull) break;
      devices = __ffsll((long long)rest);
      later = ~((2ull << (devices - 1)) - 1ull);
      if (lane_bcast((uint32_t)row, devices - 1) == 0u) break;
      Tj = lane_double(Tr, devices - 1); Pj = lane_double(Pr, devices - 1); Aj = lane_double(Ar, devices - 1);
    }
    if (whole && lane >= __ffsll((long long)whole) - 1) row = 0;  // (with more devices as well)
  }
};

// A search whose optimum is at most x, by one wave: Completion has left the rows [first, last] of lane l = d - 1 that can
// be part of a plan within x (at most kReachPad of them; lane D - 1: N alone).  Values of these cells over any number
// of stages give the optimum; then the fewest stages and, of the plans with so few, the values, as one number; then the
// walk.  Cells are taken in the order of their devices, and each is tried in front of all lanes behind it.
// Returns the fewest stages; opt: the optimum.
constexpr double kReachStage = 0x1p45;  // stages * kReachStage + value orders by stages, then values
template <int K>
__device__ __forceinline__ int reach_finish(const double *T, const double *P, const double *A, int N, int D, double M, double x, int first,
                                            int last, const double *inverse, double &opt, ReachPlan &plan, int most_stages) {
  const int lane = threadIdx.x & 63;
  const double none = __builtin_inf();
  double t[K], p[K], a[K], v[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int j = min(max(first + k, 0), N);
    t[k] = first + k <= last ? T[j] : none;
    p[k] = P[j];
    a[k] = A[j];
  }
  // first the values over any number of stages (the optimum), then stages and values of what stays within the optimum
  auto cells = [&](double bound, auto second) {
    constexpr bool SECOND = decltype(second)::value;
    // the stages behind `devices` devices and the row with sums Ti, Pi, Ai, of value vi
    auto push = [&](int devices, double Ti, double Pi, double Ai, double vi) {
      const int r = lane + 1 - devices;
      const double inv = inverse[max(r, 1) - 1], rd = (double)r, until = __builtin_fma(rd, bound, Ti), room = M + Pi;
      const double add = __builtin_fma(rd, 0.5 + CeilDiv<uint64_t>::kOffset, -1.0) - Ti;
      double base = 0.0, so_far = vi;
      if constexpr (SECOND) {
        const double s = floor(vi * (1.0 / kReachStage));
        base = __builtin_fma(s, kReachStage, kReachStage);
        so_far = __builtin_fma(-s, kReachStage, vi);
      }
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const bool ok = (r >= 1) & (t[k] <= until) & (__builtin_fma(rd, room - p[k], Ai - a[k]) >= 0.0);
        double h = __builtin_fma(t[k] + add, inv, 0x1.8p52) - 0x1.8p52;  // ceil_div
        h = dmax(so_far, h);
        if constexpr (SECOND) h += base;
        v[k] = dmin(v[k], ok ? h : none);
      }
    };
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = none;
    push(0, 0.0, 0.0, 0.0, 0.0);
    uint64_t later = (1ull << (D - 1)) - 1ull;  // lanes that are still to be sources
#pragma unroll 1
    for (;;) {
      uint64_t held[K], any = 0ull;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        held[k] = lanes(v[k] != none) & later;
        any |= held[k];
      }
      if (any == 0ull) break;
      const int from = __ffsll((long long)any) - 1;
      later &= ~((2ull << from) - 1ull);
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (K == 1 || (held[k] >> from & 1ull))
          push(from + 1, lane_double(t[k], from), lane_double(p[k], from), lane_double(a[k], from), lane_double(v[k], from));
    }
    return lane_double(v[0], D - 1);
  };
  opt = cells(x, std::false_type());
  const int stages = (int)(cells(opt, std::true_type()) * (1.0 / kReachStage));
  if (stages > most_stages) return stages;
  // the walk: of the candidates with one stage fewer and a value of at most the cell's, the smallest row, then the fewest
  // devices
  int j = N, devices = D;
  double val = opt;
  for (int s = stages; s >= 2; --s) {
    const int r = devices - (lane + 1);
    const double rd = (double)r, Tj = T[j], Pj = P[j], Aj = A[j], from = __builtin_fma(-rd, val, Tj), base = (double)(s - 1) * kReachStage;
    uint32_t best = ~0u;
    double mine = 0.0;
#pragma unroll
    for (int k = K - 1; k >= 0; --k) {
      const double w = v[k] - base;  // (of a cell with more stages: above any value; with fewer: there is none)
      const bool ok = (r >= 1) & (t[k] >= from) & (t[k] <= Tj) & (first + k < j) & (w >= 0.0) & (w <= val) &
                      (__builtin_fma(rd, M + p[k] - Pj, a[k] - Aj) >= 0.0);
      best = ok ? (uint32_t)(first + k) << 8 | (uint32_t)(lane + 1) : best;
      mine = ok ? w : mine;
    }
    const uint32_t chosen = wave_min(best);
    if (chosen == ~0u) return 0;  // (there is one)
    const int before = (int)(chosen & 255u);
    if (lane == 0) { plan.end[s - 1] = j; plan.replicas[s - 1] = devices - before; }
    val = lane_double(mine, before - 1);
    j = (int)(chosen >> 8);
    devices = before;
  }
  if (lane == 0) { plan.end[0] = j; plan.replicas[0] = devices; }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  return stages;
}

struct ReachDims { int N, D, S, cells; };  // largest of the launch
static_assert(kReachMaxBlocks < 0xFFFF, "16-bit rows");

template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void reach_kernel(const ReachIn *src, const ReachIn one, const int use_one, const ReachArgs args,
                                                           const ReachDims dims) {
  static_assert(WAVES >= 4 && WAVES <= 16, "a wave per array, and one");
  extern __shared__ __align__(16) char lds[];
  constexpr int W = (int)sizeof(ReachIn) / 4;
  __shared__ __align__(8) uint32_t s_in[W];
  __shared__ int s_flags, s_stages;
  __shared__ uint64_t s_total, s_bytes[2], s_opt;
  __shared__ uint32_t s_rows[2][WAVES][64];  // by round and wave: first row, and the window's last one << 16
  __shared__ double s_inverse[64];
  __shared__ uint32_t s_mask[3];
  __shared__ ReachPlan plan;
  const int tid = threadIdx.x, lane = tid & 63, q = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  ReachIn in = one;
  if (tid < 3) s_mask[tid] = 0u;
  if (tid == 0) s_flags = 0;
  if (wave == 3) s_inverse[lane] = 1.0 / (double)(lane + 1);
  if (!use_one && tid < W) s_in[tid] = ((const uint32_t *)(src + q))[tid];
  __syncthreads();
  if (!use_one) {
    const uint32_t mine = s_in[lane % W];
    union { ReachIn p; uint32_t u[W]; } x;
#pragma unroll
    for (int k = 0; k < W; ++k) x.u[k] = lane_bcast(mine, k);
    in = x.p;
  }
  const int N = in.N, D = in.D;
  const int entries = dims.N + 2 + kReachPad, shape = dims.S * dims.D;
  double *const sT = (double *)lds + kReachPad, *const sP = sT + entries, *const sA = sP + entries, *const value = sA + entries - kReachPad;
  uint16_t *const reach = (uint16_t *)(value + dims.cells), *const first_of = reach + shape, *const base = first_of + shape;

  // ---- sums ----
  if (wave < 3) {
    int flags = 0;
    uint32_t high = 0;
    const int64_t RANNC_GLOBAL *from = gptr(wave == 0 ? args.t : wave == 1 ? args.p : args.a) + in.first;
    int64_t RANNC_GLOBAL *save = gptr(args.save) + (int64_t)wave * args.blocks + (in.first - args.first);
    double *const s = wave == 0 ? sT : wave == 1 ? sP : sA;
    uint64_t total;
    if (N <= 64) total = reach_sums<1>(from, save, s, N, flags, high);
    else if (N <= 192) total = reach_sums<3>(from, save, s, N, flags, high);
    else if (N <= 576) total = reach_sums<9>(from, save, s, N, flags, high);
    else total = reach_sums<17>(from, save, s, N, flags, high);
    if (high >> 30) flags |= 2;
    if (flags) atomicOr(&s_flags, flags);
    if (lane < kReachPad) s[-1 - lane] = wave == 0 ? -__builtin_inf() : 0.0;
    if (lane == 0) {
      s[N + 1] = wave == 0 ? __builtin_inf() : 0.0;
      if (wave == 0) s_total = total;
      else s_bytes[wave - 1] = total;
    }
  }
  __syncthreads();
  int status = RANNC_DP_PROBLEM_OK;
  if (s_flags & 1) status = RANNC_DP_PROBLEM_NEGATIVE_INPUT;
  else if (s_flags & 2) status = RANNC_DP_PROBLEM_SUM_OVERFLOW;
  else if (s_total > (uint64_t)args.time_limit) status = RANNC_DP_PROBLEM_TIME_TOO_LARGE;
  else if (s_total >= (uint64_t)kReachMaxTime || s_bytes[0] >= (uint64_t)kReachMaxBytes || s_bytes[1] >= (uint64_t)kReachMaxBytes)
    status = kReachUndecided;

  uint64_t opt = (uint64_t)INT64_MAX;
  int n_stages = 0;
  if (status == RANNC_DP_PROBLEM_OK) {
    Reach w;
    w.T = sT; w.P = sP; w.A = sA; w.N = N; w.D = D;
    w.M = (double)min(in.M, (int64_t)(2 * kReachMaxBytes));  // (as good as unlimited)
    const uint64_t total = s_total;
    const uint64_t share = (total + (uint64_t)D - 1) / (uint64_t)D;  // of one device: no plan is better
    Completion back;
    back.T = sT; back.P = sP; back.A = sA; back.N = N; back.D = D; back.M = w.M;
    // A bound per wave and round.  lo .. hi - 1: the bounds that are left (all below fail, hi holds).
    uint64_t lo = share, hi = max(total, share);
    int round = 0;
    // The round's bounds are bound(0) <= bound(1) <= ...; holds(x, mask): sets this wave's bit if its bound does.  Returns the first one that
    // does (WAVES: none).
    auto ask = [&](auto bound, auto holds) -> int {
      holds((double)bound(wave), &s_mask[round % 3]);
      if (tid == 0) s_mask[(round + 1) % 3] = 0u;
      lds_barrier();
      const uint32_t mask = s_mask[round % 3];
      const int k = mask ? __ffs((int)mask) - 1 : WAVES;
      const uint64_t upper = k < WAVES ? bound(k) : hi, lower = k > 0 ? bound(k - 1) + 1 : lo;
      hi = upper;
      lo = max(lo, lower);
      ++round;
      return k;
    };
    // v of n bounds between lo and hi, excesses over `over` in geometric steps (of at most an eighth of the range at
    // first); every one if there are no more
    auto between = [&](uint64_t over, int v, int n) -> uint64_t {
      const uint64_t gap = hi - lo;
      if (gap <= (uint64_t)n) return min(lo + (uint64_t)v, hi - 1);
      if (round > 10) return lo + gap * (uint64_t)(v + 1) / (uint64_t)(n + 1);
      const float high = (float)(hi - over), low = fmaxf((float)(lo - over), 0.125f * high);
      const float at = low * __builtin_amdgcn_exp2f(__builtin_amdgcn_logf(high / low) * (float)(v + 1) / (float)(n + 1));
      return min(max(over + (uint64_t)at, lo), hi - 1);
    };
    int first = 1, last = 0, widest = 0;  // cells of a lane at hi (wave 0)
    // whether the cells that are left at hi are few; k: the wave that has asked for hi in this round
    auto few = [&](int k) -> bool {
      const uint32_t r = s_rows[(round - 1) & 1][k][max(D - 2 - lane, 0)];  // devices behind this lane's d: D - 1 - lane
      first = lane < D - 1 ? max((int)(r & 0xffffu), 1) : N;
      last = lane < D - 1 ? (int)(r >> 16) : N;
      const int width = lane < D ? max(last - first + 1, 0) : 0;
      widest = 1;
      int cells = 0;
#pragma unroll
      for (int n = 1; n <= kReachPad; ++n) {
        const uint64_t m = lanes(width >= n);
        if (m) widest = n;
        cells += __popcll(m);
      }
      return lanes(width > kReachPad) == 0ull && (cells <= 2 * D || lo >= hi);
    };
    auto completes = [&](double x, uint32_t *mask) {
      back.run(x, mask, wave);
      s_rows[round & 1][wave][lane] = (uint32_t)back.row | (uint32_t)(back.top & 0xffff) << 16;
    };
    auto staged = [&](double x, uint32_t *mask) {
      const int s = w.stages(x, in.S, nullptr, 0);
      if (s && lane == 0) atomicOr(mask, 1u << wave);
    };
    bool found = true, done = false;
    if (__builtin_fma((double)D, w.M - sP[N], -sA[N]) >= 0.0) {  // one stage of everything
      hi = share;
      n_stages = 1;
      if (tid == 0) { plan.end[0] = N; plan.replicas[0] = D; }
      done = true;
    } else {
      // First the excess over a share that is usual, up to eight of the chain's mean blocks over all devices together; then
      // up to everything; then between.
      constexpr float step = WAVES >= 16 ? 0.5f : WAVES >= 8 ? 1.0f : 2.5f;
      const float block = 8.0f * (float)share / (float)N;
      bool fits = false;
      for (int kind = 0;;) {
        const uint64_t from = lo;
        auto bound = [&](int v) -> uint64_t {
          if (kind == 0) return v == 0 ? share : min(share + (uint64_t)(block * __builtin_amdgcn_exp2f(step * (float)(v - (WAVES - 1)))), total);
          if (kind == 1) {
            if (v == WAVES - 1) return total;
            const float most = (float)(total - share), least = fmaxf((float)(from - share), 1.0f);
            const float at = least * __builtin_amdgcn_exp2f(__builtin_amdgcn_logf(fmaxf(most / least, 1.0f)) * (float)(v + 1) / (float)WAVES);
            return min(max(share + (uint64_t)at, from), total);
          }
          return between(share, v, WAVES);
        };
        const int k = ask(bound, completes);
        if (kind < 2 && k == WAVES) {
          found = ++kind < 2 && lo <= total;
          if (!found) break;
          continue;
        }
        kind = 2;
        if (k < WAVES) fits = few(k);
        if (fits || lo >= hi) break;
      }
      if (fits) {
        if (wave == 0) {
          double opt_at = 0.0;
          const double x = (double)hi;
          const int s = widest == 1 ? reach_finish<1>(sT, sP, sA, N, D, w.M, x, first, last, s_inverse, opt_at, plan, in.S)
                      : widest == 2 ? reach_finish<2>(sT, sP, sA, N, D, w.M, x, first, last, s_inverse, opt_at, plan, in.S)
                                    : reach_finish<kReachPad>(sT, sP, sA, N, D, w.M, x, first, last, s_inverse, opt_at, plan, in.S);
          if (lane == 0) { s_stages = s; s_opt = (uint64_t)opt_at; }
        }
        lds_barrier();
        n_stages = s_stages;
        hi = s_opt;
        done = n_stages >= 1 && n_stages <= in.S;
        if (!done) n_stages = 0;
        lds_barrier();
      }
    }
    // Many cells at the optimum, or not enough stages: level by level.
    for (int turn = 0; found && !done; ++turn) {
      if (wave == 0) {
        const int s = w.stages((double)hi, in.S, reach, dims.D);
        if (lane == 0) s_stages = s;
      }
      lds_barrier();
      n_stages = s_stages;
      lds_barrier();
      if (n_stages || turn) break;
      // the stages do not suffice there: the bound is larger
      const uint64_t over = hi;
      lo = hi + 1;
      hi = total;
      found = lo <= total && ask([&](int) { return total; }, staged) < WAVES;
      lo = over + 1;  // (every wave has asked for the same)
      while (found && lo < hi)
        ask([&](int v) { return between(over, v, WAVES); }, staged);
    }
    if (found && n_stages) {
      opt = hi;
      if (wave == 0 && !done) {
        const bool ok = n_stages == 1 || reach_plan(w, n_stages, (double)hi, reach, first_of, base, dims.D, value, dims.cells, plan);
        if (n_stages == 1 && lane == 0) { plan.end[0] = N; plan.replicas[0] = D; }
        if (!ok) status = kReachUndecided;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }
  // ---- results, by one wave ----
  if (wave != 0) return;
  if (status != RANNC_DP_PROBLEM_OK || opt == (uint64_t)INT64_MAX) {
    n_stages = 0;
    opt = (uint64_t)INT64_MAX;
  }
  const PlanResults &r = args.results;
  const bool host = r.h_flag != nullptr;
  if (lane == 0) {
    int64_t est = INT64_MAX;
    if (n_stages > 0) {
      const int64_t f = (int64_t)in.MB + n_stages - 1, best = (int64_t)opt;
      est = (best != 0 && f > INT64_MAX / best) ? INT64_MAX : f * best;
    }
    r.d_opt[q] = (int64_t)opt;
    r.d_est[q] = est;
    r.d_n_stages[q] = n_stages;
    r.d_status[q] = status;
    if (host) {
      r.h_opt[q] = (int64_t)opt;
      r.h_est[q] = est;
      r.h_n_stages[q] = n_stages;
      r.h_status[q] = status;
    }
  }
  for (int u = lane; u < args.plan_stride; u += 64) {
    const int32_t end = u < n_stages ? plan.end[u] : -1, reps = u < n_stages ? plan.replicas[u] : -1;
    const int64_t e = (int64_t)q * args.plan_stride + u;
    r.d_stage_end[e] = end;
    r.d_replicas[e] = reps;
    if (host) {
      r.h_stage_end[e] = end;
      r.h_replicas[e] = reps;
    }
  }
  if (!host) return;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");  // (of the whole wave, for the system)
  if (lane == 0) __hip_atomic_store(&r.h_flag[q], r.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

hipError_t launch_reach(const ReachIn *src, const ReachIn *host_one, int Q, const LaunchShape &sh, const ReachArgs &args, hipStream_t st) {
  if (sh.max_N > kReachMaxBlocks) return hipErrorInvalidValue;
  const ReachDims dims = {sh.max_N, sh.max_D, sh.max_S_eff, Q > 64 ? 256 : 1024};
  const size_t lds = (size_t)(dims.N + 2 + kReachPad) * 24 + (size_t)dims.cells * 8 + (size_t)dims.S * dims.D * 6;
  const ReachIn one = host_one ? *host_one : ReachIn{};
  auto go = [&](auto waves) -> hipError_t {
    constexpr int W = decltype(waves)::value;
    if (lds > 56 * 1024) {  // (with the 8 KB and more of the kernel's own, what need not be asked for)
      static std::atomic<uint64_t> asked{0};
      const hipError_t e = allow_lds(asked, (const void *)reach_kernel<W>, 144 * 1024);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(reach_kernel<W>, dim3(Q), dim3(64 * W), lds, st, src, one, host_one ? 1 : 0, args, dims);
    return hipGetLastError();
  };
  // Waves of a search, each with a bound of its own: as many as the device has places for (100 registers: four waves per
  // SIMD), and no more than eight for up to sixteen devices, whose bounds take little longer than the start of a wave.
  // Per call, 4 / 8 / 16 waves: 16 blocks at 4 devices 29 / 30 / 32 us, 96 at 16 34 / 33 / 32, 300 at 32 41 / 50 / 42,
  // 1024 at 64 99 / 65 / 65, 32 searches of 1000 at 64 148 / 119 / 105, 200 of 128 at 64 85 / 49 / 47, 512 93 / 56 / 63,
  // 1024 of 128 at 16 66 / 77 / 95, 2000 of 60 at 32 106 / 110 / 132.
  if (Q > 512) return go(std::integral_constant<int, 4>());
  if (Q > 64 || sh.max_D <= 16) return go(std::integral_constant<int, 8>());
  return go(std::integral_constant<int, 16>());
}

}  // namespace rannc
