// A min-max search over sums in LDS without its value tables: the device code shared by rannc_dp_reach.hip, which answers
// such searches with it, and rannc_dp_bound.hip, which starts from its plan.
#pragma once

#include "rannc_dp_attempts.h"
#include "rannc_dp_once.h"
#include "rannc_dp_sums.h"

#include <algorithm>
#include <type_traits>

namespace rannc {

struct ReachPlan {
  int32_t end[RANNC_DP_MAX_DEVICES], replicas[RANNC_DP_MAX_DEVICES];
};

// One bound x, by one wave; lane l holds the first block behind which e = l + 1 devices can take the rest, in any
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
          // (most rows move little: in doubling steps, then between the last two)
          bool on = l < h;
          for (int step = kReachPad; lanes(on) != 0ull; step *= 2) {
            const int mid = max(h - step, l);
            const bool f = fits(T[mid], P[mid], A[mid]);
            h = (on && f) ? mid : h;
            l = (on && !f) ? mid + 1 : l;
            on = on && f && l < h;
          }
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

struct ReachDims { int N, level_cells, level_sources, level_records, grow; };  // longest of the launch, and room for the levels
static_assert(kReachMaxBlocks < 0xFFFF, "16-bit rows");

template <int WAVES> struct ReachShared {
  int stages;
  uint64_t opt;
  uint32_t rows[2][WAVES][64];  // by round and wave: first row, and the window's last one << 16
  uint32_t kept[64];            // those of the bound that holds
  double inverse[64];
  uint32_t mask[3];
  ReachPlan plan;
  // of the levels
  int count, first[64], last[64], base[65];
  int from[RANNC_DP_MAX_DEVICES + 2];        // records of a level begin here
  uint32_t reached[RANNC_DP_MAX_DEVICES + 1];  // what the last cell was reached from, by level
};

// ---- Algorithm 1's levels among the cells that a bound U leaves ----
// Let T be the sums of all times of a block (forward and backward, no send times).  A stage of value at most U on r
// replicas has T[j] - T[i] <= r U, so a cell (s, i, d) that is part of a plan of value at most U lies in a window:
// T[i] <= d U, and the D - d devices behind can take the rest, every stage's T within its r U and its bytes within memory
// (Completion).  With a cell the windows hold every candidate of value at most U of it (what is in front of it only has to
// get there, and behind it the cell's own rest follows), and values never fall along a plan: the levels computed among the
// windows' cells alone, values above U dropped, give every value up to U, and its argmin, exactly as the full tables
// do.  That holds for both objectives, also where Algorithm 1 as printed is no minimum over plans: what it keeps in a cell
// depends on candidates of at most that value only.  So any U at which the last cell (N, D) gets a value is answered by the smallest
// one of all levels.  Where a later level could only repeat a value it is not looked for: U falls to below the best value so far,
// and the levels end when no cell is left.
// Few of the windows' cells get a value: a level is one turn of pushes (a wave to a source, a lane or several to a
// device count, the rows of its window one after the other, some 40 instructions each), a look at all cells, and two barriers.
struct LevelSpace {
  int cells, sources, records;  // of the windows, of a level, of all levels
  char *at;                     // LDS
};
constexpr size_t level_bytes(int cells, int sources, int records, bool split) {
  return (size_t)cells * (split ? 14 : 12) + (size_t)sources * (split ? 40 : 24) + (size_t)records * 8;
}
struct LevelSums { const double *T, *P, *A, *B, *C; };  // B: backward times alone; C: send times by the block in front of the cut

// forward time (with what is sent) and backward time of the stage i+1 .. j on r replicas
template <bool SPLIT, bool COMM>
__device__ __forceinline__ void level_times(const LevelSums &x, const double *inverse, int i, int j, int r, double &f, double &b) {
  const double rd = (double)r, inv = inverse[r - 1], add = __builtin_fma(rd, 0.5 + CeilDiv<uint64_t>::kOffset, -1.0);
  auto ceil_of = [&](double v) { return __builtin_fma(v + add, inv, 0x1.8p52) - 0x1.8p52; };
  const double t = x.T[j] - x.T[i];
  b = 0.0;
  if constexpr (SPLIT) {
    const double tb = x.B[j] - x.B[i];
    b = ceil_of(tb);
    f = ceil_of(t - tb);
  } else {
    f = ceil_of(t);
  }
  if constexpr (COMM) f += ceil_of(x.C[j]);
}

// By the workgroup.  kept: sh.kept holds the windows of U, or of a larger bound.  most: stages.  Found: value, stages and sh.plan.
template <int WAVES, bool SPLIT, bool COMM>
__device__ __forceinline__ LevelState reach_levels(const LevelSums &x, int N, int D, double M, double U, bool kept, int most, const LevelSpace &space,
                                                ReachShared<WAVES> &sh, double &value, int &stages) {
  constexpr int NT = 64 * WAVES;
  constexpr uint64_t kNoKey = ~0ull;
  constexpr int kPlace = 18;  // bits of a place: row << 6 | devices - 1
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint64_t *const key = (uint64_t *)space.at;  // of a cell in the level at hand: value << kPlace | place of what it comes from
  double *const front_f = (double *)(key + space.cells);  // largest forward (or the only) and backward time of the sources
  double *const front_b = front_f + 2 * space.sources;
  uint32_t *const source = (uint32_t *)(front_b + (SPLIT ? 2 * space.sources : 0));  // places
  uint32_t *const record = source + 2 * space.sources;  // places of the cells, and of what they come from
  uint32_t *const record_of = record + space.records;
  uint32_t *const cell_at = record_of + space.records;  // places of the windows' cells
  uint16_t *const index = (uint16_t *)(cell_at + space.cells);  // SPLIT: source of a cell, in the level before
  __syncthreads();
  // ---- the windows ----
  if (wave == 0) {
    if (!kept) {
      Completion back;
      back.T = x.T; back.P = x.P; back.A = x.A; back.N = N; back.D = D; back.M = M;
      if (lane == 0) sh.mask[0] = 0u;
      back.run(U, &sh.mask[0], 0);
      sh.kept[lane] = (uint32_t)back.row | (uint32_t)(back.top & 0xffff) << 16;
      if (lane < 3) sh.mask[lane] = 0u;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    const uint32_t r = sh.kept[max(D - 2 - lane, 0)];  // devices behind this lane's d: D - 1 - lane
    const int first = lane < D - 1 ? max((int)(r & 0xffffu), 1) : N, last = lane < D - 1 ? (int)(int16_t)(r >> 16) : lane < D ? N : 0;
    const int width = lane < D ? max(last - first + 1, 0) : 0;
    int run = width;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(run, o);
      if (lane >= o) run += v;
    }
    sh.first[lane] = first;
    sh.last[lane] = width ? last : first - 1;
    sh.base[lane + 1] = run;
    if (lane == 0) { sh.base[0] = 0; sh.from[0] = 0; sh.from[1] = 0; }
  }
  __syncthreads();
  const int cells = sh.base[D];
  if (cells > space.cells) return kLevelsOpen;
  for (int d = wave; d < D; d += WAVES)
    for (int e = lane; e <= sh.last[d] - sh.first[d]; e += 64) cell_at[sh.base[d] + e] = (uint32_t)(sh.first[d] + e) << 6 | (uint32_t)d;
  // a lane's devices (of the first ones several lanes, each with its share of the rows)
  const int many = D <= 8 ? 8 : D <= 16 ? 16 : D <= 32 ? 32 : 64, mine = lane & (many - 1), share = 64 / many;
  const int first = sh.first[mine], last = sh.last[mine], at = sh.base[mine] - first;
  __syncthreads();
  for (int e = tid; e < cells; e += NT) {  // level 1
    const uint32_t c = cell_at[e];
    const int j = (int)(c >> 6), d = (int)(c & 63u) + 1;
    double f, b;
    level_times<SPLIT, COMM>(x, sh.inverse, 0, j, d, f, b);
    const double v = f + b;
    key[e] = v <= U && __builtin_fma((double)d, M - x.P[j], -x.A[j]) >= 0.0 ? (uint64_t)v << kPlace : kNoKey;
  }
  double best = __builtin_inf();
  int of_best = 0;
#pragma unroll 1
  for (int s = 1;; ++s) {
    __syncthreads();
    // ---- the level's cells: sources of the next one, and the records that the plan is read from ----
    const double *const pf = front_f + ((s - 1) & 1) * space.sources, *const pb = front_b + ((s - 1) & 1) * space.sources;
    double *const nf = front_f + (s & 1) * space.sources, *const nb = front_b + (s & 1) * space.sources;
    uint32_t *const ns = source + (s & 1) * space.sources;
    const int records = sh.from[s];
    const uint64_t last_key = key[cells - 1];
    if (last_key != kNoKey && (double)(last_key >> kPlace) < best) {
      best = (double)(last_key >> kPlace);
      of_best = s;
      if (tid == 0) sh.reached[s] = (uint32_t)last_key & ((1u << kPlace) - 1u);
    }
    if (s == most) break;
    if (tid == 0) sh.count = 0;
    const double bound = best - 1.0 < U ? best - 1.0 : U;  // what a further stage has to stay within
    __syncthreads();  // (all have read the last cell and where the records begin)
    for (int e0 = 64 * wave; e0 < cells - 1; e0 += NT) {
      const int e = e0 + lane;
      const uint64_t k = e < cells - 1 ? key[e] : kNoKey;
      const bool held = k != kNoKey && (double)(k >> kPlace) <= bound;
      const uint64_t m = lanes(held);
      int place = 0;
      if (m) {
        if (lane == 0) place = atomicAdd(&sh.count, __popcll(m));
        place = (int)lane_bcast((uint32_t)place, 0) + __popcll(m & ((1ull << lane) - 1ull));
      }
      if (e < cells - 1) key[e] = kNoKey;
      if (held && place < space.sources && records + place < space.records) {
        const uint32_t c = cell_at[e], w = (uint32_t)k & ((1u << kPlace) - 1u);
        ns[place] = c;
        record[records + place] = c;
        record_of[records + place] = w;
        if constexpr (SPLIT) {
          const int j = (int)(c >> 6), d = (int)(c & 63u) + 1;
          double f, b;
          if (s == 1) {
            level_times<SPLIT, COMM>(x, sh.inverse, 0, j, d, f, b);
          } else {
            const int i = (int)(w >> 6), dp = (int)(w & 63u) + 1, p = (int)index[sh.base[dp - 1] + i - sh.first[dp - 1]];
            level_times<SPLIT, COMM>(x, sh.inverse, i, j, d - dp, f, b);
            f = dmax(f, pf[p]);
            b = dmax(b, pb[p]);
          }
          nf[place] = f;
          nb[place] = b;
        } else {
          nf[place] = (double)(k >> kPlace);
        }
      }
    }
    if (tid == 0) key[cells - 1] = kNoKey;
    __syncthreads();
    const int n = sh.count;
    if (n > space.sources || records + n > space.records) return kLevelsOpen;
    if (n == 0) break;
    if (SPLIT)
      for (int k = tid; k < n; k += NT) {
        const uint32_t c = ns[k];
        const int d = (int)(c & 63u);
        index[sh.base[d] + (int)(c >> 6) - sh.first[d]] = (uint16_t)k;
      }
    // ---- the next level: every source in front of the windows of more devices ----
    for (int k = wave; k < n; k += WAVES) {
      const uint32_t c = (uint32_t)__builtin_amdgcn_readfirstlane((int)ns[k]);
      const int i = (int)(c >> 6), d = (int)(c & 63u) + 1, r = mine + 1 - d;
      const double fs = nf[k], bs = SPLIT ? nb[k] : 0.0, Ti = x.T[i], Pi = x.P[i], Ai = x.A[i], Bi = SPLIT ? x.B[i] : 0.0;
      const double rd = (double)r, inv = sh.inverse[max(r, 1) - 1], add = __builtin_fma(rd, 0.5 + CeilDiv<uint64_t>::kOffset, -1.0);
      const double until = __builtin_fma(rd, bound, Ti), room = M + Pi;
      auto ceil_of = [&](double v) { return __builtin_fma(v + add, inv, 0x1.8p52) - 0x1.8p52; };
      int j = max(i + 1, first) + lane / many;
      bool on = r >= 1 && mine < D && j <= last;
      while (lanes(on) != 0ull) {
        const int jj = on ? j : N;
        const double Tj = x.T[jj], Pj = x.P[jj], Aj = x.A[jj];
        on = on && Tj <= until && __builtin_fma(rd, room - Pj, Ai - Aj) >= 0.0;  // (further rows take longer, and more)
        double v;
        if constexpr (SPLIT) {
          const double tb = x.B[jj] - Bi, hb = ceil_of(tb);
          double hf = ceil_of(Tj - Ti - tb);
          if constexpr (COMM) hf += ceil_of(x.C[jj]);
          v = dmax(fs, hf) + dmax(bs, hb);
        } else {
          double h = ceil_of(Tj - Ti);
          if constexpr (COMM) h += ceil_of(x.C[jj]);
          v = dmax(fs, h);
        }
        if (on && v <= bound) atomicMin((unsigned long long *)&key[at + jj], (unsigned long long)((uint64_t)v << kPlace | (uint64_t)c));
        j += share;
        on = on && j <= last;
      }
    }
    if (tid == 0) sh.from[s + 1] = records + n;
  }
  if (!of_best) return kLevelsNone;
  // ---- the plan, by one wave ----
  if (wave == 0) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    int j = N, d = D;
    uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.reached[of_best]);
    for (int s = of_best; s >= 2; --s) {
      if (lane == 0) { sh.plan.end[s - 1] = j; sh.plan.replicas[s - 1] = d - (int)(w & 63u) - 1; }
      j = (int)(w >> 6);
      d = (int)(w & 63u) + 1;
      const int begin = sh.from[s - 1], end = sh.from[s];
      for (int e0 = begin; e0 < end; e0 += 64) {
        const uint64_t m = lanes(e0 + lane < end && record[min(e0 + lane, end - 1)] == w);
        if (m) {
          w = (uint32_t)__builtin_amdgcn_readfirstlane((int)record_of[e0 + __ffsll((long long)m) - 1]);
          break;
        }
      }
    }
    if (lane == 0) { sh.plan.end[0] = j; sh.plan.replicas[0] = d; }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  value = best;
  stages = of_best;
  return kLevelsFound;
}

// The search over sums in LDS (pads in front and the infinite time behind them included), by a workgroup: optimum,
// fewest stages (0: no plan), plan.  status: kReachUndecided where it is left to the tables.  mask, inverse: made.
// window: the bound that sh.kept holds the windows of (or 0).  ASK: where many cells are left at a bound,
// that is opt, and n_stages is -1: the caller asks the levels itself.
//
// Left to the tables as soon as it seems that it will be: where the stages there are do not suffice at the optimum of any number of
// them (the smallest bound at which they do lies far above: 175 blocks at 11 devices in at most 5 stages that are 98 % full 46 us with
// tables, 96 to 215 by larger bounds, 67 to 78 left at once), and where more cells are left at the optimum than the levels
// have room for, which the windows of a bound below it tell.
template <int WAVES, bool ASK_MANY, bool ASK_FEW>
__device__ __forceinline__ void reach_search(const ReachIn &in, const double M, const uint64_t total, const double *const sT, const double *const sP,
                                             const double *const sA, const LevelSpace &space, const int grow,
                                             ReachShared<WAVES> &sh, uint64_t &opt, int &n_stages, int &status, uint64_t &window) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = in.N, D = in.D;
  const uint64_t share = (total + (uint64_t)D - 1) / (uint64_t)D;  // of one device: no plan is better
  Completion back;
  back.T = sT; back.P = sP; back.A = sA; back.N = N; back.D = D; back.M = M;
  // A bound per wave and round.  lo .. hi - 1: the bounds that are left (all below fail, hi holds).
  uint64_t lo = share, hi = max(total, share);
  int round = 0;
  // The round's bounds are bound(0) <= bound(1) <= ...; returns the first one that holds (WAVES: none).
  auto ask = [&](auto bound) -> int {
    back.run((double)bound(wave), &sh.mask[round % 3], wave);
    sh.rows[round & 1][wave][lane] = (uint32_t)back.row | (uint32_t)(back.top & 0xffff) << 16;
    if (tid == 0) sh.mask[(round + 1) % 3] = 0u;
    lds_barrier();
    const uint32_t mask = lane_bcast(sh.mask[round % 3], 0);
    const int k = mask ? __ffs((int)mask) - 1 : WAVES;
    const uint64_t upper = k < WAVES ? bound(k) : hi, lower = k > 0 ? bound(k - 1) + 1 : lo;
    hi = lane_bcast(upper, 0);  // (the same in every lane: kept in scalar registers)
    lo = lane_bcast(lower > lo ? lower : lo, 0);
    ++round;
    return k;
  };
  // v of n bounds between lo and hi, excesses over the share in geometric steps (of at most an eighth of the range at
  // first); every one if there are no more
  auto between = [&](int v, int n) -> uint64_t {
    const uint64_t gap = hi - lo;
    if (gap <= (uint64_t)n) return min(lo + (uint64_t)v, hi - 1);
    if (round > 10) return lo + gap * (uint64_t)(v + 1) / (uint64_t)(n + 1);
    const float high = (float)(hi - share), low = fmaxf((float)(lo - share), 0.125f * high);
    const float at = low * __builtin_amdgcn_exp2f(__builtin_amdgcn_logf(high / low) * (float)(v + 1) / (float)(n + 1));
    return min(max(share + (uint64_t)at, lo), hi - 1);
  };
  // a lane's window at the bound of wave k in the last round: first cell, and how many
  auto cells_of = [&](int k, int &first, int &last) -> int {
    const uint32_t r = sh.rows[(round - 1) & 1][k][max(D - 2 - lane, 0)];  // devices behind this lane's d: D - 1 - lane
    first = lane < D - 1 ? max((int)(r & 0xffffu), 1) : N;
    last = lane < D - 1 ? (int)(r >> 16) : N;
    return lane < D ? max(last - first + 1, 0) : 0;
  };
  window = 0;
  const double full = (sP[N] + sA[N] / (double)D) / ((double)in.S * M);  // of the bytes of all stages
  if (__builtin_fma((double)D, M - sP[N], -sA[N]) >= 0.0) {  // one stage of everything
    opt = share;
    n_stages = 1;
    if (tid == 0) { sh.plan.end[0] = N; sh.plan.replicas[0] = D; }
    return;
  }
  if (full > 1.0 + 0x1p-40) return;  // (what the stages hold, with all devices to each; and the rounding of that)
  if (N * D > 32768 && full > 0.75) {
    // Stages nearly full of bytes, so that the best plan of any number of stages takes more than there are, and at the bound that
    // they allow many cells are left: 1024 blocks at 64 devices, 9 stages 85 % full, tables 101 us, here 426.
    status = kReachUndecided;
    return;
  }
  // First the excess over a share that is usual, up to eight of the chain's mean blocks over all devices together; then
  // up to everything; then between.
  constexpr float step = WAVES >= 16 ? 0.5f : WAVES >= 8 ? 1.0f : 2.5f;
  const float block = 8.0f * (float)share / (float)N;
  bool few_stages = false;
#pragma unroll 1
  for (int kind = 0;;) {  // (kind grows in every turn but the last)
    const uint64_t from = lo;
    auto bound = [&](int v) -> uint64_t {
      if (kind == 0) return v == 0 ? share : min(share + (uint64_t)(block * __builtin_amdgcn_exp2f(step * (float)(v - (WAVES - 1)))), total);
      if (kind == 1) {
        if (v == WAVES - 1) return total;
        const float most = (float)(total - share), least = fmaxf((float)(from - share), 1.0f);
        const float at = least * __builtin_amdgcn_exp2f(__builtin_amdgcn_logf(fmaxf(most / least, 1.0f)) * (float)(v + 1) / (float)WAVES);
        return min(max(share + (uint64_t)at, from), total);
      }
      return between(v, WAVES);
    };
    const int k = ask(bound);
    if (kind < 2 && k == WAVES) {
      if (++kind == 2 || lo > total) return;  // no plan
      continue;
    }
    int first = 1, last = 0, widest = 0;  // cells of a lane at hi
    bool fits = false;
    if (k < WAVES) {
      const int width = cells_of(k, first, last);
      if (wave == 0) sh.kept[lane] = sh.rows[(round - 1) & 1][k][lane];
      window = hi;
      widest = 1;
      int cells = 0;
#pragma unroll
      for (int n = 1; n <= kReachPad; ++n) {
        const uint64_t m = lanes(width >= n);
        if (m) widest = n;
        cells += __popcll(m);
      }
      fits = lanes(width > kReachPad) == 0ull && (cells <= 2 * D || lo >= hi);
    }
    if (fits && widest <= 2) {
      if (wave == 0) {
        double opt_at = 0.0;
        const double x = (double)hi;
        const int s = widest == 1 ? reach_finish<1>(sT, sP, sA, N, D, M, x, first, last, sh.inverse, opt_at, sh.plan, in.S)
                                  : reach_finish<2>(sT, sP, sA, N, D, M, x, first, last, sh.inverse, opt_at, sh.plan, in.S);
        if (lane == 0) { sh.stages = s; sh.opt = (uint64_t)opt_at; }
      }
      lds_barrier();
      const int s = (int)lane_bcast((uint32_t)sh.stages, 0);
      if (s >= 1 && s <= in.S) {
        n_stages = s;
        opt = lane_bcast(sh.opt, 0);
        return;
      }
      few_stages = true;
    } else {
      if (k > 0 && k < WAVES) {  // at the optimum there are as many cells as at a bound below it, or more
        int run = cells_of(k - 1, first, last);
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) run += __shfl_xor(run, o);
        if (__builtin_amdgcn_readfirstlane(run) > space.cells) {
          status = kReachUndecided;
          return;
        }
      }
      if (!fits && kind != 2 && lo < hi) {
        kind = 2;
        continue;
      }
    }
    break;
  }
  // Many cells, though few may be reached (memory, or a long block, costs more than the share), or the stages do not suffice: the
  // levels tell, at hi and, where the stages do not suffice there, at one larger bound.
  if (few_stages ? ASK_FEW : ASK_MANY) {
    opt = hi;
    n_stages = -1;
    return;
  }
  const LevelSums sums = {sT, sP, sA, nullptr, nullptr};
#pragma unroll 1
  for (int turn = 0; turn < 2; ++turn) {
    if (few_stages && in.S * D > grow) break;
    const uint64_t U = few_stages ? min(hi + 4 * (hi - share) + (share >> 6) + 1, total) : hi;
    double v = 0.0;
    int s = 0;
    const LevelState state = reach_levels<WAVES, false, false>(sums, N, D, M, (double)U, U == hi, in.S, space, sh, v, s);
    __syncthreads();
    if (state == kLevelsFound) {
      n_stages = s;
      opt = lane_bcast((uint64_t)v, 0);
      return;
    }
    if (state == kLevelsNone && U >= total) return;  // (no plan takes longer)
    if (state == kLevelsNone && ASK_FEW) {
      opt = hi;
      n_stages = -1;
      return;
    }
    if (state == kLevelsOpen || few_stages) break;
    few_stages = true;
  }
  status = kReachUndecided;
}

// Results of search q, by the workgroup's first wave.
__device__ __forceinline__ void reach_results(const ReachIn &in, const ReachArgs &args, int q, const ReachPlan &plan, uint64_t opt, int n_stages,
                                              int status) {
  const int lane = threadIdx.x & 63;
  if (threadIdx.x >= 64) return;
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

}  // namespace rannc
