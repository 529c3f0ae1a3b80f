// gfx950 kernel behind the outer driver (Algorithm 2 of Sec. III-C): one workgroup per (n, MB) pair finds the smallest
// stage count S of its range for which a plan of EXACTLY S stages on D devices exists, that plan's value V[S][N][D] and
// the plan itself, for all three forms of the stage time (with and without send times, one objective or forward and
// backward maxima apart), without any table.
//
// A cell (s, i, d) of Algorithm 1's tables matters only if the stages s+1 .. S can still cover the blocks behind i and
// get a device each: d is one of s .. s + K - 1 with K = D - S + 1 devices to spare and one, no stage has more than K
// replicas, and i lies between the first row that S - s stages of K replicas complete and the last one that s of them
// reach, memory alone considered.  Algorithm 2 takes the smallest S that works: memory is nearly full, and few rows lie
// between the two.  What precedes such a cell in a plan is such a cell, so the recurrence among them gives the values,
// ties and argmins of the full tables: K values per row instead of D, some rows of every level instead of all.
//
// Bound by latency: a level is one round of reads, some 150 (one objective) or 350 instructions per pair of rows, LDS
// minima and a barrier.  By its own clock, us from the start: 32 blocks on 4 x 8 devices sums 3.5, rows and room 6.5, sixteen levels
// 16.5, plan 23; pairs of four nodes stop at 23, when they see that two nodes have a plan; 512 blocks 3.8, 7.8, 35, 41; 96 with the
// maxima apart 3.5, 7 to 11, 26 to 30, 28 to 32, and 37 for a pair whose first stage count has no plan.  Per call 42, 60 and 55
// us (with tables 84, 353, 523).
#include "rannc_dp_once.h"
#include "rannc_dp_sums.h"

#include <type_traits>

namespace rannc {

constexpr int kFormThreads = 1024;
constexpr int kFormMaxStages = RANNC_DP_MAX_DEVICES;
// Pairs of rows of a search, over all stage counts tried, beyond which the tables, which spread over the device, are the
// faster way.
constexpr int kFormPairs = 256 * 1024;

// KM: K rounded up to 4 or 8.
template <bool SPLIT, bool COMM, int KM>
__global__ __launch_bounds__(kFormThreads) void form_kernel(const FormArgs args) {
  constexpr int NT = kFormThreads, RS = KM + 1;  // a row's entries in LDS (an odd number: no bank conflicts)
  constexpr uint64_t kNoKey = ~0ull;
  extern __shared__ __align__(16) char lds[];
  __shared__ int s_up[kFormMaxStages + 1], s_down[kFormMaxStages + 1];                                   // the two chains of rows
  __shared__ int s_lo[kFormMaxStages + 1], s_hi[kFormMaxStages + 1], s_from[kFormMaxStages + 1], s_base[kFormMaxStages + 1];
  __shared__ int s_verdict, s_rows, s_stop[3];  // s_stop: a word for levels of either parity, written in front of a level's barrier, read behind it
  __shared__ float s_work;
  __shared__ double s_result;
  __shared__ __align__(8) uint32_t s_in[sizeof(FormIn) / 4];
  __shared__ int32_t s_end[kFormMaxStages], s_replicas[kFormMaxStages];
  const int tid = threadIdx.x, lane = tid & 63, q = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = args.N, entries = N + 1;
  double *const T = (double *)lds, *const P = T + entries, *const A = P + entries, *const TB = A + entries, *const C = TB + (SPLIT ? entries : 0);
  double *const cell = C + (COMM ? entries : 0);  // values, or with SPLIT keys, of all levels
  uint64_t *const key = (uint64_t *)cell;
  double *const pairs_f = cell + args.cells;      // SPLIT: the two maxima of a level and the one before
  uint16_t *const up = (uint16_t *)(pairs_f + (SPLIT ? 4 * kFormWide * RS : 0)), *const down = up + entries;

  // ---- sums, per sample, then of the pair's samples ----
  if (tid < 3) s_stop[tid] = 0;
  if (tid == 0) s_work = 0.0f;
  if (tid < (int)(sizeof(FormIn) / 4)) s_in[tid] = ((const uint32_t *)(args.pairs + q))[tid];
  if (wave < 3 || (SPLIT && wave == 3)) {
    int flags = 0;
    uint32_t high = 0;
    const int64_t *from = wave == 0 ? args.t : wave == 1 ? args.p : wave == 2 ? args.a : args.tb;
    double *const s = wave == 0 ? T : wave == 1 ? P : wave == 2 ? A : TB;
    if (N <= 64) reach_sums<1>(gptr(from), nullptr, s, N, flags, high);
    else if (N <= 192) reach_sums<3>(gptr(from), nullptr, s, N, flags, high);
    else if (N <= 576) reach_sums<9>(gptr(from), nullptr, s, N, flags, high);
    else reach_sums<17>(gptr(from), nullptr, s, N, flags, high);
  }
  __syncthreads();
  union { FormIn f; uint32_t u[sizeof(FormIn) / 4]; } in;
#pragma unroll
  for (int k = 0; k < (int)(sizeof(FormIn) / 4); ++k) in.u[k] = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_in[k]);
  const int D = in.f.D;
  const double samples = (double)in.f.b, M = (double)min(args.M, (int64_t)(2 * kReachMaxBytes));
  for (int e = tid; e <= N; e += NT) {
    T[e] *= samples;
    A[e] *= samples;
    if (SPLIT) TB[e] *= samples;
    if constexpr (COMM) {
      int flags = 0;
      C[e] = e >= 1 && e < N ? (double)cut_time(args.o[e - 1] * in.f.b, args.bw, flags) : 0.0;
    }
  }
  __syncthreads();
  auto fits = [&](int i, int j, double r) { return __builtin_fma(r, M + P[i] - P[j], A[i] - A[j]) >= 0.0; };
  auto ceil_of = [](double x, int r) {  // r is a compile-time number wherever this is called in a loop
    const double rd = (double)r, add = 0.5 * rd - 1.0 + rd * CeilDiv<uint64_t>::kOffset;
    return __builtin_fma(x + add, 1.0 / rd, 0x1.8p52) - 0x1.8p52;
  };
  const double none = __builtin_inf();
  auto uniform = [](int x) { return __builtin_amdgcn_readfirstlane(x); };

  // A search of fewer nodes that has found a plan, or one of as many nodes with fewer stages, makes this one needless: the
  // last wave looks for their words now and then, a read across the bus that nothing waits for until some levels later.
  uint64_t seen = 0;
  auto look = [&]() {
    if (tid >= NT - 64 && lane < args.searches) seen = __hip_atomic_load(&args.found[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  };
  auto looked = [&](int S, int word) {
    const int group = (int)(seen >> 8) & 255, stages = (int)seen & 255;
    const bool ahead = seen >> 16 == args.results.seq && (group < in.f.group || (group == in.f.group && stages < S));
    if (tid >= NT - 64 && lane < args.searches && ahead) s_stop[word] = 1;
  };
  int stages = 0, status = RANNC_DP_PROBLEM_OK;
  double value = none;
  int tried = 0;
  look();
  for (int S = in.f.lo; S <= in.f.hi; ++S) {  // (every condition below is uniform over the workgroup)
    const int K = D - S + 1;
    tried = S;
    // ---- rows that K replicas a stage reach and complete ----
    for (int i = tid; i <= N; i += NT) {
      int lo = i, hi = N, first = 0, last = i;
      while (lo < hi || first < last) {
        const int mid = (lo + hi + 1) >> 1, low = (first + last) >> 1;
        const bool f = fits(i, mid, (double)K), g = fits(low, i, (double)K);
        if (lo < hi) { if (f) lo = mid; else hi = mid - 1; }
        if (first < last) { if (g) last = low; else first = low + 1; }
      }
      up[i] = (uint16_t)lo;
      down[i] = (uint16_t)first;
    }
    __syncthreads();
    if (wave == 0) {
      for (int s = 0, row = 0; s <= S; ++s, row = up[row])
        if (lane == 0) s_up[s] = row;
    } else if (wave == 1) {
      for (int s = 0, row = N; s <= S; ++s, row = down[row])
        if (lane == 0) s_down[s] = row;
    }
    looked(S, 2);
    look();
    __syncthreads();
    if (wave == 0) {
      // the rows of every level (lane s; level 64 is the last one and has one row), its first row of the level before, and
      // where its cells begin
      bool ok = s_up[S] >= N;
      int total = 0, widest = 1;
      float work = 0.0f;
      for (int s0 = 0; s0 <= S; s0 += 64) {
        const int s = s0 + lane;
        auto low = [&](int k) { return k >= S ? N : max(k, s_down[S - k]); };
        auto high = [&](int k) { return k <= 0 ? 0 : k >= S ? N : min(s_up[k], N - (S - k)); };
        int width = 0;
        if (s >= 1 && s <= S) {
          const int l = low(s), h = high(s), before = s == 1 ? 0 : max(low(s - 1), (int)down[min(l, N)]);
          width = h - l + 1;
          s_lo[s] = l;
          s_hi[s] = h;
          s_from[s] = before;
          if (s >= 2) work += (float)max(width, 0) * (float)max(high(s - 1) - before + 1, 0);
        }
        ok = ok && lanes(s >= 1 && s <= S && width < 1) == 0ull;
        width = max(width, 0);
        int run = width;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int x = __shfl_up(run, o);
          if (lane >= o) run += x;
        }
        if (s >= 1 && s <= S) s_base[s] = (total + run - width) * RS;
        total += (int)lane_bcast((uint32_t)run, 63);
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) width = max(width, __shfl_xor(width, o));
        widest = max(widest, width);
      }
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) work += __shfl_xor(work, o);
      if (ok) work += s_work;
      const bool large = total * RS > args.cells || work > (float)(SPLIT ? kFormPairs / 2 : kFormPairs) || (SPLIT && widest > kFormWide);
      if (lane == 0) { s_verdict = !ok ? 0 : large ? 2 : 1; s_rows = total; if (ok) s_work = work; }
    }
    __syncthreads();
    const int verdict = uniform(s_verdict), all = uniform(s_rows) * RS;
    if (s_stop[2]) break;
    if (verdict == 0) { __syncthreads(); continue; }
    if (verdict == 2) { status = kReachUndecided; break; }

    // ---- level 1, and nothing found yet in the others (entries beyond the devices in use rank behind every value) ----
    for (int e = tid; e < all; e += NT) {
      if (SPLIT) {
        key[e] = kNoKey;
      } else {
        const int row = e / RS, x = e - row * RS, i = s_lo[1] + row;
        double v = x < K ? none : 0.0;
        if (i <= s_hi[1] && x < K && fits(0, i, (double)(x + 1))) {
          const double r = (double)(x + 1);
          v = ceil(T[i] / r) + (COMM ? ceil(C[i] / r) : 0.0);
        }
        cell[e] = v;
      }
    }
    if (SPLIT)
      for (int e = tid; e < (s_hi[1] - s_lo[1] + 1) * RS; e += NT) {
        const int row = e / RS, x = e - row * RS, i = s_lo[1] + row;
        const double r = (double)(x + 1);
        const bool ok = x < K && fits(0, i, r);
        double *const F = pairs_f + 2 * kFormWide * RS, *const B = F + kFormWide * RS;
        F[e] = ok ? ceil(T[i] / r) + (COMM ? ceil(C[i] / r) : 0.0) : none;
        B[e] = ok ? ceil(TB[i] / r) : none;
      }
    __syncthreads();

    // ---- levels 2 .. S ----
    bool stop = false;
    for (int s = 2; s <= S; ++s) {
      const int lo = uniform(s_lo[s]), rows = uniform(s_hi[s]) - lo + 1, from = uniform(s_from[s]), before = uniform(s_lo[s - 1]);
      const int pairs = rows * (uniform(s_hi[s - 1]) - from + 1), base = uniform(s_base[s]), base_before = uniform(s_base[s - 1]);
      const float inv_rows = 1.0f / (float)rows;
      const bool ask = (s & 3) == 2 || pairs > NT;  // (of a short level the answer is looked at when the next asking one begins)
      if (ask && pairs <= NT) looked(S, s & 1);
      if (ask) look();
      double *const F0 = pairs_f + ((s - 1) & 1) * 2 * kFormWide * RS, *const B0 = F0 + kFormWide * RS;
      double *const F1 = pairs_f + (s & 1) * 2 * kFormWide * RS, *const B1 = F1 + kFormWide * RS;
      for (int e = tid; e < pairs; e += NT) {
        int k = (int)((float)e * inv_rows);  // e / rows, corrected
        k -= k * rows > e ? 1 : 0;
        k += (k + 1) * rows <= e ? 1 : 0;
        const int i = from + k, j = lo + e - k * rows;  // the stage i+1 .. j
        if (i >= j || i < (int)down[j]) continue;
        const double t = T[j] - T[i], slack = M + P[i] - P[j], a = A[i] - A[j], c = COMM ? C[j] : 0.0;
        double h[KM];
#pragma unroll
        for (int r = 1; r <= KM; ++r) {
          h[r - 1] = ceil_of(t, r);
          if (COMM) h[r - 1] += ceil_of(c, r);
        }
        if (lanes(slack + a < 0.0) != 0ull) {  // (where one replica holds the bytes, more do)
#pragma unroll
          for (int r = 1; r <= KM; ++r) h[r - 1] = __builtin_fma((double)r, slack, a) >= 0.0 ? h[r - 1] : none;
        }
        if constexpr (!SPLIT) {
          // both sequences fall: the K values are the largest of their merge, in order
          const double *const v = cell + base_before + (i - before) * RS;
          double w[KM];
#pragma unroll
          for (int x = 0; x < KM; ++x) w[x] = dmax(v[x], h[KM - 1 - x]);
#pragma unroll
          for (int m = KM / 2; m >= 1; m /= 2)
#pragma unroll
            for (int x = 0; x < KM; ++x)
              if (!(x & m)) {
                const double p0 = w[x], p1 = w[x + m];
                w[x] = dmax(p0, p1);
                w[x + m] = dmin(p0, p1);
              }
          uint64_t *const to = key + base + (j - lo) * RS;
#pragma unroll
          for (int x = 0; x < KM; ++x)
            if (x < K) atomicMin((unsigned long long *)&to[x], (unsigned long long)__double_as_longlong(w[x]));
        } else {
          const double tb = TB[j] - TB[i];
          double g[KM], f0[KM], b0[KM];
#pragma unroll
          for (int x = 0; x < KM; ++x) {
            g[x] = ceil_of(tb, x + 1);
            f0[x] = F0[(i - before) * RS + x];
            b0[x] = B0[(i - before) * RS + x];
          }
          unsigned long long *const to = (unsigned long long *)key + base + (j - lo) * RS;
#pragma unroll
          for (int x = 0; x < KM; ++x)
            if (x < K) {
              double best = none;
              int at = 0;
#pragma unroll
              for (int y = 0; y <= x; ++y) {  // devices ascend: an equal sum keeps the earlier one
                const double v = dmax(f0[y], h[x - y]) + dmax(b0[y], g[x - y]);
                at = v < best ? y : at;
                best = v < best ? v : best;
              }
              if (best != none) {
                const uint64_t sum = (uint64_t)__double_as_longlong(best + 0x1p52) & ((1ull << 46) - 1ull);
                atomicMin(&to[x], (unsigned long long)(sum << 13 | (uint64_t)(i - before) << 3 | (uint64_t)at));
              }
            }
        }
      }
      if (pairs > NT) looked(S, s & 1);
      lds_barrier();
      stop = ask && s_stop[s & 1];
      if (stop) break;
      if constexpr (SPLIT) {
        for (int e = tid; e < rows * RS; e += NT) {  // the winners' two maxima
          const int row = e / RS, x = e - row * RS;
          const uint64_t w = key[base + e];
          double f = none, b = none;
          if (w != kNoKey) {
            const int k = (int)(w >> 3) & 1023, y = (int)w & 7, i = before + k, j = lo + row;
            const double r = (double)(x - y + 1);
            f = dmax(F0[k * RS + y], ceil((T[j] - T[i]) / r) + (COMM ? ceil(C[j] / r) : 0.0));
            b = dmax(B0[k * RS + y], ceil((TB[j] - TB[i]) / r));
          }
          F1[e] = f;
          B1[e] = b;
        }
        lds_barrier();
      }
    }
    if (stop) break;
    if (tid == 0) {
      double v;
      if (!SPLIT) {
        v = cell[s_base[S] + K - 1];
      } else if (S == 1) {
        v = pairs_f[2 * kFormWide * RS + K - 1] + pairs_f[3 * kFormWide * RS + K - 1];
      } else {
        const uint64_t w = key[s_base[S] + K - 1];
        v = w == kNoKey ? none : (double)(w >> 13);
      }
      s_result = v;
    }
    __syncthreads();
    value = s_result;
    if (value != none) {
      stages = S;
      break;
    }
    __syncthreads();
  }

  // ---- the plan, by one wave ----
  if (wave != 0) return;
  if (stages && lane == 0)
    __hip_atomic_store(&args.found[q], args.results.seq << 16 | (uint64_t)in.f.group << 8 | (uint64_t)stages, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  if (stages) {
    int j = N, x = D - stages;
    double v = value;
    bool ok = true;
    for (int s = stages; s >= 2 && ok; --s) {
      const int before = uniform(s_lo[s - 1]), first = uniform(max(s_from[s], (int)down[j])), last = min(uniform(s_hi[s - 1]), j - 1);
      int i = -1, y = 0;
      if constexpr (SPLIT) {
        const int w = uniform((int)key[uniform(s_base[s]) + (j - uniform(s_lo[s])) * RS + x]);
        i = before + (w >> 3 & 1023);
        y = w & 7;
      } else {
        // smallest row, then fewest devices in front, of the candidates of at most the cell's value
        for (int i0 = first; i0 <= last && i < 0; i0 += 64) {
          const int row = min(i0 + lane, last);
          const double *const vals = cell + uniform(s_base[s - 1]) + (row - before) * RS;
          int at = 0;  // (they fall)
#pragma unroll
          for (int k = 0; k < KM; ++k) at += ((k <= x) & (vals[k] > v)) ? 1 : 0;
          const double rd = (double)max(x - at + 1, 1), t = T[j] - T[row];
          bool within = t <= rd * v;
          if (COMM) within = ceil(t / rd) + ceil(C[j] / rd) <= v;
          const uint64_t m = lanes((i0 + lane <= last) & (at <= x) & within & fits(row, j, rd));
          if (m) {
            const int who = __ffsll((long long)m) - 1;
            i = i0 + who;
            y = (int)lane_bcast((uint32_t)at, who);
          }
        }
        if (i >= 0) v = cell[s_base[s - 1] + (i - before) * RS + y];
      }
      ok = i >= 0;
      if (lane == 0) { s_end[s - 1] = j; s_replicas[s - 1] = x - y + 1; }
      j = i;
      x = y;
    }
    if (lane == 0) { s_end[0] = j; s_replicas[0] = x + 1; }
    if (!ok) { stages = 0; status = kReachUndecided; }  // (there is one; left to the tables)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  const PlanResults &r = args.results;
  if (lane == 0) {
    r.h_opt[q] = stages ? (int64_t)value : INT64_MAX;
    r.h_n_stages[q] = status == RANNC_DP_PROBLEM_OK ? stages : tried;
    r.h_status[q] = status;
  }
  for (int u = lane; u < args.plan_stride; u += 64) {
    r.h_stage_end[(int64_t)q * args.plan_stride + u] = u < stages ? s_end[u] : -1;
    r.h_replicas[(int64_t)q * args.plan_stride + u] = u < stages ? s_replicas[u] : -1;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");  // (of the whole wave, for the system)
  if (lane == 0) __hip_atomic_store(&r.h_flag[q], r.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// (Persistent bytes do not grow with the samples.)  A search to blockIdx.y, an array to blockIdx.z; read across the bus.
__global__ __launch_bounds__(256) void form_inputs_kernel(const int64_t *per_sample, const int64_t *samples, int64_t *out, int N, int Q, int arrays) {
  const int k = blockIdx.x * 256 + threadIdx.x, q = blockIdx.y, w = blockIdx.z;
  if (k >= N || !(arrays >> w & 1)) return;
  out[((int64_t)w * Q + q) * N + k] = per_sample[(int64_t)w * N + k] * (w == 1 ? 1 : samples[q]);
}

hipError_t launch_form_inputs(const int64_t *per_sample, const int64_t *samples, int64_t *out, int N, int Q, bool comm, bool split, hipStream_t st) {
  hipLaunchKernelGGL(form_inputs_kernel, dim3((N + 255) / 256, Q, 5), dim3(256), 0, st, per_sample, samples, out, N, Q,
                     7 | (comm ? 8 : 0) | (split ? 16 : 0));
  return hipGetLastError();
}

hipError_t launch_form(int Q, int spare, const FormArgs &in, hipStream_t st) {
  if (in.N > kFormMaxBlocks || spare > 8 || spare < 1) return hipErrorInvalidValue;
  const bool split = in.tb != nullptr;
  FormArgs args = in;
  const int KM = spare <= 4 ? 4 : 8, RS = KM + 1;
  constexpr int kLds = 152 * 1024;
  const size_t sums = (size_t)(args.N + 1) * 8 * (3 + (split ? 1 : 0) + (args.o ? 1 : 0));
  const size_t rest = (split ? (size_t)4 * kFormWide * RS * 8 : 0) + (((size_t)(args.N + 1) * 4 + 7) / 8) * 8;
  // cells: a level has at most N rows, the last one has one
  const int64_t most = (int64_t)RS * (1 + (int64_t)args.N * (RANNC_DP_MAX_DEVICES - 1));
  args.cells = (int)min(most, (int64_t)((kLds - sums - rest) / 8));
  const size_t lds = sums + rest + (size_t)args.cells * 8;
  auto go = [&](auto apart, auto sends, auto width) -> hipError_t {
    constexpr bool X = decltype(apart)::value, Y = decltype(sends)::value;
    constexpr int W = decltype(width)::value;
    static std::atomic<uint64_t> asked{0};
    const hipError_t e = allow_lds(asked, (const void *)form_kernel<X, Y, W>, kLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((form_kernel<X, Y, W>), dim3(Q), dim3(kFormThreads), lds, st, args);
    return hipGetLastError();
  };
#define GO(X, Y, W)                                  \
  if (split == X && (args.o != nullptr) == Y && KM == W) \
    return go(std::integral_constant<bool, X>(), std::integral_constant<bool, Y>(), std::integral_constant<int, W>());
  GO(false, false, 4) GO(false, false, 8) GO(false, true, 4) GO(false, true, 8)
  GO(true, false, 4) GO(true, false, 8) GO(true, true, 4) GO(true, true, 8)
#undef GO
  return hipErrorInvalidValue;
}

}  // namespace rannc
