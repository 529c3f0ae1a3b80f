// gfx950 kernel that answers searches with send times, and with forward and backward maxima apart, without their value
// tables: optimum, fewest stages and the canonical plan (rannc_dp_solve_to_host), one workgroup to a search.  The tables
// themselves are made by the kernels in rannc_dp_kernels.hip and rannc_dp_split.hip, when they are asked for.
//
// The levels of rannc_dp_reach.h, among the cells that a bound leaves.  The bound comes from the plan that is best for the sums of all
// times, without what is sent, priced with send times and the two maxima: for one objective it is an upper bound by
// itself, with the two apart (Algorithm 1 as printed may miss that plan) the levels say whether it is.
//
// Bound by latency, as rannc_dp_reach.hip.  Per call, tables / this kernel: maxima apart 256 blocks at 32 devices 9.7 ms / 62 to 103 us
// (64-bit handle); with send times 531 at 8 69 / 38 to 52 us, 1000 at 6 81 / 36, 664 at 11 in at most 5 stages that are 85 % full
// 69 / 145; both 362 at 8 2.4 ms / 43 to 68.
#include "rannc_dp_attempts.h"
#include "rannc_dp_reach.h"

namespace rannc {

constexpr int kBoundThreads = 1024, kBoundWaves = kBoundThreads / 64;
constexpr int kBoundCells = 3584;    // of the windows
constexpr int kBoundSources = 384;   // of a level
constexpr int kBoundRecords = 2048;  // of all levels

template <bool SPLIT, bool COMM>
__global__ __launch_bounds__(kBoundThreads) void bound_kernel(const ReachIn *src, const ReachIn one, const int use_one, const ReachArgs args,
                                                              const ReachDims dims) {
  constexpr int NT = kBoundThreads, WAVES = kBoundWaves;
  extern __shared__ __align__(16) char lds[];
  constexpr int W = (int)sizeof(ReachIn) / 4;
  __shared__ __align__(8) uint32_t s_in[W];
  __shared__ int s_flags;
  __shared__ uint64_t s_total[4];
  __shared__ unsigned long long s_cut;
  __shared__ ReachShared<WAVES> sh;
  const int tid = threadIdx.x, lane = tid & 63, q = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  ReachIn in = one;
  if (tid < 3) sh.mask[tid] = 0u;
  if (tid == 0) { s_flags = 0; s_cut = 0ull; }
  if (tid < 4) s_total[tid] = 0ull;
  if (wave == 3) sh.inverse[lane] = 1.0 / (double)(lane + 1);
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
  const int entries = dims.N + 2 + kReachPad;
  double *const sT = (double *)lds + kReachPad, *const sP = sT + entries, *const sA = sP + entries;
  double *const sB = sA + entries, *const sC = sB + (SPLIT ? entries : 0);
  char *const rest = (char *)(sC + (COMM ? entries : 0) - kReachPad);
  const LevelSpace space = {dims.level_cells, dims.level_sources, dims.level_records, rest};

  // ---- sums ----
  {
    int flags = 0;
    uint32_t high = 0;
    const int64_t from = in.first, to = in.first - args.first;
    if (wave < 3 || (SPLIT && wave == 3)) {
      const int64_t RANNC_GLOBAL *const x = gptr(wave == 0 ? args.t : wave == 1 ? args.p : wave == 2 ? args.a : args.tb) + from;
      int64_t RANNC_GLOBAL *const save = gptr(args.save) + (int64_t)(wave < 3 ? wave : 4) * args.blocks + to;
      double *const s = wave == 0 ? sT : wave == 1 ? sP : wave == 2 ? sA : sB;
      uint64_t total;
      if (N <= 64) total = reach_sums<1>(x, save, s, N, flags, high);
      else if (N <= 192) total = reach_sums<3>(x, save, s, N, flags, high);
      else if (N <= 576) total = reach_sums<9>(x, save, s, N, flags, high);
      else total = reach_sums<17>(x, save, s, N, flags, high);
      if (high >> 30) flags |= 2;
      if (lane < kReachPad) s[-1 - lane] = wave == 0 ? -__builtin_inf() : 0.0;
      if (lane == 0) {
        s[N + 1] = wave == 0 ? __builtin_inf() : 0.0;
        s_total[wave] = total;
      }
    } else if (COMM && wave >= 4) {
      unsigned long long most = 0ull;
      for (int k = tid - 256; k < N; k += NT - 256) {
        const int64_t o = args.o[from + k];
        args.save[3 * args.blocks + to + k] = o;
        const uint64_t c = cut_time(o, in.bw, flags);
        sC[k + 1] = k + 1 < N ? (double)c : 0.0;
        if (k + 1 < N && c > most) most = c;
      }
      if (tid == 256) sC[0] = 0.0;
      if (most) atomicMax(&s_cut, most);
    }
    if (flags) atomicOr(&s_flags, flags);
  }
  __syncthreads();
  const uint64_t total = lane_bcast((uint64_t)(s_total[0] + (SPLIT ? s_total[3] : 0ull)), 0);
  int status = RANNC_DP_PROBLEM_OK;
  if (s_flags & 1) status = RANNC_DP_PROBLEM_NEGATIVE_INPUT;
  else if (s_flags & 2) status = RANNC_DP_PROBLEM_SUM_OVERFLOW;
  else if (total + s_cut > (uint64_t)args.time_limit) status = RANNC_DP_PROBLEM_TIME_TOO_LARGE;
  else if (total + s_cut >= (uint64_t)kReachMaxTime || s_total[1] >= (uint64_t)kReachMaxBytes || s_total[2] >= (uint64_t)kReachMaxBytes)
    status = kReachUndecided;

  // Where memory makes many stages of a long chain on many devices, more cells are left than the tables take time for: 1000
  // blocks at 64 devices, memory makes 13 stages, 1176 us with tables, 1732 without; 500 616 and 981.
  const double forced = (sP[N] + sA[N] / (double)D) / fmax((double)in.M, 1.0);
  if (status == RANNC_DP_PROBLEM_OK && N * D > 24576 && forced > 8.0 && forced <= 1.01 * (double)in.S) status = kReachUndecided;

  uint64_t opt = (uint64_t)INT64_MAX, window = 0;
  int n_stages = 0;
  if (status == RANNC_DP_PROBLEM_OK) {
    if (SPLIT) {
      for (int e = tid; e <= N; e += NT) sT[e] += sB[e];
      __syncthreads();
    }
    const double M = (double)min(in.M, (int64_t)(2 * kReachMaxBytes));  // (as good as unlimited)
    reach_search<WAVES, !(SPLIT && COMM), SPLIT>(in, M, total, sT, sP, sA, space, 0, sh, opt, n_stages, status, window);
    __syncthreads();
    const LevelSums all = {sT, sP, sA, sB, sC};
    auto times = [&](int i, int j, int r, double &f, double &b) { level_times<SPLIT, COMM>(all, sh.inverse, i, j, r, f, b); };
    if (status == RANNC_DP_PROBLEM_OK && n_stages == 1) {  // one stage sends nothing, and shares everything evenly: no plan is better
      double f, b;
      times(0, N, D, f, b);
      opt = (uint64_t)(f + b);
    } else if (status == RANNC_DP_PROBLEM_OK && n_stages != 0) {
      // ---- U: that plan's value here; or where many cells were left, so that it has not been looked for, the bound itself ----
      const Attempts bounds = {(double)opt, n_stages < 0, SPLIT, N <= 64 && D <= 8};
      double price = 0.0;
      if (!bounds.asked) {
        double f = 0.0, b = 0.0;
        if (lane < n_stages) times(lane ? sh.plan.end[lane - 1] : 0, sh.plan.end[lane], sh.plan.replicas[lane], f, b);
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          f = dmax(f, __shfl_xor(f, o));
          b = dmax(b, __shfl_xor(b, o));
        }
        price = f + b;
      }
      double U = bounds.first(price);
      n_stages = 0;
      opt = (uint64_t)INT64_MAX;
      status = kReachUndecided;
#pragma unroll 1
      for (int attempt = 0; U >= 0.0; ++attempt) {
        double v = 0.0;
        int s = 0;
        const bool kept = U <= (double)window;
        const LevelState state = reach_levels<WAVES, SPLIT, COMM>(all, N, D, M, U, kept, in.S, space, sh, v, s);
        if (state == kLevelsFound) {
          opt = (uint64_t)v;
          n_stages = s;
          status = RANNC_DP_PROBLEM_OK;
        }
        window = state == kLevelsOpen ? 0 : kept ? window : (uint64_t)U;
        U = bounds.next(attempt, U, state);
      }
    }
  }
  reach_results(in, args, q, sh.plan, opt, n_stages, status);
}

hipError_t launch_bound(const ReachIn *src, const ReachIn *host_one, int Q, const LaunchShape &sh, const ReachArgs &args, hipStream_t st) {
  if (sh.max_N > kBoundMaxBlocks) return hipErrorInvalidValue;
  const bool split = args.tb != nullptr, comm = args.o != nullptr;
  const int cells = std::min(kBoundCells, (sh.max_N * sh.max_D + 15) / 8 * 8);  // (a multiple of 8: aligned arrays)
  const ReachDims dims = {sh.max_N, cells, kBoundSources, kBoundRecords, 0};
  const size_t sums = (size_t)(dims.N + 2 + kReachPad) * 8 * (3 + (split ? 1 : 0) + (comm ? 1 : 0));
  const size_t levels = level_bytes(cells, kBoundSources, kBoundRecords, split);
  const ReachIn one = host_one ? *host_one : ReachIn{};
  auto go = [&](auto apart, auto sends) -> hipError_t {
    constexpr bool X = decltype(apart)::value, Y = decltype(sends)::value;
    static std::atomic<uint64_t> asked{0};
    const hipError_t e = allow_lds(asked, (const void *)bound_kernel<X, Y>, 148 * 1024);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((bound_kernel<X, Y>), dim3(Q), dim3(kBoundThreads), sums + levels, st, src, one, host_one ? 1 : 0, args, dims);
    return hipGetLastError();
  };
  if (split && comm) return go(std::true_type(), std::true_type());
  if (split) return go(std::true_type(), std::false_type());
  if (comm) return go(std::false_type(), std::true_type());
  return hipErrorInvalidValue;
}

}  // namespace rannc
