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
// Where the bound leaves many cells (a long block, or bytes that crowd at one end, cost more than an even share), or the stages
// there are do not suffice for it, Algorithm 1's levels run among the cells that a bound leaves instead (reach_levels).
//
// Bound by latency: the devices are taken one after the other, some 350 ns each (sums of a row from lanes to scalars,
// a dozen dependent double-precision instructions, the next rows from LDS), where windows are wide up to 1 us (searches through
// rows).  Per call, tables / this kernel: 96 blocks at 16 devices 56 / 22 us, 1024 at 64 275 / 59 where memory binds and
// 454 / 17 where one stage holds everything, 701 at 48 with 64-bit values 249 / 30, 2048 searches of 128 blocks 1630 / 155;
// 251 blocks whose bytes grow along the chain, at 24 devices, 94 / 81 (172 by bounds alone, without the levels); 300 at 32 in
// at most 4 stages that are 78 % full 49 / 50 (199).
#include "rannc_dp_reach.h"

namespace rannc {

template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void reach_kernel(const ReachIn *src, const ReachIn one, const int use_one, const ReachArgs args,
                                                           const ReachDims dims) {
  static_assert(WAVES >= 4 && WAVES <= 16, "a wave per array, and one");
  extern __shared__ __align__(16) char lds[];
  constexpr int W = (int)sizeof(ReachIn) / 4;
  __shared__ __align__(8) uint32_t s_in[W];
  __shared__ int s_flags;
  __shared__ uint64_t s_total, s_bytes[2];
  __shared__ ReachShared<WAVES> sh;
  const int tid = threadIdx.x, lane = tid & 63, q = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  ReachIn in = one;
  if (tid < 3) sh.mask[tid] = 0u;
  if (tid == 0) s_flags = 0;
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
  const int N = in.N;
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

  uint64_t opt = (uint64_t)INT64_MAX, window;
  int n_stages = 0;
  const LevelSpace space = {dims.level_cells, dims.level_sources, dims.level_records, (char *)value};
  if (status == RANNC_DP_PROBLEM_OK)
    reach_search<WAVES, false>(in, (double)min(in.M, (int64_t)(2 * kReachMaxBytes)) /* as good as unlimited */, lane_bcast(s_total, 0), sT, sP, sA, value, reach, first_of,
                        base, dims, space, sh, opt, n_stages, status, window);
  reach_results(in, args, q, sh.plan, opt, n_stages, status);
}

hipError_t launch_reach(const ReachIn *src, const ReachIn *host_one, int Q, const LaunchShape &sh, const ReachArgs &args, hipStream_t st) {
  if (sh.max_N > kReachMaxBlocks) return hipErrorInvalidValue;
  // Room for the levels: of few searches, which have a compute unit to themselves, what is left of its LDS; of many, so
  // much that it does not keep the workgroups that registers allow (five of four waves) from a compute unit.
  const size_t sums = (size_t)(sh.max_N + 2 + kReachPad) * 24;
  ReachDims dims = {sh.max_N, sh.max_D, sh.max_S_eff, Q > 64 ? 256 : 1024, 1024, 160, 512, Q > 8 ? 1 : 0, 32768};
  if (Q <= 64) {
    dims.level_sources = 256;
    dims.level_records = 1024;
    dims.level_cells = (int)std::min<size_t>(std::min(3584, (sh.max_N * sh.max_D + 15) / 8 * 8), (144 * 1024 - sums - level_bytes(0, dims.level_sources, dims.level_records, false)) / 12);
  }
  const size_t lds = sums + std::max((size_t)dims.cells * 8 + (size_t)dims.S * dims.D * 6,
                                     level_bytes(dims.level_cells, dims.level_sources, dims.level_records, false));
  const ReachIn one = host_one ? *host_one : ReachIn{};
  auto go = [&](auto waves) -> hipError_t {
    constexpr int W = decltype(waves)::value;
    static std::atomic<uint64_t> asked{0};
    const hipError_t e = allow_lds(asked, (const void *)reach_kernel<W>, 148 * 1024);
    if (e != hipSuccess) return e;
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
