// gfx950 kernel that answers a min-max search without its value tables: optimum, fewest stages and the canonical
// plan, for callers that want nothing else (rannc_dp_solve_to_host).  The tables themselves are made by the kernels in
// rannc_dp_kernels.hip, when they are asked for.
//
// Without send times the stage time h(i, j, r) of Sec. III-C and its bytes grow with the stage and fall with r, so for a given
// bound X the first row behind which e devices can take the rest, no stage above X, in any number of stages,
//     B(e) = min over f < e of (the beginning of the longest stage in front of B(f) on e - f replicas),
// takes D (D + 1) / 2 stages instead of N (N + 1) / 2 merges of D values per level, and the smallest X with B(D) = 0 is the
// optimum over any number of stages.  A round asks for one bound per wave.  What can be part of a plan within X are the cells
// (i, d) with B(D - d) <= i and T[i] <= d X.
//
// Exactly s stages (the cells V[s][j][d] of the tables) against any number: let s* be the fewest stages of a plan of
// value v = V[s*][N][D].  A cell (s, i, d) from which s* - s further stages reach N within v has no plan of fewer
// than s stages within v, or the whole would have fewer than s*.  For these cells "fewest stages" and
// "exactly s stages" are the same, and every candidate of such a cell of value at most v is such a cell.  The walk of
// Algorithm 1's argmin (smallest i, then smallest d', of the candidates that attain the cell's value) therefore stays
// among them, and so does the recurrence for their values.  Where a bound leaves one or two cells to a device they are all that
// is looked at (reach_finish).
//
// Where it leaves more (a long block, or bytes that crowd at one end, cost more than an even share), Algorithm 1's levels run
// among the cells that the bound leaves instead (reach_levels).  Where these are too many, or the stages do not suffice at the bound,
// the search is left to the tables (reach_search).
//
// Bound by latency: the devices are taken one after the other, some 350 ns each (sums of a row from lanes to scalars,
// a dozen dependent double-precision instructions, the next rows from LDS), where windows are wide up to 1 us (searches through
// rows).  Per call, tables / this kernel: 96 blocks at 16 devices 51 / 14 us, 1024 at 64 282 / 55 where memory binds, 2048 searches of
// 128 blocks 1720 / 163.  Slower than with tables where nothing is to spare: 60 at 24 in at most 24 stages, 23 or 24 needed, 66 / 83;
// and by what it took to find out where they are left to them: 22 at 15 without a plan 25 / 56, 1024 at 64 in 9 stages 104 / 118.
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
  const int entries = dims.N + 2 + kReachPad;
  double *const sT = (double *)lds + kReachPad, *const sP = sT + entries, *const sA = sP + entries, *const rest = sA + entries - kReachPad;

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
  const LevelSpace space = {dims.level_cells, dims.level_sources, dims.level_records, (char *)rest};
  if (status == RANNC_DP_PROBLEM_OK)
    reach_search<WAVES, false, false>(in, (double)min(in.M, (int64_t)(2 * kReachMaxBytes)) /* as good as unlimited */, lane_bcast(s_total, 0), sT, sP, sA, space, dims.grow, sh, opt,
                        n_stages, status, window);
  reach_results(in, args, q, sh.plan, opt, n_stages, status);
}

hipError_t launch_reach(const ReachIn *src, const ReachIn *host_one, int Q, const LaunchShape &sh, const ReachArgs &args, hipStream_t st) {
  if (sh.max_N > kReachMaxBlocks) return hipErrorInvalidValue;
  // Room for the levels, as much as keeps no workgroup that registers allow from a compute unit (131 of them: three waves to a SIMD):
  // one of eight or sixteen waves, three of four.
  // grow: stages times devices up to which a search of several whose stages do not suffice is asked at one larger bound; left open it
  // costs tables of its own (15 ragged searches of 32 blocks at up to 32 devices in 6 stages: 60 us without, 52 with).  By itself a search
  // is no slower with the tables.
  const size_t sums = (size_t)(sh.max_N + 2 + kReachPad) * 24;
  ReachDims dims = {sh.max_N, 1536, 256, 1024, Q > 1 ? 512 : 0};
  if (Q <= 512) {
    // (504 equal blocks at 47 devices 523 -> 318 us, 196 searches of 35 at 32 with a long one 238 -> 190; of a few searches the launch waits
    // for the one that goes on longest)
    if ((Q == 1 || Q > 64) && sh.max_N <= 1024) {
      dims.level_sources = 512;
      dims.level_records = 4096;
    }
    dims.level_cells = (int)std::min<size_t>(std::min(3584, (sh.max_N * sh.max_D + 15) / 8 * 8), (144 * 1024 - sums - level_bytes(0, dims.level_sources, dims.level_records, false)) / 12);
  }
  const size_t lds = sums + level_bytes(dims.level_cells, dims.level_sources, dims.level_records, false);
  const ReachIn one = host_one ? *host_one : ReachIn{};
  auto go = [&](auto waves) -> hipError_t {
    constexpr int W = decltype(waves)::value;
    static std::atomic<uint64_t> asked{0};
    const hipError_t e = allow_lds(asked, (const void *)reach_kernel<W>, 148 * 1024);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(reach_kernel<W>, dim3(Q), dim3(64 * W), lds, st, src, one, host_one ? 1 : 0, args, dims);
    return hipGetLastError();
  };
  // Waves of a search, each with a bound of its own: as many as the device has places for, and no more than eight for up to
  // sixteen devices, whose bounds take little longer than the start of a wave.
  // Per call, 4 / 8 / 16 waves: 16 blocks at 4 devices 24 / 21 / 22 us, 300 at 32 40 / 27 / 28, 1024 at 64 46 / 70 / 50, 32 searches of
  // 1000 at 64 192 / 103 / 95, 200 of 128 at 64 94 / 50 / 47, 512 97 / 64 / 64, 600 of 100 at 32 67 / 66 / 69, 768 of 128 at 64
  // 100 / 82 / 78, 1024 of 128 at 16 75 / 93 / 94, 2000 of 60 at 32 112 / 136 / 139.
  if (Q > 512) return go(std::integral_constant<int, 4>());
  if (Q > 64 || sh.max_D <= 16) return go(std::integral_constant<int, 8>());
  return go(std::integral_constant<int, 16>());
}

}  // namespace rannc
