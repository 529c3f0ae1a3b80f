// gfx950 kernels of Algorithm 1 as printed (RaNNC Sec. III-C): forward and backward maxima carried
// separately, candidates valued by their sum.  Level 1, the literal level kernel, the packed-key
// level kernel with its finalize step, and their launchers.  Plan recovery for this objective is
// part of the traceback kernel (rannc_dp_kernels.hip).
#include "rannc_dp_device.h"
#include <algorithm>

namespace rannc {

// ---------------------------------------------------------------------------------------
// Algorithm 1 as printed: forward and backward maxima carried separately (problems with backward
// times).  A cell keeps V = f + b together with the pair (f, b) of the first candidate, in the
// scan order (i ascending, then d' ascending), that attains the smallest sum; only that pair is
// seen by the next level.  The sum of two maxima does not separate over the two sequences, so the
// sorted-merge form does not apply: every candidate is evaluated, one wave per (64 columns, d),
// a lane per column j, as in the literal scan kernel.
// ---------------------------------------------------------------------------------------
// Level 1: the single stage 1..j on d replicas.
template <typename VT>
__global__ __launch_bounds__(64) void split_level1_kernel(const ProblemDev *__restrict__ probs) {
  const ProblemDev &pr = probs[blockIdx.z];
  const int c = blockIdx.x, d = blockIdx.y + 1;
  if (c >= pr.nch || d > pr.D) return;
  const int lane = threadIdx.x, jj = 64 * c + lane;
  if (jj >= pr.N) return;
  const int DP = pr.DP;
  const int64_t u = unit_index(pr.nch, 0, c);
  const int64_t e = (int64_t)(jj + 1) * DP + d - 1;
  if (d < (int)pr.rmin[u * 64 + lane]) return;  // stays "no plan"
  auto share = [&](int64_t x) { return (VT)(((uint64_t)x + (uint64_t)(d - 1)) / (uint64_t)d); };
  const VT f = share(pr.T[jj + 1]) + (pr.C ? share(pr.C[jj + 1]) : (VT)0);
  const VT b = share(pr.TB[jj + 1]);
  ((VT *)pr.V)[e] = f + b;
  ((VT *)pr.VF)[e] = f;
  ((VT *)pr.VB)[e] = b;
}

template <typename VT>
__global__ __launch_bounds__(64) void level_split_kernel(const ProblemDev *__restrict__ probs, const int s,
                                                         const int write_v, int32_t *__restrict__ arg_i,
                                                         int32_t *__restrict__ arg_d) {
  const ProblemDev &pr = probs[blockIdx.z];
  const int N = pr.N, D = pr.D, DP = pr.DP, nch = pr.nch;
  if (s > pr.S_eff) return;
  const int c = blockIdx.x, d = blockIdx.y + 1;
  if (c >= nch || d > D || d < s) return;
  const int lane = threadIdx.x;
  const int jj = 64 * c + lane;
  const int j = jj + 1;
  constexpr VT INF = Lim<VT>::inf;
  const int64_t lvl = (int64_t)(N + 1) * DP;
  const VT RANNC_GLOBAL *Vprev = gptr((const VT *)pr.V) + (int64_t)(s - 2) * lvl;
  const VT RANNC_GLOBAL *Fprev = gptr((const VT *)pr.VF) + (int64_t)(s - 2) * lvl;
  const VT RANNC_GLOBAL *Bprev = gptr((const VT *)pr.VB) + (int64_t)(s - 2) * lvl;
  const VT RANNC_GLOBAL *costf = gptr((const VT *)pr.cost);
  const VT RANNC_GLOBAL *costb = gptr((const VT *)pr.costb);
  const uint8_t RANNC_GLOBAL *rmin = gptr((const uint8_t *)pr.rmin);
  const uint8_t RANNC_GLOBAL *ufit = gptr((const uint8_t *)pr.ufit);
  VT best = INF, bf = INF, bb = INF;
  int bi = -1, bd = -1;
  const int i_end = min(64 * c + 63, N - 1);
  for (int i = s - 1; i <= i_end; ++i) {
    // a plan of s-1 stages over blocks 1..i exists on d-1 devices iff it exists on any fewer
    if (Vprev[(int64_t)i * DP + d - 2] == INF) continue;
    const int64_t u = unit_index(nch, i, c);
    if (!ufit[u]) continue;  // no stage of this unit fits: its table rows were never written
    const bool act = (jj >= i) && (jj < N);
    const VT RANNC_GLOBAL *uf = costf + u * 64 * D + lane;
    const VT RANNC_GLOBAL *ub = costb + u * 64 * D + lane;
    const int rmn = act ? (int)rmin[u * 64 + lane] : 255;
    for (int dp = s - 1; dp <= d - 1; ++dp) {
      const VT a = Vprev[(int64_t)i * DP + dp - 1];
      if (a == INF) continue;      // earlier stages infeasible
      if (d - dp < rmn) continue;  // does not fit device memory
      const VT f = vmax(Fprev[(int64_t)i * DP + dp - 1], uf[(d - dp - 1) * 64]);
      const VT b = vmax(Bprev[(int64_t)i * DP + dp - 1], ub[(d - dp - 1) * 64]);
      const VT v = f + b;
      if (v < best) { best = v; bf = f; bb = b; bi = i; bd = dp; }
    }
  }
  if (jj >= N || j < s) return;
  if (write_v) {
    const int64_t e = (int64_t)(s - 1) * lvl + (int64_t)j * DP + d - 1;
    ((VT *)pr.V)[e] = best;
    ((VT *)pr.VF)[e] = bf;
    ((VT *)pr.VB)[e] = bb;
  }
  const int64_t e = ((int64_t)s * (N + 1) + j) * (D + 1) + d;
  if (arg_i) arg_i[e] = bi;
  if (arg_d) arg_d[e] = bd;
}

// Fast form of the same level.  The kept candidate of a cell is the smallest (sum, i, d') in
// lexicographic order, so partial results over disjoint sets of rows combine with a 64-bit atomicMin on
// the packed triple.  Work item (one workgroup of eight waves) = some consecutive rows of one chunk's
// window, from the same work list as the merge kernel.  Per row the workgroup computes the two stage
// times of every replica count from the prefix sums ([r][lane] in LDS, conflict-free, INF where the
// stage does not fit; two buffers, so that a row costs one barrier), and the eight waves split the device
// totals d between them (d = s + wave, s + wave + 8, ...): a lane keeps the running best of its column
// for each of its wave's d in registers.  The carried maxima of the row of the previous level are held
// one d' per lane and broadcast by lane reads.  The packed winners of the level become V
// and the two carried maxima in the next level's launch, or in a launch of their own (split_apart); the key table
// of the level before is cleared there for the level after next.
//
// Bound by vector instructions (four per candidate) and, for few rows, by latency.  With the stage times
// read from their two tables (built in front), items of four rows, d' in the key and every wave holding
// the totals of the whole class, a level of the outer driver at 96 blocks (24 searches, 31 levels) read
// 63 MB and took 22.5 us on average (call 906 us), and 1024 blocks at 64 devices 9.6 ms (now 534 us and 4.9 ms).
// Packed winner of a cell: (sum, i) in one 64-bit word whose unsigned order is the lexicographic order
// of the pair.  32-bit tables: 32 + 32 bits.  64-bit tables: 48 + 16 bits, the sums stay below 2^42 - 1
// (kSplitPackedMax, a bound of the quotient as well).  d' is not carried: the level's inner loop is four
// operations per candidate without it and six with it, and split_winner finds the first d' of row
// i whose sum is the cell's value.
template <typename VT> __device__ __forceinline__ unsigned long long split_pack(VT v, uint32_t i);
template <> __device__ __forceinline__ unsigned long long split_pack<uint32_t>(uint32_t v, uint32_t i) {
  return ((unsigned long long)v << 32) | i;
}
template <> __device__ __forceinline__ unsigned long long split_pack<uint64_t>(uint64_t v, uint32_t i) {
  return (v << 16) | i;
}
template <typename VT> __device__ __forceinline__ int split_key_i(unsigned long long k) { return (int)(k & 0xFFFFull); }
template <typename VT> __device__ __forceinline__ VT split_key_v(unsigned long long k) {
  return sizeof(VT) == 4 ? (VT)(k >> 32) : (VT)(k >> 16);
}

// Stage time of a stage that does not fit: a sum with it is never below it, and orders as any other
// value.  (32-bit sums saturate; 64-bit ones must stay below the pattern of infinity.)
template <typename VT> constexpr VT split_nofit() { return sizeof(VT) == 8 ? (VT)((uint64_t)1 << 61) : Lim<VT>::inf; }
__device__ __forceinline__ uint32_t split_sum(uint32_t f, uint32_t b) { return __builtin_elementwise_add_sat(f, b); }
__device__ __forceinline__ uint64_t split_sum(uint64_t f, uint64_t b) { return f + b; }

// The key table of level s.
__device__ __forceinline__ unsigned long long RANNC_GLOBAL *split_keys(const ProblemDev &pr, int s) {
  return gptr((unsigned long long *)pr.keys) + (int64_t)(s % kSplitKeyTables) * (pr.N + 1) * pr.DP;
}

// Cell (j, d) of level s >= 2 whose packed winner is key: eight lanes look for the first d' of the winner's row
// i whose sum is the cell's value (there is one), each at every eighth d'; the lane that finds it calls
// out(value, forward, backward maximum).  inv[r] = 1 / r.  Bound by latency: one round of reads.
constexpr int kFinalizeLanes = 8;
template <typename VT, typename Out>
__device__ __forceinline__ void split_winner(const ProblemDev &pr, const int s, const int j, const int d,
                                             const unsigned long long key, const double *inv, Out out) {
  const int N = pr.N, DP = pr.DP, sub = threadIdx.x & (kFinalizeLanes - 1);
  const int i = split_key_i<VT>(key);
  const VT v = split_key_v<VT>(key);
  const int64_t lvl = (int64_t)(N + 1) * DP;
  const VT RANNC_GLOBAL *F = gptr((const VT *)pr.VF) + (int64_t)(s - 2) * lvl + (int64_t)i * DP - 1;
  const VT RANNC_GLOBAL *B = gptr((const VT *)pr.VB) + (int64_t)(s - 2) * lvl + (int64_t)i * DP - 1;
  const int rmn = (int)pr.rmin[unit_index(pr.nch, i, (j - 1) >> 6) * 64 + ((j - 1) & 63)];
  const VT xf = (VT)(pr.T[j] - pr.T[i]), xb = (VT)(pr.TB[j] - pr.TB[i]), xc = pr.C ? (VT)pr.C[j] : (VT)0;
#pragma unroll 1
  for (int d1 = s - 1 + sub; d1 - sub <= d - 1; d1 += 2 * kFinalizeLanes) {
    VT f[2], b[2];
    unsigned mine = 0;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int dp = min(d1 + u * kFinalizeLanes, d - 1);
      f[u] = F[dp];
      b[u] = B[dp];
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int dp = d1 + u * kFinalizeLanes, r = max(d - dp, 1);
      const double in = inv[r];
      f[u] = vmax(f[u], (VT)(ceil_div<VT>(xf, r, in) + (xc ? ceil_div<VT>(xc, r, in) : (VT)0)));
      b[u] = vmax(b[u], ceil_div<VT>(xb, r, in));
      if (dp <= d - 1 && r >= rmn && split_sum(f[u], b[u]) == v) mine |= 1u << u;
    }
    // the smallest d' of the two rounds of eight
    const int base = (threadIdx.x & 63) & ~(kFinalizeLanes - 1);
    const unsigned m0 = (unsigned)(__ballot(mine & 1u) >> base) & ((1u << kFinalizeLanes) - 1u);
    const unsigned m1 = (unsigned)(__ballot(mine & 2u) >> base) & ((1u << kFinalizeLanes) - 1u);
    if (m0 | m1) {
      const int u = m0 ? 0 : 1;
      if (sub == __ffs((int)(m0 ? m0 : m1)) - 1) out(v, u ? f[1] : f[0], u ? b[1] : b[0]);
      break;
    }
  }
}

// Sixty-four cells (j = 64 block .., d) of level s, by one workgroup of the level kernel's size: V and the two
// maxima in memory.  Level s - 1's key table, which nothing reads any more, is cleared for level s + 2.
constexpr int kSplitThreads = 64 * kSplitWaves;
template <typename VT>
__device__ __forceinline__ void split_winners(const ProblemDev &pr, const int s, const int block, const int d, const double *inv) {
  const int N = pr.N, DP = pr.DP;
  const int j = block * (kSplitThreads / kFinalizeLanes) + (int)(threadIdx.x / kFinalizeLanes);
  if (j > N || d > pr.D) return;
  const int64_t at = (int64_t)(d - 1) * (N + 1) + j;
  if (s > 2 && (threadIdx.x & (kFinalizeLanes - 1)) == 0) split_keys(pr, s - 1)[at] = ~0ull;
  const unsigned long long key = d >= s ? split_keys(pr, s)[at] : ~0ull;
  if (key == ~0ull) return;  // no candidate: the cell keeps "no plan" (the eight lanes of a cell agree)
  const int64_t e = (int64_t)(s - 1) * (int64_t)(N + 1) * DP + (int64_t)j * DP + d - 1;
  split_winner<VT>(pr, s, j, d, key, inv, [&](VT v, VT f, VT b) {
    ((VT *)pr.V)[e] = v;
    ((VT *)pr.VF)[e] = f;
    ((VT *)pr.VB)[e] = b;
  });
}

// Candidates d' = lo..hi of one staged row against the device totals d_k, k >= K0, of this wave
// (all of them lie above hi, so every (d', k) pair is a candidate).  Two d' at a time, written out: the lane
// reads keep the compiler from unrolling the loop itself.  (Outer driver at 96 blocks / 256 blocks alone, whole
// call: one at a time 535 / 209 us, two 521 / 203, four, which take a workgroup's registers off each compute
// unit, 552 / 219.  Totals next to each other instead of eight apart, with a sliding window of times in
// registers instead of two LDS reads per candidate: 207 us alone, but 588 for the driver, whose waves then
// wait for the one with the most candidates at every row.)  TWO: not for 64-bit values at 16 and 64 devices, where it
// takes 82 registers instead of 68, two workgroups to a compute unit instead of three, and 210 instead of 166 (500 blocks
// at 16 devices 309 instead of 268 us, 1024 at 64 11.8 instead of 9.6 ms).
template <typename VT, int KP, int K0, int U>
__device__ __forceinline__ void split_candidates(int dp, int d0, int lane, VT F, VT B, const VT *sf, const VT *sb, VT (&row_v)[KP]) {
  VT af[U], ab[U];
#pragma unroll
  for (int u = 0; u < U; ++u) { af[u] = lane_bcast(F, dp + u - 1); ab[u] = lane_bcast(B, dp + u - 1); }
  // the times of r = d_k - d' (>= 1; beyond the staged ones only for totals above D)
  const VT *const f = sf + (d0 - dp - 1) * 64 + lane, *const b = sb + (d0 - dp - 1) * 64 + lane;
#pragma unroll
  for (int k = K0; k < KP; ++k) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      row_v[k] = vmin(row_v[k], split_sum(vmax(af[u], f[(kSplitWaves * k - u) * 64]), vmax(ab[u], b[(kSplitWaves * k - u) * 64])));
  }
}
template <typename VT, int KP, int K0, bool TWO>
__device__ __forceinline__ void split_segment(int lo, int hi, int d0, int lane, VT F, VT B, const VT *sf, const VT *sb,
                                              VT (&row_v)[KP]) {
  int dp = lo;
  if constexpr (TWO) {
#pragma unroll 1
    for (; dp + 1 <= hi; dp += 2) split_candidates<VT, KP, K0, 2>(dp, d0, lane, F, B, sf, sb, row_v);
  }
#pragma unroll 1
  for (; dp <= hi; ++dp) split_candidates<VT, KP, K0, 1>(dp, d0, lane, F, B, sf, sb, row_v);
}

template <typename VT, int KP, int K0, bool TWO>
__device__ __forceinline__ void split_row(int dlo, int D, int d0, int lane, VT F, VT B, const VT *sf, const VT *sb,
                                          VT (&row_v)[KP]) {
  if constexpr (K0 < KP) {
    // d' in [d_{K0-1}, d_{K0} - 1]: exactly the totals d_k with k >= K0 lie above it
    const int lo = K0 == 0 ? dlo : max(dlo, d0 + kSplitWaves * (K0 - 1));
    const int hi = min(d0 + kSplitWaves * K0 - 1, D - 1);
    split_segment<VT, KP, K0, TWO>(lo, hi, d0, lane, F, B, sf, sb, row_v);
    split_row<VT, KP, K0 + 1, TWO>(dlo, D, d0, lane, F, B, sf, sb, row_v);
  }
}

// The rows of one work item.  KP: device totals per wave, and replica counts it computes the times of:
// the D-s+1 totals (and counts) that are left at level s, over eight waves.
// rowF, rowB: the two maxima of row i_lo at level s - 1, the next row's `stride` values behind them.
template <typename VT, int DP, int KP, typename RP>
__device__ __forceinline__ void split_rows(const ProblemDev &pr, const int s, const int c, const int i_lo, const int i_hi,
                                           VT (*sf)[DP * 64], VT (*sb)[DP * 64], const int n_buf, const RP rowF, const RP rowB,
                                           const int stride) {
  constexpr VT INF = Lim<VT>::inf;
  constexpr bool kTwo = sizeof(VT) == 4 || (DP != 16 && DP != 64);
  const int N = pr.N, D = pr.D, nch = pr.nch;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int jj = 64 * c + lane;
  const uint8_t RANNC_GLOBAL *__restrict__ rmin = gptr((const uint8_t *)pr.rmin);
  const int64_t RANNC_GLOBAL *__restrict__ T = gptr((const int64_t *)pr.T);
  const int64_t RANNC_GLOBAL *__restrict__ TB = gptr((const int64_t *)pr.TB);
  const int rl = D - s + 1;  // replicas left for stage s when s-1 devices are spent earlier
  const int d0 = s + wave;   // this wave's device totals: d0, d0 + 8, ...
  struct Row { VT F, B; int rmn; };
  auto load = [&](int i) -> Row {  // the next row's, while one is worked on (clamped into the item)
    const int ic = min(i, i_hi);
    Row r;
    r.F = rowF[(ic - i_lo) * stride + min(lane, D - 1)];  // lane q holds d' = q + 1
    r.B = rowB[(ic - i_lo) * stride + min(lane, D - 1)];
    r.rmn = rmin[unit_index(nch, ic, c) * 64 + lane];
    return r;
  };
  Row cur = load(i_lo);
  const int jc = min(jj + 1, N);  // (lanes beyond N compute times nobody looks at)
  const int64_t Tj = T[jc], TBj = TB[jc];
  // the prefix sums of the item's rows (at most 64), a row per lane: scalar loads would be waited for at
  // every barrier
  const int64_t Trow = T[min(i_lo + lane, N)], TBrow = TB[min(i_lo + lane, N)];
  VT hc[KP];       // send time of the cut behind the lane's column, per replica count of this wave
  double inv[KP];  // 1 / r
#pragma unroll
  for (int k = 0; k < KP; ++k) {
    inv[k] = 1.0 / (double)(wave + kSplitWaves * k + 1);
    hc[k] = 0;
  }
  if (pr.C) {
    const VT Cj = (VT)gptr((const int64_t *)pr.C)[jc];
#pragma unroll
    for (int k = 0; k < KP; ++k) hc[k] = ceil_div<VT>(Cj, wave + kSplitWaves * k + 1, inv[k]);
  }
  VT best_v[KP];
  uint32_t best_i[KP];
#pragma unroll
  for (int k = 0; k < KP; ++k) { best_v[k] = INF; best_i[k] = 0; }

  int buf = 0;
  for (int i = i_lo; i <= i_hi; ++i) {  // every condition below is uniform over the workgroup
    const Row r = cur;
    cur = load(i + 1);
    const bool fit = jj >= i && jj < N && r.rmn <= rl;
    // first d' with a plan of s-1 stages over blocks 1..i (finite values are a suffix of the row)
    const unsigned long long fin = __ballot(lane < D - 1 && r.F != INF);
    if (fin == 0ull || __ballot(fit) == 0ull) continue;
    const int dlo = max(s - 1, __ffsll((long long)fin));
    VT *const f = sf[buf], *const b = sb[buf];
    const double xf = (double)(VT)(Tj - (int64_t)lane_bcast((uint64_t)Trow, i - i_lo));
    const double xb = (double)(VT)(TBj - (int64_t)lane_bcast((uint64_t)TBrow, i - i_lo));
#pragma unroll
    for (int k = 0; k < KP; ++k) {
      const int n = wave + kSplitWaves * k + 1;  // replicas
      const double o = ceil_div_offset<VT>(n);
      const bool ok = fit && n >= r.rmn;
      f[(n - 1) * 64 + lane] = ok ? (VT)(CeilDiv<VT>::at(xf + o, inv[k]) + hc[k]) : split_nofit<VT>();
      b[(n - 1) * 64 + lane] = ok ? CeilDiv<VT>::at(xb + o, inv[k]) : split_nofit<VT>();
    }
    lds_barrier();
    VT row_v[KP];
#pragma unroll
    for (int k = 0; k < KP; ++k) row_v[k] = INF;
    split_row<VT, KP, 0, kTwo>(dlo, D, d0, lane, r.F, r.B, f, b, row_v);
#pragma unroll
    for (int k = 0; k < KP; ++k) {  // rows ascend: an equal sum keeps the earlier one
      const bool ok = row_v[k] < best_v[k];
      best_v[k] = ok ? row_v[k] : best_v[k];
      best_i[k] = ok ? (uint32_t)i : best_i[k];
    }
    if (n_buf == 2) buf ^= 1;  // (rewritten behind the next row's barrier, which every wave reaches after its reads)
    else lds_barrier();
  }
  if (jj >= N || jj + 1 < s) return;
  unsigned long long RANNC_GLOBAL *K = split_keys(pr, s);
#pragma unroll
  for (int k = 0; k < KP; ++k) {
    const int dk = d0 + kSplitWaves * k;
    if (dk <= D && best_v[k] < split_nofit<VT>())
      (void)__hip_atomic_fetch_min(&K[(int64_t)(dk - 1) * (N + 1) + jj + 1], split_pack<VT>(best_v[k], best_i[k]),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// items: workgroups of the grid that work on the level's items; the others, `blocks` to a device total from
// s - 2 on, finish level s - 1.  Most rows of an item: kSplitMaxRows.
// APART: level s - 1 has been finished by a launch of its own (split_apart); the grid has items only, which read
// their rows' maxima from memory, a row ahead.
template <typename VT, int DP, bool APART>
__global__ __launch_bounds__(kSplitThreads) void level_split_fast_kernel(
    const ProblemDev *__restrict__ probs, const int s, const int items, const int blocks) {
  const ProblemDev &pr = probs[blockIdx.z];
  __shared__ double inv[APART ? 1 : 65];
  if constexpr (!APART) {
    if (threadIdx.x < 64) inv[threadIdx.x + 1] = 1.0 / (double)(threadIdx.x + 1);
    if ((int)blockIdx.x >= items) {
      if (s - 1 > pr.S_eff || s == 2) return;  // (level 1 has no keys)
      __syncthreads();
      const int at = (int)blockIdx.x - items;
      split_winners<VT>(pr, s - 1, at % blocks, s - 2 + at / blocks, inv);
      return;
    }
  }
  if (s > pr.S_eff) return;
  const int N = pr.N, D = pr.D;
  const int32_t RANNC_GLOBAL *__restrict__ runs = gptr((const int32_t *)pr.runs);
  // (the item is read together with their number, at a place that every list has)
  const int count = runs[0];
  const unsigned desc = (unsigned)runs[1 + min((int)blockIdx.x, (int)max_runs(pr.nch) - 1)];
  asm volatile("" :: "s"(count), "s"(desc));
  if ((int)blockIdx.x >= count) return;
  const int c = (int)((desc >> 16) & 0x3ffu), i0 = (int)(desc & 0xffffu), rows = (int)(desc >> 26) + 1;
  if (64 * c + 64 < s) return;  // no column j >= s in this chunk
  const int i_hi = min(min(i0 + rows - 1, 64 * c + 63), N - 1);
  const int i_lo = max(i0, s - 1);
  if (i_hi < i_lo) return;
  constexpr int BUF = 4 * DP * 64 * (int)sizeof(VT) <= 64 * 1024 ? 2 : 1;
  __shared__ VT sf[BUF][DP * 64], sb[BUF][DP * 64];
  // the two maxima of the item's rows at level s - 1
  [[maybe_unused]] __shared__ VT rowF[APART ? 1 : kSplitMaxRows * DP], rowB[APART ? 1 : kSplitMaxRows * DP];
  const VT RANNC_GLOBAL *const F = gptr((const VT *)pr.VF) + ((int64_t)(s - 2) * (N + 1) + i_lo) * pr.DP;
  const VT RANNC_GLOBAL *const B = gptr((const VT *)pr.VB) + ((int64_t)(s - 2) * (N + 1) + i_lo) * pr.DP;
  if constexpr (!APART) {
    const int n = i_hi - i_lo + 1;
    if (s == 2) {
      for (int e = threadIdx.x; e < n * DP; e += kSplitThreads) {
        const int64_t at = (int64_t)(e / DP) * pr.DP + min(e % DP, pr.DP - 1);
        rowF[e] = F[at];
        rowB[e] = B[at];
      }
    } else {
      for (int e = threadIdx.x; e < n * DP; e += kSplitThreads) rowF[e] = rowB[e] = Lim<VT>::inf;
      __syncthreads();
      const unsigned long long RANNC_GLOBAL *K = split_keys(pr, s - 1);
      const int nd = D - s + 1;  // d' = s-1 .. D-1
      for (int e = (int)(threadIdx.x / kFinalizeLanes); e < n * nd; e += kSplitThreads / kFinalizeLanes) {
        const int q = e / nd, d = s - 1 + e - q * nd;
        const unsigned long long key = K[(int64_t)(d - 1) * (N + 1) + i_lo + q];
        if (key != ~0ull)
          split_winner<VT>(pr, s - 1, i_lo + q, d, key, inv, [&](VT, VT f, VT b) {
            rowF[q * DP + d - 1] = f;
            rowB[q * DP + d - 1] = b;
          });
      }
    }
    __syncthreads();
  }
#define RANNC_ROWS(K)                                                                                              \
  case K:                                                                                                          \
    if constexpr (kSplitWaves * K <= DP) {                                                                         \
      if constexpr (APART) split_rows<VT, DP, K>(pr, s, c, i_lo, i_hi, sf, sb, BUF, F, B, pr.DP);                  \
      else split_rows<VT, DP, K>(pr, s, c, i_lo, i_hi, sf, sb, BUF, (const VT *)rowF, (const VT *)rowB, (int)DP);  \
    }                                                                                                              \
    break;
  switch ((D - s + kSplitWaves) / kSplitWaves) {
    RANNC_ROWS(1) RANNC_ROWS(2) RANNC_ROWS(3) RANNC_ROWS(4)
    RANNC_ROWS(5) RANNC_ROWS(6) RANNC_ROWS(7) RANNC_ROWS(8)
    default: break;
  }
#undef RANNC_ROWS
}

// The winners of level s: of a launch's last level (those of shorter searches are done), or of every one.
template <typename VT>
__global__ __launch_bounds__(kSplitThreads) void split_finalize_kernel(const ProblemDev *__restrict__ probs, const int s, const int every) {
  const ProblemDev &pr = probs[blockIdx.z];
  if (every ? s > pr.S_eff : s != pr.S_eff) return;
  __shared__ double inv[65];
  if (threadIdx.x < 64) inv[threadIdx.x + 1] = 1.0 / (double)(threadIdx.x + 1);
  __syncthreads();
  split_winners<VT>(pr, s, blockIdx.x, blockIdx.y + 1, inv);
}

// ---------------------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------------------
hipError_t launch_split_level1(const ProblemDev *p, const LaunchShape &sh, int bits, hipStream_t st) {
  for (int q0 = 0; q0 < sh.nprob; q0 += 65535) {
    const int nq = min(65535, sh.nprob - q0);
    const dim3 grid(sh.max_nch, sh.max_D, nq);
    if (bits == 32) hipLaunchKernelGGL((split_level1_kernel<uint32_t>), grid, dim3(64), 0, st, p + q0);
    else hipLaunchKernelGGL((split_level1_kernel<uint64_t>), grid, dim3(64), 0, st, p + q0);
  }
  return hipGetLastError();
}

hipError_t launch_level_split(const ProblemDev *p, const LaunchShape &sh, int bits, int s, int write_v,
                              int32_t *arg_i, int32_t *arg_d, hipStream_t st) {
  for (int q0 = 0; q0 < sh.nprob; q0 += 65535) {
    const int nq = min(65535, sh.nprob - q0);
    const dim3 grid(sh.max_nch, sh.max_D, nq);
    if (bits == 32)
      hipLaunchKernelGGL((level_split_kernel<uint32_t>), grid, dim3(64), 0, st, p + q0, s, write_v, arg_i,
                         arg_d);
    else
      hipLaunchKernelGGL((level_split_kernel<uint64_t>), grid, dim3(64), 0, st, p + q0, s, write_v, arg_i,
                         arg_d);
  }
  return hipGetLastError();
}

// A workgroup's rows are a chain, and every workgroup pays DP x 64 atomics of 8 bytes behind it (about 5 ps
// each over the launch): as few rows as leave about this many workgroups.  Measured per call, items of
// 1 / 2 / 3 / 4 / 8 rows: 256 blocks at 32 devices (640 rows) 283 / 271 / 293 / - / - us, 400 at 32 (1 744
// rows) 796 / 559 / 540 / - / -, outer driver at 96 blocks (1 440 rows of its 32-device searches) 575 / 582 /
// 621 / - / -, 1024 at 64 (8 704 rows) 10.8 / 6.8 / 5.5 / 5.5 / 5.9 ms where memory never binds and 2.8 /
// 2.1 / 2.1 / - / 2.8 where it does, 900 at 16 (7 620 rows) 937 / 551 / 429 / 404 / 377 us, 300 at 8 (940 rows)
// 166 / 137 / 133 / 135 / 146.
int split_rows_per_item(const LaunchShape &sh, int DP) {
  const int64_t groups = DP == 8 ? 256 : DP == 64 ? 2560 : 1024;
  const int64_t rows = std::min<int64_t>(kSplitMaxRows, (sh.wide_rows + groups - 1) / groups);
  int64_t most = 0;  // rows of the largest search: its list has room for single-row items up to a size
  for (int c = 0; c < sh.max_nch; ++c) most += std::min(64 * c + 64, sh.max_N);
  return (int)std::max<int64_t>(most > kSplitSmallRows ? 4 : 1, rows);
}

// Whether every level's winners are unpacked by a launch of their own.  A row of a level is listed once per column
// chunk, so with the unpacking in the next level's launch every row is unpacked by several workgroups and once more for
// memory: work that costs a full device more than one launch fewer per level saves.  The host does not know how many
// rows the memory leaves of a chunk, about two hundred in a long chain, so the line counts chunks, times the mean
// square of the share of the devices that a level still deals with.  Per call, in the next level's launch / apart:
//   32-bit values, 64 devices (line at 4): 128 blocks (1.2) 447 / 505 us, 256 (2.3) 946 / 932, 4 searches of 40 (3.5)
//     152 / 159, of 128 (6.2) 531 / 486, 1024 blocks (9) 5.62 / 4.88 ms;
//     32 devices (6.2, several searches 10): 512 blocks (4.6) 417 / 425, 700 (6.4) 688 / 627, outer driver at 96 blocks
//     (5.9) 534 / 563, at 160 (8.9) 759 / 800, at 200 (11.8) 952 / 907, 12 searches of 128 (14) 463 / 382; 16 devices (20): 900 blocks (5) 394 / 408, 4 searches of 500 (19) 229 / 256, 20 of
//     120 (23) 201 / 191, 8 of 500 (37) 333 / 273, 100 of 40 (58) 235 / 213; 8 devices (48): 4 searches of 500 (10) 176 /
//     189, 60 of 120 (37) 240 / 245, 200 of 40 (62) 268 / 248.
//   64-bit values, whose workgroups take longer: 32 devices (3.5): 256 blocks (2.3) 258 / 287, 4 searches of 128 (4.6)
//     326 / 309; 16 devices (20): 4 searches of 500 (19) 286 / 300, 60 of 64 (35) 285 / 262, 8 of 500 (37) 439 / 407; 8
//     devices (34): 4 of 500 (10) 203 / 213, 60 of 120 (37) 305 / 281.
static bool split_apart(const LaunchShape &sh, int bits, int DP) {
  double share = 0.0;  // sum over the levels
  for (int s = 2; s <= sh.max_S_eff; ++s) share += (double)(sh.max_D - s + 1) * (sh.max_D - s + 1) / (DP * DP);
  const double line = DP == 64 ? 4.0 : DP == 32 ? (bits == 64 ? 3.5 : sh.nprob == 1 ? 6.2 : 10.0) : DP == 16 ? 20.0 : bits == 64 ? 34.0 : 48.0;
  return sh.wide_chunks * share >= line * (sh.max_S_eff - 1);
}

template <typename VT>
static void split_fast_go(const ProblemDev *p, const LaunchShape &sh, int DP, int s, int items, hipStream_t st) {
  constexpr int cells = kSplitThreads / kFinalizeLanes;
  const int blocks = (sh.max_N + cells) / cells;
  const bool apart = split_apart(sh, (int)sizeof(VT) * 8, DP);
  for (int q0 = 0; q0 < sh.nprob; q0 += 65535) {
    const int nq = min(65535, sh.nprob - q0);
    const dim3 grid((unsigned)(items + (s > 2 && !apart ? blocks * (sh.max_D - s + 3) : 0)), 1, nq), block(kSplitThreads);
#define GO(W, X)             \
  if (DP == W && apart == X) \
    hipLaunchKernelGGL((level_split_fast_kernel<VT, W, X>), grid, block, 0, st, p + q0, s, items, blocks);
    GO(8, false) GO(16, false) GO(32, false) GO(64, false)
    GO(8, true) GO(16, true) GO(32, true) GO(64, true)
#undef GO
    if (apart || s == sh.max_S_eff)
      hipLaunchKernelGGL((split_finalize_kernel<VT>), dim3(blocks, sh.max_D, nq), block, 0, st, p + q0, s, apart ? 1 : 0);
  }
}

hipError_t launch_level_split_fast(const ProblemDev *p, const LaunchShape &sh, int bits, int DP, int s,
                                   int rows_per_item, hipStream_t st) {
  const int per = rows_per_item;
  int64_t items = 0;  // upper bound on the items of any problem of the launch
  for (int c = 0; c < sh.max_nch; ++c) items += (min(64 * c + 64, sh.max_N) + per - 1) / per;
  if (per > kSplitMaxRows) return hipErrorInvalidValue;
  if (bits == 32) split_fast_go<uint32_t>(p, sh, DP, s, (int)items, st);
  else split_fast_go<uint64_t>(p, sh, DP, s, (int)items, st);
  return hipGetLastError();
}

}  // namespace rannc
