// gfx950 kernels of the compaction step of RaNNC's block-level phase (Sec. III-B) on a chain, and
// its launcher.
#include "rannc_dp_device.h"
#include "rannc_dp_once.h"

#include <algorithm>
#include <type_traits>

namespace rannc {

// ---------------------------------------------------------------------------------------
// Compaction step of the block-level phase (Sec. III-B, last step before the stage-level search),
// on a chain of G groups.  A walk: the groups as they stand are listed by ascending computation
// time (equal times by position); a listed group that is still as listed merges with the
// neighbour whose current time is smaller if the union fits the device memory; the procedure ends
// as soon as k groups are left.  When a walk ends above k groups the groups are listed again by
// their current times and walked again, until k is reached, a walk merges nothing, or the caller's
// limit on the number of walks is met.  The kernels exist so that the chain stays on the device
// between the two phases.  One workgroup, and for the walks of long chains launches over the device.
//
// The walk follows a list, but a turn of it reads and changes only its own neighbourhood: the turn
// of group v looks at its neighbours l and r and merges v with one of them, and the only turns that
// can change what it sees are those of l, r and of the groups next to them (which may pick l or r).
// So every group whose place in the list is ahead of all groups within two positions that still wait
// for their turn can take it NOW, whatever the rest of the list holds: its neighbourhood is what the
// walk in list order would show it.  The kernel takes all such turns at once, round after round; two
// turns of one round are at least three positions apart and touch different groups.  On times without
// an order along the chain the waiting groups fall by a constant share per round (about twenty rounds
// at 15 000 groups); a chain of ascending times takes one turn per round, which is the list's own
// pace.  No list is built: a place in it is the pair (time, position), compared where it is needed.
//
// State: the groups of the walk are numbered 0..n-1 in chain order, T[u] is the time of everything in
// front of group u, M[u] the bytes.  Merging only removes a boundary, so the whole state that
// changes is one bit per group (still a head), one bit (still waits) and the time of a group is
// T[next head] - T[head].  After a walk the heads are renumbered.  Stopping at k: a walk that would go
// below k has to stop at its (n-k)-th merge in list order; the merges that lie ahead of that one do not
// depend on those behind it, so the walk is taken to its end, the (n-k)-th smallest place is found
// (radix selection over (time, position)), and the merges behind it are undone.
//
// Where few turns are possible at a time, one wave goes on without barriers (kFewTurns).
//
// On times without an order along the chain a group's turn depends on few positions to either side, so a walk is first
// tried in windows, a wave to each (compact_window_walk), without barriers: walks of up to kCompactWindows groups by the
// waves of one workgroup, those of longer chains as launches over the whole device (compact_first_kernel,
// compact_walk_kernel), which leave a bit per group; a walk of which any window was too small, or which would go to k groups or below, is
// done again by one workgroup in rounds as above (a walk that stops at k by its windows, where they are large enough).
//
// Bound by latency: a round of a window is some 80 instructions and one round of LDS permutes, 0.35 us, six to nine rounds to
// a walk; a launched walk is 8 to 10 us, of which 3 are four dependent reads (words of the walk before, first
// group, sums) and the workgroup's scan.  15 000 groups to 32 blocks, per call: 19.7 ms with one lane following a sorted list
// through memory, 0.30 ms in rounds by one workgroup, 62 us here (9 the first walk and the sums, 3 x 9 the next walks,
// 22 the rest).  In rounds / here: 65 535 groups 1 110 / 115 us, 5 000 158 / 55, 1 600 129 / 72, 400 71 / 46, 64 51 / 33;
// ascending times, 15 000 groups, 14.6 ms (a turn after the other by one wave, 1 us each).
// ---------------------------------------------------------------------------------------
constexpr int kCompactSmall = 1600;     // up to here everything is in LDS and four waves do the work
constexpr int kCompactTimesLds = 16384; // up to here the times (and the bit maps) are in LDS

constexpr int kCompactWindows = 1600;  // up to here a walk of one workgroup goes in windows
// Above, a walk of a long chain gets a launch of its own (9 us; by one workgroup's windows 500 groups take as long, 1 600
// 20 us).
constexpr int kCompactLaunch = 500;

template <int MODE> struct CompactShape;  // mask of the groups a thread looks after (u = tid + b * threads)
template <> struct CompactShape<0> { using Mask = uint32_t; static constexpr int kMax = kCompactSmall; };
template <> struct CompactShape<1> { using Mask = uint32_t; static constexpr int kMax = kCompactTimesLds; };
template <> struct CompactShape<2> { using Mask = uint64_t; static constexpr int kMax = 65535; };

// inclusive sum over the workgroup of one value per thread; part: one word per wave
template <int NT, typename X> __device__ __forceinline__ X compact_scan(X v, X *part) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const X w = __shfl_up(v, o);
    if (lane >= o) v += w;
  }
  if (lane == 63) part[wave] = v;
  __syncthreads();
  X before = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w)
    if (w < wave) before += part[w];
  __syncthreads();
  return v + before;
}

// The bit maps: group u is bit u + 32, and the words in front of the first and behind the last group
// stay empty, so that a look at either end of the chain needs no test.
__device__ __forceinline__ bool compact_bit(const uint32_t *map, int u) { return (map[(u + 32) >> 5] >> (u & 31)) & 1u; }
// the groups u - 16 .. u + 15: group u is bit 16
__device__ __forceinline__ uint32_t compact_window(const uint32_t *map, int u) {
  const int b = u + 16;
  return __builtin_amdgcn_alignbit(map[(b >> 5) + 1], map[b >> 5], (uint32_t)(b & 31));
}
// next / previous head of group u (n / -1 if there is none)
__device__ __forceinline__ int compact_next(const uint32_t *head, int u, int n) {
  int w = (u + 33) >> 5;
  uint32_t m = head[w] & (~0u << ((u + 1) & 31));
  const int last = (n + 31) >> 5;  // the word of group n - 1
  while (!m && w < last) m = head[++w];
  return m ? (w << 5) + __ffs((int)m) - 1 - 32 : n;
}
__device__ __forceinline__ int compact_prev(const uint32_t *head, int u) {
  int w = (u + 32) >> 5;
  uint32_t m = head[w] & ((1u << (u & 31)) - 1u);
  while (!m && w > 1) m = head[--w];
  return m ? (w << 5) + 31 - __clz((int)m) - 32 : -1;
}

// What a turn of group v looks at: the neighbouring heads l, r = v + 1 and those behind them (-1 / n
// where the chain ends), and which of them still wait (bits: ll, l, r, rr, lll, rrr).
struct CompactAround { int l, ll, lll, r, rr, rrr; uint32_t waits; };
__device__ __forceinline__ CompactAround compact_around(const uint32_t *head, const uint32_t *waits, int v, int n) {
  CompactAround c;
  const uint32_t hw = compact_window(head, v), ww = compact_window(waits, v);
  uint32_t lo = hw & 0xFFFFu, hi = hw >> 17;  // hi: bit 0 is group v + 1
  c.r = v + 1;
  if ((__popc(lo) >= 3 || v <= 16) && (__popc(hi) >= 3 || v + 16 > n)) {
    // (the common case) everything is inside the window: bit 16 - (v - u) for a group u below v
    auto below = [&](uint32_t &m, int &u, uint32_t bit) {
      const int b = 31 - __clz((int)m);
      u = m ? v - 16 + b : -1;
      if (m && ((ww >> b) & 1u)) c.waits |= bit;
      m &= ~(1u << (b & 31));
    };
    auto above = [&](uint32_t &m, int &u, uint32_t bit) {
      const int b = __ffs((int)m) - 1;
      u = m ? v + 1 + b : n;
      if (m && ((ww >> ((17 + b) & 31)) & 1u)) c.waits |= bit;
      m &= m - 1u;
    };
    c.waits = 0;
    int r;
    below(lo, c.l, 2u); below(lo, c.ll, 1u); below(lo, c.lll, 16u);
    above(hi, r, 4u); above(hi, c.rr, 8u); above(hi, c.rrr, 32u);
  } else {
    c.l = compact_prev(head, v);
    c.ll = c.l >= 0 ? compact_prev(head, c.l) : -1;
    c.lll = c.ll >= 0 ? compact_prev(head, c.ll) : -1;
    c.rr = c.r < n ? compact_next(head, c.r, n) : n;
    c.rrr = c.rr < n ? compact_next(head, c.rr, n) : n;
    c.waits = (c.ll >= 0 && compact_bit(waits, c.ll) ? 1u : 0u) | (c.l >= 0 && compact_bit(waits, c.l) ? 2u : 0u) |
              (c.r < n && compact_bit(waits, c.r) ? 4u : 0u) | (c.rr < n && compact_bit(waits, c.rr) ? 8u : 0u) |
              (c.lll >= 0 && compact_bit(waits, c.lll) ? 16u : 0u) | (c.rrr < n && compact_bit(waits, c.rrr) ? 32u : 0u);
  }
  return c;
}

// Whether group v, which waits, takes its turn now (it is ahead of every waiting group within two
// positions), and if so whether it merges and on which side.  A group that waits is as listed: its
// successor v + 1 is a head (or the end of the chain), and so is that of every waiting neighbour.
template <typename TP, typename MP>
__device__ __forceinline__ bool compact_turn(TP T, MP M, const CompactAround &c, int v, int n, uint64_t mem, bool &join,
                                             bool &left) {
  const int l = max(c.l, 0), ll = max(c.ll, 0), rr = c.rr;
  // one round of reads
  const uint64_t Tv = T[v], Tr = T[v + 1], Tl = T[l], Trr = T[rr], Tl1 = T[ll], Tl2 = T[ll + 1], Tr2 = T[min(rr + 1, n)];
  const uint64_t Ml = M[l], Mv = M[v], Mr = M[v + 1], Mrr = M[rr];
  const uint64_t tv = Tr - Tv;
  const uint64_t tl = c.l >= 0 ? Tv - Tl : ~0ull, tr = c.r < n ? Trr - Tr : ~0ull;
  // equal times: the one further left is ahead in the list
  const bool ahead = !((c.waits & 2u) && tl <= tv) & !((c.waits & 4u) && tr < tv) & !((c.waits & 1u) && Tl2 - Tl1 <= tv) &
                     !((c.waits & 8u) && Tr2 - Trr < tv);
  left = !(tr < tl);
  join = (left ? Mr - Ml : Mrr - Mv) <= mem;
  return ahead;
}

// ---- a walk in windows ----
// What a turn sees depends on turns a few positions away, those on a few more, and so on, each ahead of the one before: on
// times without an order along the chain rarely more than twenty positions in all.  A wave takes 63 consecutive groups, one
// to a lane, with everything it needs in registers, and walks them as far as it can: a group whose turn could be
// preceded by one outside the window never gets there, and neither does what depends on it.  If the groups in the
// window's middle have all had their turns, and the head in front of them too (whose turn could remove the first one's
// boundary), what became of them is what the walk makes of them.
struct CompactWindow { uint64_t heads, self; bool whole; };  // self: boundaries removed by the turn of the group behind them
constexpr int kWindow = 63;                                  // (the last lane holds the end of the last group)
constexpr uint32_t kCompactOpen = ~0u;                       // a chunk whose window was too small
// t, m: time and bytes of the group of this lane; groups: lanes with one; the middle: lanes [first, last)
__device__ __forceinline__ CompactWindow compact_window_walk(uint64_t t, uint64_t m, int groups, bool open_left, bool open_right,
                                                             uint64_t mem, int first, int last) {
  const int lane = threadIdx.x & 63;
  const uint64_t all = (1ull << groups) - 1ull, middle = all & ((1ull << last) - (1ull << first)), in_front = (1ull << first) - 1ull;
  const uint64_t below = (1ull << lane) - 1ull, above = ~((2ull << lane) - 1ull);
  auto has = [](uint64_t mask, int u) { return (mask >> (u & 63) & 1ull) != 0ull; };
  uint64_t head = all, waits = all, self = 0ull;
  for (;;) {
    const uint64_t hf = head & in_front, needed = middle | (hf ? 1ull << (63 - __clzll((long long)hf)) : 0ull);
    if (!(waits & needed)) return {head, self, true};
    const uint64_t hb = head & below, ha = head & above;
    const int l = 63 - __clzll((long long)hb), r = __ffsll((long long)ha) - 1;  // next heads (-1: none)
    const uint64_t hb2 = hb & ~(1ull << (l & 63)), ha2 = ha & (ha - 1ull);
    const int ll = 63 - __clzll((long long)hb2), rr = __ffsll((long long)ha2) - 1;
    const uint64_t listed = has(waits, lane) ? t : ~0ull;  // place in the list; behind all others where the group is not in it any more
    const uint64_t tl = __shfl(t, l & 63), tr = __shfl(t, r & 63), kll = __shfl(listed, ll & 63), krr = __shfl(listed, rr & 63);
    const uint64_t ml = __shfl(m, l & 63), mr = __shfl(m, r & 63);
    // equal times: the one further left is ahead in the list
    const bool known = (hb2 != 0ull || !open_left) && (ha2 != 0ull || !open_right);
    const bool l_first = hb != 0ull && has(waits, l) && tl <= t, ll_first = hb2 != 0ull && kll <= t;
    const bool r_first = ha != 0ull && has(waits, r) && tr < t, rr_first = ha2 != 0ull && krr < t;
    const bool turn = has(waits, lane) && known && !(l_first | ll_first | r_first | rr_first);
    const bool left = !((ha != 0ull ? tr : ~0ull) < (hb != 0ull ? tl : ~0ull));
    const bool join = m + (left ? ml : mr) <= mem;
    const uint64_t turns = __ballot(turn), to_left = __ballot(turn & join & left), to_right = __ballot(turn & join & !left);
    if (turns == 0ull) return {head, self, false};
    const bool takes = ha != 0ull && has(to_left, r);  // the next head joins this one
    if (takes || has(to_right, lane)) {
      t += tr;
      m += mr;
    }
    // (a group that waits is as listed: its right neighbour is the next lane)
    waits &= ~(turns | __ballot(takes) | to_right << 1);
    head &= ~(to_left | to_right << 1);
    self |= to_left;
  }
}

// What becomes of `size` (at most 32) of the n groups from `at` on, by one wave: bits of heads and self, or whole = false.
// load(u, t, m): time and bytes of group u (any u; collective).  Where the window is too small for all of them, for half as
// many at a time.  (Of windows with a middle of 16 groups three in a million are too small on times without an order,
// with a middle of 32 one in a hundred.)
constexpr int kLeastMiddle = 2;
constexpr int kWindowReach = kWindow / 2 + 1;  // groups in front of `at`, and from at + size on, that load may be asked for
template <typename Load> __device__ __forceinline__ CompactWindow compact_range(int at, int size, int n, uint64_t mem, Load load) {
  const int lane = threadIdx.x & 63, end = min(at + size, n);
  CompactWindow all = {0ull, 0ull, true};
#pragma unroll 1
  for (int pos = at; pos < end;) {
    const int start = max(pos - (kWindow - size) / 2 - 1, 0), groups = min(kWindow, n - start), first = pos - start;
    uint64_t t, m;
    load(start + lane, t, m);
    const CompactWindow w = compact_window_walk(t, m, groups, start > 0, start + groups < n, mem, first, first + size);
    if (w.whole) {
      const uint64_t here = (1ull << min(size, end - pos)) - 1ull;
      all.heads |= (w.heads >> first & here) << (pos - at);
      all.self |= (w.self >> first & here) << (pos - at);
      pos += size;
    } else if (size > kLeastMiddle) {
      size /= 2;
    } else {
      all.whole = false;
      break;
    }
  }
  return all;
}

// Where the state of a chain of more than kCompactSmall groups stands in the workspace.  Sums in front of a group of the
// input: A, P, T; those of a walk's groups, by walk's parity: the input group each begins with (first), and what became
// of them, sixteen to a word: heads, self << 16 (or kCompactOpen).
struct CompactState {
  uint64_t *A, *P, *T;
  int32_t *first[2], *turn;
  uint32_t *became[2];
  uint64_t *totals;      // of times, persistent and transient bytes: upper halves, lower halves, flags
  int32_t *left;         // [w]: groups left by walk w, or -1: that walk does not count
};
constexpr int kCompactMostWalks = 24;
constexpr int kCompactChunk = 16;  // groups in the middle of a window
constexpr size_t compact_state_bytes(int G) {
  return 3 * compact_array_bytes(G, 8) + 3 * compact_array_bytes(G, 4) + 2 * compact_array_bytes(G / kCompactChunk, 4) + 9 * 8 +
         4 * (kCompactMostWalks + 1);
}
__host__ __device__ inline CompactState compact_state(void *ws, int G) {
  const size_t a8 = compact_array_bytes(G, 8), a4 = compact_array_bytes(G, 4), aw = compact_array_bytes(G / kCompactChunk, 4);
  char *const b = (char *)ws, *const c = b + 3 * a8, *const d = c + 3 * a4;
  return {(uint64_t *)b, (uint64_t *)(b + a8), (uint64_t *)(b + 2 * a8), {(int32_t *)c, (int32_t *)(c + a4)}, (int32_t *)(c + 2 * a4),
          {(uint32_t *)d, (uint32_t *)(d + aw)}, (uint64_t *)(d + 2 * aw), (int32_t *)(d + 2 * aw + 9 * 8)};
}
static_assert(compact_state_bytes(kCompactSmall + 1) <= compact_workspace_bytes(kCompactSmall + 1) &&
              compact_state_bytes(2049) <= compact_workspace_bytes(2049) && compact_state_bytes(4096) <= compact_workspace_bytes(4096) &&
              compact_state_bytes(16384) <= compact_workspace_bytes(16384) && compact_state_bytes(65535) <= compact_workspace_bytes(65535),
              "what callers have been told holds it");

// The groups that a walk has left of n, from what became of them: expand(rank, group) is called for those whose rank
// (number among the groups left) lies in [lo, hi).  Returns how many are left, or -1 where a chunk is open.
template <int NT, typename Expand>
__device__ __forceinline__ int compact_left(const uint32_t *became, int n, int lo, int hi, int *part, Expand expand) {
  const int words = (n + kCompactChunk - 1) / kCompactChunk, per = (words + NT - 1) / NT;
  const int at = min((int)threadIdx.x * per, words), end = min(at + per, words);
  int sum = 0;
  bool open = false;
#pragma unroll 4
  for (int e = at; e < end; ++e) {
    const uint32_t w = became[e];
    open |= w == kCompactOpen;
    sum += __popc(w & 0xFFFFu);
  }
  const int upto = compact_scan<NT>(sum, part);
  if (upto > lo && upto - sum < hi) {
    int rank = upto - sum;
#pragma unroll 1
    for (int e = at; e < end; ++e)
#pragma unroll 1
      for (uint32_t x = became[e] & 0xFFFFu; x; x &= x - 1u, ++rank)
        if (rank >= lo && rank < hi) expand(rank, e * kCompactChunk + __ffs((int)x) - 1);
  }
  if ((int)threadIdx.x == NT - 1) part[NT / 64] = upto;
  const bool bad = __syncthreads_or(open);
  return bad ? -1 : part[NT / 64];
}

constexpr int kCompactWalkNT = 256;
template <typename Load> __device__ __forceinline__ void compact_chunk(int at, int n, uint64_t mem, uint32_t *became, Load load) {
  const CompactWindow w = compact_range(at, kCompactChunk, n, mem, load);
  if ((threadIdx.x & 63) == 0) became[at / kCompactChunk] = w.whole ? (uint32_t)w.heads | (uint32_t)w.self << 16 : kCompactOpen;
}

// First walk of a long chain, a window to a wave, and, by the first workgroups, the sums in front of its groups.
// Every workgroup of the sums adds up what lies in front of its own 1024 groups again.
constexpr int kCompactSumsPer = 4;
__global__ __launch_bounds__(kCompactWalkNT) void compact_first_kernel(int G, int64_t mem, const int64_t *__restrict__ t_in,
                                                                       const int64_t *__restrict__ p_in,
                                                                       const int64_t *__restrict__ a_in, const CompactState st) {
  constexpr int NT = kCompactWalkNT, PER = kCompactSumsPer, U = 32;  // U: reads in flight
  __shared__ uint64_t part[NT / 64], s_front;
  __shared__ unsigned long long s_sum[2];
  __shared__ int s_flags;
  const int tid = threadIdx.x, lane = tid & 63;
  const int stretches = (G + NT * PER - 1) / (NT * PER), b = blockIdx.x;
  if (b >= 3 * stretches) {
    const int at = ((b - 3 * stretches) * (NT / 64) + (tid >> 6)) * kCompactChunk;
    if (at >= G) return;
    compact_chunk(at, G, (uint64_t)mem, st.became[1], [&](int u, uint64_t &t, uint64_t &m) {
      u = min(u, G - 1);
      t = (uint64_t)t_in[u];
      m = (uint64_t)p_in[u] + (uint64_t)a_in[u];
    });
    return;
  }
  // (the longest ones first)
  const int which = b % 3, stretch = stretches - 1 - b / 3;
  const int64_t *const in = which == 0 ? t_in : which == 1 ? p_in : a_in;
  uint64_t *const out = which == 0 ? st.T : which == 1 ? st.P : st.A;
  const int lo = stretch * NT * PER, hi = min(lo + NT * PER, G);
  if (tid < 2) s_sum[tid] = 0ull;
  if (tid == 0) s_flags = 0;
  // totals as sums of the upper and of the lower halves: neither can overflow before the check
  uint64_t high = 0, low = 0;
  int flags = 0;
  auto take = [&](int64_t v) {
    if (v < 0) flags |= 1;
    else if ((uint64_t)v >= kSumLimit) flags |= 2;
    high += (uint64_t)v >> 32;
    low += (uint32_t)v;
  };
  int64_t mine[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) mine[u] = lo + tid * PER + u < hi ? in[lo + tid * PER + u] : 0;
  for (int g0 = tid; g0 < lo; g0 += U * NT) {
    int64_t v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = in[min(g0 + u * NT, lo - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (g0 + u * NT < lo) take(v[u]);
  }
  const uint64_t upto = compact_scan<NT>((high << 32) + low, part);
  if (tid == NT - 1) s_front = upto;
  uint64_t own = 0;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    take(mine[u]);
    own += (uint64_t)mine[u];
  }
  own = compact_scan<NT>(own, part) - own;
  uint64_t run = s_front + own;  // (behind the barriers of the scan)
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int g = lo + tid * PER + u;
    if (g < hi) out[g] = run;
    run += (uint64_t)mine[u];
    if (g + 1 == G) out[G] = run;
  }
  if (stretch != stretches - 1) return;
  // ---- this workgroup has seen the whole array: what its validation needs ----
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    high += __shfl_xor(high, o);
    low += __shfl_xor(low, o);
    flags |= __shfl_xor(flags, o);
  }
  if (lane == 0) {
    atomicAdd(&s_sum[0], (unsigned long long)high);
    atomicAdd(&s_sum[1], (unsigned long long)low);
    if (flags) atomicOr(&s_flags, flags);
  }
  __syncthreads();
  if (tid < 2) st.totals[3 * which + tid] = s_sum[tid];
  if (tid == 2) st.totals[3 * which + 2] = (uint64_t)s_flags;
}

// Walk w of a long chain, w >= 2; does nothing where the one before does not count (a window was too small, nothing
// merged, or it would have gone to k groups or below: left to compact_resume_kernel).
__global__ __launch_bounds__(kCompactWalkNT) void compact_walk_kernel(int G, int k, int64_t mem, int w, const CompactState st) {
  constexpr int NT = kCompactWalkNT, kRanks = NT / 64 * kCompactChunk;  // of a workgroup
  __shared__ int part[NT / 64 + 1];
  __shared__ int group[kRanks + 2 * kWindowReach];
  const int tid = threadIdx.x, lane = tid & 63;
  const int before = w == 2 ? G : st.left[w - 2];
  const int lo = (int)blockIdx.x * kRanks - kWindowReach, hi = lo + kRanks + 2 * kWindowReach;
  int n = -1;
  if (before >= 0) {
    n = compact_left<NT>(st.became[(w - 1) & 1], before, lo, hi, part, [&](int rank, int u) { group[rank - lo] = u; });
    if (n <= k || n >= before) n = -1;
  }
  if (blockIdx.x == 0 && tid == 0) st.left[w - 1] = n;
  const int at = ((int)blockIdx.x * (NT / 64) + (tid >> 6)) * kCompactChunk;
  if (at >= n) return;
  compact_chunk(at, n, (uint64_t)mem, st.became[w & 1], [&](int u, uint64_t &t, uint64_t &m) {
    int from = G;
    if (u < n) {
      from = group[u - lo];
      if (w > 2) from = st.first[w & 1][from];
    }
    const uint64_t T = st.T[from], M = st.P[from] + st.A[from];
    if (u >= at && u < min(at + kCompactChunk, n)) st.first[(w - 1) & 1][u] = from;
    t = __shfl(T, (lane + 1) & 63) - T;
    m = __shfl(M, (lane + 1) & 63) - M;
  });
}

constexpr int kCompactFewRemoved = 256;  // walks up to here: the merge to stop at is found by comparing all pairs

template <int MODE, int NT> struct CompactShared {
  static constexpr int kMax = CompactShape<MODE>::kMax;
  static constexpr int kWords = (kMax + 31) / 32 + 3;  // a bit per group, an empty word in front and two behind
  using Mask = typename CompactShape<MODE>::Mask;
  uint64_t removed_time[kCompactFewRemoved], part[NT / 64], s_key;
  unsigned long long s_sum[4];
  uint64_t s_last[3];
  Mask look[2][NT];                   // groups a thread has to look at in this round / in the next one
  uint32_t head[kWords], waits[kWords];
  int first[kWords];                  // heads in front of a word of the bit map
  int hist[256], parti[NT / 64], few[64], removed_place[kCompactFewRemoved];
  int s_turns[3], s_flags, s_left, s_few, s_open;
};

// RESUME: n groups are left of a chain whose sums stand in `state`; the input group u begins with is from(u), for
// u <= n (a collective call is not needed).
template <int MODE, int NT, bool RESUME, typename From>
__device__ __forceinline__ void compact_body(
    CompactShared<MODE, NT> &sh, int G, int n, int k, int64_t mem, int walk, int max_walks, const int64_t *__restrict__ t_in, const int64_t *__restrict__ p_in,
    const int64_t *__restrict__ a_in, char *__restrict__ ws, const CompactState &state, From from, int32_t *n_out, int32_t *block_end,
    int64_t *t_out, int64_t *p_out, int64_t *a_out, int32_t *status) {
  constexpr int kMax = CompactShape<MODE>::kMax, kWords = CompactShared<MODE, NT>::kWords;
  using Mask = typename CompactShape<MODE>::Mask;
  constexpr int kFewTurns = 12;  // their neighbours, five each, fill a wave
  static_assert((kMax + NT - 1) / NT <= 8 * (int)sizeof(Mask), "a thread's groups fit its mask");
  extern __shared__ __align__(16) char lds[];
  auto &removed_time = sh.removed_time;
  auto &part = sh.part;
  auto &s_last = sh.s_last;
  auto &s_sum = sh.s_sum;
  auto &s_key = sh.s_key;
  auto &look = sh.look;
  auto &head = sh.head, &waits = sh.waits;
  auto &first = sh.first;
  auto &hist = sh.hist;
  auto &parti = sh.parti;
  auto &few = sh.few;
  auto &removed_place = sh.removed_place;
  auto &s_turns = sh.s_turns;
  int &s_flags = sh.s_flags, &s_left = sh.s_left, &s_few = sh.s_few, &s_open = sh.s_open;
  const int tid = threadIdx.x, lane = tid & 63;
  // arrays of G + 1 entries: times and bytes in front of a group (the bytes of the inputs as well), its
  // first input group; and which turn removed a boundary
  const int entries = RESUME && MODE == 0 ? kCompactSmall : G;
  const size_t a8 = compact_array_bytes(entries, 8), a4 = compact_array_bytes(entries, 4);
  char *const arrays = MODE == 0 ? lds : ws;
  uint64_t *const M = (uint64_t *)arrays;
  uint64_t *const T = (uint64_t *)(MODE == 0 ? lds + a8 : MODE == 1 ? lds : ws + 2 * a8);
  uint64_t *const P = RESUME ? state.P : (uint64_t *)(arrays + (MODE == 0 ? 2 : 1) * a8);
  int32_t *const orig = (int32_t *)(arrays + 3 * a8);
  int32_t *const turn = (int32_t *)(arrays + 3 * a8 + (MODE == 0 ? 1 : 2) * a4);

  if constexpr (RESUME) {
    // (in place where they stand in the workspace: a group never begins in front of its own number)
    for (int u0 = 0; u0 <= n; u0 += NT) {
      const int u = u0 + tid;
      int at = 0;
      uint64_t tv = 0, mv = 0;
      if (u <= n) { at = from(u); tv = state.T[at]; mv = state.P[at] + state.A[at]; }
      __syncthreads();
      if (u <= n) { orig[u] = at; T[u] = tv; M[u] = mv; }
    }
    __syncthreads();
  } else {
  // ---- validation, and the sums in front of every group ----
  if (tid < 4) s_sum[tid] = 0ull;
  if (tid == 0) s_flags = 0;
  __syncthreads();
  {
    // totals as sums of the upper and of the lower halves: neither can overflow before the check
    uint64_t th = 0, tl = 0, mh = 0, ml = 0;
    int flags = 0;
    auto take = [&](int64_t v, uint64_t &hi, uint64_t &lo) -> uint64_t {
      if (v < 0) flags |= 1;
      else if ((uint64_t)v >= kSumLimit) flags |= 2;
      else {
        hi += (uint64_t)v >> 32;
        lo += (uint32_t)v;
        return (uint64_t)v;
      }
      return 0;
    };
    uint64_t none = 0;
    if constexpr (MODE != 2) {
      // An array at a time through LDS: read along the chain, summed up a thread's own stretch at a
      // time (an odd number of entries: no bank conflicts), and copied to the workspace along the
      // chain again.  (Stretches read from memory touch a cache line per lane.)
      const int per = (G + NT - 1) / NT | 1, lo = min(tid * per, G), hi = min(lo + per, G);
      auto in_front = [&](uint64_t *X) {
        __syncthreads();
        uint64_t s = 0;
        for (int g = lo; g < hi; ++g) s += X[g];
        s = compact_scan<NT>(s, part) - s;
        for (int g = lo; g < hi; ++g) { const uint64_t v = X[g]; X[g] = s; s += v; }
        if (lo < hi && hi == G) X[G] = s;
        __syncthreads();
      };
      constexpr int U = 8;  // reads of an input in flight
      uint64_t *const X = T, *const Xp = MODE == 0 ? P : T, *const Xm = MODE == 0 ? M : T;
      for (int g0 = tid; g0 < G; g0 += U * NT) {
        int64_t v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = p_in[min(g0 + u * NT, G - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (g0 + u * NT < G) Xp[g0 + u * NT] = take(v[u], mh, ml);
      }
      in_front(Xp);
      if constexpr (MODE == 1) {
        for (int g = tid; g <= G; g += NT) P[g] = Xp[g];
        __syncthreads();
      }
      for (int g0 = tid; g0 < G; g0 += U * NT) {
        int64_t v[U], w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) { v[u] = p_in[min(g0 + u * NT, G - 1)]; w[u] = a_in[min(g0 + u * NT, G - 1)]; }
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (g0 + u * NT < G) Xm[g0 + u * NT] = take(v[u], none, none) + take(w[u], mh, ml);
      }
      in_front(Xm);
      if constexpr (MODE == 1) {
        for (int g = tid; g <= G; g += NT) M[g] = Xm[g];
        __syncthreads();
      }
      for (int g0 = tid; g0 < G; g0 += U * NT) {
        int64_t v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = t_in[min(g0 + u * NT, G - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (g0 + u * NT < G) X[g0 + u * NT] = take(v[u], th, tl);
      }
      in_front(X);
    } else {
      // NT entries of the three arrays at a time
      uint64_t st = 0, sp = 0, sm = 0;
      for (int g0 = 0; g0 < G; g0 += NT) {
        const int g = g0 + tid, gc = min(g, G - 1);
        const int64_t tv = t_in[gc], pv = p_in[gc], av = a_in[gc];
        uint64_t t = 0, p = 0, m = 0;
        if (g < G) {
          t = take(tv, th, tl);
          p = take(pv, mh, ml);
          m = p + take(av, mh, ml);
        }
        const uint64_t it = compact_scan<NT>(t, part), ip = compact_scan<NT>(p, part), im = compact_scan<NT>(m, part);
        if (g < G) { T[g] = st + it - t; P[g] = sp + ip - p; M[g] = sm + im - m; }
        if (tid == NT - 1) { s_last[0] = it; s_last[1] = ip; s_last[2] = im; }
        __syncthreads();
        st += s_last[0]; sp += s_last[1]; sm += s_last[2];
        __syncthreads();
      }
      if (tid == 0) { T[G] = st; P[G] = sp; M[G] = sm; }
    }
    for (int g = tid; g <= G; g += NT) orig[g] = g;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      th += __shfl_xor(th, o); tl += __shfl_xor(tl, o); mh += __shfl_xor(mh, o); ml += __shfl_xor(ml, o);
      flags |= __shfl_xor(flags, o);
    }
    if (lane == 0) {
      atomicAdd(&s_sum[0], (unsigned long long)th); atomicAdd(&s_sum[1], (unsigned long long)tl);
      atomicAdd(&s_sum[2], (unsigned long long)mh); atomicAdd(&s_sum[3], (unsigned long long)ml);
      if (flags) atomicOr(&s_flags, flags);
    }
    __syncthreads();
    flags = s_flags;
    if (s_sum[0] + (s_sum[1] >> 32) >= (kSumLimit >> 32) || s_sum[2] + (s_sum[3] >> 32) >= (kSumLimit >> 32)) flags |= 2;
    if (flags) {  // (the sums may have wrapped: they are not looked at)
      if (tid == 0) {
        *status = (flags & 1) ? RANNC_DP_PROBLEM_NEGATIVE_INPUT : RANNC_DP_PROBLEM_SUM_OVERFLOW;
        *n_out = 0;
      }
      return;
    }
  }
  }

  bool windows = true;  // none was too small so far (an order along the chain is still one in the next walk)
  for (; n > k && (max_walks <= 0 || walk <= max_walks); ++walk) {  // (n: groups as they stand)
    const int nw = (n + 31) >> 5;  // words of the bit maps that hold groups: 1 .. nw
    if (tid == 0) { s_left = 0; s_open = 0; }
    bool open = true;
    if (windows && n <= kCompactWindows) {
      // ---- the walk, in windows: 32 groups to a wave and turn ----
      if (tid == 0) { head[0] = 0u; head[nw + 1] = 0u; head[nw + 2] = 0u; }
      __syncthreads();
      for (int at = 32 * (tid >> 6); at < n; at += NT / 2) {
        const CompactWindow w = compact_range(at, 32, n, (uint64_t)mem, [&](int u, uint64_t &t, uint64_t &m) {
          const uint64_t Tu = T[min(u, n)], Mu = M[min(u, n)];
          t = __shfl(Tu, (lane + 1) & 63) - Tu;
          m = __shfl(Mu, (lane + 1) & 63) - Mu;
        });
        if (!w.whole) { if (lane == 0) s_open = 1; break; }
        const uint32_t here = (uint32_t)(n - at >= 32 ? ~0u : (1u << (n - at)) - 1u), heads = (uint32_t)w.heads & here;
        if (lane == 0) {
          head[(at + 32) >> 5] = heads;
          atomicAdd(&s_left, __popc(here & ~heads));
        }
        if (lane < 32 && at + lane < n && !(heads >> lane & 1u)) turn[at + lane] = at + lane - ((uint32_t)w.self >> lane & 1u ? 0 : 1);
      }
      __syncthreads();
      open = s_open != 0;
      windows = !open;
      __syncthreads();
      if (tid == 0 && open) s_left = 0;
    }
    if (open) {
    for (int w = tid; w < nw + 3 && w < kWords; w += NT) {
      const uint32_t all = w == 0 || w > nw ? 0u : (w == nw && (n & 31)) ? (1u << (n & 31)) - 1u : ~0u;
      head[w] = all;
      waits[w] = all;
    }
    {
      Mask mine = 0;
      for (int u = tid, b = 0; u < n; u += NT, ++b) mine |= (Mask)1 << b;
      look[0][tid] = mine;
      look[1][tid] = 0;
    }
    if (tid < 3) s_turns[tid] = tid == 2;  // ("the round before the first one had a turn")
    __syncthreads();
    // ---- the walk, in rounds ----
    int merged = 0;
    // one turn: v (and the group it merges with) no longer waits; a merge removes the second one's boundary
    auto take_turn = [&](int v, int l, bool join, bool left) {
      atomicAnd(&waits[(v + 32) >> 5], ~(1u << (v & 31)));
      if (!join) return;
      const int w = left ? l : v + 1, gone = left ? v : v + 1;
      atomicAnd(&waits[(w + 32) >> 5], ~(1u << (w & 31)));
      atomicAnd(&head[(gone + 32) >> 5], ~(1u << (gone & 31)));
      turn[gone] = v;
      ++merged;
    };
    for (int cur = 0, slot = 0;; cur ^= 1, slot = slot == 2 ? 0 : slot + 1) {
      // A: which groups take their turn now, and what it does (nothing is changed but the next round's masks)
      Mask see = look[cur][tid], go = 0, join = 0, left = 0;
      const bool over = s_turns[slot == 0 ? 2 : slot - 1] == 0;  // no turn in the round before: nobody waits any more
      look[cur][tid] = 0;
      if (over) break;
      int turns = 0;
      while (see) {
        const int b = sizeof(Mask) == 8 ? __ffsll((unsigned long long)see) - 1 : __ffs((unsigned)see) - 1;
        see &= see - 1;
        const int v = tid + b * NT;
        if (!compact_bit(waits, v)) continue;
        const CompactAround c = compact_around(head, waits, v, n);
        bool jn, lf;
        if (!compact_turn(T, M, c, v, n, (uint64_t)mem, jn, lf))
          continue;  // whoever is in front looks at this group again after its own turn
        ++turns;
        go |= (Mask)1 << b;
        if (jn) join |= (Mask)1 << b;
        if (lf) left |= (Mask)1 << b;
        auto look_again = [&](bool waiting, int u) {
          if (waiting) atomicOr(&look[cur ^ 1][u % NT], (Mask)1 << (u / NT));
        };
        look_again(c.waits & 1u, c.ll); look_again(c.waits & 2u, c.l);
        look_again(c.waits & 4u, c.r); look_again(c.waits & 8u, c.rr);
        if (jn) look_again(c.waits & (lf ? 16u : 32u), lf ? c.lll : c.rrr);
      }
      if (turns) atomicAdd(&s_turns[slot], turns);
      __syncthreads();
      // B: the turns themselves; what a turn finds around its group is not touched by the others of the round
      const int in_round = s_turns[slot];
      if (tid == 0) { s_turns[slot == 2 ? 0 : slot + 1] = 0; s_few = 0; }
      if (in_round > 0 && in_round <= kFewTurns) {
        // Few turns: whatever can follow follows from them, so the first wave goes on by itself, without
        // barriers, until more turns are possible at a time than it handles (or none).
        __syncthreads();
        while (go) {
          const int b = sizeof(Mask) == 8 ? __ffsll((unsigned long long)go) - 1 : __ffs((unsigned)go) - 1;
          go &= go - 1;
          few[atomicAdd(&s_few, 1)] = tid + b * NT;
        }
        __syncthreads();
        if (tid < 64) {
          int v = lane < in_round ? few[lane] : -1;
          for (;;) {
            // a lane per group to look at; the groups of the first pass are known to take their turn
            CompactAround c;
            bool jn = false, lf = false, act = false;
            if (v >= 0 && compact_bit(waits, v)) {
              c = compact_around(head, waits, v, n);
              act = compact_turn(T, M, c, v, n, (uint64_t)mem, jn, lf);
            }
            __builtin_amdgcn_wave_barrier();
            if (act)  // (a group may have been looked at by two lanes: the first one here takes the turn)
              act = (atomicAnd(&waits[(v + 32) >> 5], ~(1u << (v & 31))) >> (v & 31)) & 1u;
            if (act) take_turn(v, c.l, jn, lf);
            const unsigned long long turns_now = __ballot(act);
            const int many = __popcll(turns_now);
            if (many == 0) break;
            // the waiting groups around each turn are looked at next
            int next[5] = {-1, -1, -1, -1, -1};
            if (act) {
              if (c.waits & 1u) next[0] = c.ll;
              if (c.waits & 2u) next[1] = c.l;
              if (c.waits & 4u) next[2] = c.r;
              if (c.waits & 8u) next[3] = c.rr;
              if (jn && (c.waits & (lf ? 16u : 32u))) next[4] = lf ? c.lll : c.rrr;
            }
            if (many > kFewTurns) {
#pragma unroll
              for (int e = 0; e < 5; ++e)
                if (next[e] >= 0) atomicOr(&look[cur ^ 1][next[e] % NT], (Mask)1 << (next[e] / NT));
              break;
            }
            if (act) {
              const int at = 5 * __popcll(turns_now & ((1ull << lane) - 1ull));
#pragma unroll
              for (int e = 0; e < 5; ++e) few[at + e] = next[e];
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            v = lane < 5 * many ? few[lane] : -1;
          }
        }
        __syncthreads();
        continue;
      }
      while (go) {
        const int b = sizeof(Mask) == 8 ? __ffsll((unsigned long long)go) - 1 : __ffs((unsigned)go) - 1;
        go &= go - 1;
        const int v = tid + b * NT;
        const bool lf = (left >> b) & 1;
        take_turn(v, lf ? compact_prev(head, v) : -1, (join >> b) & 1, lf);
      }
      __syncthreads();
    }
    if (merged) atomicAdd(&s_left, merged);
    __syncthreads();
    }
    const int total = s_left;
    if (total == 0) break;
    // ---- stop at k groups: undo the merges behind the (n-k)-th in list order ----
    int now = n - total;
    if (now < k) {
      auto removed = [&](int u) { return !compact_bit(head, u); };
      if (total <= kCompactFewRemoved) {
        if (tid == 0) s_few = 0;
        __syncthreads();
        for (int u = tid; u < n; u += NT)
          if (removed(u)) {
            const int e = atomicAdd(&s_few, 1), v = turn[u];
            removed_time[e] = T[v + 1] - T[v];
            removed_place[e] = v << 1 | (u != v ? 1 : 0);
          }
        __syncthreads();
        if (tid < total) {
          const uint64_t tv = removed_time[tid];
          const int v = removed_place[tid];  // (one merge to a turn: no two are equal)
          int ahead = 0;
          for (int e = 0; e < total; ++e) ahead += (removed_time[e] < tv) | ((removed_time[e] == tv) & (removed_place[e] < v)) ? 1 : 0;
          const int u = (v >> 1) + (v & 1);
          if (ahead >= n - k) atomicOr(&head[(u + 32) >> 5], 1u << (u & 31));
        }
      } else {
      int want = n - k;  // the want-th smallest (time, position) among the turns that merged, 1-based
      uint64_t found = 0;  // the digits of that place so far: the time, then the position
      uint64_t top = 0;
      for (int u = tid; u < n; u += NT)
        if (removed(u)) { const int v = turn[u]; top = max(top, T[v + 1] - T[v]); }
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) top = max(top, (uint64_t)__shfl_xor(top, o));
      if (tid == 0) s_key = 0;
      __syncthreads();
      if (lane == 0) atomicMax((unsigned long long *)&s_key, (unsigned long long)top);
      __syncthreads();
      const int digits = (64 - __clzll((long long)(s_key | 1ull)) + 7) / 8;  // of the times
      uint64_t at = 0;
      for (int d = digits + 1; d >= 0; --d) {  // the last two digits are those of the position
        const bool pos = d < 2;
        const int sh = 8 * (pos ? d : d - 2);
        if (d == 1) { at = found; found = 0; }  // the time is known; now the position
        for (int e = tid; e < 256; e += NT) hist[e] = 0;
        __syncthreads();
        for (int u = tid; u < n; u += NT) {
          if (!removed(u)) continue;
          const int v = turn[u];
          const uint64_t tv = T[v + 1] - T[v];
          if (pos && tv != at) continue;
          const uint64_t key = pos ? (uint64_t)v : tv;
          if (((key >> sh) >> 8) == found) atomicAdd(&hist[(int)(key >> sh) & 255], 1);
        }
        __syncthreads();
        if (tid < 64) {  // the digit in which the want-th one lies
          int h[4], s = 0;
#pragma unroll
          for (int e = 0; e < 4; ++e) { h[e] = hist[4 * lane + e]; s += h[e]; }
          int before = s;
#pragma unroll
          for (int o = 1; o < 64; o <<= 1) {
            const int w = __shfl_up(before, o);
            if (lane >= o) before += w;
          }
          before -= s;
          if (before < want && want <= before + s) {
            int e = 0;
            while (before + h[e] < want) before += h[e++];
            s_key = ((uint64_t)(unsigned)(want - before) << 32) | (unsigned)(4 * lane + e);
          }
        }
        __syncthreads();
        want = (int)(s_key >> 32);
        found = (found << 8) | (s_key & 255u);
        __syncthreads();
      }
      for (int u = tid; u < n; u += NT) {
        if (!removed(u)) continue;
        const int v = turn[u];
        const uint64_t tv = T[v + 1] - T[v];
        if (tv > at || (tv == at && (uint64_t)v > found)) atomicOr(&head[(u + 32) >> 5], 1u << (u & 31));
      }
      }
      now = k;
      __syncthreads();
    }
    // ---- renumber the heads (every entry moves to the left, a stretch of NT entries at a time) ----
    {
      int c[(kWords + NT - 1) / NT], sum = 0;
#pragma unroll
      for (int e = 0; e < (kWords + NT - 1) / NT; ++e) {  // consecutive words per thread
        const int w = tid * ((kWords + NT - 1) / NT) + e;
        c[e] = w <= nw ? __popc(head[w]) : 0;
        sum += c[e];
      }
      int before = compact_scan<NT>(sum, parti) - sum;
#pragma unroll
      for (int e = 0; e < (kWords + NT - 1) / NT; ++e) {
        const int w = tid * ((kWords + NT - 1) / NT) + e;
        if (w <= nw) first[w] = before;
        before += c[e];
      }
    }
    __syncthreads();
    for (int u0 = 0; u0 <= n; u0 += NT) {
      const int u = u0 + tid;
      int to = -1;
      if (u < n) {
        const uint32_t w = head[(u + 32) >> 5];
        if ((w >> (u & 31)) & 1u) to = first[(u + 32) >> 5] + __popc(w & ((1u << (u & 31)) - 1u));
      } else if (u == n) {
        to = now;
      }
      uint64_t tv = 0, mv = 0;
      int ov = 0;
      if (to >= 0) { tv = T[u]; mv = M[u]; ov = orig[u]; }
      __syncthreads();
      if (to >= 0) { T[to] = tv; M[to] = mv; orig[to] = ov; }
    }
    n = now;
    __syncthreads();
  }
  // ---- result ----
  for (int u = tid; u < n; u += NT) {
    const int from = orig[u], to = orig[u + 1];
    const uint64_t p = P[to] - P[from];
    block_end[u] = to;
    t_out[u] = (int64_t)(T[u + 1] - T[u]);
    p_out[u] = (int64_t)p;
    a_out[u] = (int64_t)(M[u + 1] - M[u] - p);
  }
  if (tid == 0) { *n_out = n; *status = RANNC_DP_PROBLEM_OK; }
}

template <int MODE, int NT>
__global__ __launch_bounds__(NT) void compact_kernel(int G, int k, int64_t mem, int max_walks, const int64_t *__restrict__ t_in,
                                                     const int64_t *__restrict__ p_in, const int64_t *__restrict__ a_in,
                                                     char *__restrict__ ws, int32_t *n_out, int32_t *block_end, int64_t *t_out,
                                                     int64_t *p_out, int64_t *a_out, int32_t *status) {
  __shared__ CompactShared<MODE, NT> sh;
  compact_body<MODE, NT, false>(sh, G, G, k, mem, 1, max_walks, t_in, p_in, a_in, ws, CompactState{}, [](int u) { return u; }, n_out, block_end,
                                t_out, p_out, a_out, status);
}

// What is left to do behind `walks` launched walks of a long chain.
template <int MODE>
__global__ __launch_bounds__(1024) void compact_resume_kernel(int G, int k, int64_t mem, int max_walks, int walks, char *__restrict__ ws,
                                                              const CompactState state, int32_t *n_out, int32_t *block_end, int64_t *t_out,
                                                              int64_t *p_out, int64_t *a_out, int32_t *status) {
  constexpr int NT = 1024;
  extern __shared__ __align__(16) char lds[];
  __shared__ int part[NT / 64 + 1];
  __shared__ union { CompactShared<0, NT> small; CompactShared<MODE, NT> large; } sh;
  const int tid = threadIdx.x;
  const uint64_t *const x = state.totals;
  int flags = (int)(x[2] | x[5] | x[8]);
  if (x[0] + (x[1] >> 32) >= (kSumLimit >> 32) || x[3] + x[6] + ((x[4] + x[7]) >> 32) >= (kSumLimit >> 32)) flags |= 2;
  if (flags) {  // (the sums may have wrapped: they are not looked at)
    if (tid == 0) {
      *status = (flags & 1) ? RANNC_DP_PROBLEM_NEGATIVE_INPUT : RANNC_DP_PROBLEM_SUM_OVERFLOW;
      *n_out = 0;
    }
    return;
  }
  int done = 0, n = G;  // walks that count
  while (done + 1 < walks && state.left[done + 1] >= 0) n = state.left[++done];
  const int32_t *first = done ? state.first[done & 1] : nullptr;
  auto plain = [&](int u) { return u >= n ? G : first ? first[u] : u; };
  int at[2] = {G, G};  // of a thread's groups, where the last walk counts, whose groups nobody has gathered yet
  static_assert(kCompactSmall < 2 * NT, "two of a thread");
  bool picked = false;
  if (done == walks - 1) {
    int *const group = (int *)lds;
    const int left = compact_left<NT>(state.became[walks & 1], n, 0, kCompactSmall, part, [&](int rank, int u) { group[rank] = u; });
    picked = left >= k && left < n && left <= kCompactSmall;
    if (picked) {
#pragma unroll
      for (int e = 0; e < 2; ++e)
        if (e * NT + tid < left) at[e] = plain(group[e * NT + tid]);
      n = left;
      ++done;
    } else if (left > kCompactSmall && left >= k && left < n) {
      // (in rounds again it would take longest: 15 000 groups to 1 000 142 us, so 86; 65 535, one walk only, 566 / 111)
      int32_t *const next = state.first[(done + 1) & 1];
      compact_left<NT>(state.became[walks & 1], n, 0, left, part, [&](int rank, int u) { next[rank] = plain(u); });
      n = left;
      ++done;
      first = next;
    }
    __syncthreads();
  }
  if (n <= kCompactSmall)
    compact_body<0, NT, true>(sh.small, G, n, k, mem, done + 1, max_walks, nullptr, nullptr, nullptr, ws, state,
                              [&](int u) { return picked ? (u < NT ? at[0] : at[1]) : plain(u); }, n_out, block_end, t_out, p_out, a_out,
                              status);
  else
    compact_body<MODE, NT, true>(sh.large, G, n, k, mem, done + 1, max_walks, nullptr, nullptr, nullptr, ws, state, plain, n_out, block_end,
                                 t_out, p_out, a_out, status);
}

constexpr size_t kCompactSmallLds = 3 * compact_array_bytes(kCompactSmall, 8) + 2 * compact_array_bytes(kCompactSmall, 4);

hipError_t launch_compact(int G, int k, int64_t M, int max_walks, const int64_t *t, const int64_t *p,
                          const int64_t *a, void *ws, int32_t *n_out, int32_t *block_end, int64_t *t_out,
                          int64_t *p_out, int64_t *a_out, int32_t *status, hipStream_t st) {
  constexpr size_t kTimesLds = compact_array_bytes(kCompactTimesLds, 8);
  static_assert(kTimesLds >= kCompactSmallLds, "either form of the state");
  auto go = [&](auto width) -> hipError_t {
    constexpr int NT = decltype(width)::value;
    static std::atomic<uint64_t> asked{0};
    const hipError_t e = allow_lds(asked, (const void *)compact_kernel<0, NT>, (int)kCompactSmallLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((compact_kernel<0, NT>), dim3(1), dim3(NT), 3 * compact_array_bytes(G, 8) + 2 * compact_array_bytes(G, 4), st, G, k, M,
                       max_walks, t, p, a, (char *)ws, n_out, block_end, t_out, p_out, a_out, status);
    return hipGetLastError();
  };
  if (G <= kCompactSmall) return G <= 256 ? go(std::integral_constant<int, 256>()) : go(std::integral_constant<int, 1024>());
  // Walks with launches of their own: as long as a walk, which leaves some 35 of a hundred groups, is expected to leave more than
  // k and there are more groups than one workgroup takes as fast.
  int walks = 0;
  for (int left = G; left > kCompactLaunch && left * 2 / 5 > k && walks < kCompactMostWalks && (max_walks <= 0 || walks < max_walks); ++walks)
    left = left * 9 / 25;
  const bool times_lds = G <= kCompactTimesLds;
  static std::atomic<uint64_t> asked[3];
  if (walks == 0) {
    if (times_lds) {
      const hipError_t e = allow_lds(asked[0], (const void *)compact_kernel<1, 1024>, (int)kTimesLds);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL((compact_kernel<1, 1024>), dim3(1), dim3(1024), compact_array_bytes(G, 8), st, G, k, M, max_walks, t, p, a,
                         (char *)ws, n_out, block_end, t_out, p_out, a_out, status);
    } else {
      hipLaunchKernelGGL((compact_kernel<2, 1024>), dim3(1), dim3(1024), 0, st, G, k, M, max_walks, t, p, a, (char *)ws, n_out, block_end,
                         t_out, p_out, a_out, status);
    }
    return hipGetLastError();
  }
  const CompactState state = compact_state(ws, G);
  constexpr int kWaves = kCompactWalkNT / 64, kStretch = kCompactWalkNT * kCompactSumsPer;
  const int blocks = ((G + kCompactChunk - 1) / kCompactChunk + kWaves - 1) / kWaves, stretches = (G + kStretch - 1) / kStretch;
  hipLaunchKernelGGL(compact_first_kernel, dim3(3 * stretches + blocks), dim3(kCompactWalkNT), 0, st, G, M, t, p, a, state);
  for (int w = 2; w <= walks; ++w)
    hipLaunchKernelGGL(compact_walk_kernel, dim3(blocks), dim3(kCompactWalkNT), 0, st, G, k, M, w, state);
  if (times_lds) {
    const hipError_t e = allow_lds(asked[1], (const void *)compact_resume_kernel<1>, (int)kTimesLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(compact_resume_kernel<1>, dim3(1), dim3(1024), std::max(compact_array_bytes(G, 8), kCompactSmallLds), st, G, k, M,
                       max_walks, walks, (char *)ws, state, n_out, block_end, t_out, p_out, a_out, status);
  } else {
    const hipError_t e = allow_lds(asked[2], (const void *)compact_resume_kernel<2>, (int)kCompactSmallLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(compact_resume_kernel<2>, dim3(1), dim3(1024), kCompactSmallLds, st, G, k, M, max_walks, walks, (char *)ws, state,
                       n_out, block_end, t_out, p_out, a_out, status);
  }
  return hipGetLastError();
}

}  // namespace rannc
