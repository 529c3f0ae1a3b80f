// gfx950 kernel of the compaction step of RaNNC's block-level phase (Sec. III-B) on a chain, and
// its launcher.
#include "rannc_dp_device.h"
#include "rannc_dp_once.h"

namespace rannc {

// ---------------------------------------------------------------------------------------
// Compaction step of the block-level phase (Sec. III-B, last step before the stage-level search),
// on a chain of G groups.  A walk: the groups as they stand are listed by ascending computation
// time (equal times by position); a listed group that is still as listed merges with the
// neighbour whose current time is smaller if the union fits the device memory; the procedure ends
// as soon as k groups are left.  When a walk ends above k groups the groups are listed again by
// their current times and walked again, until k is reached, a walk merges nothing, or the caller's
// limit on the number of walks is met.  The kernel exists so that the chain stays on the device
// between the two phases.  One workgroup.
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
// Bound by latency and by one compute unit's issue rate.  15 000 groups to 32 blocks: 19.7 ms with one
// lane following a sorted list through memory, 0.30 ms here (41 us of it the sums in front of the
// groups, 115 us the first walk); 400 groups 330 -> 60 us; ascending times 20.8 -> 14.6 ms at 15 000
// groups (1 us per turn), 0.37 -> 0.39 ms at 400.
// ---------------------------------------------------------------------------------------
constexpr int kCompactSmall = 1600;     // up to here everything is in LDS and four waves do the work
constexpr int kCompactTimesLds = 16384; // up to here the times (and the bit maps) are in LDS

template <int MODE> struct CompactShape;  // threads; mask of the groups a thread looks after (u = tid + b * threads)
template <> struct CompactShape<0> { static constexpr int NT = 256; using Mask = uint32_t; static constexpr int kMax = kCompactSmall; };
template <> struct CompactShape<1> { static constexpr int NT = 1024; using Mask = uint32_t; static constexpr int kMax = kCompactTimesLds; };
template <> struct CompactShape<2> { static constexpr int NT = 1024; using Mask = uint64_t; static constexpr int kMax = 65535; };

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

template <int MODE>
__global__ __launch_bounds__(CompactShape<MODE>::NT) void compact_kernel(
    int G, int k, int64_t mem, int max_walks, const int64_t *__restrict__ t_in, const int64_t *__restrict__ p_in,
    const int64_t *__restrict__ a_in, char *__restrict__ ws, int32_t *n_out, int32_t *block_end,
    int64_t *t_out, int64_t *p_out, int64_t *a_out, int32_t *status) {
  constexpr int NT = CompactShape<MODE>::NT;
  constexpr int kMax = CompactShape<MODE>::kMax;
  constexpr int kWords = (kMax + 31) / 32 + 3;  // a bit per group, an empty word in front and two behind
  using Mask = typename CompactShape<MODE>::Mask;
  static_assert((kMax + NT - 1) / NT <= 8 * (int)sizeof(Mask), "a thread's groups fit its mask");
  extern __shared__ __align__(16) char lds[];
  __shared__ uint32_t head[kWords], waits[kWords];
  __shared__ Mask look[2][NT];        // groups a thread has to look at in this round / in the next one
  __shared__ int first[kWords];       // heads in front of a word of the bit map
  __shared__ uint64_t part[NT / 64], s_key;
  __shared__ int hist[256], parti[NT / 64], s_flags, s_turns[3], s_left;
  constexpr int kFewTurns = 12;  // their neighbours, five each, fill a wave
  __shared__ int few[64], s_few;
  __shared__ unsigned long long s_sum[4];
  [[maybe_unused]] __shared__ uint64_t s_last[3];
  const int tid = threadIdx.x, lane = tid & 63;
  // arrays of G + 1 entries: times and bytes in front of a group (the bytes of the inputs as well), its
  // first input group; and which turn removed a boundary
  const size_t a8 = compact_array_bytes(G, 8), a4 = compact_array_bytes(G, 4);
  char *const arrays = MODE == 0 ? lds : ws;
  uint64_t *const M = (uint64_t *)arrays;
  uint64_t *const P = (uint64_t *)(arrays + a8);
  int32_t *const orig = (int32_t *)(arrays + 2 * a8);
  int32_t *const turn = (int32_t *)(arrays + 2 * a8 + a4);
  uint64_t *const T = (uint64_t *)(MODE == 1 ? lds : arrays + 2 * a8 + 2 * a4);

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

  int n = G;  // groups as they stand
  for (int walk = 1; n > k && (max_walks <= 0 || walk <= max_walks); ++walk) {
    const int nw = (n + 31) >> 5;  // words of the bit maps that hold groups: 1 .. nw
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
    if (tid == 0) s_left = 0;
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
    const int total = s_left;
    if (total == 0) break;
    // ---- stop at k groups: undo the merges behind the (n-k)-th in list order ----
    int now = n - total;
    if (now < k) {
      auto removed = [&](int u) { return !compact_bit(head, u); };
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

template <int MODE>
static hipError_t compact_go(size_t lds, int G, int k, int64_t M, int max_walks, const int64_t *t, const int64_t *p,
                             const int64_t *a, void *ws, int32_t *n_out, int32_t *block_end, int64_t *t_out,
                             int64_t *p_out, int64_t *a_out, int32_t *status, hipStream_t st) {
  // more than the default 64 KiB of dynamic LDS has to be asked for
  constexpr size_t most = MODE == 0 ? 3 * compact_array_bytes(kCompactSmall, 8) + 2 * compact_array_bytes(kCompactSmall, 4)
                          : MODE == 1 ? compact_array_bytes(kCompactTimesLds, 8) : 0;
  if constexpr (most > 64 * 1024) {
    static std::atomic<uint64_t> asked{0};
    const hipError_t attr = allow_lds(asked, (const void *)compact_kernel<MODE>, (int)most);
    if (attr != hipSuccess) return attr;
  }
  if (lds > most) return hipErrorInvalidValue;
  hipLaunchKernelGGL((compact_kernel<MODE>), dim3(1), dim3(CompactShape<MODE>::NT), lds, st, G, k, M, max_walks, t, p, a,
                     (char *)ws, n_out, block_end, t_out, p_out, a_out, status);
  return hipGetLastError();
}

hipError_t launch_compact(int G, int k, int64_t M, int max_walks, const int64_t *t, const int64_t *p,
                          const int64_t *a, void *ws, int32_t *n_out, int32_t *block_end, int64_t *t_out,
                          int64_t *p_out, int64_t *a_out, int32_t *status, hipStream_t st) {
  const size_t a8 = compact_array_bytes(G, 8), a4 = compact_array_bytes(G, 4);
  if (G <= kCompactSmall)
    return compact_go<0>(3 * a8 + 2 * a4, G, k, M, max_walks, t, p, a, ws, n_out, block_end, t_out, p_out, a_out, status, st);
  if (G <= kCompactTimesLds)
    return compact_go<1>(a8, G, k, M, max_walks, t, p, a, ws, n_out, block_end, t_out, p_out, a_out, status, st);
  return compact_go<2>(0, G, k, M, max_walks, t, p, a, ws, n_out, block_end, t_out, p_out, a_out, status, st);
}

}  // namespace rannc
