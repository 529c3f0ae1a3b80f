// CPU model of the recomputing level kernel's pass list, on the functions the library itself places the
// stages with: over chain lengths and non-decreasing ends[], the windows that the rows mark are the ones that the
// definition gives, the stages of a chunk are numbered through without a gap, their passes fit the chunk's units of
// the stage-time table (whose region they use), and the items fit the list and the grid; and the item size that the
// kernels pick is the one of the rule as it is stated.  Prints the first violation.
#include "../paper_2103_16063_amd/csrc/rannc_dp_worklist.h"

#include <cstdio>
#include <random>
#include <vector>

using namespace rannc;

static int check(int N, const std::vector<uint32_t> &ends) {
  const int nch = (N + 63) / 64;
  std::vector<uint32_t> esum(N + 1, 0u);
  for (int i = 0; i < N; ++i) esum[i + 1] = esum[i] + ends[i];
  std::vector<int64_t> passes(nch, 0);
  // as the kernels do, and in 16 bits; the rows in any order (every row by its own thread)
  constexpr int kNone = 0x7fffffff;
  std::vector<int> marked(nch, kNone), full_of(nch);
  std::vector<uint16_t> marked16(nch, 0xFFFF), full16(nch);
  for (int c = 0; c < nch; ++c) full16[c] = (uint16_t)(full_of[c] = std::min(64 * c + 64, N));
  for (int k = 0; k < N; ++k) {
    const int i = N % 2 ? (int)((int64_t)k * 2 % N) : N - 1 - k;
    mark_windows(N, nch, i, i ? ends[i - 1] : 0u, ends[i], marked.data(), full_of.data());
    mark_windows(N, nch, i, i ? ends[i - 1] : 0u, ends[i], marked16.data(), full16.data());
  }
  for (int c = 0; c < nch; ++c) {
    const int b = 64 * c, last = std::min(b + 63, N - 1);
    const uint32_t X = (uint32_t)std::min(b + 64, N);
    int w = -1, full = -1;
    for (int i = 0; i <= last && w < 0; ++i)
      if (ends[i] > (uint32_t)std::max(i, b)) w = i;
    const int start = window_start(ends.data(), N, c, marked[c], kNone);
    const int start16 = window_start(ends.data(), N, c, marked16[c] == 0xFFFF ? kNone : (int)marked16[c], kNone);
    if (start != (w < 0 ? kNone : w) || start16 != start) {
      std::printf("N %d, chunk %d: window from %d and %d, not %d\n", N, c, start, start16, w);
      return 1;
    }
    if (w < 0) continue;
    for (full = w; full <= last && ends[full] < X;) ++full;
    if (std::max(full_of[c], w) != full || std::max((int)full16[c], w) != full) {
      std::printf("N %d, chunk %d: full from %d and %d, not %d\n", N, c, full_of[c], (int)full16[c], full);
      return 1;
    }
    uint32_t count = 0;
    for (int i = w; i <= last; ++i) {
      if (stages_before(esum.data(), N, c, w, full, i) != count) { std::printf("N %d, chunk %d, row %d\n", N, c, i); return 1; }
      count += std::min(ends[i], X) - (uint32_t)std::max(i, b);
    }
    if (stages_before(esum.data(), N, c, w, full, last + 1) != count) { std::printf("N %d, chunk %d, end\n", N, c); return 1; }
    passes[c] = (count + 63) / 64;
    if (passes[c] > last + 1) { std::printf("N %d, chunk %d: %lld passes\n", N, c, (long long)passes[c]); return 1; }
  }
  for (int bits : {32, 64}) {
    const int max_rows = merge_max_rows(bits);
    for (int Q : {1, 2, 24, 512})
      for (int DP : {8, 16, 32, 64})
        for (int fixed : {-1, 4, 8, 16, 32, 48, 64}) {
          LaunchShape sh = {};
          sh.nprob = Q; sh.max_N = N; sh.max_nch = nch; sh.max_D = DP; sh.max_S_eff = 2;
          int list = 0;
          const int grid = merge_grid_items(sh, fixed, 256 * merge_workgroups_per_cu(bits, DP, true), true, max_rows, &list);
          // a size the device chooses is at most max_rows, whose items fit the grid
          const int rows = list > 0 ? list : max_rows;
          int64_t items = 0;
          for (int c = 0; c < nch; ++c) items += (passes[c] + rows - 1) / rows;
          if (rows > 64 || items > grid || items > max_pass_items(nch) || kPassItemWords * (1 + items) > max_run_words(nch)) {
            std::printf("N %d, items of %d: %lld on a grid of %d\n", N, rows, (long long)items, grid);
            return 1;
          }
        }
  }
  return 0;
}

// The smallest size whose items fit the grid; if they take more than one round of workgroups, the smallest larger one that
// takes one, if that round fills half the device; else, for one large search of the recomputing form, the largest
// one that leaves one and a half rounds.
static int check_sizes(std::mt19937 &g) {
  for (int n = 0; n < 200000; ++n) {
    const int most = n % 3 == 0 ? 8 : 16, batch = n % 2 ? 1 : 1 + (int)(g() % 40), slots = 1 + (int)(g() % 1600);
    const int max_items = 1 + (int)(g() % 3000);
    const bool passes = n % 5 < 3;
    int count[16], items = (int)(g() % 6000);
    for (int k = 0; k < 16; ++k) {
      count[k] = items;
      items = items * (k + 1) / (k + 2) + (int)(g() % 3);  // (about an eighth of them have one more at a larger size)
    }
    int want = -1;
    for (int k = 0; k < most && want < 0; ++k)
      if (count[k] <= max_items) want = k;
    if (want < 0) want = most - 1;
    if ((long long)count[want] * batch > slots) {
      int one = want + 1;
      while (one < most && (long long)count[one] * batch > slots) ++one;
      if (one < most && 2ll * count[one] * batch >= slots) want = one;
      else if (passes && batch == 1)
        for (int k = most - 1; k > want; --k)
          if (2 * count[k] >= 3 * slots) { want = k; break; }
    }
    uint32_t listed = 0, round = 0, half = 0, many = 0;
    for (int k = 0; k < 32; ++k) {  // (the kernels ask with sixteen lanes' answers twice over)
      const long long then = (long long)count[k % 16] * batch;
      listed |= (uint32_t)(count[k % 16] <= max_items) << k;
      round |= (uint32_t)(then <= slots) << k;
      half |= (uint32_t)(2 * then >= slots) << k;
      many |= (uint32_t)(2 * count[k % 16] >= 3 * slots) << k;
    }
    const int got = pick_item_size(listed, round, half, many, most, passes && batch == 1);
    if (got != want) { std::printf("item size %d, not %d (of %d, %d searches, %d slots)\n", got, want, most, batch, slots); return 1; }
  }
  return 0;
}

int main() {
  std::mt19937 g(5);
  if (check_sizes(g)) return 1;
  for (int N : {1, 2, 3, 31, 63, 64, 65, 88, 127, 128, 129, 200, 251, 320, 701, 1024, 1025, 4096, 65535}) {
    for (int kind = 0; kind < 12; ++kind) {
      std::vector<uint32_t> ends(N);
      const int span = kind == 0 ? N : kind == 1 ? 0 : kind == 2 ? 1 : 1 + (int)(g() % (unsigned)std::min(N, kind % 2 ? 80 : 2000));
      uint32_t at = 0;
      for (int i = 0; i < N; ++i) {
        const uint32_t jitter = kind > 4 && span > 1 ? g() % (unsigned)span : 0;
        at = std::max(at, std::min<uint32_t>(N, i + span - std::min<uint32_t>(jitter, span)));
        if (kind >= 8 && g() % 17 == 0) at = std::max<uint32_t>(at, i);  // a block that fits no device ends every stage
        ends[i] = std::max<uint32_t>(at, i);
      }
      if (check(N, ends)) return 1;
    }
  }
  std::printf("ok\n");
  return 0;
}
