// CPU model of the level kernel's work list, on the functions the library itself cuts it with: over every
// chain length, window and item size, no item holds more rows than the kernel's array, the items cover the
// window's rows once, and the list fits the workspace and the grid.  Prints the first violation.
#include "../paper_2103_16063_amd/csrc/rannc_dp_worklist.h"

#include <cstdio>

using namespace rannc;

static int check(int bits, bool paired, int N) {
  const int max_rows = paired ? merge_max_rows(bits) : 64, nch = (N + 63) / 64;
  for (int rows = 1; rows <= max_rows; ++rows) {
    int64_t most = 0;
    for (int c = 0; c < nch; ++c) {
      int64_t most_c = 0;
      const int hi = std::min(64 * c + 63, N - 1);
      for (int lo = c > 1 ? 64 * c - 66 : 0; lo <= hi; ++lo) {  // windows in front of and inside the block
        const RunSegments g = run_segments(N, c, lo, paired);
        const int n0 = items_of_rows(g, rows), n1 = items_of_pairs(g, rows, max_rows);
        most_c = std::max<int64_t>(most_c, n0 + n1);
        const int per0 = n0 ? (g.n0 + n0 - 1) / n0 : 0, per1 = n1 ? (g.n1 + n1 - 1) / n1 : 0;
        if (paired && (per0 > merge_item_rows(bits) || 2 * per1 > merge_item_rows(bits))) {
          std::printf("%d bits, N %d, chunk %d, window from %d, items of %d: %d rows, %d pairs staged in %d\n", bits, N, c, lo,
                      rows, per0, per1, merge_item_rows(bits));
          return 1;
        }
        if (per0 > 64 || per1 > 64) { std::printf("item word: %d %d\n", per0, per1); return 1; }
        // every row of the window is a listed row or the partner 64c + 64 - p of a listed pair p = 1 .. 31
        for (int r = lo; r <= hi; ++r) {
          const bool first = (r >= g.lo0 && r < g.lo0 + g.n0) || (r >= g.lo1 && r < g.lo1 + g.n1);
          const int p = 128 * c + 64 - r;  // the row whose partner r is
          const bool second = paired && r >= 64 * c && p - 64 * c >= 1 && p - 64 * c <= 31 && p >= g.lo1 && p < g.lo1 + g.n1;
          if (!first && !second) {
            std::printf("%d bits, N %d, chunk %d, window from %d: row %d in no item\n", bits, N, c, lo, r);
            return 1;
          }
        }
      }
      // (windows further in front only have more rows in the first segment)
      const RunSegments all = run_segments(N, c, 0, paired);
      most += std::max<int64_t>(most_c, items_of_rows(all, rows) + items_of_pairs(all, rows, max_rows));
    }
    if (rows % 4 == 0) {
      if (most > max_runs(nch)) { std::printf("N %d, items of %d: %lld listed\n", N, rows, (long long)most); return 1; }
      LaunchShape one = {};
      one.nprob = 1; one.max_N = N; one.max_nch = nch; one.max_D = 64; one.max_S_eff = 2;
      int list = 0;
      const int grid = merge_grid_items(one, rows, 512, paired, max_rows, &list);
      if (list != rows || grid < most) { std::printf("N %d, items of %d: grid %d for %lld\n", N, rows, grid, (long long)most); return 1; }
    }
  }
  // the sizes the library takes itself: what the host fixes, or the largest one if the device chooses
  for (int Q : {1, 2, 16, 24, 128, 512, 2048})
    for (int DP : {8, 16, 32, 64}) {
      const int slots = 256 * merge_workgroups_per_cu(bits, DP, paired);
      LaunchShape sh = {};
      sh.nprob = Q; sh.max_N = N; sh.max_nch = nch; sh.max_D = DP; sh.max_S_eff = 2;
      int list = 0;
      const int grid = merge_grid_items(sh, -1, slots, paired, max_rows, &list);
      const int rows = list > 0 ? list : max_rows;
      int64_t items = 0;
      for (int c = 0; c < nch; ++c) {
        const RunSegments g = run_segments(N, c, 0, paired);
        items += items_of_rows(g, rows) + items_of_pairs(g, rows, max_rows);
      }
      if (rows > max_rows || grid < items) {
        std::printf("N %d, %d searches, class %d: items of %d, grid %d for %lld\n", N, Q, DP, rows, grid, (long long)items);
        return 1;
      }
    }
  return 0;
}

int main() {
  for (int bits : {32, 64})
    for (int paired : {0, 1}) {
      for (int N = 1; N <= 330; ++N)
        if (check(bits, paired != 0, N)) return 1;
      for (int N : {404, 700, 1000, 1234, 1300, 4096})
        if (check(bits, paired != 0, N)) return 1;
    }
  std::printf("ok\n");
  return 0;
}
