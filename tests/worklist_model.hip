// CPU model of the level kernel's work list of rows, on the functions the library itself cuts it with: over every
// chain length, window and item size the items cover the window's rows once, and the list fits the workspace
// and the grid.  (tests/pass_model.hip: the recomputing form's list of passes.)  Prints the first violation.
#include "../paper_2103_16063_amd/csrc/rannc_dp_worklist.h"

#include <cstdio>

using namespace rannc;

static int check(int N) {
  const int max_rows = 64, nch = (N + 63) / 64;
  for (int rows = 1; rows <= max_rows; ++rows) {
    int64_t most = 0;
    for (int c = 0; c < nch; ++c) {
      const int hi = std::min(64 * c + 63, N - 1);
      int64_t most_c = items_of_rows(run_rows(N, c, 0), rows);
      for (int lo = c > 1 ? 64 * c - 66 : 0; lo <= hi; ++lo) {  // windows in front of and inside the block
        const RunRows g = run_rows(N, c, lo);
        const int items = items_of_rows(g, rows), per = items ? (g.n + items - 1) / items : 0;
        most_c = std::max<int64_t>(most_c, items);
        if (per > rows || per > 64) { std::printf("items of %d: %d rows\n", rows, per); return 1; }
        int next = lo;  // as the kernels cut them
        for (int k = 0; k < items; ++k) {
          const int first = g.lo + k * per, take = std::max(std::min(per, g.n - k * per), 1);
          if (first > next || first + take - 1 > hi) {
            std::printf("N %d, chunk %d, window from %d, items of %d: item %d at %d\n", N, c, lo, rows, k, first);
            return 1;
          }
          next = std::max(next, first + take);
        }
        if (next != hi + 1) { std::printf("N %d, chunk %d, window from %d, items of %d: up to %d\n", N, c, lo, rows, next); return 1; }
      }
      most += most_c;
    }
    if (rows % 4 == 0) {
      if (most > max_runs(nch)) { std::printf("N %d, items of %d: %lld listed\n", N, rows, (long long)most); return 1; }
      LaunchShape one = {};
      one.nprob = 1; one.max_N = N; one.max_nch = nch; one.max_D = 64; one.max_S_eff = 2;
      int list = 0;
      const int grid = merge_grid_items(one, rows, 512, false, max_rows, &list);
      if (list != rows || grid < most) { std::printf("N %d, items of %d: grid %d for %lld\n", N, rows, grid, (long long)most); return 1; }
    }
  }
  // the sizes the library takes itself: what the host fixes, or the largest one if the device chooses
  for (int bits : {32, 64})
    for (int Q : {1, 2, 16, 24, 128, 512, 2048})
      for (int DP : {8, 16, 32, 64}) {
        const int slots = 256 * merge_workgroups_per_cu(bits, DP, false);
        LaunchShape sh = {};
        sh.nprob = Q; sh.max_N = N; sh.max_nch = nch; sh.max_D = DP; sh.max_S_eff = 2;
        int list = 0;
        const int grid = merge_grid_items(sh, -1, slots, false, max_rows, &list);
        const int rows = list > 0 ? list : max_rows;
        int64_t items = 0;
        for (int c = 0; c < nch; ++c) items += items_of_rows(run_rows(N, c, 0), rows);
        if (rows > max_rows || grid < items) {
          std::printf("N %d, %d searches, class %d: items of %d, grid %d for %lld\n", N, Q, DP, rows, grid, (long long)items);
          return 1;
        }
      }
  return 0;
}

int main() {
  for (int N = 1; N <= 330; ++N)
    if (check(N)) return 1;
  for (int N : {404, 700, 1000, 1234, 1300, 4096})
    if (check(N)) return 1;
  std::printf("ok\n");
  return 0;
}
