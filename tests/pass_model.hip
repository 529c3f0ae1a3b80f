// CPU model of the recomputing level kernel's pass list, on the functions the library itself places the
// stages with: over chain lengths and non-decreasing ends[], the stages of a chunk are numbered through
// without a gap, their passes fit the chunk's units of the stage-time table (whose region they use), and the
// items fit the list and the grid.  Prints the first violation.
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
  for (int c = 0; c < nch; ++c) {
    const int b = 64 * c, last = std::min(b + 63, N - 1);
    const uint32_t X = (uint32_t)std::min(b + 64, N);
    int w = -1, full = -1;
    for (int i = 0; i <= last && w < 0; ++i)
      if (ends[i] > (uint32_t)std::max(i, b)) w = i;
    if (w < 0) continue;
    for (full = w; full <= last && ends[full] < X;) ++full;
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

int main() {
  std::mt19937 g(5);
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
