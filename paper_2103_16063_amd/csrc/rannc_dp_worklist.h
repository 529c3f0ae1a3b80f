// Rules that cut the rows of a launch of the sorted-merge level kernel into work items: used by the
// kernel that writes the list (setup_kernel), by the host that sizes the grid, and by their model on the
// CPU.
#pragma once

#include "rannc_dp_internal.h"

#include <algorithm>

namespace rannc {

// The rows of one chunk's window that the work list of rows cuts (setup_kernel): n rows from lo on.
struct RunRows { int lo, n; };
__host__ __device__ inline RunRows run_rows(int N, int c, int lo) {
  const int last = 64 * c + 63, hi = last < N - 1 ? last : N - 1;
  return {lo, lo <= hi ? hi - lo + 1 : 0};
}
__host__ __device__ inline int items_of_rows(const RunRows &g, int rows) { return (g.n + rows - 1) / rows; }

// Items of a chunk if every stage of it fits, in items of at most `rows` rows, or passes (the recomputing form's passes
// of 64 stages that fit; the host does not know which ones do): in front of the chunk's diagonal block a row has at
// most one pass, and in the block two rows, p and 64 - p, have one together.
inline int items_at_most(int N, int c, int rows, bool passes) {
  if (!passes) return items_of_rows(run_rows(N, c, 0), rows);
  const int columns = std::min(64, N - 64 * c);
  return (64 * c + rows - 1) / rows + (std::min(columns, 33) + rows - 1) / rows;
}

// What the recomputing form's list knows of a chunk (rannc_dp_kernels.hip, pass_entries): its first row whose
// stages reach the chunk's end, the passes and the items in front of it, and the passes of an item.
struct PassChunk { uint32_t full, base, start, per; };

// Stages that fit in rows w .. i-1 of chunk c, for i up to the chunk's last row + 1; w: the first row with one,
// full: the first row from w on whose stages reach the chunk's end.  esum[i] is the sum of ends[0 .. i-1]
// (below 2^32: N <= 65535; the differences are taken modulo 2^32).
template <typename EP>
__host__ __device__ inline uint32_t stages_before(EP esum, int N, int c, uint32_t w, uint32_t full, uint32_t i) {
  const uint32_t b = 64u * (uint32_t)c, X = b + 64u < (uint32_t)N ? b + 64u : (uint32_t)N;
  const uint32_t up = b > w ? b : w, m = up < i ? up : i;  // rows w .. m-1 begin at b, the others at themselves
  const uint32_t starts = (m - w) * b + (i * (i - 1u)) / 2u - (m * (m - 1u)) / 2u;
  return esum[i < full ? i : full] - esum[w] + (i > full ? (i - full) * X : 0u) - starts;
}

// A row's part in the windows of the chunks: row i is the first whose stages end behind `first` (the last block that
// fits behind the row before it; 0 for row 0) and up to `end`, its own.  window[c] becomes the first row that reaches
// into chunk c, full[c] (before: the row behind the chunk's last) the first whose stages reach the chunk's end.
template <typename WP, typename FP>
__host__ __device__ inline void mark_windows(int N, int nch, int i, uint32_t first, uint32_t end, WP window, FP full) {
  for (int c = i ? (int)(first + 63u) >> 6 : 0; c < nch && 64u * (uint32_t)c < end; ++c) window[c] = i;
  for (int c = i ? (int)(first >> 6) : 0; c < nch; ++c) {
    const uint32_t X = (uint32_t)(64 * c + 64 < N ? 64 * c + 64 : N);
    if (X > end) break;
    if ((i == 0 || X > first) && i < (int)full[c]) full[c] = i;
  }
}
// The window's first row: the marked one (none: any number above 64 c), or, if the chunk's first block fits no device by
// itself, the first later row with a stage; `none` if there is none.
template <typename EP>
__host__ __device__ inline int window_start(EP ends, int N, int c, int marked, int none) {
  if (marked <= 64 * c) return marked;
  const int last = 64 * c + 63 < N - 1 ? 64 * c + 63 : N - 1;
  for (int i = 64 * c + 1; i <= last; ++i)
    if (ends[i] > (uint32_t)i) return i;
  return none;
}

// The item size, in fours, less one: from the sizes 4 (k + 1), k < most, as bits of what holds for them: their items fit the
// grid (listed), take at most one round of workgroups over the launch (round), at least half of one (half), at least
// one and a half (many; only looked at for one large search of the recomputing form, `lone`).
__host__ __device__ inline int pick_item_size(uint32_t listed, uint32_t round, uint32_t half, uint32_t many, int most, bool lone) {
  const uint32_t all = (1u << most) - 1u;
  const int pick = listed & all ? __builtin_ctz(listed & all) : most - 1;
  if ((round >> pick) & 1u) return pick;
  const uint32_t above = all & ~((2u << pick) - 1u);
  if ((round & above) && ((half >> __builtin_ctz(round & above)) & 1u)) return __builtin_ctz(round & above);
  // the largest items that still leave one and a half rounds, by the passes that are really there (the host, which
  // fixes the size for a launch over many searches, cannot see the pruning of a single one)
  if (lone && (many & above)) return 31 - __builtin_clz(many & above);
  return pick;
}

// rows of the searches of a launch if nothing is pruned (every chunk c holds rows 0 .. 64c+63)
inline int64_t merge_launch_rows(const LaunchShape &sh) {
  int64_t all_rows = 0;
  for (int c = 0; c < sh.max_nch; ++c) all_rows += std::min(64 * c + 64, sh.max_N);
  return all_rows * sh.nprob;
}

// Grid of the sorted-merge level kernel = items of the largest search of the launch if nothing is
// pruned.  rows_per_item > 0: in items of that size.  Otherwise in the size that suits the launch
// as a whole: 4-row items (most workgroups) while that leaves the device short of work, larger ones
// (fewer folds and atomics per row) when the launch is full anyway.  The work list then takes the
// smallest item size that fits this grid.
// rows_for_list: what launch_setup is to be given as rows_per_item (the size the host fixed, or -1)
inline int merge_grid_items(const LaunchShape &sh, int rows_per_item, int slots, bool paired, int max_rows, int *rows_for_list) {
  // items of the largest search of the launch if nothing is pruned (a pruned window has no more rows or passes, so no more
  // items at any size)
  auto items_at = [&](int rows) {
    int64_t items = 0;
    for (int c = 0; c < sh.max_nch; ++c) items += items_at_most(sh.max_N, c, rows, paired);
    return std::max<int64_t>(1, items);
  };
  int rows = std::min(rows_per_item, max_rows);
  *rows_for_list = rows;
  if (rows <= 0) {
    const int64_t launch_rows = merge_launch_rows(sh);
    rows = launch_rows >= kMergeRows16From ? 16 : launch_rows >= kMergeRows8From ? 8 : kMergeMinRows;
    // A launch of the recomputing form over several searches with many rounds of workgroups: the
    // largest items that still fill the device one and a quarter times if nothing is pruned, the same
    // size for every search of the launch.  Clearing the tile and the atomics are paid per item (2048 searches of
    // 128 blocks, with earlier forms of the kernel: 16 -> 64 rows 157 -> 115 us per level; one and a quarter rounds
    // 2.13 ms for all levels, two 2.13, three 2.25; over ragged batches of 100 to 1 500 searches within 5 %).
    if (paired && sh.nprob > 1 && items_at(rows) * sh.nprob > slots)
      for (int r = max_rows; r > rows; r -= 4)
        if (4 * items_at(r) * sh.nprob >= 5ll * slots) { rows = r; *rows_for_list = r; break; }
  }
  return (int)items_at(rows);
}

// Workgroups of the sorted-merge level kernel that one compute unit holds at a time (by the
// registers of its four waves, one per SIMD; see the kernel's resource usage).
inline int merge_workgroups_per_cu(int bits, int DP, bool recompute) {
  if (bits == 32) {
    if (recompute) return DP == 64 ? 4 : DP == 32 ? 6 : 8;
    return DP == 64 ? 3 : DP == 32 ? 4 : DP == 16 ? 6 : 8;
  }
  if (recompute) return DP == 64 ? 3 : DP == 32 ? 5 : 8;
  return DP == 64 ? 2 : DP == 32 ? 3 : DP == 16 ? 4 : 8;
}

// One-launch kernel, a workgroup per search and per compute unit: whether its rounds leave little of the device
// idle, a lone round a quarter of it, several a sixteenth of the whole.
inline bool one_launch_rounds_full(int searches, int cus) {
  const int64_t places = ((int64_t)searches + cus - 1) / cus * cus;
  return places == cus ? 4ll * searches >= 3ll * cus : 16ll * searches >= 15 * places;
}

}  // namespace rannc
