// Internal declarations shared by the host orchestration and the gfx950 kernels of the
// stage-level partition search.  Not part of the public ABI (see include/rannc_dp.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rannc {

// ---------------------------------------------------------------------------------------
// Table layout in HBM.
//
// Indices follow the recurrence of Sec. III-C: a stage holds blocks i+1..j (0 <= i < j <= N)
// and runs on r = d - d' replicas.  The level kernel keeps one output column j per lane, so
// the stage-time table is cut into UNITS: unit (i, c) holds predecessor row i for the 64
// columns jj = j-1 in [64c, 64c+63], all D replica counts, as a contiguous block
//
//     cost[(unit(i,c) * D + (r-1)) * 64 + (jj - 64c)]         stage time h(i,j,r), INF if r < rmin
//     rmin[ unit(i,c) * 64      + (jj - 64c)]                 uint8: smallest r whose stage fits
//                                                             memory (the m <= M rule), 255 = none
//
// so that one wavefront reads a unit with D coalesced 256-byte (32-bit values) or 512-byte
// (64-bit) requests out of one contiguous 16 KiB / 32 KiB region.  Row i has units for the
// chunks that can hold a j > i, c = i/64 .. nch-1 (nch = ceil(N/64)); units are numbered row by
// row.  Lanes with jj < i or jj >= N are padding: never written, never read.
//
//     V[(s-1)*(N+1)*DP + j*DP + (d-1)]     level s >= 1, DP = 8/16/32/64 >= D; entries d > D hold 0
//
// The d-fastest layout of V makes the row V[s-1][i][.] one contiguous, wave-uniform read.
// ---------------------------------------------------------------------------------------

// number of units in rows i' < i
__host__ __device__ inline int64_t units_before(int nch, int i) {
  const int64_t g = i >> 6;
  return 64LL * (g * nch - g * (g - 1) / 2) + (int64_t)(i - 64 * g) * (nch - g);
}
__host__ __device__ inline int64_t unit_index(int nch, int i, int c) {
  return units_before(nch, i) + (c - (i >> 6));
}

// upper bound on the number of work items ("runs") of one level: every chunk's rows cut into
// groups of at least 4 rows (chunk c has at most 64(c+1) rows), or, for a search of at most
// kSplitSmallRows rows, into items of one or two rows (split_rows_per_item)
constexpr int kSplitSmallRows = 16384;
__host__ __device__ inline int64_t max_runs(int nch) {
  const int64_t by4 = 8LL * nch * (nch + 1), rows = 32LL * nch * (nch + 1);
  const int64_t small = rows < kSplitSmallRows + nch ? rows : kSplitSmallRows + nch;
  return by4 > small ? by4 : small;
}
// words of the list: one per item and the count, or kPassItemWords per item of at least four passes (a
// chunk has at most 64c + 33)
constexpr int kPassItemWords = 8;
__host__ __device__ inline int max_pass_items(int nch) { return 8 * nch * (nch - 1) + 9 * nch; }
__host__ __device__ inline int64_t max_run_words(int nch) {
  const int64_t passes = kPassItemWords * (1 + (int64_t)max_pass_items(nch));
  return passes > max_runs(nch) + 1 ? passes : max_runs(nch) + 1;
}

// Sorted-merge level kernel: waves per work item; a wave takes 1, 2, 4, ... of the item's rows.  The
// host sizes the grid for items of 16 rows when the searches of a launch together hold at least
// kMergeRows16From rows (unpruned), of 8 from kMergeRows8From, of 4 below.
constexpr int kMergeWaves = 4;
constexpr int kMergeMinRows = 4;
// Largest work item of the recomputing form, in passes.  64-bit values, 32 / 64 passes: 600 searches of 200 blocks at 64
// devices 1802 / 1689 us a call, at 16 devices 552 / 547; 200 of them at 16 devices 267 / 273, at 8 209 / 215; single
// searches the same.
__host__ __device__ constexpr int merge_max_rows(int bits) { return bits == 64 ? 32 : 64; }
constexpr int kMergeRows8From = 6144;
constexpr int kMergeRows16From = 16384;
// From this many rows (unpruned) in a launch on, a search without a communication term has its
// stage times recomputed in the level kernel (RANNC_DP_ALGO_AUTO), which also saves building their
// table.  Measured per call, table against recomputed: 1024 blocks at 64 devices 357 / 305 us where
// memory binds and 773 / 466 us where it does not, 701 at 48 261 / 211, 400 (1 744 rows) at 64 193 / 154, at 16
// 120 / 109.  The line was drawn with kernels that were level at 1 000 rows; with these the recomputing form is ahead
// below it as well: 300 blocks (940 rows) at 64 179 / 144, 251 at 24 124 / 110, 96 at 16 105 / 95.
constexpr int kRecomputeRowsFrom = 1024;

__host__ __device__ inline int dp_class(int D) { return D <= 8 ? 8 : D <= 16 ? 16 : D <= 32 ? 32 : 64; }

struct ProblemDev {
  int32_t N, D, S_eff, MB;
  int32_t DP;   // padded device dimension of a V row
  int32_t nch;  // 64-wide column chunks
  int32_t bits; // 32 or 64: width of the values in cost and V
  int32_t q;    // index of the problem in the caller's batch (outputs go there)
  int64_t M;
  int64_t time_limit;          // limits.max_total_time_ns
  const int64_t *t, *p, *a;    // caller's inputs (DEVICE), N entries each
  const int64_t *tb;           // caller's backward block times (DEVICE), or null: one time per block (min-max search)
  int64_t *TB;                 // prefix sums of tb, N+1 entries; null when tb is null
  void *costb;                 // backward stage-time table, layout of cost; null when tb is null
  void *VF, *VB;               // largest forward / backward stage time of the plan behind each V entry
                               // (layout of V); null when tb is null
  void *keys;                  // kSplitKeyTables x [DP][N+1] uint64: packed (value, i) winners of a level;
                               // only with tb and a time bound the packing can hold, else null
  const int64_t *o;            // caller's bytes per cut (DEVICE), N entries, or null: no communication term
  int64_t bw;                  // bandwidth in bytes per microsecond (>= 1 when o is given)
  int64_t *T, *P, *A;          // prefix sums, N+1 entries each
  int64_t *C;                  // C[j] = ns to send the bytes of the cut after block j at one replica
                               // (C[0] = C[N] = 0), N+1 entries; null when o is null
  uint8_t *rmin;
  void *cost;
  void *V;
  uint8_t *ufit;               // per unit: 1 if any of its stages fits for some r <= D
  uint32_t *ends;              // recomputing level kernel (else null): N entries ends[], then N + 1 running sums of
                               // them (pass_entries; they use the words that C would)
  int32_t *wlo;                // [nch] smallest row i with a stage (i, j in chunk) that fits for some
                               // r <= D; 0x7fffffff if none; behind it, with ends, four words per chunk (PassChunk)
  int32_t *runs;               // runs[0] = count, then ((rows - 1) << 26 | c << 16 | first row) per work item;
                               // with ends, from word kPassItemWords on, kPassItemWords words per work item: first
                               // pass, c | (passes - 1) << 16, first and last row << 16 of its first four passes
  int32_t *status;             // RANNC_DP_PROBLEM_*
  int64_t *res;                // res[0] = opt (int64, INT64_MAX if none), res[1] = n_stages
};

// Result arrays of a batch, on the device and (h_*, or null) in pinned host memory; h_flag[q] = seq is
// stored behind the results of search q.
struct PlanResults {
  int64_t *d_opt, *d_est;
  int32_t *d_n_stages, *d_status, *d_stage_end, *d_replicas;
  int64_t *h_opt, *h_est;
  int32_t *h_n_stages, *h_status, *h_stage_end, *h_replicas;
  uint64_t *h_flag, seq;
};

// Outer driver: what Algorithm 2's loops over a solved batch need, and where the result goes (rec: 6
// int64 {q, S, bad status, 0, V, estimate}, then 2*stride int32 of plan; device memory or pinned host
// memory; flag (or null) = seq is stored behind it).
struct FormStageIn {
  int Q, N, devices_per_node;
  int64_t *rec;
  uint64_t *flag, seq;
};

struct LaunchShape {
  int nprob;     // problems in the launch (blockIdx.z runs over them)
  int max_N;     // largest N among them
  int max_nch;   // largest nch among them
  int max_D;
  int max_S_eff;
  int64_t wide_rows;  // rows (unpruned) of the searches of its widest device-count class
  int wide_chunks;    // and their column chunks
};

// Kernel launchers (rannc_dp_kernels.hip, rannc_dp_split.hip, rannc_dp_compact.hip).  All enqueue on `st` and return the launch status.
// `probs` points at the first ProblemDev of the launch; problems of one launch are contiguous.
// parts: 1 = fits-in-memory tables (rmin, ufit) and level 1 of V, 2 = the stage-time table, 3 = both
hipError_t launch_build(const ProblemDev *probs, const LaunchShape &sh, int bits, int DP, int parts, hipStream_t st);
// launch_build for the searches whose level kernel recomputes the stage times: parts = 1, and the entries of the
// pass list that launch_setup has laid out
hipError_t launch_build_passes(const ProblemDev *probs, const LaunchShape &sh, int bits, int DP, hipStream_t st);
// prefix sums, validation, initial V, windows and work list of the searches of a launch.
// rows_per_item: > 0 fixed, -1 chosen on the device for the sorted-merge kernel (the smallest item size
// whose item count fits max_items)
// slots: workgroups of the level kernel that the device holds at a time
// paired: the list for the level kernel that recomputes the stage times (passes of stages that fit)
// src: the descriptors, in device memory (probs itself) or in pinned host memory the device can read;
// the launch then also stores them to probs.  host_one: for a launch over one search, its descriptor in
// host memory (passed by value instead), or null
hipError_t launch_setup(const ProblemDev *src, ProblemDev *probs, int Q, int rows_per_item, int max_items, int slots, bool paired,
                        int max_rows, const ProblemDev *host_one, hipStream_t st);
// launch_setup and launch_build (parts 1 or 3), and with the split objective launch_split_level1, as one launch
// (where can_prepare says so)
bool can_prepare(const LaunchShape &sh);
hipError_t launch_prepare(const ProblemDev *src, ProblemDev *probs, const LaunchShape &sh, int bits, int DP, int parts,
                          int rows_per_item, int max_items, int slots, bool paired, int max_rows, bool split, bool comm,
                          const ProblemDev *host_one, hipStream_t st);
int merge_rows_per_item(int rows_per_wave);
// recompute: the level kernel computes the stage times from the prefix sums instead of reading
// their table (where can_recompute_times says so)
// items: merge_grid_items of the launch, the value launch_setup was given
// host_one: for a launch over one search, a host copy of its descriptor (passed by value), or null
hipError_t launch_level_merge(const ProblemDev *probs, const LaunchShape &sh, int bits, int s,
                              bool recompute, int items, const ProblemDev *host_one, hipStream_t st);
// whole search of problems with N <= small_max_blocks() in one launch, one workgroup each
int small_max_blocks();
// direct: the stage times are recomputed from the prefix sums and no table is written (only where
// small_can_recompute says so, and only for searches without a communication term);
// max_total_time: the largest total time a search of the launch can have without being flagged
bool small_can_recompute(int bits, int DP, int64_t max_total_time);
// whether the level kernel can recompute the stage times
bool can_recompute_times(int bits, int64_t max_total_time);
// src: as in launch_setup.  results: the launch also recovers the plans of its searches and writes them there
// (and to the host's mirror with h_flag), or null.  cus: compute units of the device
hipError_t launch_solve_small(const ProblemDev *src, ProblemDev *probs, int Q, int bits, int DP, bool direct, int64_t *d_opt,
                              int32_t *d_n_stages, int64_t *d_est, int32_t *d_status, const ProblemDev *host_one,
                              int plan_stride, const PlanResults *results, int cus, hipStream_t st);
hipError_t launch_level_scan(const ProblemDev *probs, const LaunchShape &sh, int bits, int s,
                             int write_v, int32_t *arg_i, int32_t *arg_d, hipStream_t st);
// Algorithm 1 with forward and backward maxima carried separately (problems with tb != null):
// level 1 from the two tables, then one launch per level s >= 2.  write_v = 0: only the argmin
// arrays (canonical layout of ONE problem) are written.
hipError_t launch_split_level1(const ProblemDev *probs, const LaunchShape &sh, int bits, hipStream_t st);
hipError_t launch_level_split(const ProblemDev *probs, const LaunchShape &sh, int bits, int s, int write_v,
                              int32_t *arg_i, int32_t *arg_d, hipStream_t st);
// needs the key table and the work list made by launch_setup(..., split_rows_per_item(), ...); with
// 64-bit tables only for time bounds up to kSplitPackedMax (the packed winner holds 42 value bits)
constexpr int64_t kSplitPackedMax = (1LL << 42) - 2;
// rows per work item of a launch; the level launcher is given the same value
int split_rows_per_item(const LaunchShape &sh, int DP);
constexpr int kSplitMaxRows = 16;
// key tables of a search: of the level in flight, of the one before, and one that is cleared for the next
constexpr int kSplitKeyTables = 3;
hipError_t launch_level_split_fast(const ProblemDev *probs, const LaunchShape &sh, int bits, int DP, int s,
                                   int rows_per_item, hipStream_t st);
// (any of the outputs may be null: the choice itself is kept with the search)
hipError_t launch_select(const ProblemDev *probs, int Q, int64_t *d_opt, int32_t *d_n_stages,
                         int64_t *d_est, int32_t *d_status, hipStream_t st);
// d_levels: per problem (caller's order) the exact stage count to recover, 0 = the best one; or null
// lds_bytes > 0: the kernel that first copies what the walk reads into LDS; every problem of the
// launch must be a min-max search with traceback_lds_bytes(...) <= lds_bytes <= kTracebackLdsMax
constexpr int kTracebackLdsMax = 150 * 1024;
int64_t traceback_lds_bytes(int N, int DP, int S_eff, int bits);
// form_stage != null: the outer driver's loops over the values of the batch are run first, and only the
// plan of the search they choose is recovered, by one workgroup
// results != null: choose = the stage count of every search is chosen here (launch_select is not
// needed); h_flag != null = the results also go to the host's mirror
hipError_t launch_traceback(const ProblemDev *probs, int Q, int plan_stride, int32_t *d_stage_end,
                            int32_t *d_replicas, const int32_t *d_levels, int64_t lds_bytes,
                            const FormStageIn *form_stage, const PlanResults *results, bool choose, hipStream_t st);
hipError_t launch_level_values(const ProblemDev *probs, int Q, int stride, int64_t *d_out, hipStream_t st);
// Min-max searches without send times answered without their tables (rannc_dp_reach.hip): optimum, fewest stages,
// plan, by one workgroup each.  Copies of the inputs go to `save` (times, persistent, transient bytes; there is room for five arrays
// of `blocks` entries, the searches one after the other), from which the tables can be made later.
constexpr int kReachMaxBlocks = 4096;   // the sums of a search are held in LDS
constexpr int kReachUndecided = -1;     // status of a search that is left to the tables
struct ReachIn {
  int32_t N, D, S, MB;
  int64_t M;
  int64_t first;  // index of its first block in the input arrays
  int64_t bw;     // bytes per microsecond between stages, where the batch has send times
};
struct ReachArgs {
  const int64_t *t, *p, *a, *o, *tb;  // DEVICE; o, tb: of launch_bound, or null
  int64_t *save;
  int64_t blocks, first;  // of the batch: entries of a saved array, index of the first block
  int64_t time_limit;
  int plan_stride;
  PlanResults results;
};
// src: the descriptors in memory the device can read (pinned); host_one: of a launch over one search, by value, or null
hipError_t launch_reach(const ReachIn *src, const ReachIn *host_one, int Q, const LaunchShape &sh, const ReachArgs &args, hipStream_t st);
// The same for searches with send times, or with forward and backward maxima apart (rannc_dp_bound.hip); bytes per cut and
// backward times are saved as the fourth and fifth array.
constexpr int kBoundMaxBlocks = 1024;  // (the LDS: up to five arrays of sums, and room for the levels)
hipError_t launch_bound(const ReachIn *src, const ReachIn *host_one, int Q, const LaunchShape &sh, const ReachArgs &args, hipStream_t st);
// The outer driver's searches, each the smallest stage count of lo..hi with a plan of exactly so many stages on D devices,
// and that plan (rannc_dp_form.hip): one workgroup each, results in pinned host memory.
constexpr int kFormMaxBlocks = 1024, kFormMaxSpare = 8;  // spare: devices of a node
constexpr int kFormWide = 256;  // split objective: rows of a level
struct FormIn {
  int32_t D, lo, hi, group;  // group: searches of as many nodes; of a smaller group a plan is taken first
  int64_t b;                 // samples of a microbatch
};
struct FormArgs {
  const int64_t *t, *p, *a, *o, *tb;  // per sample, in memory the device can read; o, tb: or null
  const FormIn *pairs;
  int64_t M, bw;
  int N, searches, plan_stride, cells;
  uint64_t *found;      // pinned host memory, a word per search: results.seq << 16 | group << 8 | stages of its plan
  PlanResults results;  // h_opt, h_n_stages (of a search left to the tables: the stage count that is open), h_status,
                        // h_stage_end, h_replicas, h_flag
};
// spare: largest D - lo + 1 of the pairs
hipError_t launch_form(int Q, int spare, const FormArgs &args, hipStream_t st);
// The inputs of all Q searches of the outer driver, one after the other, from its own per sample: five arrays of N entries (times,
// persistent, transient bytes, bytes per cut, backward times) to as many of Q * N; samples[q] of search q.
hipError_t launch_form_inputs(const int64_t *per_sample, const int64_t *samples, int64_t *out, int N, int Q, bool comm, bool split, hipStream_t st);
// compaction step of the block-level phase on a chain of G groups.  Chains of up to kCompactLds groups are held in the LDS of one
// workgroup; longer ones keep arrays in the workspace: three of 8 bytes and three of 4 of G + 1 entries, and a word per
// sixteen groups for what the last two walks have left (compact_state in rannc_dp_compact.hip)
constexpr size_t compact_array_bytes(int G, int entry) { return ((size_t)(G + 1) * entry + 255) / 256 * 256; }
// (the size callers have been given since the first version of the step; more than the arrays need)
constexpr int kCompactLds = 1600;
constexpr size_t compact_order_bytes(int G) {
  size_t P = 1;
  while (P < (size_t)G) P <<= 1;
  return (P * 4 + 255) / 256 * 256;
}
constexpr size_t compact_workspace_bytes(int G) {
  const size_t a8 = (((size_t)G * 8 + 255) / 256) * 256, a4 = (((size_t)G * 4 + 255) / 256) * 256;
  return 2 * compact_order_bytes(G) + (G > kCompactLds ? 3 * a8 + 4 * a4 : 0);
}
hipError_t launch_compact(int G, int k, int64_t M, int max_walks, const int64_t *t, const int64_t *p,
                          const int64_t *a, void *ws, int32_t *n_out, int32_t *block_end, int64_t *t_out,
                          int64_t *p_out, int64_t *a_out, int32_t *status, hipStream_t st);
hipError_t launch_export(const ProblemDev *prob, int which, int bits, void *d_dst, hipStream_t st);


}  // namespace rannc
