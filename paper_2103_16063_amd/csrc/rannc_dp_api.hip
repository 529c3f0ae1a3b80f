// Host orchestration behind the C ABI of include/rannc_dp.h: argument checks, workspace
// layout, and the sequence of kernel launches of one search (prefix sums and tables, one
// launch per DP level, final selection, plan recovery).  Nothing here computes any part of the
// recurrence; that is all in the kernel files (rannc_dp_kernels.hip, rannc_dp_split.hip; without tables rannc_dp_reach.hip,
// rannc_dp_bound.hip, rannc_dp_form.hip; rannc_dp_compact.hip).
#include "../../include/rannc_dp.h"
#include "rannc_dp_internal.h"
#include "rannc_dp_worklist.h"

#include <algorithm>
#include <atomic>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

using rannc::LaunchShape;
using rannc::ProblemDev;

namespace {

constexpr size_t kAlign = 256;
constexpr int64_t kNarrowMax = 4294967294LL;  // largest total time a 32-bit table can hold
constexpr int kStagingSlots = 2;

inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

struct Sizes {  // bytes of one problem's regions inside the workspace
  size_t prefix, wlo, runs, ufit, misc, rmin, cost, V, keys;
  bool split;  // split objective: a fifth prefix array, a second stage-time table, two more value tables
  size_t total() const {
    return prefix * (split ? 5 : 4) + wlo + runs + ufit + misc + rmin + cost * (split ? 2 : 1) +
           V * (split ? 3 : 1) + keys;
  }
};

// A batch of few searches can run as ONE group: its V rows are padded to the widest device-count class of
// the batch, so that every launch covers all of its searches.  A level then costs one launch instead of
// one per class (3 us of the host each) and no stream is forked and joined (20 us a class).  The price is
// paid by the narrower searches: their merges are as wide as their own level needs anyway, but they run
// in the wide kernel, with fewer workgroups per compute unit and longer rows to copy and clear.  It
// grows with their rows, the saving with the number of classes.  So a batch is a group while the narrower
// searches have at most this many rows (unpruned): the first number for a batch of two classes, the second
// more for every further class.  Measured over 550 batches of 2 to 64 searches of 16 to 1024 blocks, one
// group / class by class: 4 x 160 blocks at 8 and 4 at 64 devices 154 / 187 us, 24 searches of the
// outer driver at 384 blocks 334 / 372, 16 x 256 at each of 8, 16 and 32 221 / 277, 2 x 96 at each class
// 141 / 269; beyond the lines 15 x 400 at 8 and one at 32 261 / 180, 2 x 1024 at each class 1230 / 753, 63 x
// 1024 at 8 and one at 64 7350 / 1085.  With 64-bit values or the split objective the wide kernels
// are slower still: 4 x 200 at 8 and 4 at 64, 64-bit, 290 / 246; 15 x 128 at 16 and one at 32, split, 412 / 295.
constexpr int kOneGroupMax = 64;  // searches
struct GroupRows { int two, more; };
constexpr GroupRows kGroupRows[3][3] = {  // widest class: 16, 32, 64 devices
    {{20480, 0}, {10240, 25600}, {5632, 1792}},  // 32-bit values
    {{10240, 0}, {7168, 7168}, {1408, 1408}},    // 64-bit values
    {{3584, 0}, {1792, 1792}, {768, 768}},       // split objective
};

int64_t search_rows(int N) {  // chunk c holds rows 0 .. 64c+63
  const int64_t full = N / 64;
  return 32 * full * (full + 1) + (N % 64 ? N : 0);
}

// the class whose width all searches of the batch would run at as a group, or 0: too many searches
int widest_class(const rannc_dp_batch_t *b) {
  if (b->n_problems > kOneGroupMax) return 0;
  int D = 1;
  for (int q = 0; q < b->n_problems; ++q) D = std::max(D, b->n_devices[q]);
  return rannc::dp_class(D);
}

// the class whose width all searches of the batch run at, or 0: each at that of its own class
int group_dp(const rannc_dp_batch_t *b, int bits, bool split) {
  const int widest = widest_class(b);
  int64_t narrower = 0;
  int classes = 0;  // as a mask, 8 | 16 | 32 | 64
  for (int q = 0; q < b->n_problems && widest; ++q) {
    const int own = rannc::dp_class(b->n_devices[q]);
    classes |= own;
    if (own < widest) narrower += search_rows(b->n_blocks[q]);
  }
  if (classes == widest) return widest;
  const GroupRows &most = kGroupRows[split ? 2 : bits == 64 ? 1 : 0][widest == 16 ? 0 : widest == 32 ? 1 : 2];
  return narrower <= most.two + (int64_t)(__builtin_popcount(classes) - 2) * most.more ? widest : 0;
}

// false on arithmetic overflow
bool problem_sizes(int N, int D, int DP, int S_eff, int bits, bool split, bool packed, Sizes *o) {
  const int nch = (N + 63) / 64;
  const size_t esz = bits / 8;
  const unsigned __int128 rows = (unsigned __int128)rannc::units_before(nch, N) * 64;
  const unsigned __int128 cost = rows * (unsigned)D * esz;
  const unsigned __int128 V = (unsigned __int128)S_eff * (unsigned)(N + 1) * (unsigned)DP * esz;
  if (cost > ((unsigned __int128)1 << 46) || V > ((unsigned __int128)1 << 46)) return false;
  o->prefix = align_up((size_t)(N + 1) * 8);
  o->wlo = align_up((size_t)nch * 20);  // the windows, and four words per chunk for the recomputing level kernel
  o->runs = align_up((size_t)rannc::max_run_words(nch) * 4);
  o->ufit = align_up((size_t)rannc::units_before(nch, N));
  o->misc = align_up(64);  // status word, result pair
  o->rmin = align_up((size_t)rows);
  o->cost = align_up((size_t)cost);
  o->V = align_up((size_t)V);
  o->split = split;
  o->keys = (split && packed) ? align_up((size_t)(N + 1) * (size_t)DP * 8 * rannc::kSplitKeyTables) : 0;
  return true;
}

bool limits_ok(const rannc_dp_limits_t *l) {
  return l && l->max_problems >= 1 && l->max_blocks >= 1 && l->max_blocks <= 65535 &&
         l->max_devices >= 1 && l->max_devices <= RANNC_DP_MAX_DEVICES && l->max_stages >= 1 &&
         l->max_total_time_ns >= 0 && (l->flags & ~RANNC_DP_FLAG_SPLIT_OBJECTIVE) == 0 && l->algo >= RANNC_DP_ALGO_AUTO &&
         l->algo <= RANNC_DP_ALGO_RECOMPUTE && l->rows_per_wave >= 0 && l->rows_per_wave <= 16 &&
         l->one_launch_small >= 0 && l->one_launch_small <= 2 && l->single_stream >= 0 && l->single_stream <= 1 &&
         l->reserved == 0;
}

bool split_of(const rannc_dp_limits_t *l) { return (l->flags & RANNC_DP_FLAG_SPLIT_OBJECTIVE) != 0; }
// split objective: can the winners of a level be packed into 64-bit words (see the level kernel)
bool packed_of(const rannc_dp_limits_t *l) { return l->max_total_time_ns <= rannc::kSplitPackedMax; }
int bits_of(const rannc_dp_limits_t *l) { return l->max_total_time_ns <= kNarrowMax ? 32 : 64; }

size_t header_bytes(int Q) { return align_up((size_t)Q * sizeof(ProblemDev)); }
// the copies of the inputs behind the searches' regions, from which tables are made later: up to five arrays
size_t saved_bytes(size_t blocks) { return align_up(5 * 8 * blocks) + kAlign; }

// Host-side validation of the batch descriptors against the limits.
int check_batch(const rannc_dp_limits_t *l, const rannc_dp_batch_t *b) {
  if (!b || b->n_problems < 1) return RANNC_DP_INVALID_ARG;
  if (!b->n_blocks || !b->n_devices || !b->max_stages || !b->n_microbatches || !b->mem_capacity ||
      !b->block_offset)
    return RANNC_DP_INVALID_ARG;
  if (b->n_problems > l->max_problems) return RANNC_DP_LIMIT_EXCEEDED;
  if (b->block_offset[0] < 0) return RANNC_DP_INVALID_ARG;
  if ((b->bandwidth_bytes_per_us == nullptr) != (b->cut_bytes == nullptr)) return RANNC_DP_INVALID_ARG;
  for (int q = 0; q < b->n_problems; ++q) {
    if (b->n_blocks[q] < 1 || b->n_devices[q] < 1 || b->max_stages[q] < 1 ||
        b->n_microbatches[q] < 1 || b->mem_capacity[q] < 0)
      return RANNC_DP_INVALID_ARG;
    if (b->bandwidth_bytes_per_us && b->bandwidth_bytes_per_us[q] < 1) return RANNC_DP_INVALID_ARG;
    if (b->block_offset[q + 1] - b->block_offset[q] != (int64_t)b->n_blocks[q])
      return RANNC_DP_INVALID_ARG;
    if (b->n_blocks[q] > l->max_blocks || b->n_devices[q] > l->max_devices ||
        std::min(b->max_stages[q], std::min(b->n_blocks[q], b->n_devices[q])) > l->max_stages)
      return RANNC_DP_LIMIT_EXCEEDED;
  }
  return RANNC_DP_OK;
}

struct ResultLayout {  // offsets of the arrays of one result buffer
  size_t opt, est, n_stages, status, stage_end, replicas, total;
  ResultLayout(size_t Q, size_t stride) {
    auto a8 = [](size_t x) { return (x + 7) / 8 * 8; };
    opt = 0;
    est = opt + 8 * Q;
    n_stages = est + 8 * Q;
    status = n_stages + a8(4 * Q);
    stage_end = status + a8(4 * Q);
    replicas = stage_end + a8(4 * Q * stride);
    total = replicas + a8(4 * Q * stride);
  }
};

// batches of up to this many searches write their results to host memory themselves
constexpr int kPollMaxProblems = 64;

}  // namespace

struct rannc_dp {
  rannc_dp_limits_t lim;
  int bits;
  char *ws;
  size_t ws_bytes;
  // Pinned host memory, one allocation: staging for the per-problem descriptors, reused round-robin, and
  // behind it the mirror the kernels write a small batch's results into.  (A mirror allocated by the first
  // call that wants one made that call wait for it: first call of a
  // handle at 16 / 96 / 251 blocks 50 / 82 / 134 us, here 27 / 59 / 109.)
  char *pin, *pin_dev;               // pin_dev: the address the device uses, or null
  char *staging[kStagingSlots];
  char *staging_dev[kStagingSlots];  // or null
  hipEvent_t staging_free[kStagingSlots];
  bool staging_used[kStagingSlots];
  size_t staging_bytes;
  int next_slot;
  // state of the last successful solve
  bool solved;
  bool unchosen;  // its stage counts have not been chosen: plan recovery has that done first
  int Q;
  std::vector<ProblemDev> host_probs;  // in device order: grouped by DP class
  std::vector<int32_t> pos_of;         // position of the caller's problem q in that order
  ProblemDev *d_probs;
  // timing
  bool timing;
  hipEvent_t ev[4];
  bool ev_valid;
  int level_launches;
  // Device-count classes are independent chains of launches: with more than one class in a batch
  // the others run on streams of the handle (default priority), forked from and joined to the
  // caller's stream with events.  Off while per-phase timing is on (the phases are timed on the
  // caller's stream) and with RANNC_DP_STREAMS=0.
  char *res_pin;         // the mirror: inside pin, or (a longer plan stride) an allocation of its own
  char *res_pin_dev;     // its device address, or null
  size_t res_pin_bytes;
  bool res_pin_own;
  uint64_t seq;          // of the calls that poll for their results
  char *fs_pin;          // pinned host mirror of the outer driver's device scratch (grown on demand)
  char *fs_pin_dev;      // the address the device reads and writes the mirror through, or null
  size_t fs_pin_bytes;
  hipStream_t aux[3];
  hipEvent_t fork_ev, join_ev[3];
  bool multi_stream;
  int n_cus;  // compute units of the device the handle was created on
  rannc_dp_solve_info_t info;  // of the last successful solve
  bool no_times[4];  // per device-count class of the last solve: the stage-time table was not built
  int tune_spw;  // > 0: override of the rows-per-wave heuristic (RANNC_DP_ROWS_PER_WAVE)
  int fused_small;  // one-launch kernel for classes of small searches: 1 = where it pays (default),
                    // 0 = never, 2 = whenever N <= 128 (RANNC_DP_FUSED_SMALL)
  int64_t call_total_bound;  // > 0 during the outer driver's solve: no search's total time exceeds it
  // The last batch, where it was answered without its tables (solved, but not tabled): what makes them when they are
  // asked for.  Its inputs are at ws + saved_at (times, persistent, transient bytes, bytes per cut, backward times), or, of
  // the outer driver, they come from its own per sample (`sample`, the same arrays, and how many samples each search has).
  bool tabled;
  // They may still be under way on the stream of the call that asked for them: behind this event they are there.
  hipEvent_t tables_ev;
  bool tables_pending;
  // Whether the last call brought its results to the host, and whether its tables were asked for behind it.  Then the next call to the host makes its own at once: a program that reads them
  // behind every call pays for one search each, not for one without tables and one with them (a call and rannc_dp_traceback, the
  // stream waited for: 96 blocks at 16 devices 96 -> 86 us, 1024 at 64 360 -> 323).
  bool to_host, asked;
  int direct;  // searches of it that were
  // A call on the handle has been recorded into a graph, whose replays read the tables of whatever call came before
  // them, or write them: from then on every call makes its tables.
  bool recorded;
  struct {
    std::vector<int32_t> N, D, S, MB;
    std::vector<int64_t> M, off, bw, sample;
    bool comm, split;
    int64_t total_bound;
    size_t saved_at;
  } kept;
};

extern "C" {

const char *rannc_dp_strerror(int status) {
  switch (status) {
    case RANNC_DP_OK: return "ok";
    case RANNC_DP_INVALID_ARG: return "invalid argument";
    case RANNC_DP_LIMIT_EXCEEDED: return "problem exceeds the limits of the handle";
    case RANNC_DP_WORKSPACE_TOO_SMALL: return "workspace too small for this batch";
    case RANNC_DP_OVERFLOW: return "size computation overflow";
    case RANNC_DP_HIP_ERROR: return "HIP runtime error";
    case RANNC_DP_BAD_STATE: return "no solved batch on this handle";
    case RANNC_DP_NO_HOST_MEMORY: return "out of host memory";
    default: return "unknown status";
  }
}

size_t rannc_dp_workspace_bytes(const rannc_dp_limits_t *l) {
  if (!limits_ok(l)) return 0;
  Sizes sz;
  const int S_eff = std::min(l->max_stages, std::min(l->max_blocks, l->max_devices));
  if (!problem_sizes(l->max_blocks, l->max_devices, rannc::dp_class(l->max_devices), S_eff, bits_of(l), split_of(l),
                     packed_of(l), &sz))
    return 0;
  const unsigned __int128 tot =
      (unsigned __int128)sz.total() * (unsigned)l->max_problems + header_bytes(l->max_problems) +
      saved_bytes((size_t)l->max_blocks * (size_t)l->max_problems);
  if (tot > ((unsigned __int128)1 << 47)) return 0;
  return (size_t)tot;
}

size_t rannc_dp_workspace_bytes_for(const rannc_dp_limits_t *l, const rannc_dp_batch_t *b) {
  if (!limits_ok(l) || check_batch(l, b) != RANNC_DP_OK) return 0;
  size_t tot = header_bytes(l->max_problems) + saved_bytes((size_t)(b->block_offset[b->n_problems] - b->block_offset[0]));
  const int all = widest_class(b);  // (room for the group, whichever way the batch then runs)
  for (int q = 0; q < b->n_problems; ++q) {
    Sizes sz;
    const int S_eff = std::min(b->max_stages[q], std::min(b->n_blocks[q], b->n_devices[q]));
    if (!problem_sizes(b->n_blocks[q], b->n_devices[q], all ? all : rannc::dp_class(b->n_devices[q]), S_eff, bits_of(l),
                       split_of(l), packed_of(l), &sz))
      return 0;
    tot += sz.total();
    if (tot > ((size_t)1 << 47)) return 0;
  }
  return tot;
}

int rannc_dp_create(const rannc_dp_limits_t *l, void *d_workspace, size_t workspace_bytes,
                    rannc_dp_t **out) {
  if (out) *out = nullptr;
  if (!out || !limits_ok(l) || !d_workspace || ((uintptr_t)d_workspace % kAlign) != 0)
    return RANNC_DP_INVALID_ARG;
  if (workspace_bytes < header_bytes(l->max_problems)) return RANNC_DP_WORKSPACE_TOO_SMALL;
  rannc_dp *h = new (std::nothrow) rannc_dp();
  if (!h) return RANNC_DP_NO_HOST_MEMORY;
  h->lim = *l;
  h->bits = bits_of(l);
  h->ws = (char *)d_workspace;
  h->ws_bytes = workspace_bytes;
  h->staging_bytes = header_bytes(l->max_problems);
  h->next_slot = 0;
  h->solved = false;
  h->unchosen = false;
  h->tabled = false;
  h->tables_pending = false;
  h->to_host = h->asked = false;
  h->direct = 0;
  h->recorded = false;
  h->Q = 0;
  h->timing = false;
  h->ev_valid = false;
  h->level_launches = 0;
  h->tune_spw = l->rows_per_wave;
  for (int k = 0; k < 4; ++k) h->no_times[k] = false;
  h->call_total_bound = 0;
  {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) {
      (void)hipGetLastError();
      cus = 256;
    }
    h->n_cus = cus;
  }
  if (const char *e = std::getenv("RANNC_DP_ROWS_PER_WAVE")) h->tune_spw = std::atoi(e);
  h->fused_small = l->one_launch_small == 1 ? 0 : l->one_launch_small == 2 ? 2 : 1;
  if (const char *e = std::getenv("RANNC_DP_FUSED_SMALL")) h->fused_small = std::atoi(e);
  h->d_probs = (ProblemDev *)h->ws;
  h->res_pin_own = false;
  h->seq = 0;
  h->fs_pin = nullptr;
  h->fs_pin_dev = nullptr;
  h->fs_pin_bytes = 0;
  h->multi_stream = l->single_stream == 0;
  if (const char *e = std::getenv("RANNC_DP_STREAMS")) h->multi_stream = std::atoi(e) != 0;
  int made_ev_s = 0, made_ev = 0, made_aux = 0, made_join = 0;
  bool made_fork = false, made_tables = false;
  bool ok = true;
  {
    const size_t polled = (size_t)std::min(l->max_problems, kPollMaxProblems);
    h->res_pin_bytes = ResultLayout(polled, (size_t)std::min(l->max_stages, RANNC_DP_MAX_DEVICES)).total + 8 * polled;
    const size_t res_at = kStagingSlots * h->staging_bytes;
    ok = hipHostMalloc((void **)&h->pin, res_at + h->res_pin_bytes, hipHostMallocMapped | hipHostMallocPortable) == hipSuccess;
    if (!ok) {
      h->pin = nullptr;
    } else if (hipHostGetDevicePointer((void **)&h->pin_dev, h->pin, 0) != hipSuccess) {
      (void)hipGetLastError();
      h->pin_dev = nullptr;
    }
    for (int k = 0; k < kStagingSlots && ok; ++k) {
      h->staging_used[k] = false;
      h->staging[k] = h->pin + k * h->staging_bytes;
      h->staging_dev[k] = h->pin_dev ? h->pin_dev + k * h->staging_bytes : nullptr;
    }
    if (ok) {
      h->res_pin = h->pin + res_at;
      h->res_pin_dev = h->pin_dev ? h->pin_dev + res_at : nullptr;
      std::memset(h->res_pin, 0, h->res_pin_bytes);
    }
  }
  for (int k = 0; k < kStagingSlots && ok; ++k) {
    ok = hipEventCreateWithFlags(&h->staging_free[k], hipEventDisableTiming) == hipSuccess;
    if (ok) ++made_ev_s;
  }
  for (int k = 0; k < 4 && ok; ++k) {
    ok = hipEventCreate(&h->ev[k]) == hipSuccess;
    if (ok) ++made_ev;
  }
  for (int k = 0; k < 3 && ok; ++k) {
    ok = hipStreamCreateWithFlags(&h->aux[k], hipStreamNonBlocking) == hipSuccess;
    if (ok) ++made_aux;
  }
  for (int k = 0; k < 3 && ok; ++k) {
    ok = hipEventCreateWithFlags(&h->join_ev[k], hipEventDisableTiming) == hipSuccess;
    if (ok) ++made_join;
  }
  if (ok) {
    ok = hipEventCreateWithFlags(&h->fork_ev, hipEventDisableTiming) == hipSuccess;
    made_fork = ok;
  }
  if (ok) {
    ok = hipEventCreateWithFlags(&h->tables_ev, hipEventDisableTiming) == hipSuccess;
    made_tables = ok;
  }
  if (!ok) {
    for (int k = 0; k < made_aux; ++k) (void)hipStreamDestroy(h->aux[k]);
    for (int k = 0; k < made_join; ++k) (void)hipEventDestroy(h->join_ev[k]);
    if (made_fork) (void)hipEventDestroy(h->fork_ev);
    if (made_tables) (void)hipEventDestroy(h->tables_ev);
    if (h->pin) (void)hipHostFree(h->pin);
    for (int k = 0; k < made_ev_s; ++k) (void)hipEventDestroy(h->staging_free[k]);
    for (int k = 0; k < made_ev; ++k) (void)hipEventDestroy(h->ev[k]);
    delete h;
    (void)hipGetLastError();
    return RANNC_DP_HIP_ERROR;
  }
  *out = h;
  return RANNC_DP_OK;
}

void rannc_dp_destroy(rannc_dp_t *h) {
  if (!h) return;
  for (int k = 0; k < kStagingSlots; ++k) {
    if (h->staging_used[k]) (void)hipEventSynchronize(h->staging_free[k]);
    (void)hipEventDestroy(h->staging_free[k]);
  }
  for (int k = 0; k < 4; ++k) (void)hipEventDestroy(h->ev[k]);
  for (int k = 0; k < 3; ++k) {
    (void)hipStreamSynchronize(h->aux[k]);
    (void)hipStreamDestroy(h->aux[k]);
    (void)hipEventDestroy(h->join_ev[k]);
  }
  (void)hipEventDestroy(h->fork_ev);
  if (h->tables_pending) (void)hipEventSynchronize(h->tables_ev);  // (they may be made from the outer driver's mirror)
  (void)hipEventDestroy(h->tables_ev);
  if (h->fs_pin) (void)hipHostFree(h->fs_pin);
  if (h->res_pin_own) (void)hipHostFree(h->res_pin);
  (void)hipHostFree(h->pin);
  delete h;
}

int rannc_dp_set_timing(rannc_dp_t *h, int enabled) {
  if (!h) return RANNC_DP_INVALID_ARG;
  h->timing = enabled != 0;
  return RANNC_DP_OK;
}

int rannc_dp_get_timing(rannc_dp_t *h, float *out_ms, int32_t *out_level_launches) {
  if (!h || !out_ms) return RANNC_DP_INVALID_ARG;
  if (!h->ev_valid) return RANNC_DP_BAD_STATE;
  if (hipEventSynchronize(h->ev[3]) != hipSuccess) return RANNC_DP_HIP_ERROR;
  for (int k = 0; k < 3; ++k)
    if (hipEventElapsedTime(&out_ms[k], h->ev[k], h->ev[k + 1]) != hipSuccess) return RANNC_DP_HIP_ERROR;
  if (out_level_launches) *out_level_launches = h->level_launches;
  return RANNC_DP_OK;
}

// chosen != null: the caller waits for the batch before the handle is used again, and the plan recovery
// behind it can choose the stage counts; *chosen = whether that has been done here already.
// results != null: a solve that is one launch over few searches recovers their plans there as well;
// *recovered = whether it has.
// info_only: nothing is launched, and only what rannc_dp_solve_info reports is found out.
// part != null: the batch is a part of another one, whose arrays of blocks it has and in whose results its searches have
// their places.
struct BatchPart { std::vector<int32_t> place; std::vector<int64_t> first; };  // in the results; of the blocks
static int solve_impl(rannc_dp_t *h, const rannc_dp_batch_t *b, void *hip_stream, int64_t *d_opt, int32_t *d_n_stages,
                      int64_t *d_est_iter_ns, int32_t *d_status, bool *chosen, int32_t plan_stride = 0,
                      const rannc::PlanResults *results = nullptr, bool *recovered = nullptr, bool info_only = false,
                      const BatchPart *part = nullptr) {
  int rc = check_batch(&h->lim, b);
  if (rc != RANNC_DP_OK) return rc;
  if (!b->time_ns || !b->param_bytes || !b->act_bytes) return RANNC_DP_INVALID_ARG;
  const bool split = split_of(&h->lim);
  if (split != (b->time_bwd_ns != nullptr)) return RANNC_DP_INVALID_ARG;
  hipStream_t st = (hipStream_t)hip_stream;
  const int Q = b->n_problems;

  // ---- device order: problems grouped by the padded device dimension their kernels are
  //      specialised for, so that one launch covers a contiguous slice of descriptors --------
  static const int kClasses[4] = {8, 16, 32, 64};
  std::vector<ProblemDev> probs;
  std::vector<int32_t> pos_of;
  try {
    probs.resize(Q);
    pos_of.resize(Q);
  } catch (...) {
    return RANNC_DP_NO_HOST_MEMORY;
  }
  // (a handle told to run every small search as one launch keeps the classes apart: the form of that
  // kernel depends on the class)
  int all = h->fused_small == 2 ? 0 : group_dp(b, h->bits, split);
  if (all) {
    // a workspace sized for another batch can hold these searches only at their own classes' widths
    size_t need = header_bytes(h->lim.max_problems);
    for (int q = 0; q < Q && all; ++q) {
      Sizes sz;
      const int S_eff = std::min(b->max_stages[q], std::min(b->n_blocks[q], b->n_devices[q]));
      if (!problem_sizes(b->n_blocks[q], b->n_devices[q], all, S_eff, h->bits, split, packed_of(&h->lim), &sz) ||
          need + sz.total() > h->ws_bytes)
        all = 0;
      else need += sz.total();
    }
  }
  auto dp_of = [&](int q) { return all ? all : rannc::dp_class(b->n_devices[q]); };
  int cls_start[5] = {0, 0, 0, 0, 0};
  for (int q = 0; q < Q; ++q)
    for (int k = 0; k < 4; ++k)
      if (dp_of(q) == kClasses[k]) ++cls_start[k + 1];
  for (int k = 0; k < 4; ++k) cls_start[k + 1] += cls_start[k];
  {
    int next[4] = {cls_start[0], cls_start[1], cls_start[2], cls_start[3]};
    for (int q = 0; q < Q; ++q)
      for (int k = 0; k < 4; ++k)
        if (dp_of(q) == kClasses[k]) pos_of[q] = next[k]++;
  }

  // ---- workspace layout -------------------------------------------------------------
  LaunchShape shape[4];
  std::memset(shape, 0, sizeof(shape));
  size_t off = header_bytes(h->lim.max_problems);
  for (int q = 0; q < Q; ++q) {
    const int N = b->n_blocks[q], D = b->n_devices[q];
    const int S_eff = std::min(b->max_stages[q], std::min(N, D));
    Sizes sz;
    if (!problem_sizes(N, D, dp_of(q), S_eff, h->bits, split, packed_of(&h->lim), &sz)) return RANNC_DP_OVERFLOW;
    if (off + sz.total() > h->ws_bytes) return RANNC_DP_WORKSPACE_TOO_SMALL;
    ProblemDev &p = probs[pos_of[q]];
    std::memset(&p, 0, sizeof(p));
    p.N = N; p.D = D; p.S_eff = S_eff; p.MB = b->n_microbatches[q];
    p.DP = dp_of(q);
    p.nch = (N + 63) / 64;
    p.bits = h->bits;
    p.q = part ? part->place[q] : q;
    p.M = b->mem_capacity[q];
    p.time_limit = h->lim.max_total_time_ns;
    const int64_t first = part ? part->first[q] : b->block_offset[q];
    p.t = b->time_ns + first;
    p.p = b->param_bytes + first;
    p.a = b->act_bytes + first;
    p.o = b->cut_bytes ? b->cut_bytes + first : nullptr;
    p.bw = b->cut_bytes ? b->bandwidth_bytes_per_us[q] : 0;
    char *base = h->ws + off;
    p.T = (int64_t *)base; base += sz.prefix;
    p.P = (int64_t *)base; base += sz.prefix;
    p.A = (int64_t *)base; base += sz.prefix;
    p.C = b->cut_bytes ? (int64_t *)base : nullptr;
    p.ends = (uint32_t *)base;  // (where the level kernel recomputes the stage times: set below)
    base += sz.prefix;
    if (split) {
      p.tb = b->time_bwd_ns + first;
      p.TB = (int64_t *)base; base += sz.prefix;
    }
    p.wlo = (int32_t *)base; base += sz.wlo;
    p.runs = (int32_t *)base; base += sz.runs;
    p.ufit = (uint8_t *)base; base += sz.ufit;
    p.status = (int32_t *)base;
    p.res = (int64_t *)(base + 16); base += sz.misc;
    p.rmin = (uint8_t *)base; base += sz.rmin;
    p.cost = base; base += sz.cost;
    p.V = base; base += sz.V;
    if (split) {
      p.costb = base; base += sz.cost;
      p.VF = base; base += sz.V;
      p.VB = base; base += sz.V;
      if (sz.keys) { p.keys = base; base += sz.keys; }
    }
    off += sz.total();
    for (int k = 0; k < 4; ++k)
      if (p.DP == kClasses[k]) {
        LaunchShape &sh = shape[k];
        sh.nprob++;
        sh.max_N = std::max(sh.max_N, p.N);
        sh.max_nch = std::max(sh.max_nch, p.nch);
        sh.max_D = std::max(sh.max_D, p.D);
        sh.max_S_eff = std::max(sh.max_S_eff, p.S_eff);
        if (rannc::dp_class(D) == p.DP) {
          for (int c = 0; c < p.nch; ++c) sh.wide_rows += std::min(64 * c + 64, N);
          sh.wide_chunks += p.nch;
        }
      }
  }

  const bool scan = h->lim.algo == RANNC_DP_ALGO_SCAN;
  // split objective: packed-key kernel wherever a cell's winner fits a 64-bit word (all 32-bit
  // handles, 64-bit ones up to 2^42 - 2 ns); RANNC_DP_ALGO_SCAN and larger time bounds take the
  // literal one
  const bool split_fast = split && !scan && packed_of(&h->lim);
  // what the host knows about the total time of a search of this batch: the handle's bound, or the
  // outer driver's own sum over the inputs it has just scaled
  const int64_t total_bound = h->call_total_bound > 0 ? std::min(h->call_total_bound, h->lim.max_total_time_ns)
                                                      : h->lim.max_total_time_ns;
  // stage times recomputed inside the level kernel instead of read from their table: where it
  // applies, on request, or (AUTO) for the classes whose launches are large enough to be bound by
  // throughput
  const bool can_recompute = !scan && !split && !b->cut_bytes && rannc::can_recompute_times(h->bits, total_bound);
  bool recompute_cls[4];
  for (int k = 0; k < 4; ++k)
    recompute_cls[k] = can_recompute && (h->lim.algo == RANNC_DP_ALGO_RECOMPUTE ||
                                         (h->lim.algo == RANNC_DP_ALGO_AUTO &&
                                          rannc::merge_launch_rows(shape[k]) >= rannc::kRecomputeRowsFrom));
  for (int q = 0; q < Q; ++q)
    for (int k = 0; k < 4; ++k)
      if (probs[q].DP == kClasses[k] && !recompute_cls[k]) probs[q].ends = nullptr;

  bool fused[4] = {false, false, false, false};
  bool fused_direct[4] = {false, false, false, false};  // one-launch kernel that recomputes the stage times
  // estimated time of a class of few small searches (us): as one launch with recomputed stage times
  // (< 0: that kernel does not apply) and as launches per level
  double est_one[4] = {-1.0, -1.0, -1.0, -1.0}, est_levels[4] = {0.0, 0.0, 0.0, 0.0};
  auto levels_us = [&](const LaunchShape &sh) {
    return h->bits == 64 ? 26.9 + 4.7 * (sh.max_S_eff - 1) + 0.023 * sh.max_N : 24.3 + 4.1 * (sh.max_S_eff - 1) + 0.033 * sh.max_N;
  };
  for (int k = 0; k < 4; ++k) {
    const LaunchShape &sh = shape[k];
    if (!sh.nprob) continue;
    // Small searches: everything in one launch, one workgroup per search, where that measured
    // faster than the launches per level (MI355X; N = 16..128, D = 8..64, 1..512 searches per class).
    {
      const int64_t rows = std::min(sh.max_N, 64) + (sh.max_nch > 1 ? sh.max_N : 0);
      const int levels = sh.max_S_eff - 1;
      const int cls = kClasses[k];
      // the launches per level of a few small searches: 14 us in front of the levels, 4.4 us a level
      const double launches_us = 14.0 + 4.4 * levels;
      const bool direct_ok = !scan && !split && !b->cut_bytes && h->lim.algo != RANNC_DP_ALGO_MERGE &&
                             rannc::small_can_recompute(h->bits, cls, total_bound);
      const bool heavy = h->bits / 8 * cls >= 256;  // the variants that run eight waves per search
      bool tiny;
      if (direct_ok) {
        // Stage times recomputed: the levels read nothing from memory.  The kernel runs a level as
        // passes of 64 stages that fit, sixteen waves at a time; the host counts the passes of the
        // triangular and rectangular blocks, which the stages that fit cannot exceed by much.  Least-squares
        // fit over whole calls (N = 16..128, D = 8, 16, 32, S = 3..D, memory for an even share twice, six and
        // thirty times, 1 and 6 searches; 426 shapes, rms 11 us): 24 us + 0.08 us per table row in front,
        // then per level a constant and a price per pass that follow the width of the merge the level still
        // needs (32 / 16 / 8 inputs), the passes of the first round of sixteen dearer than the later ones.  The
        // launches per level on the same sweep: 24 us + 4.1 us per level + 0.03 us per block.  The choice is
        // 0.7 % above the better of the two on average (64-bit values 1.9 %).
        auto tri = [](int W) {
          int lg = 0;
          while ((1 << lg) < W) ++lg;
          return (W / 2 + (64 >> lg)) >> (6 - lg);
        };
        int passes = tri(std::min(sh.max_N, 64));
        if (sh.max_N > 64) {
          int lg = 0;
          while ((1 << lg) < sh.max_N - 64) ++lg;
          passes += (64 >> (6 - lg)) + tri(sh.max_N - 64);
        }
        const double work = 0.17 * std::min(passes, 16) + 0.105 * std::max(passes - 16, 0);
        const bool w64 = h->bits == 64;  // the same fit on 64-bit values (rms 22 us; eight waves at 32 devices)
        double us = 24.3 + (w64 ? 0.090 : 0.079) * (double)rows;
        for (int s = 2; s <= sh.max_S_eff; ++s) {
          const int rl = sh.max_D - s + 1;
          if (w64) us += rl <= 8 ? 0.43 + 0.26 * work : rl <= 16 ? 0.67 + 0.53 * work : 0.73 + 1.19 * work;
          else us += rl <= 8 ? 0.42 + 0.20 * work : rl <= 16 ? 0.84 + 0.37 * work : 0.76 + 0.65 * work;
        }
        est_one[k] = us;
        // Up to a search to a compute unit the one launch takes as long as one search; the launches per level take longer
        // with every search of theirs, in proportion to the devices that a level still deals with (66 to 128 blocks, 8
        // stages, 8 to 127 searches: 0.2 to 0.26 us a search at 8 devices, 0.35 to 0.6 at 32).  8 stages, 64 searches of 80
        // blocks at 16 devices: one launch 76 us, levels 98; 127 of 100 at 8 devices 79 and 114; 48 of 80 at 32 devices 95
        // and 106, 64 of 128 143 and 131.  (Beside other classes the launches per level hide behind one another.)
        const double share = levels * (sh.max_D - 0.5 * sh.max_S_eff) / cls;
        const double more = sh.nprob == Q && sh.nprob < 128 ? (sh.nprob - 1) * share * (0.035 + 1.4e-5 * sh.max_N * cls) : 0.0;
        tiny = us <= levels_us(sh) + more;
      } else if (heavy) {
        // 64 devices, or 64-bit values from 32 devices on, stage times from the table: a level costs
        // about 7 us plus 1.7 us per pass of eight rows, more than a launch; only two or three levels
        // are cheaper in one launch
        tiny = rows <= (h->bits == 64 ? 16 : 32) && (7.0 + 1.7 * (double)((rows + 7) / 8)) * levels <= launches_us;
      } else {
        // stage times from the table, sixteen waves (sweep over N = 8..128, D = 8, 16, S = 2..D)
        tiny = rows <= 64 && rows * levels <= (h->bits == 64 ? 240 : 480);
      }
      // Hundreds of searches: the launches per level are throughput-bound as well.  One launch where it
      // recomputes the stage times (256 searches of 96 blocks and 32 devices 129 us against 187 us of launches
      // per level, 1024 of them 407 against 437 us), and where neither side does (1024 such searches with send
      // times 1.25 against 1.96 ms; not 64 devices, 32-bit values and more than 64 blocks: 3.5 against 3.3 ms).  Where
      // only the levels recompute -- 64 devices -- they are the faster ones (1024 searches of 24 blocks: 232 us
      // against 426 us).  A workgroup that has a compute unit to itself and more than 64 blocks leaves much of the
      // device idle in a last round that is not full (one_launch_rounds_full: 100 blocks, 64-bit values, 64 devices,
      // send times, one launch / levels: 256 searches 1.60 / 1.74 ms, 300 2.50 / 1.99, 400 2.79 / 2.59, 768 4.67 /
      // 4.80, 1100 7.17 / 6.80; 32 devices, times recomputed: 200 198 / 218 us, 256 202 / 228, 300 331 / 309, 520
      // 471 / 392, 768 506 / 514).  From 32 devices and 65 blocks on only for a class alone: beside the levels of other
      // classes its workgroups stand in their way (2048 searches of 128 blocks in four classes: 1.79 against
      // 1.69 ms).  Where it recomputes the times one launch is ahead from fewer searches on (8 stages of 64 blocks
      // and 32 devices: 64 searches 66 against 82 us; of 128 blocks and 16 devices: 64 searches level, 128 of
      // them 116 against 133 us).
      const bool alone = sh.nprob == Q;
      const int many = !direct_ok ? 256 : sh.max_N <= 64 ? 64 : 128;
      const bool one_per_cu = h->bits == 64 && (cls == 64 || (cls == 32 && direct_ok));
      const bool batch = sh.nprob >= many && (direct_ok || !recompute_cls[k]) &&
                         (cls <= 16 || sh.max_N <= 64 ||
                          (alone && (one_per_cu ? rannc::one_launch_rounds_full(sh.nprob, h->n_cus) : cls < 64)));
      fused[k] = !scan && !split && sh.max_N <= rannc::small_max_blocks() &&
                 (h->fused_small == 1 ? (batch || tiny) : h->fused_small == 2);
      fused_direct[k] = fused[k] && direct_ok;
      est_levels[k] = levels_us(sh);
    }
  }
  // Classes in the shadow of the longest one.  The classes of a batch run side by side on streams
  // of their own, so the call takes as long as its longest class -- or as long as the host needs to
  // enqueue everything: a class of launches per level costs the host some 3 us per launch (outer
  // driver at 128 blocks: 118 launches, 0.385 ms per call for 0.27 ms of device time).  A class of
  // few searches that is not the longest and would finish as ONE launch within the longest class's
  // time takes the one-launch kernel even where its own launches per level would be faster.
  bool share_stream = true;  // the one-launch classes besides the first share one stream
  if (h->fused_small == 1 && h->multi_stream && !h->timing) {
    double longest = 0.0;
    int crit = -1;
    for (int k = 0; k < 4; ++k) {
      if (!shape[k].nprob) continue;
      const double t = fused[k] && est_one[k] >= 0.0 ? est_one[k] : est_levels[k];
      if (t > longest) { longest = t; crit = k; }
    }
    for (int k = 0; k < 4; ++k)
      if (shape[k].nprob && k != crit && !fused[k] && est_one[k] >= 0.0 && est_one[k] <= longest &&
          shape[k].nprob <= 64 && shape[k].max_N <= rannc::small_max_blocks())
        fused[k] = fused_direct[k] = true;
    double sum = 0.0;
    for (int k = 0; k < 4; ++k)
      if (shape[k].nprob && fused[k] && k != crit && est_one[k] >= 0.0) sum += est_one[k];
    share_stream = sum <= longest;
  }
  auto report = [&]() {
    int kernel_of[4];
    for (int k = 0; k < 4; ++k) {
      kernel_of[k] = fused[k]           ? (fused_direct[k] ? RANNC_DP_KERNEL_ONE_LAUNCH_RECOMPUTE : RANNC_DP_KERNEL_ONE_LAUNCH)
                     : split_fast       ? RANNC_DP_KERNEL_SPLIT
                     : split            ? RANNC_DP_KERNEL_SPLIT_SCAN
                     : scan             ? RANNC_DP_KERNEL_SCAN
                     : recompute_cls[k] ? RANNC_DP_KERNEL_MERGE_RECOMPUTE
                                        : RANNC_DP_KERNEL_MERGE_TABLE;
      h->info.n_problems[k] = 0;
      h->info.level_kernel[k] = RANNC_DP_KERNEL_NONE;
    }
    for (int q = 0; q < Q; ++q) {  // reported by the searches' own classes, also where they ran as one group
      int own = 0, ran = 0;
      while (kClasses[own] != rannc::dp_class(b->n_devices[q])) ++own;
      while (kClasses[ran] != dp_of(q)) ++ran;
      h->info.n_problems[own]++;
      h->info.level_kernel[own] = kernel_of[ran];
    }
  };
  if (info_only) {
    report();
    return RANNC_DP_OK;
  }

  // ---- descriptors to the device ---------------------------------------------------
  const int slot = h->next_slot;
  h->next_slot = (slot + 1) % kStagingSlots;
  if (h->staging_used[slot] && hipEventSynchronize(h->staging_free[slot]) != hipSuccess)
    return RANNC_DP_HIP_ERROR;
  const size_t probs_bytes = (size_t)Q * sizeof(ProblemDev);
  std::memcpy(h->staging[slot], probs.data(), probs_bytes);
  h->solved = false;
  // one group: its first launch reads the descriptors out of the staging memory and stores them
  const bool in_place = all != 0 && h->staging_dev[slot] != nullptr;
  h->staging_used[slot] = false;
  if (!in_place) {
    if (hipMemcpyAsync(h->ws, h->staging[slot], probs_bytes, hipMemcpyHostToDevice, st) != hipSuccess ||
        hipEventRecord(h->staging_free[slot], st) != hipSuccess) {
      (void)hipGetLastError();
      return RANNC_DP_HIP_ERROR;
    }
    h->staging_used[slot] = true;
  }
  auto staging_read = [&]() -> bool {  // behind the launch that has read the staging memory
    if (!in_place || chosen) return true;  // (a caller that waits has the slot back by then)
    h->staging_used[slot] = hipEventRecord(h->staging_free[slot], st) == hipSuccess;
    return h->staging_used[slot];
  };

  // ---- kernels ---------------------------------------------------------------------------
  ProblemDev *const dp = h->d_probs;
  const ProblemDev *const src = in_place ? (const ProblemDev *)h->staging_dev[slot] : dp;
  bool ok = true;
  const bool timing = h->timing;
  h->ev_valid = false;
  h->level_launches = 0;
  if (timing) ok = ok && hipEventRecord(h->ev[0], st) == hipSuccess;
  // one stream per device-count class: the largest class stays on the caller's stream
  hipStream_t cs[4] = {st, st, st, st};
  int n_aux = 0;
  if (h->multi_stream && !timing) {
    // (the other classes that run as ONE launch each share a stream where together they stay within
    // the longest class's time: every stream costs a wait on the fork event and one on its join
    // event, 10 us of host time each)
    bool first = true;
    int shared = -1;
    for (int k = 3; k >= 0; --k) {
      if (!shape[k].nprob) continue;
      if (first) { first = false; continue; }
      if (fused[k] && share_stream) {
        if (shared < 0) shared = n_aux++;
        cs[k] = h->aux[shared];
      } else {
        cs[k] = h->aux[n_aux++];
      }
    }
    if (n_aux > 0) {
      ok = ok && hipEventRecord(h->fork_ev, st) == hipSuccess;  // descriptors are on the device
      for (int a = 0; a < n_aux && ok; ++a) ok = hipStreamWaitEvent(h->aux[a], h->fork_ev, 0) == hipSuccess;
    }
  }
  int merge_items[4] = {1, 1, 1, 1};
  for (int k = 0; k < 4 && ok; ++k) {
    const LaunchShape &sh = shape[k];
    if (!sh.nprob) continue;
    ProblemDev *cp = dp + cls_start[k];
    const hipStream_t st = cs[k];  // this class's stream
    if (fused[k]) continue;
    // Rows per item of the level kernel: chosen on the device from the size of the windows unless
    // the handle fixes it, or the host does for a launch of many rounds (merge_grid_items).
    const int slots = h->n_cus * rannc::merge_workgroups_per_cu(h->bits, kClasses[k], recompute_cls[k]);
    const int max_rows = recompute_cls[k] ? rannc::merge_max_rows(h->bits) : 64;
    int rows_for_list = -1;
    if (split) rows_for_list = rannc::split_rows_per_item(sh, kClasses[k]);
    else
      merge_items[k] = rannc::merge_grid_items(sh, rannc::merge_rows_per_item(h->tune_spw), slots, recompute_cls[k],
                                               max_rows, &rows_for_list);
    const ProblemDev *host_one = sh.nprob == 1 ? &probs[cls_start[k]] : nullptr;
    const int parts = recompute_cls[k] || split_fast ? 1 : 3;
    // Tables of several searches as two launches, sums and builder, where the one launch pays more for the sums, which each
    // of its workgroups forms again, or for the waves it keeps on the stores.  Per call with send times, as one launch /
    // two: up to sixteen searches of more than 512 blocks (4 of 1000, 8 devices 124 / 108 us, 32 devices 158 / 144; 7 of
    // 500 104 / 102, 30 of 1000 231 / 234); more than 64 (whose descriptors are copied to the device in front of the
    // first launch, which takes as long) of up to 256 blocks (64 of 100 at 8 devices 91 / 101, 66 103 / 98, 100 of 130 at
    // 16 172 / 165, 300 of 160 at 8 311 / 278, at 32 969 / 936, 64-bit values 1773 / 1581; 100 of 500 at 8 375 / 388),
    // and at 64 devices (512 of 128 blocks 583 / 546, 64-bit values 1024 / 878).
    const bool apart = parts == 3 && ((sh.nprob > 1 && sh.nprob <= 16 && sh.max_N > 512) ||
                                      (sh.nprob > 64 && (sh.max_N <= 256 || kClasses[k] == 64)));
    if (rannc::can_prepare(sh) && !apart) {
      ok = rannc::launch_prepare(src + cls_start[k], cp, sh, h->bits, kClasses[k], parts, rows_for_list, merge_items[k], slots,
                                 recompute_cls[k], max_rows, split, b->cut_bytes != nullptr, host_one, st) == hipSuccess;
      ok = ok && staging_read();
    } else {
      ok = rannc::launch_setup(src + cls_start[k], cp, sh.nprob, rows_for_list, merge_items[k], slots, recompute_cls[k],
                               max_rows, host_one, st) == hipSuccess;
      ok = ok && staging_read();
      ok = ok && (recompute_cls[k] ? rannc::launch_build_passes(cp, sh, h->bits, kClasses[k], st)
                                   : rannc::launch_build(cp, sh, h->bits, kClasses[k], parts, st)) == hipSuccess;
      if (split) ok = ok && rannc::launch_split_level1(cp, sh, h->bits, st) == hipSuccess;
    }
  }
  if (timing) ok = ok && hipEventRecord(h->ev[1], st) == hipSuccess;
  int max_levels = 0, in_one = 0;
  for (int k = 0; k < 4; ++k) in_one += fused[k] && shape[k].nprob == Q ? 1 : 0;
  const bool recover = results && in_one && !timing;
  if (recovered) *recovered = recover;
  for (int k = 0; k < 4; ++k) {
    if (fused[k]) {
      ok = ok && rannc::launch_solve_small(src + cls_start[k], dp + cls_start[k], shape[k].nprob, h->bits, kClasses[k], fused_direct[k], d_opt,
                                           d_n_stages, d_est_iter_ns, d_status,
                                           shape[k].nprob == 1 ? &probs[cls_start[k]] : nullptr, plan_stride,
                                           recover ? results : nullptr, h->n_cus, cs[k]) == hipSuccess;
      ok = ok && staging_read();
      h->level_launches++;
    } else {
      max_levels = std::max(max_levels, shape[k].max_S_eff);
    }
  }
  for (int s = 2; s <= max_levels && ok; ++s) {
    for (int k = 0; k < 4 && ok; ++k) {
      const LaunchShape &sh = shape[k];
      if (!sh.nprob || sh.max_S_eff < s || fused[k]) continue;
      const hipStream_t st = cs[k];
      if (split_fast)
        ok = rannc::launch_level_split_fast(dp + cls_start[k], sh, h->bits, kClasses[k], s,
                                            rannc::split_rows_per_item(sh, kClasses[k]), st) == hipSuccess;
      else if (split)
        ok = rannc::launch_level_split(dp + cls_start[k], sh, h->bits, s, 1, nullptr, nullptr, st) ==
             hipSuccess;
      else if (scan)
        ok = rannc::launch_level_scan(dp + cls_start[k], sh, h->bits, s, 1, nullptr, nullptr, st) ==
             hipSuccess;
      else
        ok = rannc::launch_level_merge(dp + cls_start[k], sh, h->bits, s, recompute_cls[k], merge_items[k],
                                       // measured: c4 (64 devices) 0.410 -> 0.401 ms; c3, c2 (32, 16 devices,
                                       // launches of 4-6 us) 1-2 us slower per solve with the larger argument block
                                       sh.nprob == 1 && kClasses[k] == 64 ? &probs[cls_start[k]] : nullptr, st) == hipSuccess;
      h->level_launches++;
    }
  }
  if (timing) ok = ok && hipEventRecord(h->ev[2], st) == hipSuccess;
  bool choose_later = chosen && all && !timing;
  for (int k = 0; k < 4; ++k) choose_later = choose_later && !(shape[k].nprob && fused[k]);
  if (chosen) *chosen = !choose_later;
  for (int k = 0; k < 4 && ok; ++k)
    if (shape[k].nprob && !fused[k] && !choose_later)
      ok = rannc::launch_select(dp + cls_start[k], shape[k].nprob, d_opt, d_n_stages, d_est_iter_ns,
                                d_status, cs[k]) == hipSuccess;
  for (int a = 0; a < n_aux && ok; ++a)  // join: the caller's stream continues after every class
    ok = hipEventRecord(h->join_ev[a], h->aux[a]) == hipSuccess &&
         hipStreamWaitEvent(st, h->join_ev[a], 0) == hipSuccess;
  if (timing) ok = ok && hipEventRecord(h->ev[3], st) == hipSuccess;
  if (!ok) {
    (void)hipGetLastError();
    // nothing of this solve may still run on the handle's streams when the caller sees the error
    for (int a = 0; a < n_aux; ++a) (void)hipStreamSynchronize(h->aux[a]);
    return RANNC_DP_HIP_ERROR;
  }
  h->ev_valid = timing;
  for (int k = 0; k < 4; ++k) h->no_times[k] = fused[k] ? fused_direct[k] : recompute_cls[k] || split_fast;
  report();
  h->host_probs.swap(probs);
  h->pos_of.swap(pos_of);
  h->Q = Q;
  h->solved = true;
  h->tabled = true;
  h->unchosen = choose_later;
  return RANNC_DP_OK;
}

// The last batch as it was answered without its tables, over the copies of its inputs.
static rannc_dp_batch_t kept_batch(const rannc_dp_t *h) {
  rannc_dp_batch_t b = {};
  b.n_problems = h->Q;
  b.n_blocks = h->kept.N.data(); b.n_devices = h->kept.D.data(); b.max_stages = h->kept.S.data();
  b.n_microbatches = h->kept.MB.data(); b.mem_capacity = h->kept.M.data(); b.block_offset = h->kept.off.data();
  const int64_t blocks = h->kept.off[h->Q];
  b.time_ns = (const int64_t *)(h->ws + h->kept.saved_at);
  b.param_bytes = b.time_ns + blocks;
  b.act_bytes = b.param_bytes + blocks;
  if (h->kept.comm) {
    b.cut_bytes = b.act_bytes + blocks;
    b.bandwidth_bytes_per_us = h->kept.bw.data();
  }
  if (h->kept.split) b.time_bwd_ns = b.act_bytes + 2 * blocks;
  return b;
}

// Its tables, in the workspace in front of the copies; or what they will be made with.
static int solve_kept(rannc_dp_t *h, const rannc_dp_batch_t &b, hipStream_t st, bool info_only) {
  const size_t ws_bytes = h->ws_bytes;
  h->ws_bytes = h->kept.saved_at;
  h->call_total_bound = h->kept.total_bound;
  const int rc = solve_impl(h, &b, st, nullptr, nullptr, nullptr, nullptr, nullptr, 0, nullptr, nullptr, info_only);
  h->call_total_bound = 0;
  h->ws_bytes = ws_bytes;
  return rc;
}

// Whether the caller's stream is being recorded into a graph; the handle remembers that it was.
static bool recording(rannc_dp_t *h, hipStream_t st) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &status) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  if (status != hipStreamCaptureStatusNone) h->recorded = true;
  return status != hipStreamCaptureStatusNone;
}

// Enqueues what makes the tables of the last batch, if it was answered without them; work on this stream comes behind them, and
// work that a later call puts on another stream waits for them (tables_ev).  Where the caller's stream is being recorded they
// are made on a stream of the handle, and waited for: the recording holds what it would hold behind a call that had made them.
static int ensure_tables(rannc_dp_t *h, void *hip_stream) {
  hipStream_t st = (hipStream_t)hip_stream;
  const bool aside = recording(h, st);
  h->asked = h->to_host;
  if (!h->solved || (h->tabled && !h->tables_pending)) return RANNC_DP_OK;
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  if (aside && hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) {
    (void)hipGetLastError();
    return RANNC_DP_HIP_ERROR;
  }
  int rc = RANNC_DP_OK;
  if (!h->tabled) {
    if (aside) st = h->aux[0];
    const rannc_dp_batch_t b = kept_batch(h);
    if (!h->kept.sample.empty()) {  // (through the driver's mirror, which no call uses until it has waited for this)
      const int N = h->kept.N[0];
      const int64_t *const from = (const int64_t *)h->fs_pin_dev;
      if (from) std::memcpy(h->fs_pin, h->kept.sample.data(), 8 * h->kept.sample.size());
      if (!from || rannc::launch_form_inputs(from, from + 5 * (size_t)N, (int64_t *)(h->ws + h->kept.saved_at), N, h->Q, h->kept.comm,
                                             h->kept.split, st) != hipSuccess)
        rc = RANNC_DP_HIP_ERROR;
    }
    if (rc == RANNC_DP_OK) rc = solve_kept(h, b, st, false);
    if (rc == RANNC_DP_OK && hipEventRecord(h->tables_ev, st) != hipSuccess) rc = RANNC_DP_HIP_ERROR;
    h->solved = true;
    h->tabled = rc == RANNC_DP_OK;
    if (h->tabled) h->tables_pending = true;
    else (void)hipStreamSynchronize(st);  // nothing of it runs on, and it can be asked for again
  } else {
    const hipError_t e = hipEventQuery(h->tables_ev);
    if (e == hipSuccess) h->tables_pending = false;
    else if (e != hipErrorNotReady || (!aside && hipStreamWaitEvent(st, h->tables_ev, 0) != hipSuccess)) rc = RANNC_DP_HIP_ERROR;
    else (void)hipGetLastError();
  }
  if (rc == RANNC_DP_OK && aside && h->tables_pending) {
    if (hipEventSynchronize(h->tables_ev) == hipSuccess) h->tables_pending = false;
    else rc = RANNC_DP_HIP_ERROR;
  }
  if (aside) (void)hipThreadExchangeStreamCaptureMode(&mode);
  if (rc != RANNC_DP_OK) (void)hipGetLastError();
  return rc;
}

int rannc_dp_solve(rannc_dp_t *h, const rannc_dp_batch_t *b, void *hip_stream, int64_t *d_opt,
                   int32_t *d_n_stages, int64_t *d_est_iter_ns, int32_t *d_status) {
  if (!h || !d_opt || !d_n_stages) return RANNC_DP_INVALID_ARG;
  (void)recording(h, (hipStream_t)hip_stream);
  h->to_host = h->asked = false;
  h->direct = 0;
  return solve_impl(h, b, hip_stream, d_opt, d_n_stages, d_est_iter_ns, d_status, nullptr);
}

constexpr int kTracebackStagedMaxProblems = 64;
// outer driver: inputs of up to this many bytes are read by the kernels out of the pinned host mirror
constexpr size_t kFsReadInPlaceMax = 32 << 10;

int rannc_dp_solve_info(rannc_dp_t *h, rannc_dp_solve_info_t *out) {
  if (!h || !out) return RANNC_DP_INVALID_ARG;
  if (!h->solved) return RANNC_DP_BAD_STATE;
  if (!h->tabled) {  // answered without tables: what they will be made with
    const int rc = solve_kept(h, kept_batch(h), nullptr, true);
    if (rc != RANNC_DP_OK) return rc;
  }
  *out = h->info;
  return RANNC_DP_OK;
}

int rannc_dp_answered_without_tables(rannc_dp_t *h) {
  if (!h) return RANNC_DP_INVALID_ARG;
  if (!h->solved) return RANNC_DP_BAD_STATE;
  return h->direct;
}

static int traceback_impl(rannc_dp_t *h, void *hip_stream, const int32_t *d_levels, int32_t plan_stride,
                          int32_t *d_stage_end, int32_t *d_replicas,
                          const rannc::FormStageIn *form_stage,
                          const rannc::PlanResults *results = nullptr, bool choose = false) {
  if (!h || !d_stage_end || !d_replicas || plan_stride < 1) return RANNC_DP_INVALID_ARG;
  if (!h->solved) return RANNC_DP_BAD_STATE;
  // A few small min-max searches: the walk runs out of LDS (one round of reads instead of one
  // memory round trip per stage).  Many searches fill the device anyway, and a workgroup that holds
  // most of a compute unit's LDS would then only lower the number in flight.
  int64_t lds_bytes = 0;
  bool staged = h->Q <= kTracebackStagedMaxProblems;
  for (int q = 0; q < h->Q; ++q) {
    const ProblemDev &p = h->host_probs[q];
    if (p.S_eff > plan_stride) return RANNC_DP_INVALID_ARG;
    const int64_t need = rannc::traceback_lds_bytes(p.N, p.DP, p.S_eff, p.bits);
    staged = staged && !p.VF && need <= rannc::kTracebackLdsMax;
    lds_bytes = std::max(lds_bytes, need);
  }
  if (!staged) lds_bytes = 0;
  // The outer driver chooses one search and stage count itself and leaves those of the other searches
  // open.  (Done again by every recovery until the next solve: a call may be recorded and never run.)
  if ((h->unchosen && !form_stage && !choose &&
       rannc::launch_select(h->d_probs, h->Q, nullptr, nullptr, nullptr, nullptr, (hipStream_t)hip_stream) != hipSuccess) ||
      rannc::launch_traceback(h->d_probs, h->Q, plan_stride, d_stage_end, d_replicas, d_levels, lds_bytes, form_stage,
                              results, choose, (hipStream_t)hip_stream) != hipSuccess) {
    (void)hipGetLastError();
    return RANNC_DP_HIP_ERROR;
  }
  if (choose) h->unchosen = false;
  return RANNC_DP_OK;
}

int rannc_dp_traceback_at(rannc_dp_t *h, void *hip_stream, const int32_t *d_levels, int32_t plan_stride,
                          int32_t *d_stage_end, int32_t *d_replicas) {
  if (!h || !d_stage_end || !d_replicas || plan_stride < 1) return RANNC_DP_INVALID_ARG;
  const int rc = ensure_tables(h, hip_stream);
  if (rc != RANNC_DP_OK) return rc;
  return traceback_impl(h, hip_stream, d_levels, plan_stride, d_stage_end, d_replicas, nullptr);
}

int rannc_dp_traceback(rannc_dp_t *h, void *hip_stream, int32_t plan_stride, int32_t *d_stage_end,
                       int32_t *d_replicas) {
  return rannc_dp_traceback_at(h, hip_stream, nullptr, plan_stride, d_stage_end, d_replicas);
}

// ---- solve + plan recovery + results in host memory, as one call --------------------------------
namespace {

// Waits until every flag word holds seq: the last kernel of the call stores them behind its results
// in pinned host memory, which the host sees some microseconds before the stream reports completion.
// The stream is asked now and then, so that a failed launch ends the wait.
int wait_flags(hipStream_t st, const uint64_t *flags, int n, uint64_t seq) {
  for (int q = 0; q < n; ++q) {
    for (unsigned spins = 1; __atomic_load_n(&flags[q], __ATOMIC_ACQUIRE) != seq; ++spins) {
      __builtin_ia32_pause();
      if (spins % 8192) continue;
      const hipError_t e = hipStreamQuery(st);
      if (e == hipErrorNotReady) { (void)hipGetLastError(); continue; }
      if (e != hipSuccess || __atomic_load_n(&flags[q], __ATOMIC_ACQUIRE) != seq) {
        (void)hipGetLastError();
        return RANNC_DP_HIP_ERROR;
      }
    }
  }
  // (the runtime retires a stream's finished commands when it is asked to wait)
  if (seq % 64 == 0 && hipStreamSynchronize(st) != hipSuccess) {
    (void)hipGetLastError();
    return RANNC_DP_HIP_ERROR;
  }
  return RANNC_DP_OK;
}

}  // namespace

namespace {

// Whether the kernels are left to the library, and whether a call makes tables to the library alone.
bool library_chooses(const rannc_dp_t *h) {
  return !h->recorded && !h->asked && h->lim.algo == RANNC_DP_ALGO_AUTO && h->tune_spw == 0 && h->fused_small == 1 && !h->timing && h->staging_dev[h->next_slot];
}

// Where the copies of a batch's inputs go: behind the regions that its tables take.  False: the workspace has no such room,
// or none for the tables themselves (which then find that out).  shape(q): blocks, devices, stages of search q.
struct SearchShape { int N, D, S; };
extern "C++" template <typename Shape> bool room_for_inputs(const rannc_dp_t *h, int Q, Shape shape, size_t blocks, size_t *saved_at) {
  size_t need = header_bytes(h->lim.max_problems), last = 0;
  SearchShape before = {};
  for (int q = 0; q < Q; ++q) {
    const SearchShape x = shape(q);
    if (!q || x.N != before.N || x.D != before.D || x.S != before.S) {
      Sizes sz;
      if (!problem_sizes(x.N, x.D, rannc::dp_class(x.D), std::min(x.S, std::min(x.N, x.D)), h->bits, split_of(&h->lim), packed_of(&h->lim), &sz))
        return false;
      last = sz.total();
      before = x;
    }
    need += last;
  }
  const size_t saved = saved_bytes(blocks);
  if (need + saved > h->ws_bytes) return false;
  *saved_at = (h->ws_bytes - saved + kAlign) / kAlign * kAlign;
  return true;
}

// Whether a batch can be answered without its tables: searches that the kernels hold.
bool reach_applies(const rannc_dp_t *h, const rannc_dp_batch_t *b, size_t *saved_at) {
  if (!library_chooses(h) || !b->time_ns || !b->param_bytes || !b->act_bytes || split_of(&h->lim) != (b->time_bwd_ns != nullptr)) return false;
  const bool bound = b->time_bwd_ns || b->cut_bytes;
  if (bound && b->n_problems > kPollMaxProblems) return false;
  int longest = 0, widest = 0;
  for (int q = 0; q < b->n_problems; ++q) {
    longest = std::max(longest, b->n_blocks[q]);
    widest = std::max(widest, b->n_devices[q] * std::min(b->max_stages[q], b->n_devices[q]));
  }
  if (longest > (bound ? rannc::kBoundMaxBlocks : rannc::kReachMaxBlocks)) return false;
  // Every stage boundary sends, so where memory makes many of them the plan that the bound is taken from is a loose one, and the
  // levels take longer than the tables: 130 blocks at 12 devices in at most 12 stages 77 us with tables, 148 without; 400 at 24 in
  // 12 91 and 85, at 64 125 and 651.  With few devices or stages they do not: 260 at 6 in 6 53 and 45, 1000 at 12 in 4 62 and 41.
  // Up to 128 blocks the tables are one launch with one objective: 12 blocks at 6 devices 23 us, without tables 30; 130 at 6 in 6 49 and 55.
  if (b->cut_bytes && (widest > 64 || (!b->time_bwd_ns && longest <= 160))) return false;
  return room_for_inputs(h, b->n_problems, [&](int q) { return SearchShape{b->n_blocks[q], b->n_devices[q], b->max_stages[q]}; },
                         (size_t)(b->block_offset[b->n_problems] - b->block_offset[0]), saved_at);
}

// Enqueues the searches and keeps what makes their tables later.  The caller waits for them.
int reach_impl(rannc_dp_t *h, const rannc_dp_batch_t *b, hipStream_t st, int32_t plan_stride, const rannc::PlanResults &r, size_t saved_at) {
  const int Q = b->n_problems;
  const int slot = h->next_slot;
  if (h->staging_used[slot] && hipEventSynchronize(h->staging_free[slot]) != hipSuccess) {
    (void)hipGetLastError();
    return RANNC_DP_HIP_ERROR;
  }
  h->staging_used[slot] = false;
  h->solved = false;
  static_assert(sizeof(rannc::ReachIn) <= sizeof(ProblemDev), "the staging memory holds a descriptor per search");
  rannc::ReachIn *const in = (rannc::ReachIn *)h->staging[slot];
  LaunchShape sh = {};
  sh.nprob = Q;
  for (int q = 0; q < Q; ++q) {
    const int N = b->n_blocks[q], D = b->n_devices[q], S = std::min(b->max_stages[q], std::min(N, D));
    in[q] = {N, D, S, b->n_microbatches[q], b->mem_capacity[q], b->block_offset[q], b->cut_bytes ? b->bandwidth_bytes_per_us[q] : 1};
    sh.max_N = std::max(sh.max_N, N);
    sh.max_D = std::max(sh.max_D, D);
    sh.max_S_eff = std::max(sh.max_S_eff, S);
  }
  rannc::ReachArgs args = {};
  args.t = b->time_ns; args.p = b->param_bytes; args.a = b->act_bytes; args.o = b->cut_bytes; args.tb = b->time_bwd_ns;
  args.save = (int64_t *)(h->ws + saved_at);
  args.first = b->block_offset[0];
  args.blocks = b->block_offset[Q] - args.first;
  args.time_limit = h->lim.max_total_time_ns;
  args.plan_stride = plan_stride;
  args.results = r;
  const auto launch = args.o || args.tb ? rannc::launch_bound : rannc::launch_reach;
  if (launch((const rannc::ReachIn *)h->staging_dev[slot], Q == 1 ? in : nullptr, Q, sh, args, st) != hipSuccess) {
    (void)hipGetLastError();
    return RANNC_DP_HIP_ERROR;
  }
  h->ev_valid = false;
  h->level_launches = 0;
  try {
    h->kept.N.assign(b->n_blocks, b->n_blocks + Q);
    h->kept.D.assign(b->n_devices, b->n_devices + Q);
    h->kept.S.assign(b->max_stages, b->max_stages + Q);
    h->kept.MB.assign(b->n_microbatches, b->n_microbatches + Q);
    h->kept.M.assign(b->mem_capacity, b->mem_capacity + Q);
    h->kept.off.resize(Q + 1);
    for (int q = 0; q <= Q; ++q) h->kept.off[q] = b->block_offset[q] - b->block_offset[0];
    if (b->cut_bytes) h->kept.bw.assign(b->bandwidth_bytes_per_us, b->bandwidth_bytes_per_us + Q);
  } catch (...) {
    return RANNC_DP_NO_HOST_MEMORY;
  }
  h->kept.sample.clear();
  h->kept.comm = b->cut_bytes != nullptr;
  h->kept.split = b->time_bwd_ns != nullptr;
  h->kept.total_bound = 0;
  h->kept.saved_at = saved_at;
  return RANNC_DP_OK;
}

}  // namespace

int rannc_dp_solve_to_host(rannc_dp_t *h, const rannc_dp_batch_t *b, void *hip_stream, int32_t plan_stride,
                           void *d_results, void *h_results, size_t results_bytes) {
  if (!h || !b || !d_results || !h_results || plan_stride < 1 || ((uintptr_t)d_results % 8) || ((uintptr_t)h_results % 8))
    return RANNC_DP_INVALID_ARG;
  int rc = check_batch(&h->lim, b);
  if (rc != RANNC_DP_OK) return rc;
  const int Q = b->n_problems;
  for (int q = 0; q < Q; ++q)
    if (std::min(b->max_stages[q], std::min(b->n_blocks[q], b->n_devices[q])) > plan_stride) return RANNC_DP_INVALID_ARG;
  const ResultLayout at((size_t)Q, (size_t)plan_stride);
  if (results_bytes < at.total) return RANNC_DP_INVALID_ARG;
  hipStream_t st = (hipStream_t)hip_stream;
  char *d = (char *)d_results;
  rannc::PlanResults r = {};
  r.d_opt = (int64_t *)(d + at.opt); r.d_est = (int64_t *)(d + at.est);
  r.d_n_stages = (int32_t *)(d + at.n_stages); r.d_status = (int32_t *)(d + at.status);
  r.d_stage_end = (int32_t *)(d + at.stage_end); r.d_replicas = (int32_t *)(d + at.replicas);
  bool poll = Q <= kPollMaxProblems;
  const size_t need = at.total + 8 * (size_t)Q;
  if (poll && h->res_pin_bytes < need) {  // a longer stride than any plan of the handle
    char *grown = nullptr;
    if (hipHostMalloc((void **)&grown, need, hipHostMallocMapped | hipHostMallocPortable) != hipSuccess) {
      (void)hipGetLastError();
      return RANNC_DP_NO_HOST_MEMORY;
    }
    if (h->res_pin_own) (void)hipHostFree(h->res_pin);  // (no earlier call is under way: they all waited)
    h->res_pin_own = true;
    h->res_pin = grown;
    h->res_pin_bytes = need;
    std::memset(h->res_pin, 0, need);
    if (hipHostGetDevicePointer((void **)&h->res_pin_dev, h->res_pin, 0) != hipSuccess) {
      (void)hipGetLastError();
      h->res_pin_dev = nullptr;
    }
  }
  poll = poll && h->res_pin_dev;
  uint64_t *flags = nullptr;
  if (poll) {
    char *m = h->res_pin_dev;
    r.h_opt = (int64_t *)(m + at.opt); r.h_est = (int64_t *)(m + at.est);
    r.h_n_stages = (int32_t *)(m + at.n_stages); r.h_status = (int32_t *)(m + at.status);
    r.h_stage_end = (int32_t *)(m + at.stage_end); r.h_replicas = (int32_t *)(m + at.replicas);
    r.h_flag = (uint64_t *)(m + at.total);
    r.seq = ++h->seq;
    flags = (uint64_t *)(h->res_pin + at.total);
    // (a call of another layout may have left a result here that equals seq, which starts at 1)
    std::memset(flags, 0, 8 * (size_t)Q);
  }
  // the tables of a batch, or of a part of this one, and its results
  auto by_tables = [&](const rannc_dp_batch_t *which, const BatchPart *part) -> int {
    bool chosen = false, recovered = false;
    int rc = solve_impl(h, which, hip_stream, r.d_opt, r.d_n_stages, r.d_est, r.d_status, &chosen, plan_stride, poll ? &r : nullptr, &recovered, false, part);
    if (rc == RANNC_DP_OK && !recovered)
      rc = traceback_impl(h, hip_stream, nullptr, plan_stride, r.d_stage_end, r.d_replicas, nullptr, &r, !chosen);
    if (rc == RANNC_DP_OK && !poll &&
        (hipMemcpyAsync(h_results, d_results, at.total, hipMemcpyDeviceToHost, st) != hipSuccess ||
         hipStreamSynchronize(st) != hipSuccess)) {
      (void)hipGetLastError();
      rc = RANNC_DP_HIP_ERROR;
    }
    if (rc != RANNC_DP_OK) {
      (void)hipStreamSynchronize(st);  // the staging memory may be refilled by the next call
      return rc;
    }
    if (poll && part)
      for (size_t k = 0; k < part->place.size() && rc == RANNC_DP_OK; ++k) rc = wait_flags(st, flags + part->place[k], 1, r.seq);
    else if (poll)
      rc = wait_flags(st, flags, Q, r.seq);
    if (rc == RANNC_DP_OK && poll) std::memcpy(h_results, h->res_pin, at.total);
    return rc;
  };
  size_t saved_at = 0;
  const bool direct = reach_applies(h, b, &saved_at);
  h->to_host = true;
  h->asked = false;
  h->direct = 0;
  if (!direct) return by_tables(b, nullptr);
  rc = reach_impl(h, b, st, plan_stride, r, saved_at);
  if (rc == RANNC_DP_OK && !poll &&
      (hipMemcpyAsync(h_results, d_results, at.total, hipMemcpyDeviceToHost, st) != hipSuccess || hipStreamSynchronize(st) != hipSuccess)) {
    (void)hipGetLastError();
    rc = RANNC_DP_HIP_ERROR;
  }
  if (rc == RANNC_DP_OK && poll) rc = wait_flags(st, flags, Q, r.seq);
  if (rc != RANNC_DP_OK) {
    (void)hipStreamSynchronize(st);
    return rc;
  }
  const int32_t *const status = (const int32_t *)((poll ? h->res_pin : (const char *)h_results) + at.status);
  const int open = (int)std::count(status, status + Q, rannc::kReachUndecided);
  if (open) r.seq = ++h->seq;  // left to the tables
  if (open == Q) return by_tables(b, nullptr);
  if (open) {
    // Those of the open searches alone, in front of the copies of the inputs, as a batch of their own.  (With one of them in a
    // batch of many all tables would be made: 2 047 of 128 blocks and one of bytes beyond the kernel's range 1 790 us, so 290; 63 and one 323, so 121.)
    BatchPart part;
    std::vector<int32_t> N, D, S, MB;
    std::vector<int64_t> M, off, bw;
    try {
      off.push_back(0);
      for (int q = 0; q < Q; ++q) {
        if (status[q] != rannc::kReachUndecided) continue;
        part.place.push_back(q);
        part.first.push_back(b->block_offset[q]);
        N.push_back(b->n_blocks[q]); D.push_back(b->n_devices[q]); S.push_back(b->max_stages[q]); MB.push_back(b->n_microbatches[q]);
        M.push_back(b->mem_capacity[q]);
        off.push_back(off.back() + b->n_blocks[q]);
        bw.push_back(b->cut_bytes ? b->bandwidth_bytes_per_us[q] : 1);
      }
    } catch (...) {
      return RANNC_DP_NO_HOST_MEMORY;
    }
    rannc_dp_batch_t some = *b;
    some.n_problems = open;
    some.n_blocks = N.data(); some.n_devices = D.data(); some.max_stages = S.data(); some.n_microbatches = MB.data();
    some.mem_capacity = M.data(); some.block_offset = off.data();
    if (b->cut_bytes) some.bandwidth_bytes_per_us = bw.data();
    const size_t ws_bytes = h->ws_bytes;
    h->ws_bytes = saved_at;
    rc = by_tables(&some, &part);
    h->ws_bytes = ws_bytes;
    h->solved = false;  // (what stands in the workspace is a part)
    if (rc != RANNC_DP_OK) return rc;
  } else if (poll) {
    std::memcpy(h_results, h->res_pin, at.total);
  }
  h->Q = Q;
  h->solved = true;
  h->direct = Q - open;
  h->tabled = false;
  h->unchosen = false;
  return RANNC_DP_OK;
}

int rannc_dp_level_values(rannc_dp_t *h, void *hip_stream, int32_t stride, int64_t *d_values) {
  if (!h || !d_values || stride < 1) return RANNC_DP_INVALID_ARG;
  if (!h->solved) return RANNC_DP_BAD_STATE;
  const int rc = ensure_tables(h, hip_stream);
  if (rc != RANNC_DP_OK) return rc;
  for (int q = 0; q < h->Q; ++q)
    if (h->host_probs[q].S_eff > stride) return RANNC_DP_INVALID_ARG;
  if (rannc::launch_level_values(h->d_probs, h->Q, stride, d_values, (hipStream_t)hip_stream) != hipSuccess) {
    (void)hipGetLastError();
    return RANNC_DP_HIP_ERROR;
  }
  return RANNC_DP_OK;
}

// ---- Algorithm 2 ("form_stage"): host-level driver over one batched solve ---------------------
namespace {

struct FsPair { int n, MB; int64_t b; };

// the (n, MB) pairs Algorithm 2 can visit, in its order; false if the input is invalid
bool fs_pairs(const rannc_dp_form_stage_in_t *in, std::vector<FsPair> *out, int *max_D) {
  if (!in || in->n_blocks < 1 || in->n_nodes < 1 || in->devices_per_node < 1 || in->batch_size < 1 ||
      in->mem_capacity < 0 || in->reserved != 0)
    return false;
  if (in->cut_bytes_per_sample && in->bandwidth_bytes_per_us < 1) return false;
  *max_D = 0;
  for (int64_t n = 1; n <= in->n_nodes; n *= 2) {
    const int64_t D = (int64_t)in->devices_per_node * n;
    if (D > RANNC_DP_MAX_DEVICES) return false;
    *max_D = (int)D;
    const int64_t R = in->n_nodes / n;
    for (int64_t MB = 1; MB <= in->batch_size / R; MB *= 2) {
      if (out) out->push_back({(int)n, (int)MB, in->batch_size / R / MB});
      if (MB > (1 << 29)) break;
    }
  }
  return true;
}

size_t fs_scratch(int Q, int N, int stride) {
  size_t b = 0;
  b += 5 * align_up((size_t)Q * N * 8);       // scaled time, param, act, cut bytes, backward time
  b += 2 * align_up((size_t)Q * 8);           // opt, (n_stages + status as int32 pairs)
  b += 2 * align_up((size_t)Q * stride * 4);  // plans of the batch
  b += align_up(6 * 8 + (size_t)stride * 8);  // result record and the chosen plan (travels down)
  return b;
}

}  // namespace

namespace {

// The outer driver without the tables of its searches.  False: left to them, with whatever is wrong with the inputs.
// *rc: status of the call otherwise.
bool form_direct(rannc_dp_t *h, const rannc_dp_form_stage_in_t *in, const std::vector<FsPair> &pairs, int max_D, hipStream_t st,
                 rannc_dp_form_stage_out_t *out, int32_t *stage_end, int32_t *replicas, int32_t plan_stride, int *rc) {
  const int N = in->n_blocks, Q = (int)pairs.size(), per = in->devices_per_node;
  const bool comm = in->cut_bytes_per_sample != nullptr, split = in->time_bwd_per_sample_ns != nullptr;
  if (Q > kPollMaxProblems || N > rannc::kFormMaxBlocks || per > rannc::kFormMaxSpare || !h->fs_pin_dev || !h->res_pin_dev)
    return false;
  size_t saved_at = 0;
  if (!room_for_inputs(h, Q, [&](int q) { return SearchShape{N, per * pairs[q].n, per * pairs[q].n}; }, (size_t)Q * N, &saved_at)) return false;
  // ---- inputs within the exact range of the kernel, and persistent bytes alone: the fewest stages that hold them ----
  int64_t samples = 0;  // of the largest microbatch
  for (const FsPair &p : pairs) samples = std::max(samples, p.b);
  constexpr int64_t kBytes = (int64_t)1 << 46, kTime = (int64_t)1 << 44;
  int64_t time = 0, param = 0, act = 0, cut = 0, stage = 0;
  int fewest = 1;
  for (int k = 0; k < N; ++k) {
    const int64_t t = in->time_per_sample_ns[k], a = in->act_bytes_per_sample[k], p = in->param_bytes[k];
    const int64_t o = comm ? in->cut_bytes_per_sample[k] : 0, tb = split ? in->time_bwd_per_sample_ns[k] : 0;
    if (t < 0 || a < 0 || p < 0 || o < 0 || tb < 0 || t >= kTime || tb >= kTime || a >= kBytes || p >= kBytes || o >= kBytes) return false;
    time += t + tb;
    act += a;
    param += p;
    cut = std::max(cut, o);
    if (time >= kTime || act >= kBytes || param >= kBytes) return false;
    if (stage + p > in->mem_capacity) { stage = 0; ++fewest; }
    stage += p;  // (a block that fits no device by itself: more stages than there are, or none that the kernel finds)
  }
  if ((__int128)time * samples >= kTime || (__int128)act * samples >= kBytes || (__int128)cut * samples >= kBytes) return false;
  const int64_t send = comm ? (int64_t)(((__int128)cut * samples * 1000 + in->bandwidth_bytes_per_us - 1) / in->bandwidth_bytes_per_us) : 0;
  if (time * samples + send >= kTime || time * samples + send > h->lim.max_total_time_ns) return false;
  // ---- the searches whose stage counts can hold the chain ----
  const int stride = std::min(max_D, N);
  int64_t *const arrays = (int64_t *)h->fs_pin;  // per sample; the scratch's mirror has room for them and the descriptors
  const size_t arrays_bytes = 5 * 8 * (size_t)N;
  rannc::FormIn *const desc = (rannc::FormIn *)(h->fs_pin + arrays_bytes);
  int of[kPollMaxProblems], searches = 0;
  const size_t found_at = arrays_bytes + (size_t)Q * sizeof(rannc::FormIn);
  if (found_at + 8 * (size_t)Q > h->fs_pin_bytes) return false;
  for (int q = 0; q < Q; ++q) {
    const int lo = per * (pairs[q].n - 1) + 1, hi = std::min(per * pairs[q].n, N);
    if (hi < lo || hi < fewest) continue;
    desc[searches] = {per * pairs[q].n, std::max(lo, fewest), hi, __builtin_ctz((unsigned)pairs[q].n), pairs[q].b};
    of[searches++] = q;
  }
  const ResultLayout at((size_t)std::max(searches, 1), (size_t)stride);
  if (at.total + 8 * (size_t)searches > h->res_pin_bytes) return false;
  std::memcpy(arrays, in->time_per_sample_ns, 8 * (size_t)N);
  std::memcpy(arrays + N, in->param_bytes, 8 * (size_t)N);
  std::memcpy(arrays + 2 * N, in->act_bytes_per_sample, 8 * (size_t)N);
  if (comm) std::memcpy(arrays + 3 * N, in->cut_bytes_per_sample, 8 * (size_t)N);
  if (split) std::memcpy(arrays + 4 * N, in->time_bwd_per_sample_ns, 8 * (size_t)N);
  h->solved = false;
  h->ev_valid = false;
  h->level_launches = 0;
  const char *const m = h->res_pin;
  if (searches) {
    const int64_t *const dev = (const int64_t *)h->fs_pin_dev;
    rannc::FormArgs args = {};
    args.t = dev; args.p = dev + N; args.a = dev + 2 * N;
    args.o = comm ? dev + 3 * N : nullptr;
    args.tb = split ? dev + 4 * N : nullptr;
    args.pairs = (const rannc::FormIn *)(h->fs_pin_dev + arrays_bytes);
    args.M = in->mem_capacity; args.bw = comm ? in->bandwidth_bytes_per_us : 1;
    args.N = N; args.searches = searches; args.plan_stride = stride;
    char *const d = h->res_pin_dev;
    args.results.h_opt = (int64_t *)(d + at.opt);
    args.results.h_n_stages = (int32_t *)(d + at.n_stages);
    args.results.h_status = (int32_t *)(d + at.status);
    args.results.h_stage_end = (int32_t *)(d + at.stage_end);
    args.results.h_replicas = (int32_t *)(d + at.replicas);
    args.results.h_flag = (uint64_t *)(d + at.total);
    args.results.seq = ++h->seq;
    args.found = (uint64_t *)(h->fs_pin_dev + found_at);
    std::memset(h->fs_pin + found_at, 0, 8 * (size_t)searches);
    std::memset(h->res_pin + at.total, 0, 8 * (size_t)searches);  // (as in rannc_dp_solve_to_host)
    if (rannc::launch_form(searches, per, args, st) != hipSuccess) {
      (void)hipGetLastError();
      *rc = RANNC_DP_HIP_ERROR;
      return true;
    }
  }
  bool kept = true;
  try {
    h->kept.N.assign(Q, N);
    h->kept.D.resize(Q); h->kept.S.resize(Q); h->kept.MB.resize(Q); h->kept.off.resize(Q + 1);
    h->kept.sample.assign(5 * (size_t)N + (size_t)Q, 0);
    h->kept.M.assign(Q, in->mem_capacity);
    h->kept.bw.assign(Q, in->bandwidth_bytes_per_us);
  } catch (...) {
    kept = false;
  }
  if (kept) {
    for (int q = 0; q < Q; ++q) {
      h->kept.D[q] = h->kept.S[q] = per * pairs[q].n;
      h->kept.MB[q] = pairs[q].MB;
      h->kept.sample[5 * (size_t)N + q] = pairs[q].b;
      h->kept.off[q] = (int64_t)q * N;
    }
    h->kept.off[Q] = (int64_t)Q * N;
    std::memcpy(h->kept.sample.data(), arrays, (split ? 5 : comm ? 4 : 3) * 8 * (size_t)N);
    h->kept.comm = comm;
    h->kept.split = split;
    int64_t forward = 0;
    for (int k = 0; k < N; ++k) forward += in->time_per_sample_ns[k];
    h->kept.total_bound = std::max<int64_t>(forward * samples, 0);
    h->kept.saved_at = saved_at;
  }
  if (searches) *rc = wait_flags(st, (const uint64_t *)(m + at.total), searches, h->seq);
  else *rc = hipStreamSynchronize(st) == hipSuccess ? RANNC_DP_OK : RANNC_DP_HIP_ERROR;
  if (*rc == RANNC_DP_OK && !kept) *rc = RANNC_DP_NO_HOST_MEMORY;
  if (*rc != RANNC_DP_OK) {
    (void)hipStreamSynchronize(st);
    (void)hipGetLastError();
    return true;
  }
  // ---- Algorithm 2's loops: the first n with a plan, its fewest stages, the smallest estimate, the first search ----
  const int64_t *const value = (const int64_t *)(m + at.opt);
  const int32_t *const n_stages = (const int32_t *)(m + at.n_stages), *const status = (const int32_t *)(m + at.status);
  int pick = -1;
  int64_t best = 0;
  for (int k0 = 0, k1; k0 < searches && pick < 0; k0 = k1) {  // (n ascends)
    int open = INT32_MAX;  // fewest stages that a search of this n has left open
    for (k1 = k0; k1 < searches && pairs[of[k1]].n == pairs[of[k0]].n; ++k1) {
      if (status[k1] != RANNC_DP_PROBLEM_OK) { open = std::min(open, n_stages[k1]); continue; }
      if (n_stages[k1] == 0) continue;
      const int64_t f = (int64_t)pairs[of[k1]].MB + n_stages[k1] - 1;
      const int64_t est = value[k1] != 0 && f > INT64_MAX / value[k1] ? INT64_MAX : f * value[k1];
      if (pick < 0 || n_stages[k1] < n_stages[pick] || (n_stages[k1] == n_stages[pick] && est < best)) { pick = k1; best = est; }
    }
    if (open != INT32_MAX && (pick < 0 || open <= n_stages[pick])) return false;
  }
  h->Q = Q;
  h->solved = true;
  h->direct = Q;
  h->tabled = false;
  h->unchosen = false;
  std::memset(out, 0, sizeof(*out));
  for (int u = 0; u < plan_stride; ++u) stage_end[u] = replicas[u] = -1;
  if (pick < 0) return true;
  const FsPair &p = pairs[of[pick]];
  out->feasible = 1;
  out->n = p.n;
  out->devices = per * p.n;
  out->replica_factor = in->n_nodes / p.n;
  out->n_stages = n_stages[pick];
  out->n_microbatches = p.MB;
  out->stage_time_ns = value[pick];
  out->est_iter_ns = best;
  const int32_t *const se = (const int32_t *)(m + at.stage_end) + (size_t)pick * stride, *const rp = (const int32_t *)(m + at.replicas) + (size_t)pick * stride;
  for (int u = 0; u < std::min(stride, (int)plan_stride); ++u) { stage_end[u] = se[u]; replicas[u] = rp[u]; }
  return true;
}

}  // namespace

int32_t rannc_dp_form_stage_problems(const rannc_dp_form_stage_in_t *in) {
  std::vector<FsPair> pairs;
  int max_D = 0;
  try {
    if (!fs_pairs(in, &pairs, &max_D)) return 0;
  } catch (...) {
    return 0;
  }
  return (int32_t)pairs.size();
}

size_t rannc_dp_form_stage_scratch_bytes(const rannc_dp_form_stage_in_t *in) {
  const int Q = rannc_dp_form_stage_problems(in);
  int max_D = 0;
  if (Q == 0 || !fs_pairs(in, nullptr, &max_D)) return 0;
  return fs_scratch(Q, in->n_blocks, max_D);
}

int rannc_dp_form_stage(rannc_dp_t *h, const rannc_dp_form_stage_in_t *in, void *hip_stream,
                        void *d_scratch, size_t scratch_bytes, rannc_dp_form_stage_out_t *out,
                        int32_t *stage_end, int32_t *replicas, int32_t plan_stride) {
  if (!h || !in || !out || !stage_end || !replicas || !d_scratch) return RANNC_DP_INVALID_ARG;
  if (!in->time_per_sample_ns || !in->act_bytes_per_sample || !in->param_bytes) return RANNC_DP_INVALID_ARG;
  std::vector<FsPair> pairs;
  int max_D = 0;
  std::vector<int64_t> hbw, hM, hoff;
  const bool comm = in->cut_bytes_per_sample != nullptr;
  std::vector<int32_t> hN, hD, hS, hMB;
  const int N = in->n_blocks;
  try {
    if (!fs_pairs(in, &pairs, &max_D)) return RANNC_DP_INVALID_ARG;
  } catch (...) {
    return RANNC_DP_NO_HOST_MEMORY;
  }
  const int Q = (int)pairs.size();
  if (Q == 0) return RANNC_DP_INVALID_ARG;
  const bool split = in->time_bwd_per_sample_ns != nullptr;
  if (split != split_of(&h->lim)) return RANNC_DP_INVALID_ARG;
  const int stride = max_D;
  if (plan_stride < std::min(stride, N)) return RANNC_DP_INVALID_ARG;
  // before anything is sized by them (the batched solve would refuse the same)
  if (N > h->lim.max_blocks || max_D > h->lim.max_devices || Q > h->lim.max_problems ||
      std::min(N, max_D) > h->lim.max_stages)
    return RANNC_DP_LIMIT_EXCEEDED;
  const size_t need = fs_scratch(Q, N, stride);
  if (scratch_bytes < need) return RANNC_DP_WORKSPACE_TOO_SMALL;
  if (((uintptr_t)d_scratch % kAlign) != 0) return RANNC_DP_INVALID_ARG;
  hipStream_t st = (hipStream_t)hip_stream;
  // pinned host mirror of the device scratch: same layout, so inputs go up and results come down
  // in one copy each
  const size_t pin_need = need + 8;  // and the flag word behind it
  if (h->tables_pending) {  // they may be made from the mirror
    if (hipEventSynchronize(h->tables_ev) != hipSuccess) {
      (void)hipGetLastError();
      return RANNC_DP_HIP_ERROR;
    }
    h->tables_pending = false;
  }
  if (h->fs_pin_bytes < pin_need) {
    if (h->fs_pin) {
      if (hipStreamSynchronize(st) != hipSuccess) return RANNC_DP_HIP_ERROR;  // an earlier call's copies
      (void)hipHostFree(h->fs_pin);
      h->fs_pin = nullptr;
      h->fs_pin_dev = nullptr;
      h->fs_pin_bytes = 0;
    }
    if (hipHostMalloc((void **)&h->fs_pin, pin_need, hipHostMallocMapped | hipHostMallocPortable) != hipSuccess) {
      (void)hipGetLastError();
      h->fs_pin = nullptr;
      return RANNC_DP_NO_HOST_MEMORY;
    }
    h->fs_pin_bytes = pin_need;
    std::memset(h->fs_pin, 0, pin_need);
    // the device's view of the mirror; without one the call copies in both directions
    if (hipHostGetDevicePointer((void **)&h->fs_pin_dev, h->fs_pin, 0) != hipSuccess) {
      (void)hipGetLastError();
      h->fs_pin_dev = nullptr;
    }
  }
  const bool may = library_chooses(h);
  h->to_host = true;
  h->asked = false;
  h->direct = 0;
  int direct = RANNC_DP_OK;
  if (may && form_direct(h, in, pairs, max_D, st, out, stage_end, replicas, plan_stride, &direct)) return direct;
  try {
    if (comm) hbw.assign(Q, in->bandwidth_bytes_per_us);
    hM.assign(Q, in->mem_capacity); hoff.resize(Q + 1);
    hN.assign(Q, N); hD.resize(Q); hS.resize(Q); hMB.resize(Q);
  } catch (...) {
    return RANNC_DP_NO_HOST_MEMORY;
  }
  // layout of the scratch (device) and of its mirror (host)
  const size_t a_in = align_up((size_t)Q * N * 8);
  const size_t o_t = 0;
  const size_t o_p = o_t + a_in, o_a = o_t + 2 * a_in, o_o = o_t + 3 * a_in, o_b = o_t + 4 * a_in;
  const size_t o_opt = o_t + 5 * a_in;
  const size_t o_ns = o_opt + align_up((size_t)Q * 8);
  const size_t o_se = o_ns + align_up((size_t)Q * 8);
  const size_t o_rp = o_se + align_up((size_t)Q * stride * 4);
  const size_t o_rec = o_rp + align_up((size_t)Q * stride * 4);
  char *dev = (char *)d_scratch, *pin = h->fs_pin;
  int64_t *ht = (int64_t *)(pin + o_t), *hp = (int64_t *)(pin + o_p), *ha = (int64_t *)(pin + o_a);
  int64_t *ho = (int64_t *)(pin + o_o), *hb = (int64_t *)(pin + o_b);
  // per-microbatch inputs of every (n, MB): b samples on one pipeline replica
  const __int128 lim = (__int128)1 << 62;
  __int128 max_total = 0;  // largest total time of a search (forward, no communication term: what the
                           // kernels that care about it are restricted to)
  for (int q = 0; q < Q; ++q) {
    __int128 total = 0;
    hD[q] = in->devices_per_node * pairs[q].n;
    hS[q] = hD[q];
    hMB[q] = pairs[q].MB;
    hoff[q] = (int64_t)q * N;
    for (int k = 0; k < N; ++k) {
      const int64_t ts = in->time_per_sample_ns[k], as = in->act_bytes_per_sample[k];
      if (ts < 0 || as < 0 || in->param_bytes[k] < 0) return RANNC_DP_INVALID_ARG;
      if ((__int128)ts * pairs[q].b >= lim || (__int128)as * pairs[q].b >= lim) return RANNC_DP_OVERFLOW;
      ht[(size_t)q * N + k] = ts * pairs[q].b;
      total += (__int128)ts * pairs[q].b;
      ha[(size_t)q * N + k] = as * pairs[q].b;
      hp[(size_t)q * N + k] = in->param_bytes[k];
      if (split) {
        const int64_t tb = in->time_bwd_per_sample_ns[k];
        if (tb < 0) return RANNC_DP_INVALID_ARG;
        if ((__int128)tb * pairs[q].b >= lim) return RANNC_DP_OVERFLOW;
        hb[(size_t)q * N + k] = tb * pairs[q].b;
      }
      if (comm) {
        const int64_t os = in->cut_bytes_per_sample[k];
        if (os < 0) return RANNC_DP_INVALID_ARG;
        if ((__int128)os * pairs[q].b > (lim - 1) / 1000) return RANNC_DP_OVERFLOW;
        ho[(size_t)q * N + k] = os * pairs[q].b;
      }
    }
    max_total = std::max(max_total, total);
  }
  hoff[Q] = (int64_t)Q * N;
  // The block arrays in use are contiguous: one copy up.  Small inputs (the paper's 32 blocks: 18 KB) are
  // not copied at all: the mirror is pinned host memory that the device reads through the same address,
  // which costs the kernels a bus round trip and saves the call a copy in front of its first kernel.
  const size_t in_bytes = o_t + (split ? 5 : comm ? 4 : 3) * a_in;
  char *pin_dev = h->fs_pin_dev;
  const bool in_place = pin_dev && in_bytes <= kFsReadInPlaceMax;
  if (!in_place && hipMemcpyAsync(dev, pin, in_bytes, hipMemcpyHostToDevice, st) != hipSuccess) {
    (void)hipGetLastError();
    return RANNC_DP_HIP_ERROR;
  }
  const char *src = in_place ? pin_dev : dev;
  int64_t *d_opt = (int64_t *)(dev + o_opt);
  int32_t *d_ns = (int32_t *)(dev + o_ns), *d_st = d_ns + Q;
  int32_t *d_se = (int32_t *)(dev + o_se), *d_rp = (int32_t *)(dev + o_rp);
  // the result record and the chosen plan behind it are written by the kernels straight into the
  // mirror (they only write it): no copy down, the wait for the stream is all that is left
  int64_t *d_rec = (int64_t *)((pin_dev ? pin_dev : dev) + o_rec);
  rannc_dp_batch_t b;
  b.n_problems = Q;
  b.n_blocks = hN.data(); b.n_devices = hD.data(); b.max_stages = hS.data();
  b.n_microbatches = hMB.data(); b.mem_capacity = hM.data(); b.block_offset = hoff.data();
  b.time_ns = (const int64_t *)(src + o_t); b.param_bytes = (const int64_t *)(src + o_p);
  b.act_bytes = (const int64_t *)(src + o_a);
  b.bandwidth_bytes_per_us = comm ? hbw.data() : nullptr;
  b.cut_bytes = comm ? (const int64_t *)(src + o_o) : nullptr;
  b.time_bwd_ns = split ? (const int64_t *)(src + o_b) : nullptr;
  // Everything on the device, in stream order: the batched search, then one launch that runs Algorithm
  // 2's loops over the values V[S][N][D] of every search and S (first n, then first S with a feasible
  // MB; among those the smallest (MB + S - 1) * V, the first found among equals), recovers the plan of
  // the chosen (n, MB, S) and writes record, plan and flag word into the mirror.
  rannc::FormStageIn f = {};
  f.Q = Q; f.N = N; f.devices_per_node = in->devices_per_node;
  f.rec = d_rec;
  if (pin_dev) {
    f.flag = (uint64_t *)(pin_dev + need);
    f.seq = ++h->seq;
    std::memset(pin + need, 0, 8);  // an earlier call's inputs may have stood here
  }
  bool chosen = false;
  h->call_total_bound = max_total < lim ? (int64_t)max_total : 0;
  int rc = solve_impl(h, &b, hip_stream, d_opt, d_ns, nullptr, d_st, &chosen);
  h->call_total_bound = 0;
  if (rc == RANNC_DP_OK) rc = traceback_impl(h, hip_stream, nullptr, stride, d_se, d_rp, &f);
  if (rc != RANNC_DP_OK) {
    (void)hipStreamSynchronize(st);  // the mirror may be refilled by the next call
    return rc;
  }
  if (pin_dev) {
    rc = wait_flags(st, (const uint64_t *)(pin + need), 1, f.seq);
    if (rc != RANNC_DP_OK) return rc;
  } else if (hipMemcpyAsync(pin + o_rec, dev + o_rec, 6 * 8 + (size_t)stride * 8, hipMemcpyDeviceToHost, st) != hipSuccess ||
             hipStreamSynchronize(st) != hipSuccess) {
    (void)hipGetLastError();
    return RANNC_DP_HIP_ERROR;
  }
  const int64_t *rec = (const int64_t *)(pin + o_rec);
  const int stq = (int)rec[2];
  if (stq == RANNC_DP_PROBLEM_NEGATIVE_INPUT) return RANNC_DP_INVALID_ARG;
  if (stq != RANNC_DP_PROBLEM_OK) return RANNC_DP_OVERFLOW;  // sums or times beyond the handle's width
  std::memset(out, 0, sizeof(*out));
  for (int u = 0; u < plan_stride; ++u) stage_end[u] = replicas[u] = -1;
  const int q_sel = (int)rec[0], S_sel = (int)rec[1];
  if (q_sel < 0) return RANNC_DP_OK;  // infeasible: out->feasible = 0
  const int32_t *hse = (const int32_t *)(rec + 6), *hrp = hse + stride;
  out->feasible = 1;
  out->n = pairs[q_sel].n;
  out->devices = hD[q_sel];
  out->replica_factor = in->n_nodes / pairs[q_sel].n;
  out->n_stages = S_sel;
  out->n_microbatches = pairs[q_sel].MB;
  out->stage_time_ns = rec[4];
  out->est_iter_ns = rec[5];
  for (int u = 0; u < std::min(stride, (int)plan_stride); ++u) { stage_end[u] = hse[u]; replicas[u] = hrp[u]; }
  return RANNC_DP_OK;
}

size_t rannc_dp_compact_workspace_bytes(int32_t n_groups) {
  if (n_groups < 1 || n_groups > 65535) return 0;
  return rannc::compact_workspace_bytes(n_groups);
}

int rannc_dp_compact(void *hip_stream, int32_t n_groups, int32_t k, int32_t max_walks, int64_t mem_capacity,
                     const int64_t *d_time_ns, const int64_t *d_param_bytes, const int64_t *d_act_bytes,
                     void *d_workspace, size_t workspace_bytes, int32_t *d_n_blocks, int32_t *d_block_end,
                     int64_t *d_time_out, int64_t *d_param_out, int64_t *d_act_out, int32_t *d_status) {
  if (n_groups < 1 || n_groups > 65535 || k < 1 || max_walks < 0 || mem_capacity < 0) return RANNC_DP_INVALID_ARG;
  if (!d_time_ns || !d_param_bytes || !d_act_bytes || !d_workspace || !d_n_blocks || !d_block_end ||
      !d_time_out || !d_param_out || !d_act_out || !d_status)
    return RANNC_DP_INVALID_ARG;
  if (((uintptr_t)d_workspace % kAlign) != 0) return RANNC_DP_INVALID_ARG;
  if (workspace_bytes < rannc::compact_workspace_bytes(n_groups)) return RANNC_DP_WORKSPACE_TOO_SMALL;
  if (rannc::launch_compact(n_groups, k, mem_capacity, max_walks, d_time_ns, d_param_bytes, d_act_bytes,
                            d_workspace, d_n_blocks, d_block_end, d_time_out, d_param_out, d_act_out, d_status,
                            (hipStream_t)hip_stream) != hipSuccess) {
    (void)hipGetLastError();
    return RANNC_DP_HIP_ERROR;
  }
  return RANNC_DP_OK;
}

// ---- compaction for callers that cannot allocate: workspace in a static device array ----------
namespace {

constexpr size_t kCompactStaticBytes = rannc::compact_workspace_bytes(RANNC_DP_COMPACT_STATIC_MAX_GROUPS);
// Workspace of rannc_dp_compact_static.  Every device the library runs on holds its own copy at its
// own address until the process ends; host code never uses this name as an address (it is only a
// handle for hipGetSymbolAddress), kernels get the looked-up pointer as an argument.
static __device__ __align__(256) unsigned char scratch[kCompactStaticBytes];

constexpr int kMaxDevicesPerProcess = 64;
std::atomic<void *> scratch_of_device[kMaxDevicesPerProcess];

// Device address of `scratch` on the current device, looked up once per device.
int static_scratch(void **out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevicesPerProcess) {
    (void)hipGetLastError();
    return RANNC_DP_HIP_ERROR;
  }
  void *ptr = scratch_of_device[dev].load(std::memory_order_acquire);
  if (!ptr) {
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
      (void)hipGetLastError();
      return RANNC_DP_HIP_ERROR;
    }
    scratch_of_device[dev].store(ptr, std::memory_order_release);  // two racing threads store the same address
  }
  *out = ptr;
  return RANNC_DP_OK;
}

}  // namespace

int rannc_dp_compact_static(void *hip_stream, int32_t n_groups, int32_t k, int32_t max_walks, int64_t mem_capacity,
                            const int64_t *d_time_ns, const int64_t *d_param_bytes, const int64_t *d_act_bytes,
                            int32_t *d_n_blocks, int32_t *d_block_end, int64_t *d_time_out, int64_t *d_param_out,
                            int64_t *d_act_out, int32_t *d_status) {
  if (n_groups < 1 || k < 1 || max_walks < 0 || mem_capacity < 0) return RANNC_DP_INVALID_ARG;
  if (n_groups > RANNC_DP_COMPACT_STATIC_MAX_GROUPS) return RANNC_DP_LIMIT_EXCEEDED;
  if (!d_time_ns || !d_param_bytes || !d_act_bytes || !d_n_blocks || !d_block_end || !d_time_out ||
      !d_param_out || !d_act_out || !d_status)
    return RANNC_DP_INVALID_ARG;
  void *ws = nullptr;
  const int rc = static_scratch(&ws);
  if (rc != RANNC_DP_OK) return rc;
  // the kernel initialises every word of the workspace it later reads, so nothing has to be cleared
  if (rannc::launch_compact(n_groups, k, mem_capacity, max_walks, d_time_ns, d_param_bytes, d_act_bytes, ws,
                            d_n_blocks, d_block_end, d_time_out, d_param_out, d_act_out, d_status,
                            (hipStream_t)hip_stream) != hipSuccess) {
    (void)hipGetLastError();
    return RANNC_DP_HIP_ERROR;
  }
  return RANNC_DP_OK;
}

int rannc_dp_read_table(rannc_dp_t *h, int which, int32_t problem, void *d_dst, size_t bytes,
                        void *hip_stream) {
  if (!h || !d_dst) return RANNC_DP_INVALID_ARG;
  if (!h->solved) return RANNC_DP_BAD_STATE;
  if (problem < 0 || problem >= h->Q) return RANNC_DP_INVALID_ARG;
  const int made = ensure_tables(h, hip_stream);
  if (made != RANNC_DP_OK) return made;
  const int pos = h->pos_of[problem];
  const ProblemDev &p = h->host_probs[pos];
  const size_t tri = (size_t)p.N * (size_t)(p.N + 1) / 2 * (size_t)p.D;
  const size_t cells = (size_t)(p.S_eff + 1) * (size_t)(p.N + 1) * (size_t)(p.D + 1);
  size_t want = 0;
  switch (which) {
    case RANNC_DP_TABLE_COST_BWD:
      if (!p.costb) return RANNC_DP_INVALID_ARG;
      want = tri * 8;
      break;
    case RANNC_DP_TABLE_MAX_FWD:
    case RANNC_DP_TABLE_MAX_BWD:
      if (!p.VF) return RANNC_DP_INVALID_ARG;
      want = cells * 8;
      break;
    case RANNC_DP_TABLE_COST: want = tri * 8; break;
    case RANNC_DP_TABLE_FIT: want = tri; break;
    case RANNC_DP_TABLE_V: want = cells * 8; break;
    case RANNC_DP_TABLE_ARG_I:
    case RANNC_DP_TABLE_ARG_D: want = cells * 4; break;
    default: return RANNC_DP_INVALID_ARG;
  }
  if (bytes != want) return RANNC_DP_INVALID_ARG;
  hipStream_t st = (hipStream_t)hip_stream;
  bool ok = true;
  int cls = 0;
  while (cls < 3 && p.DP != (8 << cls)) ++cls;
  if (h->no_times[cls] && (which == RANNC_DP_TABLE_COST || which == RANNC_DP_TABLE_COST_BWD || which == RANNC_DP_TABLE_ARG_I || which == RANNC_DP_TABLE_ARG_D)) {
    // the solve recomputed the stage times instead of tabulating them: tabulate this search's now
    LaunchShape one;
    one.nprob = 1; one.max_N = p.N; one.max_nch = p.nch; one.max_D = p.D; one.max_S_eff = p.S_eff; one.wide_rows = 0; one.wide_chunks = 0;
    ok = rannc::launch_build(h->d_probs + pos, one, p.bits, p.DP, 2, st) == hipSuccess;
  }
  ok = ok && rannc::launch_export(h->d_probs + pos, which, p.bits, d_dst, st) == hipSuccess;
  if (which == RANNC_DP_TABLE_ARG_I || which == RANNC_DP_TABLE_ARG_D) {
    LaunchShape sh;
    sh.nprob = 1; sh.max_N = p.N; sh.max_nch = p.nch; sh.max_D = p.D; sh.max_S_eff = p.S_eff; sh.wide_rows = 0; sh.wide_chunks = 0;
    int32_t *ai = which == RANNC_DP_TABLE_ARG_I ? (int32_t *)d_dst : nullptr;
    int32_t *ad = which == RANNC_DP_TABLE_ARG_D ? (int32_t *)d_dst : nullptr;
    for (int s = 2; s <= p.S_eff && ok; ++s)
      ok = (p.VF ? rannc::launch_level_split(h->d_probs + pos, sh, p.bits, s, 0, ai, ad, st)
                 : rannc::launch_level_scan(h->d_probs + pos, sh, p.bits, s, 0, ai, ad, st)) == hipSuccess;
  }
  if (!ok) {
    (void)hipGetLastError();
    return RANNC_DP_HIP_ERROR;
  }
  return RANNC_DP_OK;
}

}  // extern "C"
