// gfx950 kernels of the stage-level partition search (RaNNC Sec. III-C, Algorithm 1).
//
// One wavefront is 64 lanes; in every kernel that touches the stage-time table a lane owns one
// output column j (blocks 1..j covered), so table rows are read with coalesced requests and no
// value ever has to cross lanes.  All arithmetic is exact unsigned integer arithmetic.
//
// A problem whose inputs failed validation (status word != 0) still runs through the table and
// level kernels: every access stays inside the problem's own regions, and its values are never
// reported (the final selection, the plan recovery and the exports check the status word).
#include "rannc_dp_device.h"
#include "rannc_dp_once.h"
#include "rannc_dp_worklist.h"

#include <type_traits>

namespace rannc {

// ---------------------------------------------------------------------------------------
// Stage-time and fits-in-memory tables: h(i,j,r) and the m(i,j,r) <= M rule of Sec. III-C for
// every stage (i,j) and replica count r.  One wave per unit (row i, 64-column chunk c), four
// rows per workgroup; a lane
// owns one j and writes its D entries, each store instruction covering 64 consecutive columns
// of one contiguous unit.  Memory is non-increasing in r, so the fit rule is stored as the
// smallest fitting r and folded into the time table as INF below it (within units that hold at
// least one fitting stage; the others keep only their rmin bytes).  Row i = 0 is also level 1
// of the DP (one stage on d devices), written here.
// ---------------------------------------------------------------------------------------
constexpr int kBuildWaves = 4;

// ceil(x / r) for every r = 1..DP of a 32-bit x, without integer division: for odd r one
// double-precision add and one fused multiply-add whose low word is the quotient (the derivation
// stands at CeilDiv), for even r an add and a shift from ceil(x / (r/2)).
template <int DP>
__device__ __forceinline__ void ceil_div_all(uint32_t x, uint32_t (&q)[DP + 1]) {
  const double xf = (double)x;
  double magic = 0x1.8p52;
  asm("" : "+v"(magic));  // one register for all entries instead of a literal per instruction
#pragma unroll
  for (int r = 1; r <= DP; ++r) {
    if (r & 1) {
      const double add = (double)r / 2.0 - 1.0 + (double)r * 0x1p-18;
      const double y = __builtin_fma(xf + add, 1.0 / (double)r, magic);
      q[r] = (uint32_t)__double_as_longlong(y);
    } else {
      q[r] = (q[r / 2] + 1u) >> 1;
    }
  }
}

// The D entries of one stage (i,j): ceil(tij / r) (+ ceil(cj / r) with the communication term), INF
// below rmin.  NODIV: 32-bit values take the division-free form above (the table builder was bound
// by the quarter-rate integer multiplies of 64 divisions by constants per stage, not by its stores;
// the one-launch kernel, which has 128 registers per lane, keeps the integer form).  Otherwise r is
// a compile-time constant after unrolling, so the divisions are multiplications.
template <typename VT, int DP, bool COMM, bool NODIV>
__device__ __forceinline__ void build_rows(VT tij, VT cj, int rmin, int D, VT RANNC_GLOBAL *crow, VT *lds1) {
  constexpr bool FAST = NODIV && sizeof(VT) == 4;
  [[maybe_unused]] uint32_t qt[DP + 1], qc[DP + 1];
  if constexpr (FAST) {
    ceil_div_all<DP>((uint32_t)tij, qt);
    if (COMM) ceil_div_all<DP>((uint32_t)cj, qc);
  }
  auto entry = [&](const int r) -> VT {  // r is a compile-time number wherever this is called
    VT h;
    if constexpr (FAST) {
      h = qt[r];
      if (COMM) h += qc[r];
    } else {
      const VT q = tij / (VT)r;
      h = q + (VT)(q * (VT)r != tij);  // ceil
      if (COMM) {
        const VT qq = cj / (VT)r;
        h += qq + (VT)(qq * (VT)r != cj);
      }
    }
    return (r >= rmin) ? h : Lim<VT>::inf;
  };
  // one straight run of stores per destination; r <= D is a scalar test (every r keeps its own
  // code: the quotient arrays stay in registers only with compile-time indices)
  if (crow) {
#pragma unroll
    for (int r = 1; r <= DP; ++r)
      if (r <= D) crow[(r - 1) * 64] = entry(r);
  }
  if (lds1) {
#pragma unroll
    for (int r = 1; r <= DP; ++r)
      if (r <= D) lds1[r - 1] = entry(r);
  }
}

// ---------------------------------------------------------------------------------------
// Passes of the recomputing level kernel.
//
// ends[i] is the last block a stage that starts behind block i can take and still fit (for some r <= D;
// i itself if not even one block fits).  Memory grows with the stage, so the stages (i, j) of row i
// that fit are exactly j = i+1 .. ends[i], and ends[] never decreases.  The level kernel works on the stages
// that fit and on nothing else: those of chunk c, row by row from the window's first row on, are numbered
// through, and a PASS is sixty-four of them in a row, a lane each, whatever rows they come from.  (With a
// pass per row, two rows to a pass in the diagonal block, 20 % of the lanes idled at 1024 blocks where a
// stage spans 115 of them, 26 % over the searches of 128 blocks that span 46, half where the last
// chunk is a third full.)
//
// Stages of the chunk in rows w .. i-1, with X = min(64c+64, N) and the first row `full` whose stages reach X:
//     sum over those rows of min(ends, X) - max(row, 64c)
// in closed form from the running sums of ends[] (stages_before).
//
// Per pass 64 words { row, column in the chunk << 16, smallest r that fits << 22 }, all ones behind the
// chunk's last stage, then the 64 stages' times at one replica.  They live in the region of the
// stage-time table, which a search that recomputes the times does not build (a table that is asked for
// later replaces them, and the next solve writes them again).
// ---------------------------------------------------------------------------------------
template <typename VT> constexpr int pass_bytes() { return 64 * (4 + (int)sizeof(VT)); }

__device__ __forceinline__ uint32_t *pass_chunks(const ProblemDev &pr) { return (uint32_t *)pr.wlo + pr.nch; }

// The entries of row i in chunk c, by one wave; fits: the lane's stage fits, from rmin replicas on.
// w, rec, esum: the chunk's window, its share of the list and the running sums of ends[].
template <typename VT, typename EP>
__device__ __forceinline__ void pass_entries(const ProblemDev &pr, int i, int c, int lane, bool fits, int rmin, VT tij, int w,
                                             const PassChunk &rec, EP esum) {
  const int N = pr.N, b = 64 * c, hi = min(b + 63, N - 1);
  if (i < w) return;
  const uint32_t full = rec.full, base = rec.base, start = rec.start, per = rec.per;
  const uint32_t first = stages_before(esum, N, c, (uint32_t)w, full, (uint32_t)i);
  const uint32_t all = stages_before(esum, N, c, (uint32_t)w, full, (uint32_t)hi + 1u);
  char *const passes = (char *)pr.cost + (int64_t)base * pass_bytes<VT>();
  auto word_at = [&](uint32_t at) { return (uint32_t *)(passes + (int64_t)(at >> 6) * pass_bytes<VT>()) + (at & 63u); };
  if (fits) {
    const uint32_t at = first + (uint32_t)(b + lane - max(i, b)), q = at >> 6;
    *word_at(at) = (uint32_t)i | (uint32_t)lane << 16 | (uint32_t)rmin << 22;
    ((VT *)(passes + (int64_t)q * pass_bytes<VT>() + 256))[at & 63u] = tij;
    // the work list: the rows of an item's first passes, one for each wave, and the item itself
    const bool begins = (at & 63u) == 0u, ends = (at & 63u) == 63u || at == all - 1u;
    if (begins || ends) {
      const uint32_t item = q / per, slot = q - item * per;
      uint32_t *const list = (uint32_t *)pr.runs + kPassItemWords * (1 + start + item);
      if (begins && slot == 0) {
        const uint32_t n = min(per, ((all + 63u) >> 6) - q);
        list[0] = base + q;
        list[1] = (uint32_t)c | (n - 1u) << 16;
      }
      if (slot < (uint32_t)kMergeWaves) {
        if (begins) ((uint16_t *)(list + 2 + slot))[0] = (uint16_t)i;
        if (ends) ((uint16_t *)(list + 2 + slot))[1] = (uint16_t)i;
      }
    }
  }
  if (i == hi) {
    const uint32_t at = all + (uint32_t)lane;
    if ((at >> 6) == ((all - 1u) >> 6)) *word_at(at) = ~0u;
  }
}

// One unit (row i, chunk c) of the tables, by one wave.  T, P, A, Cc may live in global memory or in
// LDS; Cc (per-cut send time at one replica, Cc[N] = 0) is null when there is no communication
// term.  Returns whether any stage of the unit fits.  Row 0's entries are level 1 of V: with
// lds_level1 given they go to LDS, row (j - row0) with row stride ls, and the caller copies them to
// the value table (a lane's D values are a row of V, so writing them from here would scatter every
// store instruction over 64 cache lines).  with_times = false: only the fits-in-memory part (rmin,
// ufit) and level 1 are produced, for searches whose level kernel recomputes the stage times.
// stages: what the lists of stages that fit want to know of the lane's stage.
template <typename VT> struct UnitStages { bool fits; int rmin; VT tij; };
template <typename VT, int DP, bool NODIV = false>
__device__ __forceinline__ bool build_unit(const ProblemDev &pr, const int64_t *T, const int64_t *P,
                                           const int64_t *A, const int64_t *Cc, int i, int c, int lane,
                                           VT *lds_level1, int ls, int row0, const int64_t *TBp = nullptr,
                                           const bool with_times = true, UnitStages<VT> *stages = nullptr) {
  const int N = pr.N, D = pr.D, nch = pr.nch;
  const int jj = 64 * c + lane;
  const bool valid = (jj >= i) && (jj < N);
  const int j = valid ? jj + 1 : i + 1;  // padding lanes compute a harmless in-range stage
  const int64_t Tij = T[j] - T[i];
  const int64_t Pij = P[j] - P[i];
  const int64_t Aij = A[j] - A[i];
  // smallest r with Pij + ceil(Aij / r) <= M, using ceil(a/r) <= k  <=>  a <= k*r
  int rmin = 255;
  if (Pij <= pr.M) {
    const int64_t slack = pr.M - Pij;
    if (Aij <= slack) rmin = 1;
    else if (slack > 0) {
      const int need = ceil_ratio((uint64_t)Aij, (uint64_t)slack, __builtin_amdgcn_rcpf((float)slack));
      if (need <= D) rmin = need;
    }
  }
  const bool fits = valid && rmin <= D;
  const bool unit_fits = __ballot(fits) != 0ull;
  const int64_t u = unit_index(nch, i, c);
  if (lane == 0) pr.ufit[u] = (uint8_t)unit_fits;
  if (stages) *stages = {fits, rmin, (VT)Tij};
  if (!valid) return unit_fits;
  pr.rmin[u * 64 + lane] = (uint8_t)rmin;
  // A unit in which no stage fits for any r is never read (every reader consults ufit or rmin
  // first): only those are written.  Row 0 also carries level 1 and is always written.
  if (!unit_fits && i != 0) return unit_fits;
  if (!with_times && !(i == 0 && lds_level1)) return unit_fits;
  VT RANNC_GLOBAL *crow = with_times ? gptr((VT *)pr.cost) + u * 64 * D + lane : nullptr;
  VT *lds1 = (i == 0 && lds_level1) ? lds_level1 + (j - row0) * ls : nullptr;
  const VT tij = (VT)Tij;
  if (Cc)  // wave-uniform: with the stage's own send time at one replica (0 for j = N)
    build_rows<VT, DP, true, NODIV>(tij, (VT)Cc[j], rmin, D, crow, lds1);
  else
    build_rows<VT, DP, false, NODIV>(tij, (VT)0, rmin, D, crow, lds1);
  if (TBp && with_times)  // split objective: the backward times get a table of their own (never a send time)
    build_rows<VT, DP, false, NODIV>((VT)(TBp[j] - TBp[i]), (VT)0, rmin, D,
                              gptr((VT *)pr.costb) + u * 64 * D + lane, nullptr);
  return unit_fits;
}

// parts: 1 = fits-in-memory tables and level 1 of V only, 3 = those and the stage-time table,
// 2 = the stage-time table alone (added later to a search that was solved without it)
// A wave takes `rows` consecutive rows of one chunk, one after the other: one row when the
// stage-time table is written (64 row stores per unit keep it busy), several when only the
// fits-in-memory part is (a unit is then 65 bytes of output, and a launch of one wave per unit is
// bound by the rate at which waves can be started).
// (The several-rows variant is held to the registers of four waves per SIMD: its time goes into the
// latency of many short units, and the 64 quotients of row 0, the only row that needs them there,
// would otherwise halve the waves in flight at 64 devices.)
template <typename VT, int DP, int ROWS>
__global__ __launch_bounds__(64 * kBuildWaves) __attribute__((amdgpu_waves_per_eu(ROWS > 1 ? 4 : 1)))
void build_kernel(const ProblemDev *__restrict__ probs, const int parts, const int pr_many) {
  // Workgroups go to the eight XCDs round-robin in the order of their linear index.  A launch over
  // several searches has grid = (searches, row groups, chunks): the search runs fastest and every
  // XCD gets rows of every chunk (with the chunk fastest and two chunks per search, the XCDs with
  // even numbers would get the triangle of chunk 0 and the others the three times larger chunk 1:
  // config 5, fits-in-memory part, 59 -> 39 us).  One search: grid = (chunks, row groups, 1).
  const bool many = pr_many != 0;
  const ProblemDev &pr = probs[many ? blockIdx.x : 0];
  const int lane = threadIdx.x & 63;
  const int i0 = (blockIdx.y * kBuildWaves + (int)(threadIdx.x >> 6)) * ROWS, c = many ? blockIdx.z : blockIdx.x;
  __shared__ VT tile[64 * (DP + 1)];  // level 1 of this chunk (only the wave that holds row 0 uses it)
  if (c >= pr.nch) return;
  auto one_row = [&](const int i) {
    const bool level1 = i == 0 && (parts & 1);
    (void)build_unit<VT, DP, true>(pr, pr.T, pr.P, pr.A, pr.C, i, c, lane, level1 ? tile : nullptr, DP + 1, 64 * c + 1,
                                   pr.TB, (parts & 2) != 0);
    if (level1) {
      // rows j = 64c+1 .. of level 1 are contiguous in V: written with consecutive lanes on
      // consecutive words (columns d > D keep the zeros of the fill)
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      const int D = pr.D, nrow = min(64, pr.N - 64 * c);
      VT RANNC_GLOBAL *v1 = gptr((VT *)pr.V) + (int64_t)(64 * c + 1) * DP;
      for (int e = lane; e < nrow * DP; e += 64) {
        const int row = e / DP, col = e % DP;
        if (col < D) v1[e] = tile[row * (DP + 1) + col];
      }
    }
  };
  if constexpr (ROWS == 1) {
    // straight-line: the wave ends behind its last store without waiting for it
    if (i0 < pr.N && c >= (i0 >> 6)) one_row(i0);
  } else {
#pragma unroll 1
    for (int i = i0; i < min(i0 + ROWS, pr.N); ++i) {
      if (c < (i >> 6)) break;  // the rows from here on have no column in this chunk
      one_row(i);
    }
  }
}

// whether bytes P (not divided) + ceil(A / D) fit M
__device__ __forceinline__ bool fits_at(uint64_t P, uint64_t A, uint64_t M, int D) {
  if (P > M) return false;
  const uint64_t slack = M - P;
  return A <= slack * (uint64_t)D || __umul64hi(slack, (uint64_t)D) != 0;  // ceil(A/D) <= slack  <=>  A <= slack D
}

// Of row i the first chunk without a stage that fits (row 0 has its units written in any case, and a chunk's last row
// closes the chunk's passes).  end: the row's last block that fits.
__device__ __forceinline__ int row_units_behind(int i, int end, int N) {
  return max((end + 63) >> 6, (i >> 6) + (i == 0 || i == min(i | 63, N - 1) ? 1 : 0));
}

// The units of row i from chunk `behind` on, "fits nowhere" for all of their stages: one wave, or `parts` of them.
// FEW: at most sixteen chunks, one wave.  (The loops make the compiler spill eighty more scalar registers in
// prepare_kernel: 96 blocks 11.3 -> 13.6 us.)
template <bool FEW>
__device__ __forceinline__ void units_that_fit_nowhere(const ProblemDev &pr, int i, int behind, int part, int parts) {
  const int lane = threadIdx.x & 63, from = max(behind, i >> 6), rest = pr.nch - from;
  if (rest <= 0) return;
  const int64_t u = unit_index(pr.nch, i, from);
  typedef uint32_t Quad __attribute__((ext_vector_type(4)));
  Quad RANNC_GLOBAL *const rm = (Quad RANNC_GLOBAL *)(gptr(pr.rmin) + u * 64);
  uint8_t RANNC_GLOBAL *const uf = gptr(pr.ufit) + u;
  if constexpr (FEW) {
    if (lane < 4 * rest) rm[lane] = Quad{~0u, ~0u, ~0u, ~0u};
    if (lane < rest) uf[lane] = 0;
  } else {
    for (int e = 64 * part + lane; e < 4 * rest; e += 64 * parts) rm[e] = Quad{~0u, ~0u, ~0u, ~0u};
    for (int e = 64 * part + lane; e < rest; e += 64 * parts) uf[e] = 0;
  }
}

// Level 1: one stage on d devices, an entry per thread and turn (a thread keeps its d), by workgroup `group` of `groups`
// of nt threads.  C, TB: looked at with send (comm) and backward (bwd) times.
template <typename VT>
__device__ __forceinline__ void level_one(const ProblemDev &pr, const int64_t *T, const int64_t *P, const int64_t *A, const int64_t *C,
                                          const int64_t *TB, bool comm, bool bwd, int group, int groups, int nt) {
  constexpr VT INF = Lim<VT>::inf;
  const int N = pr.N, D = pr.D, VD = pr.DP, tid = threadIdx.x, d = (tid & (VD - 1)) + 1;
  const double inv = 1.0 / (double)d;
  auto share = [&](int64_t x) -> VT {
    if constexpr (sizeof(VT) == 4) return ceil_div<VT>((VT)x, d, inv);
    else return (VT)(((uint64_t)x + (uint64_t)(d - 1)) / (uint64_t)d);
  };
  auto *const V = gptr((VT *)pr.V), *const VF = gptr((VT *)pr.VF), *const VB = gptr((VT *)pr.VB);
  const int per = nt / VD;  // rows of a turn
  for (int j = group * per + tid / VD; j <= N; j += groups * per) {
    const int64_t e = (int64_t)j * VD + d - 1;
    const bool fit = j > 0 && d <= D && fits_at((uint64_t)P[j], (uint64_t)A[j], (uint64_t)pr.M, d);
    const VT none = d <= D ? INF : (VT)0;  // (padding columns hold 0, so that padded rows stay sorted)
    VT f = 0, b = 0;
    if (fit) {
      f = share(T[j]);
      if (comm) f += share(C[j]);
      if (bwd) b = share(TB[j]);
    }
    V[e] = fit ? f + b : none;
    if (bwd) {
      VF[e] = fit ? f : none;
      VB[e] = fit ? b : none;
    }
  }
}

// The same for the searches of more than kSetupLdsN blocks whose level kernel recomputes the stage times: the
// fits-in-memory part, level 1 and the entries of the pass list.  `parts` waves to a row, which take the row's units that
// hold a stage that fits in turn; the others, most of a long chain, hold only "fits nowhere" and are written
// 16 bytes to a lane.  The workgroups behind `groups` write level 1.  A wave to eight rows of one chunk was bound by
// the rate at which waves start: 64 searches of 1100 blocks 151 us, now 83; 16 of 2000 154, now 42; one of 4096 at 8
// devices 41, now 17.
constexpr int kPassBuildThreads = 64 * kBuildWaves;
template <typename VT>
__global__ __launch_bounds__(kPassBuildThreads) void build_passes_kernel(const ProblemDev *__restrict__ probs, const int groups,
                                                                         const int parts) {
  const ProblemDev &pr = probs[blockIdx.y];
  const int N = pr.N, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if ((int)blockIdx.x >= groups) {
    level_one<VT>(pr, pr.T, pr.P, pr.A, nullptr, nullptr, false, false, (int)blockIdx.x - groups, (int)gridDim.x - groups, kPassBuildThreads);
    return;
  }
  const int id = (int)blockIdx.x * kBuildWaves + wave, i = id / parts, part = id - i * parts;
  if (i >= N) return;
  const bool listed = pr.S_eff > 1;
  const uint32_t *const esum = pr.ends + N;
  const int own = i >> 6;
  const int behind = row_units_behind(i, (int)pr.ends[i], N);
  for (int c = own + part; c < behind; c += parts) {
    UnitStages<VT> st;
    (void)build_unit<VT, 8, true>(pr, pr.T, pr.P, pr.A, nullptr, i, c, lane, nullptr, 0, 0, nullptr, false, &st);
    if (!listed) continue;
    const int w = pr.wlo[c];
    const uint32_t *const r = pass_chunks(pr) + 4 * c;
    const PassChunk rec = {r[0], r[1], r[2], r[3]};
    pass_entries<VT>(pr, i, c, lane, st.fits, st.rmin, st.tij, w, rec, esum);
  }
  units_that_fit_nowhere<false>(pr, i, behind, part, parts);
}

// ---------------------------------------------------------------------------------------
// Everything a search needs in front of its tables, one launch: prefix sums T, P, A of the block
// inputs (the sums over a stage's members that stand in for profile(), Sec. IV-D), input validation,
// the windows and the work list of the level kernels (workgroup 0 of a search), and the initial state
// of V (the other workgroups of the search).
//
// Window of the level kernels: wlo[c] = first row i that holds a stage into chunk c that fits for
// some r <= D (0x7fffffff if none).  Rows below it are never visited.  Memory grows with the stage,
// so row i <= 64c has such a stage iff the one that ends at the chunk's first column fits, and if row
// 64c has one then so has every row from the first such row on: a search, sixteen probes at a time.  (If the chunk's
// first block fits no device by itself, the first later block that does starts the window.)
//
// Work list of the level kernels: the rows wlo[c] .. min(64c+63, N-1) of every chunk, cut into
// items of consecutive rows, listed chunk by chunk.  A compact list keeps the workgroups that have
// work at the front of the grid.  The number of rows of an item travels in the top bits of its
// descriptor: (rows - 1) << 26 | c << 16 | first row.  rows > 0: items of that many rows.
// rows = -1 (sorted-merge level kernel): the smallest multiple of 4 (up to 64) whose item count
// fits max_items, the grid the host launches (sized for the rows of an unpruned search: small
// items, i.e. many workgroups and a short critical path, when pruning leaves few rows; large ones,
// i.e. fewer folds and atomics per row, when the launch is full anyway; and never a workgroup
// without an item in a launch over many searches).  If that launch needs more than one round of
// workgroups (`slots` run at a time, `batch` searches in the launch), the smallest item size that
// brings it down to one round is taken instead, provided the round still fills half the device:
// the round is then as full as it can be, and no compute unit is left with one workgroup more
// than its neighbours.  (For a launch of many rounds, hundreds of searches, the host fixes the item
// size for all of them: merge_grid_items.)
// paired (the level kernel that recomputes the stage times): the list is of passes instead of rows
// (pass_entries), an item of at most that many passes of one chunk; workgroup 0 finds ends[], its
// running sums and every chunk's share of the list (setup_passes), build_passes_kernel writes the entries.
//
// Searches of up to kSetupLdsN blocks come here only where hundreds of them build tables at 64 devices
// (prepare_kernel takes the others).  Bound by latency, a chain of memory round trips and barriers: with send times 22
// us at 2048 blocks and 39 at 4096, a list of passes 19 and 35.
// ---------------------------------------------------------------------------------------
constexpr int kSetupThreads = 256;

// The descriptor of a search, by the first kernel that runs for it.  For a few searches the host does
// not copy the descriptors to the device: `src` is its pinned staging memory, each workgroup fetches
// its descriptor from there once, and the workgroup that owns the search (`keep`) stores it where the
// later kernels read it (dst; src == dst: it is there already).  A copy in front of the first kernel
// costs the host 6 us and the stream 4.  The words go through LDS into scalar registers, so that the
// fields stay wave-uniform.  lds: sizeof(ProblemDev) bytes.
// one: the descriptor itself as a kernel argument (launches over one search: no read from the host at
// all, 1 us), used if use_one.
__device__ __forceinline__ ProblemDev fetch_problem(const ProblemDev *src, ProblemDev *dst, bool keep, uint32_t *lds,
                                                    const ProblemDev &one, int use_one) {
  constexpr int W = (int)sizeof(ProblemDev) / 4;
  static_assert(W <= 64 && sizeof(ProblemDev) % 8 == 0, "a word per lane");
  if (use_one) {
    if (keep && threadIdx.x == 0) *dst = one;
    return one;
  }
  if (threadIdx.x < W / 2) {
    const uint64_t w = ((const uint64_t *)src)[threadIdx.x];
    ((uint64_t *)lds)[threadIdx.x] = w;
    if (keep && src != dst) ((uint64_t *)dst)[threadIdx.x] = w;
  }
  __syncthreads();
  const uint32_t mine = lds[min((int)(threadIdx.x & 63), W - 1)];
  union { ProblemDev p; uint32_t u[W]; } x;
#pragma unroll
  for (int k = 0; k < W; ++k) x.u[k] = (uint32_t)__builtin_amdgcn_readlane((int)mine, k);
  return x.p;
}
constexpr int kSetupLdsN = 1024;  // up to this many blocks the windows are searched in LDS

// Inclusive sums over the workgroup of NW values per thread.  Values stay below 2^62; the upper halves
// of all partial sums are collected in `high`: the total reaches 2^62 iff one of them has bit 30 or 31 set
// (later sums may then wrap: the search is flagged and its values are not looked at).
template <int NW> __device__ __forceinline__ void setup_scan(uint64_t (&v)[NW], uint64_t (*part)[4], uint32_t &high) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const uint64_t x = __shfl_up(v[w], o);
      if (lane >= o) v[w] += x;
      high |= (uint32_t)(v[w] >> 32);
    }
  }
  if (lane == 63)
#pragma unroll
    for (int w = 0; w < NW; ++w) part[wave][w] = v[w];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kSetupThreads / 64 - 1; ++k)
    if (k < wave)
#pragma unroll
      for (int w = 0; w < NW; ++w) { v[w] += part[k][w]; high |= (uint32_t)(v[w] >> 32); }
}

__device__ void setup_fill(const ProblemDev &pr, int levels_done, int64_t t0, int64_t stride) {
  // every V entry behind the first levels_done levels "no plan" (padding columns d > D hold 0 so that padded rows stay sorted)
  typedef uint32_t Quad __attribute__((ext_vector_type(4)));
  if (pr.keys) {  // packed winners of the split level kernel: "none"
    const int64_t nk = (int64_t)(pr.N + 1) * pr.DP * kSplitKeyTables;
    for (int64_t e = t0; e < nk; e += stride) ((unsigned long long *)pr.keys)[e] = ~0ull;
  }
  void *tabs[3] = {pr.V, pr.VF, pr.VB};
  const int words = pr.DP * (pr.bits / 32), used = pr.D * (pr.bits / 32);  // of a row, 32-bit
  const int64_t quads = (int64_t)pr.S_eff * (pr.N + 1) * words / 4;
  for (int w = 0; w < (pr.VF ? 3 : 1); ++w) {
    Quad RANNC_GLOBAL *V = (Quad RANNC_GLOBAL *)gptr((uint32_t *)tabs[w]);
    for (int64_t e = t0 + levels_done * ((int64_t)(pr.N + 1) * words / 4); e < quads; e += stride) {
      const int at = (int)((4 * e) & (words - 1));
      Quad q;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t inf = pr.bits == 32 ? Lim<uint32_t>::inf : (k & 1) ? (uint32_t)(Lim<uint64_t>::inf >> 32) : 0u;
        q[k] = at + k < used ? inf : 0u;
      }
      V[e] = q;
    }
  }
}

// The last block of the largest stage behind block i for which fits(j) holds (i if there is none; the empty
// stage fits).
template <typename F> __device__ __forceinline__ int prepare_end(int i, int N, F fits) {
  int lo = i, hi = N;
  while (__any(lo < hi)) {
    const int mid = (lo + hi + 1) >> 1;  // lo itself once they meet
    if (fits(mid)) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// pick_item_size by one wave: lane k < 16 holds the number of items of size 4 (k + 1).
__device__ __forceinline__ int wave_item_size(int cnt, int most, int max_items, int batch, int slots, bool passes) {
  const long long then = (long long)cnt * batch;
  return pick_item_size((uint32_t)__ballot(cnt <= max_items), (uint32_t)__ballot(then <= slots), (uint32_t)__ballot(2 * then >= slots),
                        (uint32_t)__ballot(2 * cnt >= 3 * slots), most, passes && batch == 1);
}

// ends[], its running sums, the windows and every chunk's share of the pass list (see pass_entries) of a search of more
// than kSetupLdsN blocks, by one workgroup.  pool: LDS of kSetupPool words; marks: of 2 nch 16-bit words.  bad: the sums
// P, A may have wrapped.
//
// Bound by latency, a chain of dependent reads per step of the search for the ends: the sums Z (prepare_kernel) of up to
// kSetupZ blocks are held in LDS; of longer chains every 64th row's end is found first and bounds the others.  A thread
// searches for eight rows at a time.  (Two rows at a time out of memory, and the windows by binary searches in what had been
// written, took the launch 26 us at 1100 blocks, 35 at 2048, 66 at 4096; now 17, 19 and 35.)
constexpr int kSetupZ = 4096;
constexpr int kSetupPool = kSetupZ + 1;
static_assert(kSetupPool >= 2 * (kSetupLdsN + 1) + 1024, "room for two sums and the windows of a list of rows");

__device__ __forceinline__ void setup_passes(const ProblemDev &pr, uint64_t *pool, uint16_t *marks, bool bad, int rows, int max_items,
                                             int batch, int slots, int most) {
  constexpr int U = 8;  // consecutive rows of a thread
  __shared__ uint32_t part[kSetupThreads / 64], behind[kSetupThreads / 64];
  __shared__ int count[16];
  const int N = pr.N, D = pr.D, nch = pr.nch, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t M = (uint64_t)pr.M;
  const uint64_t RANNC_GLOBAL *const P = gptr((const uint64_t *)pr.P), *const A = gptr((const uint64_t *)pr.A);
  uint32_t RANNC_GLOBAL *const ends = gptr(pr.ends), *const esum = ends + N;
  uint16_t *const window = marks, *const full_of = marks + nch;
  for (int c = tid; c < nch; c += kSetupThreads) {
    window[c] = 0xFFFF;  // (no row: N <= 65535)
    full_of[c] = (uint16_t)min(64 * c + 64, N);
  }
  if (tid < 16) count[tid] = 0;
  uint32_t carry = 0, before_base = 0;
  // bound(i): a block up to which the stage behind block i is known to fit (or i), and one behind which it does not;
  // key(i), fits(key, j): whether the stage i+1..j fits
  auto find_ends = [&](auto bound, auto key, auto fits) {
    for (int base = 0; base < N; base += U * kSetupThreads) {
      const int i0 = base + U * tid;
      int lo[U], hi[U];
      decltype(key(0)) of[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = min(i0 + u, N - 1);
        lo[u] = hi[u] = i;
        if (!bad && i0 + u < N) bound(i, lo[u], hi[u]);
        of[u] = key(i);
      }
      bool more = true;
      while (__any(more)) {
        more = false;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int mid = (lo[u] + hi[u] + 1) >> 1;  // lo itself once they meet
          if (fits(of[u], mid)) lo[u] = mid;
          else hi[u] = mid - 1;
          hi[u] = max(hi[u], lo[u]);
          more = more || lo[u] < hi[u];
        }
      }
      uint32_t sum = 0;
#pragma unroll
      for (int u = 0; u < U; ++u) sum += i0 + u < N ? (uint32_t)lo[u] : 0u;
      uint32_t run = sum;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t x = __shfl_up(run, o);
        if (lane >= o) run += x;
      }
      if (lane == 63) { part[wave] = run; behind[wave] = (uint32_t)lo[U - 1]; }
      __syncthreads();
      uint32_t before = __shfl_up((uint32_t)lo[U - 1], 1);  // the end of the row in front of this thread's
      if (lane == 0) before = wave == 0 ? before_base : behind[wave - 1];
      uint32_t at = carry + run - sum;
#pragma unroll
      for (int k = 0; k < kSetupThreads / 64; ++k) {
        if (k < wave) at += part[k];
        carry += part[k];
      }
      before_base = behind[kSetupThreads / 64 - 1];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u;
        if (i < N) {
          const uint32_t end = (uint32_t)lo[u];
          ends[i] = end;
          esum[i] = at;
          at += end;
          mark_windows(N, nch, i, before, end, window, full_of);
          before = end;
        }
      }
      __syncthreads();
    }
  };
  const bool small = P[N] < (1ull << 55) && A[N] < (1ull << 60);
  const uint64_t DM = __umul64hi(M, (uint64_t)D) ? ~0ull : M * (uint64_t)D;
  auto Z_of = [&](int j) { return (uint64_t)D * P[j] + A[j]; };  // (below 2^62 where `small`)
  auto limit = [&](uint64_t z) { return z + DM < z ? ~0ull : z + DM; };
  if (small && N <= kSetupZ) {
    for (int i = tid; i <= N; i += kSetupThreads) pool[i] = Z_of(i);
    __syncthreads();
    find_ends([&](int, int &, int &hi) { hi = N; }, [&](int i) { return limit(pool[i]); },
              [&](uint64_t most_z, int j) { return pool[j] <= most_z; });
  } else {
    struct Sums { uint64_t P, A; };
    auto fits = [&](const Sums &s, int j) { return fits_at(P[j] - s.P, A[j] - s.A, M, D); };
    int *const coarse = (int *)pool;  // the ends of rows 0, 64, ...
    for (int c0 = 0; c0 < nch; c0 += kSetupThreads) {
      if (c0 + 64 * wave >= nch) break;
      const int c = min(c0 + tid, nch - 1);
      const Sums s = {P[64 * c], A[64 * c]};
      const int end = bad ? 64 * c : prepare_end(64 * c, N, [&](int j) { return fits(s, j); });
      if (c0 + tid < nch) coarse[c] = end;
    }
    __syncthreads();
    auto bound = [&](int i, int &lo, int &hi) {  // (ends never decrease)
      const int c = i >> 6;
      lo = max(i, coarse[c]);
      hi = c + 1 < nch ? coarse[c + 1] : N;
    };
    if (small)
      find_ends(bound, [&](int i) { return limit(Z_of(i)); }, [&](uint64_t most_z, int j) { return Z_of(j) <= most_z; });
    else
      find_ends(bound, [&](int i) { return Sums{P[i], A[i]}; }, fits);
  }
  if (tid == 0) esum[N] = carry;
  __syncthreads();  // (the ends in memory are visible to the whole workgroup; pool is free)
  int *const cpass = (int *)pool;
  for (int c = tid; c < nch; c += kSetupThreads) {
    const int last = min(64 * c + 63, N - 1);
    const int w = window_start(ends, N, c, window[c] == 0xFFFF ? kNoRow : (int)window[c], kNoRow);
    uint32_t all = 0, full = 0;
    if (w != kNoRow) {
      full = (uint32_t)max((int)full_of[c], w);
      all = stages_before(esum, N, c, (uint32_t)w, full, (uint32_t)last + 1u);
    }
    pr.wlo[c] = w;
    pass_chunks(pr)[4 * c] = full;
    cpass[c] = (int)((all + 63u) >> 6);
  }
  __syncthreads();
  if (rows <= 0) {
    // thread t counts the items of candidate size 4 (t % 16 + 1) over the chunks t / 16, t / 16 + 16, ...
    const int k = tid % 16, r = 4 * (k + 1);
    int cnt = 0;
    for (int c = tid / 16; c < nch; c += kSetupThreads / 16) cnt += (cpass[c] + r - 1) / r;
    if (cnt) atomicAdd(&count[k], cnt);
    __syncthreads();
    rows = 4 * (wave_item_size(count[k], most, max_items, batch, slots, true) + 1);
  }
  // passes and items in front of every chunk; the passes of a chunk dealt evenly over its items
  if (wave == 0) {
    uint32_t passes = 0, items = 0;
    for (int c0 = 0; c0 < nch; c0 += 64) {
      const int c = c0 + lane;
      const uint32_t np = c < nch ? (uint32_t)cpass[c] : 0u, ni = (np + (uint32_t)rows - 1u) / (uint32_t)rows;
      uint32_t p = np, t = ni;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t x = __shfl_up(p, o), y = __shfl_up(t, o);
        if (lane >= o) { p += x; t += y; }
      }
      if (c < nch) {
        uint32_t *const rec = pass_chunks(pr) + 4 * c;
        rec[1] = passes + p - np;
        rec[2] = items + t - ni;
        rec[3] = ni ? (np + ni - 1u) / ni : 1u;
      }
      passes += (uint32_t)__shfl(p, 63);
      items += (uint32_t)__shfl(t, 63);
    }
    if (lane == 0) pr.runs[0] = (int32_t)items;
  }
}

__global__ __launch_bounds__(kSetupThreads) void setup_kernel(const ProblemDev *src, ProblemDev *probs, int rows,
                                                             int max_items, int batch, int slots, int paired,
                                                             int max_rows, const ProblemDev one, int use_one) {
  __shared__ __align__(8) uint32_t desc[sizeof(ProblemDev) / 4];
  const ProblemDev pr = fetch_problem(src + blockIdx.y, probs + blockIdx.y, blockIdx.x == 0, desc, one, use_one);
  const int N = pr.N, tid = threadIdx.x;
  if (blockIdx.x > 0) {
    setup_fill(pr, 0, (int64_t)(blockIdx.x - 1) * kSetupThreads + tid, (int64_t)(gridDim.x - 1) * kSetupThreads);
    return;
  }
  // Entries per thread and tile.  Two keep the kernel, and with it the workgroups that fill V, at four
  // waves per SIMD: over 1024 searches of 128 blocks that takes 40 us instead of 71 with four entries.
  constexpr int U = 2;
  __shared__ uint64_t part[kSetupThreads / 64][4], last[4];
  __shared__ __align__(16) uint64_t pool[kSetupPool];
  uint64_t *const sP = pool, *const sA = pool + kSetupLdsN + 1;
  __shared__ int flags;
  __shared__ unsigned long long max_cut;
  if (tid == 0) { flags = 0; max_cut = 0ull; sP[0] = 0; sA[0] = 0; }
  const int64_t RANNC_GLOBAL *in[4] = {gptr(pr.t), gptr(pr.p), gptr(pr.a), gptr(pr.tb)};
  int64_t RANNC_GLOBAL *out[4] = {gptr(pr.T), gptr(pr.P), gptr(pr.A), gptr(pr.TB)};
  const bool bwd = pr.tb != nullptr;  // backward times only with the split objective
  const bool in_lds = N <= kSetupLdsN;
  int myflags = 0;
  if (tid == 0) {
    out[0][0] = out[1][0] = out[2][0] = 0;
    if (bwd) out[3][0] = 0;
    if (pr.o) pr.C[0] = 0;
  }
  uint64_t carry[4] = {0, 0, 0, 0};
  unsigned long long mc = 0ull;
  uint32_t high = 0;
  auto sums = [&](auto nw) {  // NW arrays
    constexpr int NW = decltype(nw)::value;
    for (int base = 0; base < N; base += U * kSetupThreads) {
      const int k0 = base + U * tid;
      uint64_t v[NW][U], sum[NW];
#pragma unroll
      for (int w = 0; w < NW; ++w)
#pragma unroll
        for (int u = 0; u < U; ++u) v[w][u] = (uint64_t)in[w][min(k0 + u, N - 1)];
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        sum[w] = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          uint64_t x = k0 + u < N ? v[w][u] : 0;
          if ((int64_t)x < 0) { myflags |= 1; x = 0; }
          if (x >= kSumLimit) { myflags |= 2; x = 0; }
          v[w][u] = x;
          sum[w] += x;
          high |= (uint32_t)(sum[w] >> 32);
        }
      }
      uint64_t run[NW];
#pragma unroll
      for (int w = 0; w < NW; ++w) run[w] = sum[w];
      __syncthreads();  // (part and last are free again)
      setup_scan<NW>(run, part, high);
      if (tid == kSetupThreads - 1)
#pragma unroll
        for (int w = 0; w < NW; ++w) last[w] = run[w];
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        uint64_t at = carry[w] + run[w] - sum[w];  // in front of this thread's entries
#pragma unroll
        for (int u = 0; u < U; ++u) {
          at += v[w][u];
          high |= (uint32_t)(at >> 32);
          if (k0 + u < N) {
            out[w][k0 + u + 1] = (int64_t)at;
            if (in_lds && w == 1) sP[k0 + u + 1] = at;
            if (in_lds && w == 2) sA[k0 + u + 1] = at;
          }
        }
      }
      __syncthreads();
#pragma unroll
      for (int w = 0; w < NW; ++w) carry[w] += last[w];
    }
  };
  if (bwd) sums(std::integral_constant<int, 4>());
  else sums(std::integral_constant<int, 3>());
  if (high >> 30) myflags |= 2;
  if (pr.o)  // per-cut send time; the last block has no follower
#pragma unroll 1
    for (int k = tid; k < N; k += kSetupThreads) {
      const uint64_t c = cut_time(pr.o[k], pr.bw, myflags);
      pr.C[k + 1] = (k + 1 < N) ? (int64_t)c : 0;
      if (k + 1 < N && c > mc) mc = c;
    }
  if (pr.o) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) mc = max(mc, (unsigned long long)__shfl_xor(mc, o));
    if (mc && (tid & 63) == 0) atomicMax(&max_cut, mc);
  }
  if (myflags) atomicOr(&flags, myflags);
  __syncthreads();  // the sums in memory are visible to the whole workgroup as well
  if (tid == 0) {
    int st = RANNC_DP_PROBLEM_OK;
    if (flags & 1) st = RANNC_DP_PROBLEM_NEGATIVE_INPUT;
    else if (flags & 2) st = RANNC_DP_PROBLEM_SUM_OVERFLOW;
    else if (carry[0] + (bwd ? carry[3] : 0ull) + max_cut > (uint64_t)pr.time_limit)
      st = RANNC_DP_PROBLEM_TIME_TOO_LARGE;  // a value is at most forward + send + backward time of all blocks
    *pr.status = st;
  }

  // ---- windows ----
  __shared__ int start[1025];  // nch <= 1024 (N <= 65535)
  if (paired) {
    // (sums that may have wrapped: no stage fits)
    setup_passes(pr, pool, (uint16_t *)start, flags != 0, rows, max_items, batch, slots, max_rows / 4);
    return;
  }
  RunRows *const seg = (RunRows *)(pool + 2 * (kSetupLdsN + 1));  // every chunk's window
  static_assert(sizeof(RunRows) == sizeof(uint64_t), "a chunk to a word");
  constexpr int NC = 16;  // candidate item sizes 4, 8, ..., 64 rows, up to max_rows
  const int most = max_rows / 4;
  __shared__ int count[NC];
  const int nch = pr.nch, D = pr.D;
  const uint64_t M = (uint64_t)pr.M;
  auto window = [&](auto P, auto A) {
    // sixteen lanes per chunk: sixteen probes at a time
    const int sub = tid & 15;
    for (int c = tid >> 4; c < ((nch + 15) & ~15); c += kSetupThreads / 16) {
      const int cc = min(c, nch - 1);
      const int j = 64 * cc + 1;  // the chunk's first column, for the rows up to 64c
      const uint64_t Pj = P[j], Aj = A[j];
      int lo = 64 * cc, below = -1;  // the smallest row known to fit (if 64c does), the largest known not to
      const bool some = fits_at(Pj - P[lo], Aj - A[lo], M, D);
      while (__ballot(some && lo - below > 1) != 0ull) {
        const int width = max((lo - below + 15) >> 4, 1);
        const int at = min(below + (sub + 1) * width, lo);
        const bool fits = fits_at(Pj - P[max(at, 0)], Aj - A[max(at, 0)], M, D);
        const unsigned m = (unsigned)(__ballot(fits) >> (tid & 48)) & 0xFFFFu;
        const int f = m ? __ffs((int)m) - 1 : 15;  // (the last probe is lo, which fits)
        if (some && lo - below > 1) {
          const int next = min(below + (f + 1) * width, lo);
          below += f * width;
          lo = next;
        }
      }
      if (!some) {  // the chunk's first block fits no device by itself: the first later one that does
        const int hi = min(64 * cc + 63, N - 1);
        for (++lo; lo <= hi; ++lo)
          if (fits_at(P[lo + 1] - P[lo], A[lo + 1] - A[lo], M, D)) break;
        if (lo > hi) lo = kNoRow;
      }
      if (c < nch && sub == 0) {
        pr.wlo[c] = lo;
        seg[c] = run_rows(N, c, lo);
      }
    }
  };
  if (in_lds) window((const uint64_t *)sP, (const uint64_t *)sA);
  else window((const uint64_t RANNC_GLOBAL *)out[1], (const uint64_t RANNC_GLOBAL *)out[2]);
  __syncthreads();

  // ---- work list ----
  int32_t *const runs = pr.runs;  // (read once: the stores below would make the compiler fetch it again)
  if (rows <= 0) {
    if (tid < NC) count[tid] = 0;
    __syncthreads();
    // thread t counts the items of candidate size 4 (t % 16 + 1) over the chunks t / 16, t / 16 + 16, ...
    {
      const int k = tid % NC, r = 4 * (k + 1);
      int cnt = 0;
      for (int c = tid / NC; c < nch; c += kSetupThreads / NC) {
        cnt += items_of_rows(seg[c], r);
      }
      if (cnt) atomicAdd(&count[k], cnt);
    }
    __syncthreads();
    rows = 4 * (wave_item_size(count[tid % NC], most, max_items, batch, slots, false) + 1);
  }
  // per chunk: its items, the rows dealt evenly over them (33 rows in items of up to 16: three items of 11,
  // not 16 + 16 + 1)
  for (int c = tid; c < nch; c += kSetupThreads) start[c + 1] = items_of_rows(seg[c], rows);
  __syncthreads();
  if (tid == 0) {
    int sum = 0;
    start[0] = 0;
    for (int c = 1; c <= nch; ++c) { sum += start[c]; start[c] = sum; }
    runs[0] = sum;
  }
  __syncthreads();
  const int total = start[nch];
  for (int e = tid; e < total; e += kSetupThreads) {
    int lo = 0, hi = nch - 1;  // the chunk whose items contain e: start[c] <= e < start[c + 1]
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (start[mid + 1] <= e) lo = mid + 1;
      else hi = mid;
    }
    const int c = lo, k = e - start[c];
    const RunRows g = seg[c];
    const int items = start[c + 1] - start[c], per = (g.n + items - 1) / items;
    const int take = max(min(per, g.n - k * per), 1);  // (never below one row: the word stays well-formed)
    runs[1 + e] = ((take - 1) << 26) | (c << 16) | (g.lo + k * per);
  }
}

// ---------------------------------------------------------------------------------------
// setup_kernel and build_kernel as ONE launch, for searches of up to kSetupLdsN blocks (and, with the split
// objective, its level 1): the first `groups` workgroups of a search each form the prefix sums, the ends
// and the chunks' shares of the pass list for themselves, in LDS, and then build their share of the tables;
// the first of them also writes what later launches read.  The other workgroups fill V.  Nothing is
// exchanged between workgroups.  Bound by latency: one round of reads, the sums, ten steps of the search
// for the ends, a few barriers, the tables.  The two launches took 7 + 5 us at 96 blocks, 8 + 7 at 251 and 14 +
// 28 at 1024 (where the second one reads the sums back from memory).
// ---------------------------------------------------------------------------------------
constexpr int kPrepareChunks = kSetupLdsN / 64;
struct PrepareIn { int groups, parts, rows, max_items, batch, slots, paired, max_rows; };

// Inclusive prefix sums of one array by one wave, PER (odd: no bank conflicts) consecutive entries per
// lane, into s[1 .. N]; flags and high as in setup_kernel.
template <int PER>
__device__ __forceinline__ void prepare_sums(const int64_t RANNC_GLOBAL *in, int64_t *s, int N, int &flags, uint32_t &high) {
  const int lane = threadIdx.x & 63, i0 = lane * PER;
  uint64_t v[PER], sum = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) v[k] = (uint64_t)in[min(i0 + k, N - 1)];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    uint64_t x = i0 + k < N ? v[k] : 0;
    if ((int64_t)x < 0) { flags |= 1; x = 0; }
    if (x >= kSumLimit) { flags |= 2; x = 0; }
    sum += x;
    v[k] = sum;
    high |= (uint32_t)(sum >> 32);
  }
  uint64_t run = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t x = __shfl_up(run, o);
    if (lane >= o) run += x;
    high |= (uint32_t)(run >> 32);
  }
  run -= sum;  // in front of this lane's entries
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (i0 + k < N) {
      s[i0 + k + 1] = (int64_t)(run + v[k]);
      high |= (uint32_t)((run + v[k]) >> 32);
    }
  if (lane == 0) s[0] = 0;
}

// ceil(x / r) for x, r < 2^16 (the sum's half keeps the product off the whole numbers by more than its error)
__device__ __forceinline__ int prepare_ceil(int x, int r, float inv) { return (int)(((float)(x + r - 1) + 0.5f) * inv); }

// TIMES: the stage-time tables as well (DP then is the class they are unrolled for; otherwise any).
// NT: threads of a workgroup, 1024 for one search (a thread per row, a unit or two per wave: 24 -> 19 us at
// 1024 blocks), 256 for several (five workgroups to a compute unit instead of one: the sweep of 2048 searches of 128
// blocks 1854 -> 1741 us a call; 7 of 500 blocks at 8 devices 89 -> 79, with send times 115 -> 103).
template <typename VT, int DP, bool TIMES, int NT>
__global__ __launch_bounds__(NT) void prepare_kernel(const ProblemDev *src, ProblemDev *probs, const PrepareIn in,
                                                               const ProblemDev one, int use_one) {
  constexpr int WAVES = NT / 64;
  __shared__ __align__(8) uint32_t desc[sizeof(ProblemDev) / 4];
  __shared__ int s_flags, s_w[kPrepareChunks], s_full[kPrepareChunks];
  __shared__ PassChunk s_rec[kPrepareChunks];
  __shared__ unsigned long long s_max_cut;
  __shared__ uint32_t s_part[WAVES];
  extern __shared__ __align__(16) char lds[];
  const ProblemDev pr = fetch_problem(src + blockIdx.y, probs + blockIdx.y, blockIdx.x == 0, desc, one, use_one);
  const int N = pr.N, D = pr.D, nch = pr.nch, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if ((int)blockIdx.x >= in.groups) {
    setup_fill(pr, 1, (int64_t)(blockIdx.x - in.groups) * NT + tid, (int64_t)(gridDim.x - in.groups) * NT);
    return;
  }
  const bool bwd = pr.tb != nullptr, comm = pr.o != nullptr, writes = blockIdx.x == 0;
  int64_t *const sT = (int64_t *)lds, *const sP = sT + (N + 1), *const sA = sP + (N + 1);
  int64_t *const sTB = sA + (N + 1), *const sC = sTB + (bwd ? N + 1 : 0);
  uint64_t *const sZ = (uint64_t *)(sC + (comm ? N + 1 : 0));
  uint32_t *const sE = (uint32_t *)(sZ + (N + 1)), *const esum = sE + N;
  if (tid == 0) { s_flags = 0; s_max_cut = 0ull; }
  if (tid < kPrepareChunks) { s_w[tid] = kNoRow; s_full[tid] = min(64 * tid + 64, N); }  // (the row behind the chunk's last)
  int flags = 0;
  uint32_t high = 0;
  if (wave < 3 || bwd) {  // a wave per array
    const int64_t *from = wave == 0 ? pr.t : wave == 1 ? pr.p : wave == 2 ? pr.a : pr.tb;
    int64_t *to = wave == 0 ? sT : wave == 1 ? sP : wave == 2 ? sA : sTB;
    if (N <= 64) prepare_sums<1>(gptr(from), to, N, flags, high);
    else if (N <= 192) prepare_sums<3>(gptr(from), to, N, flags, high);
    else if (N <= 320) prepare_sums<5>(gptr(from), to, N, flags, high);
    else if (N <= 576) prepare_sums<9>(gptr(from), to, N, flags, high);
    else prepare_sums<17>(gptr(from), to, N, flags, high);
  }
  static_assert(kSetupLdsN <= 17 * 64, "entries of a lane");
  if (high >> 30) flags |= 2;
  __syncthreads();  // (s_flags is set)
  if (comm) {  // per-cut send time; the last block has no follower
    unsigned long long mc = 0ull;
#pragma unroll 1
    for (int k = tid; k < N; k += NT) {
      const uint64_t c = cut_time(pr.o[k], pr.bw, flags);
      sC[k + 1] = k + 1 < N ? (int64_t)c : 0;
      if (k + 1 < N && c > mc) mc = c;
    }
    if (tid == 0) sC[0] = 0;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) mc = max(mc, (unsigned long long)__shfl_xor(mc, o));
    if (mc && lane == 0) atomicMax(&s_max_cut, mc);
  }
  if (flags) atomicOr(&s_flags, flags);
  __syncthreads();
  flags = s_flags;
  if (writes) {
    if (tid == 0) {
      int st = RANNC_DP_PROBLEM_OK;
      if (flags & 1) st = RANNC_DP_PROBLEM_NEGATIVE_INPUT;
      else if (flags & 2) st = RANNC_DP_PROBLEM_SUM_OVERFLOW;
      else if ((uint64_t)sT[N] + (bwd ? (uint64_t)sTB[N] : 0ull) + s_max_cut > (uint64_t)pr.time_limit)
        st = RANNC_DP_PROBLEM_TIME_TOO_LARGE;  // a value is at most forward + send + backward time of all blocks
      *pr.status = st;
    }
    for (int e = tid; e <= N; e += NT) {
      pr.T[e] = sT[e]; pr.P[e] = sP[e]; pr.A[e] = sA[e];
      if (bwd) pr.TB[e] = sTB[e];
      if (comm) pr.C[e] = sC[e];
    }
  }

  // ---- ends, windows, the chunks' shares of the list ----
  {
    // A stage fits on D devices iff D bytes_not_divided + divided ones <= D M: one difference of the sums Z =
    // D P + A, where neither they nor D M wrap.
    const uint64_t M = (uint64_t)pr.M;
    const bool bad = flags != 0;  // (the sums may have wrapped: no stage fits)
    const bool small = (uint64_t)sP[N] < (1ull << 55) && (uint64_t)sA[N] < (1ull << 60);
    const uint64_t DM = __umul64hi(M, (uint64_t)D) ? ~0ull : M * (uint64_t)D;
    if (small) {
      for (int i = tid; i <= N; i += NT) sZ[i] = (uint64_t)D * (uint64_t)sP[i] + (uint64_t)sA[i];
      __syncthreads();
    }
    for (int i0 = 0; i0 < N; i0 += NT) {
      if (i0 + 64 * wave >= N) break;
      const int i = min(i0 + tid, N - 1);
      int e = i;
      if (!bad && small) {
        const uint64_t Zi = sZ[i];
        e = prepare_end(i, N, [&](int j) { return sZ[j] - Zi <= DM; });
      } else if (!bad) {
        const uint64_t Pi = (uint64_t)sP[i], Ai = (uint64_t)sA[i];
        e = prepare_end(i, N, [&](int j) { return fits_at((uint64_t)sP[j] - Pi, (uint64_t)sA[j] - Ai, M, D); });
      }
      if (i0 + tid < N) sE[i] = (uint32_t)e;
    }
    __syncthreads();
    const int Q = (N + NT - 1) / NT;  // consecutive rows of a thread
    uint32_t sum = 0;
    for (int i = Q * tid; i < min(Q * tid + Q, N); ++i) {
      const uint32_t end = sE[i], before = i ? sE[i - 1] : 0u;
      sum += end;
      mark_windows(N, nch, i, before, end, s_w, s_full);
    }
    uint32_t run = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t x = __shfl_up(run, o);
      if (lane >= o) run += x;
    }
    if (lane == 63) s_part[wave] = run;
    __syncthreads();
    uint32_t at = run - sum;
    for (int q = 0; q < wave; ++q) at += s_part[q];
    for (int i = Q * tid; i < min(Q * tid + Q, N); ++i) {
      esum[i] = at;
      at += sE[i];
      if (i == N - 1) esum[N] = at;
    }
    if (tid < nch) {
      const int c = tid;
      const int w = window_start(sE, N, c, s_w[c], kNoRow);
      s_w[c] = w;
      if (w != kNoRow) s_full[c] = max(s_full[c], w);
      if (writes) pr.wlo[c] = w;
    }
    __syncthreads();
  }
  int rows = in.rows;
  if (in.paired) {
    if (wave == 0) {
      uint32_t np = 0;
      if (lane < nch && s_w[lane] != kNoRow)
        np = (stages_before(esum, N, lane, (uint32_t)s_w[lane], (uint32_t)s_full[lane], (uint32_t)min(64 * lane + 64, N)) + 63u) >> 6;
      if (rows <= 0) {  // lane k counts the items of size 4 (k + 1)
        const int r = 4 * (lane & 15) + 4;
        const float inv = 1.0f / (float)r;
        int cnt = 0;
        for (int c = 0; c < nch; ++c) cnt += prepare_ceil((int)lane_bcast(np, c), r, inv);
        rows = 4 * (wave_item_size(cnt, in.max_rows / 4, in.max_items, in.batch, in.slots, true) + 1);
      }
      const uint32_t ni = (np + (uint32_t)rows - 1u) / (uint32_t)rows;
      uint32_t p = np, t = ni;
#pragma unroll
      for (int o = 1; o < kPrepareChunks; o <<= 1) {
        const uint32_t x = __shfl_up(p, o), y = __shfl_up(t, o);
        if (lane >= o) { p += x; t += y; }
      }
      if (lane < nch) s_rec[lane] = {(uint32_t)s_full[lane], p - np, t - ni, ni ? (np + ni - 1u) / ni : 1u};
      if (writes && lane == kPrepareChunks - 1) pr.runs[0] = (int32_t)t;
    }
    __syncthreads();
  }

  // ---- tables: of a row the units that hold a stage that fits, `parts` waves to a row; the others hold only
  // "fits nowhere" ----
  const bool passes = in.paired && pr.S_eff > 1;
  for (int id = (int)blockIdx.x * WAVES + wave; id < N * in.parts; id += in.groups * WAVES) {  // wave-uniform
    const int i = id / in.parts, part = id - i * in.parts;
    const int own = i >> 6;
    const int behind = row_units_behind(i, (int)sE[i], N);
    for (int c = own + part; c < behind; c += in.parts) {
      UnitStages<VT> st;
      (void)build_unit<VT, DP, true>(pr, sT, sP, sA, comm ? sC : nullptr, i, c, lane, nullptr, 0, 0, bwd ? sTB : nullptr, TIMES,
                                     &st);
      if (passes) pass_entries<VT>(pr, i, c, lane, st.fits, st.rmin, st.tij, s_w[c], s_rec[c], esum);
    }
    if (part == 0) units_that_fit_nowhere<true>(pr, i, behind, 0, 1);
  }
  level_one<VT>(pr, sT, sP, sA, sC, sTB, comm, bwd, (int)blockIdx.x, in.groups, NT);
  if (in.paired || !writes) return;

  // ---- work list of rows (of the first workgroup; nch <= 16) ----
  int32_t *const runs = pr.runs;
  __shared__ int start[kPrepareChunks + 1];
  if (wave == 0) {
    const int n0 = lane < nch ? run_rows(N, lane, s_w[lane]).n : 0;
    if (rows <= 0) {
      const int r = 4 * (lane & 15) + 4;
      const float inv = 1.0f / (float)r;
      int cnt = 0;
      for (int c = 0; c < nch; ++c) cnt += prepare_ceil((int)lane_bcast((uint32_t)n0, c), r, inv);
      rows = 4 * (wave_item_size(cnt, in.max_rows / 4, in.max_items, in.batch, in.slots, false) + 1);
    }
    int run = (n0 + rows - 1) / rows;
    const int mine = run;
#pragma unroll
    for (int o = 1; o < kPrepareChunks; o <<= 1) {
      const int x = __shfl_up(run, o);
      if (lane >= o) run += x;
    }
    if (lane < nch) start[lane] = run - mine;
    if (lane == kPrepareChunks - 1) { start[nch] = run; runs[0] = run; }
  }
  __syncthreads();
  for (int c = 0; c < nch; ++c) {
    const RunRows g = run_rows(N, c, s_w[c]);
    const int items = start[c + 1] - start[c], per = items ? (g.n + items - 1) / items : 0;
    for (int k = tid; k < items; k += NT) {
      const int take = max(min(per, g.n - k * per), 1);  // (never below one row: the word stays well-formed)
      runs[1 + start[c] + k] = ((take - 1) << 26) | (c << 16) | (g.lo + k * per);
    }
  }
}

// ---------------------------------------------------------------------------------------
// DP level s >= 2, sorted-merge form.
//
// For a fixed stage (i,j) the recurrence of Sec. III-C needs, for every device total d,
//     W[d] = min over d' + r = d of max(a[d'], c[r]),   a[d'] = V[s-1][i][d'], c[r] = h(i,j,r)
// (INF where r does not fit).  Both sequences are non-increasing: giving one more device to
// the last stage of a plan can only lower its time and its memory, and h, m are non-increasing
// in r.  For such sequences, W[d] <= x  <=>  (number of a's > x) + (number of c's > x) <= d-2,
// i.e. W[d] is the (d-1)-th largest element of the merged multiset {a[1..]} U {c[1..]}.  A wave
// therefore merges the two sorted D-vectors with a bitonic network held in registers
// (DP*(log2 DP + 1) max/min operations instead of D^2/2 max-min pairs) and folds the result into
// a per-lane running minimum over i.  V[s][j][d] = min over i of W[d] is then the value the
// five nested loops of Algorithm 1 produce; which (i,d') attains it is recovered where it is
// needed (traceback, table export) by the first-match scan, not carried here.
//
// Only replica counts r <= D-s+1 can occur at level s (s-1 devices are spent on the earlier
// stages); the larger ones rank below position D-1 of the merge, so they are not read.
//
// Work item (one workgroup of four waves) = 4 to 64 consecutive rows of one chunk's window,
// taken from the work list; wave w takes rows i0+w, i0+w+4, ... one after the other and keeps the
// running minimum over them in registers (one value array for the row in flight, one for the
// minimum: three waves per SIMD, i.e. three workgroups per compute unit, whose memory, merge and
// fold phases overlap).  A lane owns column jj = 64c + lane.  a[] is wave-uniform (one row of
// V[s-1], scalar loads), c[] comes from coalesced reads of one contiguous unit; the flags of the
// next row are fetched while the current one is merged.  The four waves then fold their minima
// together in LDS, and one transposed pass of device-scope atomicMin into V[s] (pre-filled with
// INF) combines the items of a chunk: min is order-independent, so the result is deterministic.
// ---------------------------------------------------------------------------------------
// Sorting a bitonic sequence (descending, then ascending) of H values into descending order.
// A bitonic sequence of LEN = F * m values, read as F rows of m, has this property for any F: sorting
// each of the m columns leaves F bitonic rows, every value of a row >= every value of the next one (a
// 0/1 bitonic sequence puts its zeros into cyclically consecutive places, so the zero counts of the
// columns differ by at most one and the rows with both values come out bitonic; Nakatani et al., K-way
// bitonic sort).  With F = 3 a column is max3 / med3 / min3: one instruction per value for log2(3) =
// 1.58 binary levels, where the binary form pays one per level.  LEN is the product of twos and threes
// that costs least for H, with LEN - H places in front that count as infinite: a column with such a
// place needs fewer operations, or none.  H = 64: 246 instead of 384 operations, 56: 220, 48: 183, 40:
// 138, 32: 100 instead of 160, 24: 72, 16: 45 instead of 64, 8: 16 instead of 24.  64-bit values have no
// three-operand form: there the columns are pairs, of the power of two above H.
__device__ __forceinline__ uint32_t vmed3(uint32_t a, uint32_t b, uint32_t c) {
  uint32_t r;
  asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// position p of the sequence is x[AT + p]; the first PAD positions are the infinite ones (not stored)
template <int LEN, int PAD, int AT, typename VT, int H> __device__ __forceinline__ void bitonic_rows(VT (&)[H]) {}
template <int LEN, int PAD, int AT, int F, int... REST, typename VT, int H>
__device__ __forceinline__ void bitonic_rows(VT (&x)[H]) {
  if constexpr (LEN > 1 && PAD < LEN) {
    constexpr int m = LEN / F;
    static_assert(m * F == LEN, "the factors multiply to the length");
#pragma unroll
    for (int q = 0; q < m; ++q) {
      if constexpr (F == 2) {
        if (q >= PAD) {
          const VT a = x[AT + q], b = x[AT + q + m];
          x[AT + q] = vmax(a, b);
          x[AT + q + m] = vmin(a, b);
        }
      } else {
        if (q >= PAD) {
          const VT a = x[AT + q], b = x[AT + q + m], c = x[AT + q + 2 * m];
          x[AT + q] = vmax(vmax(a, b), c);
          x[AT + q + m] = vmed3(a, b, c);
          x[AT + q + 2 * m] = vmin(vmin(a, b), c);
        } else if (q + m >= PAD) {
          const VT a = x[AT + q + m], b = x[AT + q + 2 * m];
          x[AT + q + m] = vmax(a, b);
          x[AT + q + 2 * m] = vmin(a, b);
        }
      }
    }
    bitonic_rows<m, (PAD < m ? PAD : m), AT, REST...>(x);
    bitonic_rows<m, (PAD < m ? 0 : PAD - m < m ? PAD - m : m), AT + m, REST...>(x);
    if constexpr (F == 3) bitonic_rows<m, (PAD < 2 * m ? 0 : PAD - 2 * m), AT + 2 * m, REST...>(x);
  }
}
template <typename VT, int H> __device__ __forceinline__ void bitonic_sort(VT (&x)[H]) {
  static_assert(H % 8 == 0 && H >= 8 && H <= 64, "merge widths");
  if constexpr (sizeof(VT) == 8) {
    if constexpr (H == 8) bitonic_rows<8, 0, 0, 2, 2, 2>(x);
    else if constexpr (H == 16) bitonic_rows<16, 0, 0, 2, 2, 2, 2>(x);
    else if constexpr (H <= 32) bitonic_rows<32, 32 - H, H - 32, 2, 2, 2, 2, 2>(x);
    else bitonic_rows<64, 64 - H, H - 64, 2, 2, 2, 2, 2, 2>(x);
  } else {
    if constexpr (H == 8) bitonic_rows<9, 1, -1, 3, 3>(x);
    else if constexpr (H == 16) bitonic_rows<18, 2, -2, 2, 3, 3>(x);
    else if constexpr (H == 24) bitonic_rows<27, 3, -3, 3, 3, 3>(x);
    else if constexpr (H <= 48) bitonic_rows<54, 54 - H, H - 54, 2, 3, 3, 3>(x);
    else bitonic_rows<81, 81 - H, H - 81, 3, 3, 3, 3>(x);
  }
}

// Width of the merge.  The first s-2 entries of a[] are INF (s-1 stages need s-1 devices) and only
// rl = D-s+1 replica counts and device totals are left, so the merge of a[sig .. sig+H-1] with c[1..H]
// for any H >= rl gives every value the level needs: its t-th output is W[d] for d - 1 = t + 1 + sig
// (the sig skipped entries are the sig largest of the full merge).  sig = min(s-2, DP-H) skips only
// INF and stays inside the row of DP entries.  H is rl rounded up to a multiple of eight.
__device__ __forceinline__ int merge_shift(int s, int DP, int H) { return min(s - 2, DP - H); }

// One row's sorted merge: x := the H largest elements of merge(a, c), sorted descending, for the
// lane's stage (`arow` points at a[sig]); all INF for a lane without work (`off` = INF there, 0
// elsewhere).
//
// x[H-1-m] = c[m+1]: reversed, so that max(a, x) is a bitonic sequence.  H is a compile-time number, so
// that the reads of a row are one straight run of independent loads; inside the last group of eight
// the row index is clamped to rl-1 (the repeated value keeps the sequence sorted, stays below rank
// D-1, and costs no memory traffic).  `unit` points at the lane's column, or for a lane without work
// at the column of a lane that has some (every load instruction then touches only lines that are
// needed); such a lane is switched off by folding `off` into the first maximum, which makes its whole
// result INF.
template <typename VT, int H, typename AP>
__device__ __forceinline__ void row_merge(VT (&x)[H], const VT RANNC_GLOBAL *__restrict__ unit, AP arow, VT off, int rl) {
#pragma unroll
  for (int m = 0; m < H; ++m) x[H - 1 - m] = unit[(m <= H - 8 ? m : min(m, rl - 1)) * 64];  // H-8 <= rl-1; wave-uniform clamp
#pragma unroll
  for (int q = 0; q < H; ++q) {
    if constexpr (std::is_same<AP, const VT RANNC_GLOBAL *>::value) x[q] = vmax(vmax_su(arow[q], x[q]), off);
    else x[q] = vmax(vmax(arow[q], x[q]), off);
  }
  bitonic_sort(x);
}

// The same for a level kernel that recomputes the stage times instead of reading their table (no
// communication term; 32-bit values here, 64-bit ones at DirectArith<uint64_t>): the lane's stage has total
// time tij, fits from rmn replicas on (255: never, or a lane without work), and c[r] = ceil(tij / r),
// INF for r < rmn.
//
// ceil(x / r) for r = odd * 2^k, k <= 3, is ONE double-precision instruction, run with the rounding mode set
// to "towards +infinity":
//     y = x * (inv * 2^-53) + 2^(k - 1)      a fused multiply-add, inv just below 1/odd
// The sum lies in [2^(k-1), 2^k), where doubles are multiples of 2^(k-53): the rounding takes x * inv / 2^k up
// to the next whole number and leaves that in the mantissa field of y.  inv lies below 1/odd by less than
// 2^-50 of it (and is exact for odd = 1), so x * inv / 2^k falls short of x / r by less than x / r * 2^-50:
// less than 2^-18 for x < 2^32, 2^-10 for x <= 2^40.  If x / r is a whole number the ceiling takes it back up to
// that number; if not, its fraction is at least 1/64 and stays positive.  Four counts up to 64 have k > 3:
// ceil(x / 2r) = ceil(ceil(x / r) / 2), an add and a shift.  (With the default rounding, odd counts took an
// addition and a fused multiply-add and even ones an addition and a shift of the odd quotient: twice the
// instructions.  That form is still the table builder's, which is bound by its stores.  1024 blocks at 64
// devices: 514 -> 479 us a call where memory never binds, 346 -> 334 where it does.)
// The reciprocals live in scalar register pairs for the whole kernel (an instruction takes one scalar
// operand; 1/2, 1, 2 and 4 need no register): the rows of V[s-1] come out of LDS, so the scalar registers
// are free for them.
// INF below rmn: a per-lane bit mask (bit r-1 set for r < rmn), folded into the entries.  Lanes without
// work are not looked at afterwards, and in almost every pass the others fit on one replica already
// (persistent bytes, which no replica shares, are the larger part): such a pass skips the mask.
template <int HMAX> struct DirectConsts {
  double inv[HMAX / 2];  // 2^-53 times a number just below 1 / (2k + 1)
};
// Also sets the rounding mode of the wave's double-precision instructions, for the rest of the kernel: no
// other one in the kernels that call this rounds.  (In assembly, so that the compiler does not set the
// mode back in front of them; every quotient depends on the registers written behind it.)
template <int HMAX> __device__ __forceinline__ void direct_consts_init(DirectConsts<HMAX> &k) {
  asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 2, 2), 1" ::);  // towards +infinity
#pragma unroll
  for (int q = 0; q < HMAX / 2; ++q) {
    k.inv[q] = 0x1p-53 * (q == 0 ? 1.0 : 1.0 / (double)(2 * q + 1) * (1.0 - 0x1p-51));
    asm volatile("" : "+s"(k.inv[q]));  // a register, not an immediate
  }
}

template <typename VT> struct DirectArith;
template <> struct DirectArith<uint32_t> {
  static __device__ __forceinline__ uint32_t quotient(double y) { return (uint32_t)__double_as_longlong(y); }
  // 0 or INF from bit (m & 31) of the mask word
  static __device__ __forceinline__ uint32_t inf_if(int word, int m) {
    return (uint32_t)__builtin_amdgcn_sbfe(word, m & 31, 1);
  }
};
// 64-bit values: for stage times up to 2^40 (the caller's bound on a search's total time guarantees it)
template <> struct DirectArith<uint64_t> {
  static __device__ __forceinline__ uint64_t quotient(double y) {
    return (uint64_t)__double_as_longlong(y) & ((1ull << 52) - 1ull);
  }
  static __device__ __forceinline__ uint64_t inf_if(int word, int m) {
    return (uint64_t)((uint32_t)__builtin_amdgcn_sbfe(word, m & 31, 1) & (uint32_t)(Lim<uint64_t>::inf >> 32)) << 32;
  }
};
// largest stage time the 64-bit form is exact for
constexpr int64_t kDirectWideMaxTime = (int64_t)1 << 40;

// x[H-1-M] := max(x[H-1-M], c[M+1]) for every entry: x[] holds the lane's row a[sig ..] and becomes the
// bitonic sequence of the merge.  q8[n - 1]: the quotient of 8n, n odd.
template <typename VT, int H, int HMAX, int M = 0>
__device__ __forceinline__ void direct_entries(VT (&x)[H], double tij, const DirectConsts<HMAX> &k, VT (&q8)[H / 8]) {
  if constexpr (M < H) {
    constexpr int R = M + 1, CTZ = __builtin_ctz(R), SH = CTZ < 3 ? CTZ : 3, ODD = R >> CTZ;
    VT h;
    if constexpr (CTZ <= 3) h = DirectArith<VT>::quotient(__builtin_fma(tij, k.inv[ODD / 2], 0.5 * (1 << SH)));
    else h = (q8[ODD - 1] + (VT)((1 << (CTZ - 3)) - 1)) >> (CTZ - 3);
    if constexpr (CTZ == 3) q8[ODD - 1] = h;
    x[H - 1 - M] = vmax(x[H - 1 - M], h);
    // (all quotients at once would take twice the registers)
    if constexpr (M % (32 / (int)sizeof(VT)) == 32 / (int)sizeof(VT) - 1) __builtin_amdgcn_sched_barrier(0);
    direct_entries<VT, H, HMAX, M + 1>(x, tij, k, q8);
  }
}

// act: the lane has work (x of the others is not looked at)
template <typename VT, int H, int HMAX>
__device__ __forceinline__ void row_merge_direct(VT (&x)[H], VT tij, int rmn, bool act, const DirectConsts<HMAX> &k) {
  VT q8[H / 8];
  direct_entries<VT, H, HMAX>(x, (double)tij, k, q8);
  if (__ballot(act && rmn > 1) != 0ull) {
    // bit r-1 set for r < rmn: these replica counts do not fit
    const unsigned long long below = rmn > 64 ? ~0ull : ((1ull << (rmn - 1)) - 1ull);
    const int mlo = (int)(uint32_t)below, mhi = (int)(uint32_t)(below >> 32);
#pragma unroll
    for (int m = 0; m < H; ++m) x[H - 1 - m] = vmax(x[H - 1 - m], DirectArith<VT>::inf_if(m < 32 ? mlo : mhi, m));
  }
  bitonic_sort(x);
}

// The passes of one work item of the recomputing level kernel (see pass_entries), wave w the passes w, w+4, ...
// A wave fetches what a pass needs while it works on the one before: the words two passes ahead, the times and the
// few rows of V[s-1] that the words name one pass ahead, a value per lane.  When its turn comes the rows are put into LDS
// and every lane reads its own back, four values at a time.  A pass with more rows than that (the end of a
// diagonal block, stages of few blocks) has each lane read its row from memory.  The waves of the item
// share nothing but the tile, so that the loop starts one round of loads after the item is known.  (With
// everything an item reads copied to LDS by the whole workgroup first, a launch without any row to work
// on took 5.5 us at 1024 blocks, where an empty one takes 1.8, and 15 us over 512 searches of 128 blocks.)
// Every pass's merge goes straight into the item's LDS tile: a running minimum in registers costs as many
// instructions per pass as the LDS does, and as many registers as the merge itself.
// H: width of the merge (multiple of eight, at least rl); LS: row stride of the tile, whose entry t is
// output t of the merge.  near: first and last row of this wave's first pass.  mine: kNearWords values.
// Returns whether any pass of this wave had work.
constexpr int kNearWords = 4 * (64 + 4);

template <typename VT, int H, int LS, int HMAX>
__device__ __forceinline__ bool merge_passes(VT *tile, VT *mine, const VT RANNC_GLOBAL *__restrict__ V, const char RANNC_GLOBAL *__restrict__ passes,
                                             const int N, const int D, const int DP, const int s, const int n,
                                             const uint32_t near, const int lane, const int wave, const DirectConsts<HMAX> &k) {
  constexpr VT INF = Lim<VT>::inf;
  constexpr int E = 16 / (int)sizeof(VT);  // values per 16 bytes
  constexpr int AS = H + E, NT = 64 * kMergeWaves;  // row stride in LDS: 16-byte aligned, rows on different banks
  constexpr int HP = H <= 8 ? 8 : H <= 16 ? 16 : H <= 32 ? 32 : 64, PER = 64 / HP;  // rows a load covers
  constexpr int LOADS = HP == 64 ? 4 : 2, NEAR = LOADS * PER;
  static_assert(NEAR * AS <= kNearWords, "the near rows fit their LDS");
  typedef VT Values __attribute__((ext_vector_type(E)));
  typedef VT ValuesAny __attribute__((ext_vector_type(E), aligned(sizeof(VT))));  // (a[sig] is any value of the row)
  const int sig = merge_shift(s, DP, H), rl = D - s + 1, top = D - 2 - sig;
  const VT RANNC_GLOBAL *__restrict__ Vprev = V + (int64_t)(s - 2) * (int64_t)(N + 1) * DP + sig;
  const int sub = lane / HP, t_of = lane % HP;
  struct Rows { int lo, hi; VT a[LOADS]; };
  auto fetch_word = [&](int x) -> uint32_t {
    return ((const uint32_t RANNC_GLOBAL *)(passes + min(x, n - 1) * pass_bytes<VT>()))[lane];
  };
  auto fetch_time = [&](int x) -> VT {
    return ((const VT RANNC_GLOBAL *)(passes + min(x, n - 1) * pass_bytes<VT>() + 256))[lane];
  };
  auto fetch_rows = [&](int lo, int hi) -> Rows {
    Rows r;
    r.lo = lo; r.hi = hi;
#pragma unroll
    for (int q = 0; q < LOADS; ++q) r.a[q] = Vprev[(int64_t)min(lo + q * PER + sub, hi) * DP + min(t_of, H - 1)];
    return r;
  };
  uint32_t next_word = fetch_word(wave), after = fetch_word(wave + kMergeWaves);
  VT next_time = fetch_time(wave);
  Rows next_rows = fetch_rows((int)(near & 0xffffu), (int)(near >> 16));
  typedef uint32_t Quad __attribute__((ext_vector_type(4)));
  static_assert(64 * LS * sizeof(VT) % 16 == 0, "the tile is cleared 16 bytes at a time");
  constexpr uint32_t inf_lo = (uint32_t)INF, inf_hi = (uint32_t)((uint64_t)INF >> (sizeof(VT) == 8 ? 32 : 0));
  for (int e = threadIdx.x; e < 64 * LS / E; e += NT) ((Quad *)tile)[e] = Quad{inf_lo, inf_hi, inf_lo, inf_hi};
  lds_barrier();  // (the loads stay in flight)
  bool any = false;
#pragma unroll 1
  for (int x = wave; x < n; x += kMergeWaves) {
    const uint32_t word = next_word;
    const VT tij = next_time;
    const Rows r = next_rows;
    next_word = after;
    next_time = fetch_time(x + kMergeWaves);
    after = fetch_word(x + 2 * kMergeWaves);
    {
      const int last = 63 - __clzll((long long)__ballot(next_word != ~0u));  // (lane 0 has a stage)
      next_rows = fetch_rows((int)(lane_bcast(next_word, 0) & 0xffffu), (int)(lane_bcast(next_word, last) & 0xffffu));
    }
    const int row = min((int)(word & 0xffffu), r.hi), col = (int)(word >> 16) & 63, rmn = (int)(word >> 22);
    VT alast, w[H];
    if (r.hi - r.lo < NEAR) {
      if (t_of < H) {
#pragma unroll
        for (int q = 0; q < LOADS; ++q) mine[(q * PER + sub) * AS + t_of] = r.a[q];
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      const VT *from = mine + (row - r.lo) * AS;
      alast = from[top];
#pragma unroll
      for (int g = 0; g < H / E; ++g) {
        const Values v = *(const Values *)&from[E * g];
#pragma unroll
        for (int u = 0; u < E; ++u) w[E * g + u] = v[u];
      }
    } else {
      const VT RANNC_GLOBAL *from = Vprev + (int64_t)row * DP;
      alast = from[top];
#pragma unroll
      for (int g = 0; g < H / E; ++g) {
        const ValuesAny v = *(const ValuesAny RANNC_GLOBAL *)(from + E * g);
#pragma unroll
        for (int u = 0; u < E; ++u) w[E * g + u] = v[u];
      }
      __builtin_amdgcn_s_waitcnt(0x0f70);  // (vmcnt(0) here, or the compiler waits where the two branches meet)
    }
    // an (s-1)-stage plan on at most D-1 devices covers blocks 1..row iff the last of them is finite
    // (behind the chunk's last stage rmn is above any rl)
    const bool act = rmn <= rl && row >= s - 1 && alast != INF;
    if (__ballot(act) == 0ull) continue;
    any = true;
    row_merge_direct<VT, H>(w, tij, rmn, act, k);
    if (act) {
#pragma unroll
      for (int t = 0; t < H; ++t) atomicMin(&tile[col * LS + t], w[t]);
    }
  }
  return any;
}

// Waves per SIMD the level kernel is compiled for: the two value arrays of the widest 32-bit case
// fit the 168 registers of three waves per SIMD (the compiler left alone takes one more).  The
// recomputing form holds one array: as many as its workgroups per compute unit (merge_workgroups_per_cu).  Left
// alone, the 64-bit forms for up to 32 and 16 values took 98 and 66 registers, one workgroup per compute unit fewer
// than the size of the items counts on (1024 blocks at 32 devices where memory never binds 300 -> 271 us a call).
// (64-bit values at 64 devices: loop-invariant addresses and one time, 20 bytes, go to scratch.  With addresses formed
// for every load and the times asked for behind the merge nothing does, and the call takes 741 us instead of 726.)
// (Table form on 64-bit values at 8 devices: 76 registers left alone, six workgroups to a compute unit; asked for seven
// waves it takes 60, and eight run: 600 searches of 200 blocks with send times 946 -> 873 us a call, 100 of 500 434 -> 417.)
template <typename VT, int HMAX, bool DIRECT> constexpr int merge_waves_per_simd() {
  if (DIRECT && sizeof(VT) == 4) return HMAX == 64 ? 4 : HMAX == 48 ? 5 : 6;
  if (DIRECT) return HMAX >= 48 ? 3 : HMAX == 32 ? 5 : 8;
  return HMAX == 64 ? 3 : sizeof(VT) == 8 && HMAX == 8 ? 7 : 1;
}

// The rows i0+wave, i0+wave+4, ... <= i_hi of one work item, folded into acc (running minimum of the
// sorted merges).  Returns whether any row had work.
// ROWFOLD: the sorted merge of every row goes straight into the lane's row of the workgroup's LDS
// tile instead of a running minimum in registers (64-bit values at DP = 64: two value arrays would
// take all 256 registers of a wave and leave one wave per SIMD).
template <typename VT, int H, bool ROWFOLD, int HMAX>
__device__ __forceinline__ bool merge_rows(VT (&acc)[HMAX], VT *tile_lane, const ProblemDev &pr, const int s,
                                           const int c, const int i0, const int i_hi, const int lane,
                                           const int wave) {
  constexpr VT INF = Lim<VT>::inf;
  const int N = pr.N, D = pr.D, DP = pr.DP, nch = pr.nch;
  const int sig = merge_shift(s, DP, H);
  const int jj = 64 * c + lane;
  const int64_t lvl = (int64_t)(N + 1) * DP;
  const VT RANNC_GLOBAL *__restrict__ Vprev = gptr((const VT *)pr.V) + (int64_t)(s - 2) * lvl;
  const VT RANNC_GLOBAL *__restrict__ cost = gptr((const VT *)pr.cost);
  const uint8_t RANNC_GLOBAL *__restrict__ rmin = gptr((const uint8_t *)pr.rmin);
  const int rl = D - s + 1;  // replicas left for stage s when s-1 devices are spent earlier
  // Flags of a row: it can contribute if its row of V[s-1] holds a finite plan and the lane's
  // stage fits with at most rl replicas.  Only the loads happen here; the values are looked at one
  // iteration later, so that the wait for them never stands between a row and its own unit reads.
  // The loads are unconditional (rows outside the item are clamped to a row inside it, every column
  // of a unit has its rmin byte in memory): a load inside a branch would be waited for where the
  // branch ends.
  struct Flags { VT alast; int rmn; int64_t ubase; };
  auto load_flags = [&](int i) -> Flags {
    const int ic = min(max(i, s - 1), i_hi);
    Flags f;
    f.ubase = unit_index(nch, ic, c);
    f.alast = Vprev[(int64_t)ic * DP + D - 1];
    f.rmn = rmin[f.ubase * 64 + lane];
    return f;
  };
  bool any = false;
  int i = i0 + wave;
  Flags cur = load_flags(i);
  while (i <= i_hi) {  // wave-uniform
    const bool act = i >= s - 1 && cur.alast != INF && jj >= i && jj < N && cur.rmn <= rl;
    const int64_t ubase = cur.ubase;
    cur = load_flags(i + kMergeWaves);  // the next row's
    const unsigned long long work = __ballot(act);
    if (work != 0ull) {
      any = true;
      VT x[H];
      const int col = act ? lane : __ffsll((long long)work) - 1;  // a lane without work reads a needed column
      row_merge<VT, H, const VT RANNC_GLOBAL *>(x, cost + ubase * 64 * D + col, Vprev + (int64_t)i * DP + sig,
                                                act ? (VT)0 : INF, rl);
      if constexpr (ROWFOLD) {
        if (act) {
#pragma unroll
          for (int t = 0; t < H; ++t) atomicMin(&tile_lane[t], x[t]);
        }
      } else {
#pragma unroll
        for (int t = 0; t < H; ++t) acc[t] = vmin(acc[t], x[t]);
      }
    }
    i += kMergeWaves;
  }
  return any;
}

// HMAX: the widest merge this kernel holds registers for (the host takes the smallest one that covers
// the launch: narrow levels run with more waves per SIMD); each search takes the width it needs.
template <typename VT, int HMAX, bool DIRECT>
__device__ __forceinline__ void level_merge_body(const ProblemDev &pr, const int s, const int item) {
  // What the workgroup needs of the descriptor, and then of the list, is asked for at once and waited for
  // once: left alone, the compiler reads each field where it is first used, behind the exits in front of
  // it, and a launch starts with a chain of six scalar reads.  (Not in the table form: behind an asm statement the
  // compiler no longer reads the rows of V[s-1] into scalar registers, 1024 searches of 128 blocks, 64-bit values,
  // 32 devices 181 -> 264 us per level.)
  const int S_eff = pr.S_eff, N = pr.N, D = pr.D, DP = pr.DP, nch = pr.nch;
  const int32_t RANNC_GLOBAL *__restrict__ runs = gptr((const int32_t *)pr.runs);
  VT RANNC_GLOBAL *const V = gptr((VT *)pr.V);
  const char RANNC_GLOBAL *__restrict__ passes = gptr((const char *)pr.cost);
  if constexpr (DIRECT) asm volatile("" :: "s"(S_eff), "s"(N), "s"(D), "s"(DP), "s"(nch), "s"(runs), "s"(V), "s"(passes));
  if (s > S_eff) return;
  int c, i0 = 0, i_hi = 0, n = 0;
  [[maybe_unused]] uint32_t near = 0;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int count = runs[0];
  if constexpr (DIRECT) {
    typedef uint32_t Item __attribute__((ext_vector_type(8)));
    const Item it = *(const Item RANNC_GLOBAL *)((const uint32_t RANNC_GLOBAL *)runs +
                                                 kPassItemWords * (1 + min(item, max_pass_items(nch) - 1)));  // (a place that every list has)
    asm volatile("" :: "s"(count), "s"(it));
    if (item >= count) return;
    c = (int)(it[1] & 0xffffu);
    n = (int)(it[1] >> 16) + 1;
    near = wave == 0 || n < 2 ? it[2] : wave == 1 || n < 3 ? it[3] : wave == 2 || n < 4 ? it[4] : it[5];
    passes += (int64_t)it[0] * pass_bytes<VT>();
  } else {
    if (item >= count) return;
    const unsigned desc = (unsigned)runs[1 + item];
    c = (int)((desc >> 16) & 0x3ffu);
    i0 = (int)(desc & 0xffffu);
    i_hi = min(min(i0 + (int)(desc >> 26), 64 * c + 63), N - 1);
    if (i_hi < s - 1) return;
  }
  if (64 * c + 64 < s) return;  // no column j >= s in this chunk
  const int lane = threadIdx.x & 63;
  constexpr VT INF = Lim<VT>::inf;
  VT RANNC_GLOBAL *Vcur = V + (int64_t)(s - 1) * (int64_t)(N + 1) * DP;

  // acc[t] = running minimum over this wave's rows of the sorted merge
  constexpr bool ROWFOLD = DIRECT || (sizeof(VT) == 8 && HMAX >= 48);  // rows fold into the tile while the row loop runs
  constexpr int NT = 64 * kMergeWaves;
  constexpr int LS = HMAX + 1;
  __shared__ __align__(16) VT tile[64 * LS];
  [[maybe_unused]] VT acc[HMAX];
  if constexpr (ROWFOLD) {
    if constexpr (!DIRECT) {  // (the recomputing form clears the tile behind its first loads)
      for (int e = threadIdx.x; e < 64 * LS; e += NT) tile[e] = INF;
      __syncthreads();
    }
  } else {
#pragma unroll
    for (int t = 0; t < HMAX; ++t) acc[t] = INF;
  }
  bool any = false;
  const int ng = (D - s + 1 + 7) >> 3;  // width of the merge in groups of eight
  if constexpr (DIRECT) {
    DirectConsts<HMAX> k;
    direct_consts_init(k);
    __shared__ __align__(16) VT rows_in[kMergeWaves * kNearWords];
    VT *const mine = rows_in + wave * kNearWords;
#define RANNC_ROWS(K)                                                                          \
  case K:                                                                                      \
    if constexpr (8 * K <= HMAX)                                                               \
      any = merge_passes<VT, 8 * K, LS, HMAX>(tile, mine, V, passes, N, D, DP, s, n, near, lane, wave, k); \
    break;
    switch (ng) {
      RANNC_ROWS(1) RANNC_ROWS(2) RANNC_ROWS(3) RANNC_ROWS(4)
      RANNC_ROWS(5) RANNC_ROWS(6) RANNC_ROWS(7) RANNC_ROWS(8)
      default: break;
    }
#undef RANNC_ROWS
  } else {
#define RANNC_ROWS(K)                                                                               \
  case K:                                                                                           \
    if constexpr (8 * K <= HMAX)                                                                    \
      any = merge_rows<VT, 8 * K, ROWFOLD>(acc, tile + lane * LS, pr, s, c, i0, i_hi, lane, wave);  \
    break;
    switch (ng) {
      RANNC_ROWS(1) RANNC_ROWS(2) RANNC_ROWS(3) RANNC_ROWS(4)
      RANNC_ROWS(5) RANNC_ROWS(6) RANNC_ROWS(7) RANNC_ROWS(8)
      default: break;
    }
#undef RANNC_ROWS
  }

  // acc[t] is W[d = t+2+sig]; V rows are indexed by d-1 = t+1+sig.  Fold the waves in LDS, then
  // write transposed so that one atomic instruction covers consecutive d of one column.
  if constexpr (ROWFOLD) {
    if (__syncthreads_or(any) == 0) return;
  } else {
    for (int e = threadIdx.x; e < 64 * LS; e += NT) tile[e] = INF;
    if (__syncthreads_or(any) == 0) return;
    if (any) {
#pragma unroll
      for (int t = 0; t < HMAX; ++t)
        if (t < 8 * ng) atomicMin(&tile[lane * LS + t], acc[t]);  // folding INF in is a no-op
    }
    __syncthreads();
  }
  const int sig = merge_shift(s, DP, 8 * ng);
  constexpr int WT = HMAX > 32 ? 64 : HMAX > 16 ? 32 : HMAX;  // threads per column
  constexpr int RPP = NT / WT;                                // columns per pass
  const int t = threadIdx.x & (WT - 1);
  if (t >= HMAX || t + 1 + sig > D - 1) return;
  for (int row = threadIdx.x / WT; row < 64; row += RPP) {
    const VT v = tile[row * LS + t];
    const int j = 64 * c + row + 1;
    if (j <= N && j >= s && v != INF) global_min(&Vcur[(int64_t)j * DP + t + 1 + sig], v);
  }
}

template <typename VT, int HMAX, bool DIRECT>
__global__ __launch_bounds__(64 * kMergeWaves) __attribute__((amdgpu_waves_per_eu(merge_waves_per_simd<VT, HMAX, DIRECT>())))
void level_merge_kernel(const ProblemDev *__restrict__ probs, const int s, const int search_major) {
  // Workgroups go to the eight XCDs round-robin in the order of their linear index.  With the items
  // of a search next to each other (search_major) and, say, four items per search, item k of every
  // search lands on XCDs k and k + 4: the XCDs with the long items finish last and those with the
  // empty ones idle (config 5: 176 against 121 us per level).  In a launch of the recomputing form
  // over several searches the search index therefore runs fastest: every XCD gets every kind of item.
  if (search_major) level_merge_body<VT, HMAX, DIRECT>(probs[blockIdx.z], s, (int)blockIdx.x);
  else level_merge_body<VT, HMAX, DIRECT>(probs[blockIdx.x], s, (int)blockIdx.z);
}

// The same for a launch over ONE search, with the descriptor as a kernel argument: a workgroup then
// starts with its fields in scalar registers instead of fetching them through the descriptor
// array's pointer, one memory round trip less in a launch that consists of a few of them.
template <typename VT, int HMAX, bool DIRECT>
__global__ __launch_bounds__(64 * kMergeWaves) __attribute__((amdgpu_waves_per_eu(merge_waves_per_simd<VT, HMAX, DIRECT>())))
void level_merge_one_kernel(const ProblemDev pr, const int s) {
  level_merge_body<VT, HMAX, DIRECT>(pr, s, (int)blockIdx.x);
}

// ---------------------------------------------------------------------------------------
// DP level s >= 2, literal form: one thread per cell (j, d) scans every split point i
// (ascending) and every device count d' of the earlier stages (ascending), skipping infeasible
// predecessors and stages that do not fit, and keeps the first strict minimum -- the loops of
// Algorithm 1 as written.  Used as the reference level kernel (RANNC_DP_ALGO_SCAN) and to
// produce the (i, d') tables for export.  With write_v = 0 the value table is left alone and
// only the argmin arrays (canonical [(L+1)][N+1][D+1] layout of one problem) are written.
// ---------------------------------------------------------------------------------------
template <typename VT>
__global__ __launch_bounds__(64) void level_scan_kernel(const ProblemDev *__restrict__ probs, const int s,
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
  const VT *__restrict__ Vprev = (const VT *)pr.V + (int64_t)(s - 2) * lvl;
  const VT *__restrict__ cost = (const VT *)pr.cost;
  VT best = INF;
  int bi = -1, bd = -1;
  const int i_end = min(64 * c + 63, N - 1);
  for (int i = s - 1; i <= i_end; ++i) {
    const bool act = (jj >= i) && (jj < N);
    const int64_t u = unit_index(nch, i, c);
    const VT *__restrict__ unit = cost + u * 64 * D + lane;
    const int rmn = act ? (int)pr.rmin[u * 64 + lane] : 255;
    for (int dp = s - 1; dp <= d - 1; ++dp) {
      const VT a = Vprev[(int64_t)i * DP + dp - 1];
      if (a == INF) continue;  // earlier stages infeasible
      if (d - dp < rmn) continue;  // does not fit device memory
      const VT h = unit[(d - dp - 1) * 64];
      const VT v = vmax(a, h);
      if (v < best) { best = v; bi = i; bd = dp; }
    }
  }
  if (jj >= N || j < s) return;
  if (write_v) ((VT *)pr.V)[(int64_t)(s - 1) * lvl + (int64_t)j * DP + d - 1] = best;
  const int64_t e = ((int64_t)s * (N + 1) + j) * (D + 1) + d;
  if (arg_i) arg_i[e] = bi;
  if (arg_d) arg_d[e] = bd;
}

// ---------------------------------------------------------------------------------------
// Final choice of the stage count: opt = min over s of V[s][N][D], smallest s among equals.
// One wave per problem, lane s-1 reads V[s][N][D] (S_eff <= D <= 64).
// ---------------------------------------------------------------------------------------
// one wave: lane s-1 brings V[s][N][D] (INT64_MAX beyond S_eff or if the status is bad)
struct Chosen { int64_t opt, est; int n_stages, status; };
__device__ __forceinline__ Chosen select_finish(const ProblemDev &pr, int64_t v, int st, int64_t *d_opt,
                                                int32_t *d_n_stages, int64_t *d_est, int32_t *d_status) {
  const int lane = threadIdx.x & 63;
  const int q = pr.q;
  // the minimum; the first lane that holds it has the fewest stages
  const int64_t best = (int64_t)wave_min((uint64_t)v);  // (no value is negative)
  const int bs = best == INT64_MAX ? 0 : __ffsll((long long)__ballot(v == best));
  Chosen c = {best, INT64_MAX, bs, st};
  if (bs > 0) {
    const int64_t f = (int64_t)pr.MB + bs - 1;
    c.est = (best != 0 && f > INT64_MAX / best) ? INT64_MAX : f * best;
  }
  if (lane == 0) {
    pr.res[0] = best;
    pr.res[1] = bs;
    if (d_opt) d_opt[q] = best;
    if (d_n_stages) d_n_stages[q] = bs;
    if (d_est) d_est[q] = c.est;
    if (d_status) d_status[q] = st;
  }
  return c;
}

// one wave
__device__ __forceinline__ Chosen select_body(const ProblemDev &pr, int64_t *d_opt, int32_t *d_n_stages, int64_t *d_est,
                                              int32_t *d_status) {
  const int lane = threadIdx.x & 63;
  const int st = *pr.status;  // (asked for together with the values)
  int64_t v = INT64_MAX;
  if (lane < pr.S_eff) {
    const int64_t lvl = (int64_t)(pr.N + 1) * pr.DP;
    const int64_t cell = (int64_t)pr.N * pr.DP + pr.D - 1;
    if (pr.bits == 32) {
      const uint32_t u = ((const uint32_t *)pr.V)[lane * lvl + cell];
      v = (u == Lim<uint32_t>::inf) ? INT64_MAX : (int64_t)u;
    } else {
      const uint64_t u = ((const uint64_t *)pr.V)[lane * lvl + cell];
      v = (u == Lim<uint64_t>::inf) ? INT64_MAX : (int64_t)u;
    }
  }
  if (st != 0) v = INT64_MAX;
  return select_finish(pr, v, st, d_opt, d_n_stages, d_est, d_status);
}

__global__ __launch_bounds__(64) void select_kernel(const ProblemDev *__restrict__ probs,
                                                    int64_t *d_opt, int32_t *d_n_stages,
                                                    int64_t *d_est, int32_t *d_status) {
  select_body(probs[blockIdx.x], d_opt, d_n_stages, d_est, d_status);
}

// ---------------------------------------------------------------------------------------
// Plan recovery (Algorithm 1's return value: the stage boundaries and replica counts behind the
// optimal table value).
// One workgroup per problem walks from (s*, N, D) down to level 1.  At each cell it finds the
// lexicographically smallest (i, d') with max(V[s-1][i][d'], h(i,j,d-d')) equal to the cell's
// value v: the candidate that the ascending scan with strict "<" of Algorithm 1 would have kept.
// v is the minimum over all candidates, so "equal" is "at most".  A lane owns a split point i.  The stage
// (i, j) takes at most v from some replica count r on (its time and its bytes fall with r), and V[s-1][i][.]
// falls with d': row i holds a candidate iff V[s-1][i][d - r] <= v, and its first one is the smallest d' with
// V[s-1][i][d'] <= v.  r follows from the time alone where one replica holds the bytes, so a lane asks for the
// rmin byte and for the eight values up to V[s-1][i][d - r] at once; the first candidate lies among them
// unless the row is flat for longer, and then only the first row with a candidate is looked at further.
// Value and prefix sum of the chosen row travel to the next step through LDS.
// Bound by latency: one round trip and one barrier per stage.  (Eight probes of the whole row and then
// eight reads of the eighth it lies in were two: 1.9 us a stage out of memory at 64 devices, now 1.6; what stands in
// front of the walk and behind it 8.0 us, now 5.3, 1024 blocks in one stage.)
// The plan and what else the host is told stay in LDS until one wave writes all of it.
// ---------------------------------------------------------------------------------------
constexpr int kTracebackThreads = 1024;

// What the waves of a plan recovery exchange: per step the smallest key ((i << 8) | d') found, in three
// words of which one is cleared while another is in use (one barrier per step), and the value and prefix
// sum of each wave's first match; then the plan.
struct TracebackLds {
  unsigned int key[3];
  uint64_t value[2][kTracebackThreads / 64];
  int64_t T[2][kTracebackThreads / 64];
  Chosen chosen;
  int ns;  // stages of the plan, 0: none
  int32_t end[RANNC_DP_MAX_DEVICES], replicas[RANNC_DP_MAX_DEVICES];
};

// The smallest r with ceil(x / r) + ceil(C / r) <= v, or more than `most`; inv_v: about 1 / v; hc: lane r - 1 of
// the wave holds ceil(C / r) (only with C).
template <typename VT>
__device__ __forceinline__ int least_replicas(uint64_t x, uint64_t C, VT v, float inv_v, uint64_t hc, int most) {
  if (v == 0) return x == 0 && C == 0 ? 1 : most + 1;
  int r = ceil_ratio(x + C, v, inv_v);
  if (C) {  // two ceilings may need some more
    for (bool done = false; __any(!done);) {
      const uint64_t c = __shfl(hc, min(r, 64) - 1);
      done = done || r > most || (c <= (uint64_t)v && at_most_times(x, (VT)(v - (VT)c), (uint32_t)r));
      if (!done) ++r;
    }
  }
  return r;
}

// forced > 0: the plan of exactly `forced` stages (Algorithm 1's own answer V[S][|B|][D]), if that level
// holds one; forced = 0: the best level chosen by the solve, or here (choose: select_body, by the first
// wave); forced < 0: no plan wanted.  The first wave leaves ns and, chosen here or read (results), what
// else the host is told in sh; every wave learns ns behind a barrier.
template <typename VT>
__device__ __forceinline__ int traceback_stages(const ProblemDev &pr, TracebackLds &sh, int forced, const PlanResults &results,
                                                bool choose) {
  if (threadIdx.x < 64) {
    const int64_t lvl = (int64_t)(pr.N + 1) * pr.DP, cell = (int64_t)pr.N * pr.DP + pr.D - 1;
    Chosen c;
    if (choose) {
      c = select_body(pr, results.d_opt, results.d_n_stages, results.d_est, results.d_status);
    } else {
      c = {INT64_MAX, INT64_MAX, (int)pr.res[1], *pr.status};
      if (results.h_flag) {
        c.opt = results.d_opt[pr.q];
        c.est = results.d_est[pr.q];
      }
    }
    int ns = forced < 0 || c.status != 0 ? 0 : c.n_stages;
    if (forced > 0 && c.status == 0)
      ns = forced <= pr.S_eff && gptr((const VT *)pr.V)[(int64_t)(forced - 1) * lvl + cell] != Lim<VT>::inf ? forced : 0;
    if (threadIdx.x == 0) { sh.chosen = c; sh.ns = ns; }
  }
  if (threadIdx.x < 3) sh.key[threadIdx.x] = 0xFFFFFFFFu;
  __syncthreads();
  return sh.ns;
}

// The walk over the levels, by the whole workgroup.  at: where the tables are (row(s, i): V[s][i][1 ..]).
template <typename VT, typename At>
__device__ __forceinline__ void traceback_walk(const At &at, int N, int D, int ns, TracebackLds &sh) {
  const int tid = threadIdx.x, lane = tid & 63, nt = blockDim.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int j = N, d = D;
  VT v = at.row(ns, N)[D - 1];
  int64_t Tj = at.sum(N);
  int step = 0;
  for (int s = ns; s >= 2; --s) {
    const uint64_t Cj = at.send(j);  // send time of the cut after block j (0 for j = N)
    const int first = max(s - 1, at.first(j));
    const int low = s - 2, most = d - (s - 1);      // V[..][low] is d' = s-1; replicas left for this stage
    const float inv_v = __builtin_amdgcn_rcpf((float)v);
    uint64_t hc = 0;
    if (Cj) hc = (Cj + (uint64_t)lane) / (uint64_t)(lane + 1);
    unsigned key = 0xFFFFFFFFu;
    for (int i0 = first; i0 < j && key == 0xFFFFFFFFu; i0 += nt) {  // rows ascend: the first match is the smallest
      const int b = step % 3, p = step & 1;
      if (i0 + 64 * wave < j) {  // (the window rarely fills the workgroup; the other waves would only take issue slots)
        const int i = min(i0 + tid, j - 1);
        const auto row = at.row(s - 1, i);  // row[d' - 1]
        const int rmn = at.least(i, j);
        const int64_t Ti = at.sum(i);
        const int rt = least_replicas<VT>((uint64_t)(Tj - Ti), Cj, v, inv_v, hc, most);
        int base = max(d - min(rt, d) - 8, 0);  // eight values, up to V[..][d - rt] if that exists
        VT a[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) a[k] = row[base + k];
        const int top = d - max(rt, rmn) - 1;
        bool ok = top >= low && i0 + tid < j;
        if (__any(ok && top < base)) {  // the bytes need more replicas than the time
          if (ok && top < base) {
            base = max(top - 7, 0);
#pragma unroll
            for (int k = 0; k < 8; ++k) a[k] = row[base + k];
          }
        }
        unsigned within = 0;  // (non-increasing: the upper ones)
#pragma unroll
        for (int k = 0; k < 8; ++k) within |= a[k] <= v ? 1u << k : 0u;
        ok = ok && ((within >> ((top - base) & 31)) & 1u);
        const unsigned long long m = __ballot(ok);
        if (m != 0ull && lane == __ffsll((long long)m) - 1) {
          while ((within & 1u) && base > 0) {  // the row is flat here: further down
            base = max(base - 8, 0);
            within = 0;
#pragma unroll
            for (int k = 0; k < 8; ++k) a[k] = row[base + k];
#pragma unroll
            for (int k = 0; k < 8; ++k) within |= a[k] <= v ? 1u << k : 0u;
          }
          // (the first place that holds a value of at most v; below a window without one, the window above's first)
          const int k = within ? __ffs((int)within) - 1 : 8;
          VT mine = a[0];
#pragma unroll
          for (int u = 1; u < 8; ++u) mine = k == u ? a[u] : mine;
          if (k == 8) mine = row[base + 8];
          atomicMin(&sh.key[b], ((unsigned)i << 8) | (unsigned)(base + k + 1));
          sh.value[p][wave] = (uint64_t)mine;
          sh.T[p][wave] = Ti;
        }
      }
      lds_barrier();
      key = sh.key[b];
      if (tid == 0) sh.key[(step + 2) % 3] = 0xFFFFFFFFu;  // the word of the step before: everybody has read it
      ++step;
      if (key != 0xFFFFFFFFu) {
        const int from = ((int)(key >> 8) - i0) >> 6;  // the wave whose first match it was
        v = (VT)sh.value[p][from];
        Tj = sh.T[p][from];
      }
    }
    if (key == 0xFFFFFFFFu) {  // tables inconsistent: report no plan rather than walk on
      if (tid == 0) sh.ns = 0;
      return;
    }
    const int i_sel = (int)(key >> 8), d_sel = (int)(key & 255u);
    if (tid == 0) { sh.end[s - 1] = j; sh.replicas[s - 1] = d - d_sel; }
    j = i_sel;
    d = d_sel;
  }
  if (tid == 0) { sh.end[0] = j; sh.replicas[0] = d; }
}

// STAGED: everything the walk reads (the levels of V below the plan's, T, C, the window bounds, the
// fits-in-memory bytes) is first copied into the workgroup's LDS with one round of independent reads,
// and the walk then runs out of LDS.  Otherwise the window bounds and, up to kTracebackSums of them, the
// prefix sums are (out of memory they would be another round trip).
// lds: traceback_lds_bytes() bytes (not STAGED: up to kTracebackSums + 1 sums, and nch words).
constexpr int kTracebackSums = 2048;

template <typename VT, bool STAGED>
__device__ void traceback_body(const ProblemDev &pr, TracebackLds &sh, int forced, char *lds, const PlanResults &results, bool choose) {
  const int N = pr.N, D = pr.D, DP = pr.DP, nch = pr.nch;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int64_t lvl = (int64_t)(N + 1) * DP;
  const VT RANNC_GLOBAL *Vg = gptr((const VT *)pr.V);
  using VP = std::conditional_t<STAGED, const VT *, const VT RANNC_GLOBAL *>;
  using CP = std::conditional_t<STAGED, const int64_t *, const int64_t RANNC_GLOBAL *>;
  using RP = std::conditional_t<STAGED, const uint8_t *, const uint8_t RANNC_GLOBAL *>;
  typedef uint32_t Quad __attribute__((ext_vector_type(4)));
  VP V;
  CP C = nullptr;
  RP rmin;
  const int64_t *T;
  const int32_t *wlo;
  [[maybe_unused]] VT *Vl = (VT *)lds;
  const bool sums = STAGED || N <= kTracebackSums;
  // (the first wave looks for the stage count meanwhile)
  if constexpr (STAGED) {
    const int64_t nT = (((int64_t)(N + 1) * 8 + 31) / 32) * 32;
    char *w = lds + (int64_t)pr.S_eff * lvl * (int64_t)sizeof(VT);  // room for every level
    int64_t *Tl = (int64_t *)w; w += nT;
    int64_t *Cl = (int64_t *)w; w += nT;
    int32_t *Wl = (int32_t *)w; w += (((int64_t)nch * 4 + 31) / 32) * 32;
    uint8_t *Rl = (uint8_t *)w;
    // (every array starts on a 256-byte boundary of the workspace)
    if (tid >= 64) {
      for (int e = tid - 64; e <= N; e += nt - 64) {
        Tl[e] = pr.T[e];
        if (pr.C) Cl[e] = pr.C[e];
      }
      for (int e = tid - 64; e < nch; e += nt - 64) Wl[e] = pr.wlo[e];
      const Quad RANNC_GLOBAL *rsrc = (const Quad RANNC_GLOBAL *)gptr((const uint8_t *)pr.rmin);
      for (int64_t e = tid - 64; e < units_before(nch, N) * 4; e += nt - 64) ((Quad *)Rl)[e] = rsrc[e];
    }
    V = Vl; T = Tl; rmin = Rl; wlo = Wl;
    if (pr.C) C = Cl;
  } else {
    V = Vg;
    rmin = gptr((const uint8_t *)pr.rmin);
    int64_t *Tl = (int64_t *)lds;
    int32_t *Wl = (int32_t *)(Tl + (sums ? N + 1 : 0));
    if (tid >= 64) {
      if (sums)
        for (int e = tid - 64; e <= N; e += nt - 64) Tl[e] = pr.T[e];
      for (int e = tid - 64; e < nch; e += nt - 64) Wl[e] = pr.wlo[e];
    }
    T = Tl;
    wlo = Wl;
    if (pr.C) C = gptr((const int64_t *)pr.C);
  }
  const int ns = traceback_stages<VT>(pr, sh, forced, results, choose);
  if (ns == 0) return;
  if constexpr (STAGED) {
    // 16-byte copies (a level of V is a multiple of 32 bytes), eight reads in flight per lane (index
    // clamped instead of tested, so that no branch separates them)
    const Quad RANNC_GLOBAL *src = (const Quad RANNC_GLOBAL *)Vg;
    const int64_t nquad = (int64_t)ns * lvl * (int64_t)sizeof(VT) / 16;
    for (int64_t e0 = tid; e0 < nquad; e0 += 8 * (int64_t)nt) {
      Quad r[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) r[k] = src[min(e0 + k * (int64_t)nt, nquad - 1)];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (e0 + k * (int64_t)nt < nquad) ((Quad *)Vl)[e0 + k * (int64_t)nt] = r[k];
    }
    __syncthreads();
  }
  struct Tables {
    VP V;
    CP C;
    RP rmin;
    const int64_t *T, *Tg;
    const int32_t *wlo;
    int64_t lvl;
    int DP, nch;
    __device__ __forceinline__ VP row(int s, int i) const { return V + (int64_t)(s - 1) * lvl + (int64_t)i * DP; }
    __device__ __forceinline__ int64_t sum(int i) const { return T ? T[i] : Tg[i]; }
    __device__ __forceinline__ uint64_t send(int j) const { return C ? (uint64_t)C[j] : 0ull; }
    __device__ __forceinline__ int first(int j) const { return min(wlo[(j - 1) >> 6], j); }  // earlier rows hold no stage that fits
    __device__ __forceinline__ int least(int i, int j) const {
      return (int)rmin[unit_index(nch, i, (j - 1) >> 6) * 64 + ((j - 1) & 63)];
    }
  };
  traceback_walk<VT>(Tables{V, C, rmin, sums ? T : nullptr, pr.T, wlo, lvl, DP, nch}, N, D, ns, sh);
}

// Plan recovery for the split objective: the candidate kept by a cell is the first one, in scan
// order, whose sum equals the cell's value.  All threads of the workgroup evaluate the candidates
// of one cell, numbered in scan order and several per thread with their reads in flight together; the
// smallest matching number wins.
template <typename VT>
__device__ void traceback_split_body(const ProblemDev &pr, TracebackLds &sh, int forced, const PlanResults &results, bool choose) {
  constexpr VT INF = Lim<VT>::inf;
  const int N = pr.N, D = pr.D, DP = pr.DP, nch = pr.nch;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int64_t lvl = (int64_t)(N + 1) * DP;
  const VT RANNC_GLOBAL *V = gptr((const VT *)pr.V), *VF = gptr((const VT *)pr.VF), *VB = gptr((const VT *)pr.VB);
  const int64_t RANNC_GLOBAL *T = gptr((const int64_t *)pr.T), *TB = gptr((const int64_t *)pr.TB);
  const uint8_t RANNC_GLOBAL *rmin = gptr((const uint8_t *)pr.rmin);
  // the stage times are valued from the prefix sums (the level kernel has not built their tables)
  __shared__ double inv[64];
  if (tid < 64) inv[tid] = 1.0 / (double)(tid + 1);
  const bool quick = pr.time_limit <= kCeilDivMax;
  const int ns = traceback_stages<VT>(pr, sh, forced, results, choose);
  if (ns == 0) return;
  auto share = [&](int64_t x, int r) -> VT {
    if (quick) return ceil_div<VT>((VT)x, r, inv[r - 1]);
    return (VT)(((uint64_t)x + (uint64_t)(r - 1)) / (uint64_t)r);
  };
  int j = N, d = D, step = 0;
  VT v = V[(int64_t)(ns - 1) * lvl + (int64_t)N * DP + D - 1];
  for (int s = ns; s >= 2; --s, ++step) {
    const int b = step % 3, p = step & 1;
    const int jj = j - 1, c = jj >> 6;
    const int64_t Tj = T[j], TBj = TB[j], Cj = pr.C ? pr.C[j] : 0;
    const int nd = d - (s - 1);                       // d' = s-1 .. d-1
    const int from = max(s - 1, min(pr.wlo[c], j));   // earlier rows hold no stage that fits
    const int total = (j - from) * nd;                // i = from .. j-1
    const float inv_nd = 1.0f / (float)nd;
    unsigned mine = 0xFFFFFFFFu;
    VT sum_v = 0;
    constexpr int U = 2;
    for (int e0 = tid; e0 < total && mine == 0xFFFFFFFFu; e0 += U * nt) {
      VT f[U], g[U];
      int64_t Ti[U], TBi[U];
      int rm[U], row[U], dd[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = min(e0 + u * nt, total - 1);
        int q = (int)((float)e * inv_nd);  // e / nd, corrected
        q -= q * nd > e ? 1 : 0;
        q += (q + 1) * nd <= e ? 1 : 0;
        row[u] = from + q;
        dd[u] = s - 1 + e - q * nd;
        const int64_t pc = (int64_t)(s - 2) * lvl + (int64_t)row[u] * DP + dd[u] - 1;
        f[u] = VF[pc];
        g[u] = VB[pc];
        rm[u] = (int)rmin[unit_index(nch, row[u], c) * 64 + (jj & 63)];
        Ti[u] = T[row[u]];
        TBi[u] = TB[row[u]];
      }
#pragma unroll
      for (int u = U - 1; u >= 0; --u) {
        // (few candidates get past what their parts alone allow: neither the earlier stages nor this one may take
        // more than v)
        const int r = d - dd[u];
        const uint64_t x = (uint64_t)(Tj - Ti[u]) + (uint64_t)(TBj - TBi[u]) + (uint64_t)Cj;
        if (f[u] == INF || f[u] + g[u] > v || r < rm[u] || !at_most_times(x, (uint64_t)v, (uint32_t)r)) continue;
        const VT hf = share(Tj - Ti[u], r) + (Cj ? share(Cj, r) : (VT)0), hb = share(TBj - TBi[u], r);
        if ((VT)(vmax(f[u], hf) + vmax(g[u], hb)) == v) {  // (i, d') ascends with e
          mine = ((unsigned)row[u] << 8) | (unsigned)dd[u];
          sum_v = f[u] + g[u];
        }
      }
    }
    const unsigned key_mine = mine;
    unsigned best = mine;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) best = min(best, (unsigned)__shfl_xor(best, o));
    if (best != 0xFFFFFFFFu && key_mine == best) {  // (candidates are distinct: one lane)
      atomicMin(&sh.key[b], best);
      sh.value[p][tid >> 6] = (uint64_t)sum_v;
      sh.T[p][tid >> 6] = (int64_t)best;
    }
    if (best == 0xFFFFFFFFu && (tid & 63) == 0) sh.T[p][tid >> 6] = -1;
    __syncthreads();
    const unsigned key = sh.key[b];
    if (tid == 0) sh.key[(step + 2) % 3] = 0xFFFFFFFFu;
    if (key == 0xFFFFFFFFu) {  // tables inconsistent: report no plan rather than walk on
      if (tid == 0) sh.ns = 0;
      return;
    }
    for (int w = 0; w < nt / 64; ++w)
      if (sh.T[p][w] == (int64_t)key) v = (VT)sh.value[p][w];
    const int i_sel = (int)(key >> 8), d_sel = (int)(key & 255u);
    if (tid == 0) { sh.end[s - 1] = j; sh.replicas[s - 1] = d - d_sel; }
    j = i_sel;
    d = d_sel;
  }
  if (tid == 0) { sh.end[0] = j; sh.replicas[0] = d; }
}

// Outer driver (Algorithm 2 "form_stage" of Sec. III-C), the loops over the solved batch: node
// counts n = 1, 2, 4, ... in turn, for each the stage counts S ascending over
// (devices_per_node*(n-1), devices_per_node*n], and for the first S that any search of that n can
// realise (V[S][N][D] finite), the search with the smallest (MB + S - 1) * V, the first one in
// batch order among equals.  That is the lexicographic minimum of (n, S, estimate, search index)
// over all feasible (search, S) pairs, S inside the range of the search's n: one wave, a lane per
// search (in rounds of 64) reads its values straight from the value tables (all reads of a lane
// are independent), then one reduction over the wave.
// Writes the record {q, S, first bad status in batch order or 0, 0, V, estimate} and the plan area
// behind it (-1 everywhere; the plan recovery, in the same launch, fills in the chosen search's).
// q = -1: infeasible.  Returns the chosen search's place in probs (-1: none) and its S.
struct FormStageChoice { int at, S; };
__device__ __forceinline__ FormStageChoice form_stage_choose(const ProblemDev *__restrict__ probs, const FormStageIn &f,
                                                             int stride) {
  constexpr int NONE = 0x7fffffff;
  constexpr int kMaxRange = 64;  // devices_per_node <= RANNC_DP_MAX_DEVICES
  const int lane = threadIdx.x & 63;
  int32_t *plan = (int32_t *)(f.rec + 6);
  for (int u = lane; u < 2 * stride; u += 64) plan[u] = -1;
  int bad_q = NONE, bad_st = 0;
  int best_k = NONE, best_q = NONE, best_p = -1;  // k = n << 16 | S
  int64_t best_e = INT64_MAX, best_v = 0;
  for (int p = lane; p < f.Q; p += 64) {
    const ProblemDev &pr = probs[p];
    const int q = pr.q;
    const int st = *pr.status;
    if (st != 0) {
      if (q < bad_q) { bad_q = q; bad_st = st; }
      continue;
    }
    const int n = pr.D / f.devices_per_node;
    const int64_t mb = pr.MB;
    const int lo = f.devices_per_node * (n - 1) + 1;
    const int hi = min(min(f.devices_per_node * n, f.N), pr.S_eff);
    const int64_t lvl = (int64_t)(pr.N + 1) * pr.DP, cell = (int64_t)pr.N * pr.DP + pr.D - 1;
    // the first S of the range that this search can realise (a smaller S always wins for one n);
    // eight values in flight at a time
    for (int S0 = lo; S0 <= hi && S0 < lo + kMaxRange; S0 += 8) {
      int64_t v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int64_t e = (min(S0 + k, hi) - 1) * lvl + cell;
        if (pr.bits == 32) {
          const uint32_t u = ((const uint32_t *)pr.V)[e];
          v[k] = (u == Lim<uint32_t>::inf) ? INT64_MAX : (int64_t)u;
        } else {
          const uint64_t u = ((const uint64_t *)pr.V)[e];
          v[k] = (u == Lim<uint64_t>::inf) ? INT64_MAX : (int64_t)u;
        }
      }
      int64_t val = INT64_MAX;
      int S = 0;
#pragma unroll
      for (int k = 7; k >= 0; --k)
        if (S0 + k <= hi && S0 + k < lo + kMaxRange && v[k] != INT64_MAX) { val = v[k]; S = S0 + k; }
      if (S == 0) continue;
      const int64_t m = mb + S - 1;
      const int64_t e = (val != 0 && m > INT64_MAX / val) ? INT64_MAX : m * val;
      const int k = n << 16 | S;
      if (k < best_k || (k == best_k && (e < best_e || (e == best_e && q < best_q)))) {
        best_k = k; best_e = e; best_v = val; best_q = q; best_p = p;
      }
      break;
    }
  }
  // the smallest n and S, then the smallest estimate, then the first search of the batch
  auto least = [](auto v) { return (decltype(v))wave_min((std::make_unsigned_t<decltype(v)>)v); };  // (no value is negative)
  const int k_min = least(best_k);
  const int64_t e_min = least(best_k == k_min ? best_e : INT64_MAX);
  const int q_min = least(best_k == k_min && best_e == e_min ? best_q : NONE);
  if (__any(bad_q != NONE)) {
    const int first = least(bad_q);
    const unsigned long long m = __ballot(bad_q == first);
    bad_st = __shfl(bad_st, __ffsll((long long)m) - 1);
    bad_q = first;
  }
  const int winner = __ffsll((long long)__ballot(best_q == q_min)) - 1;
  best_k = k_min; best_e = e_min; best_q = q_min;
  best_p = (int)lane_bcast((uint32_t)best_p, winner);
  best_v = (int64_t)lane_bcast((uint64_t)best_v, winner);
  const bool found = bad_q == NONE && best_q != NONE;
  if (lane == 0) {
    f.rec[0] = found ? best_q : -1;
    f.rec[1] = found ? (best_k & 0xffff) : 0;
    f.rec[2] = bad_q == NONE ? 0 : bad_st;
    f.rec[3] = 0;
    f.rec[4] = found ? best_v : 0;
    f.rec[5] = found ? best_e : 0;
  }
  FormStageChoice c;
  c.at = found ? best_p : -1;
  c.S = found ? (best_k & 0xffff) : 0;
  return c;
}

// The plan to the caller's arrays, and behind the outer driver's record or to the host's mirror of the
// results (both may live in host memory: they are only written here), then the flag word that tells the host,
// which polls it.  One wave writes all of it: the release of the flag word then waits for its own stores
// (with every wave of the workgroup fencing the system this took 4.8 us instead of 1.8).
__device__ __forceinline__ void plan_out(const ProblemDev &pr, int plan_stride, int32_t *se, int32_t *rp, const TracebackLds &sh,
                                         const FormStageIn &f, const PlanResults &r) {
  __syncthreads();
  const int lane = threadIdx.x, q = pr.q;
  if (lane >= 64) return;
  int32_t *const plan = f.rec ? (int32_t *)(f.rec + 6) : nullptr;
  const bool host = r.h_flag != nullptr;
  if (host && lane == 0) {
    r.h_opt[q] = sh.chosen.opt;
    r.h_est[q] = sh.chosen.est;
    r.h_n_stages[q] = sh.chosen.n_stages;
    r.h_status[q] = sh.chosen.status;
  }
  for (int u = lane; u < plan_stride; u += 64) {
    const int32_t end = u < sh.ns ? sh.end[u] : -1, reps = u < sh.ns ? sh.replicas[u] : -1;
    se[u] = end;
    rp[u] = reps;
    if (plan) { plan[u] = end; plan[plan_stride + u] = reps; }
    if (host) {
      r.h_stage_end[(int64_t)q * plan_stride + u] = end;
      r.h_replicas[(int64_t)q * plan_stride + u] = reps;
    }
  }
  uint64_t *const flag = f.rec ? f.flag : host ? &r.h_flag[q] : nullptr;
  if (!flag) return;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");  // (of the whole wave, for the system)
  if (lane == 0) __hip_atomic_store(flag, f.rec ? f.seq : r.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The whole workgroup: the first wave makes the choice; false (and the record is complete) if there is none.
__device__ __forceinline__ bool form_stage_picked(const ProblemDev *__restrict__ probs, const FormStageIn &f, int stride,
                                                  FormStageChoice &pick) {
  if (threadIdx.x < 64) {
    const FormStageChoice c = form_stage_choose(probs, f, stride);
    if (threadIdx.x == 0) pick = c;
  }
  __syncthreads();
  if (pick.at >= 0) return true;
  if (threadIdx.x == 0 && f.flag) {  // (the first wave has written the record and an empty plan)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
    __hip_atomic_store(f.flag, f.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  return false;
}

__global__ __launch_bounds__(kTracebackThreads) void traceback_kernel(
    const ProblemDev *__restrict__ probs, int plan_stride, int32_t *d_stage_end, int32_t *d_replicas,
    const int32_t *__restrict__ d_levels, const FormStageIn fs, const PlanResults results, int choose) {
  __shared__ TracebackLds sh;
  __shared__ FormStageChoice pick;
  __shared__ __align__(16) char sums[8 * (kTracebackSums + 1) + 4096];  // and the window bounds: nch <= 1024 words
  if (fs.rec && !form_stage_picked(probs, fs, plan_stride, pick)) return;
  const ProblemDev pr = probs[fs.rec ? pick.at : (int)blockIdx.x];  // by value: no reloads after the plan stores
  const int forced = fs.rec ? pick.S : d_levels ? d_levels[pr.q] : 0;
  if (pr.VF) {  // split objective: first-match over all candidates
    if (pr.bits == 32) traceback_split_body<uint32_t>(pr, sh, forced, results, choose != 0);
    else traceback_split_body<uint64_t>(pr, sh, forced, results, choose != 0);
  } else if (pr.bits == 32) {
    traceback_body<uint32_t, false>(pr, sh, forced, sums, results, choose != 0);
  } else {
    traceback_body<uint64_t, false>(pr, sh, forced, sums, results, choose != 0);
  }
  plan_out(pr, plan_stride, d_stage_end + (int64_t)pr.q * plan_stride, d_replicas + (int64_t)pr.q * plan_stride, sh, fs, results);
}

// Plan recovery out of LDS, for launches of few, small min-max searches (the host checks that every
// search of the launch fits traceback_lds_bytes() into the dynamic LDS it passes).
__global__ __launch_bounds__(kTracebackThreads) void traceback_lds_kernel(
    const ProblemDev *__restrict__ probs, int plan_stride, int32_t *d_stage_end, int32_t *d_replicas,
    const int32_t *__restrict__ d_levels, const FormStageIn fs, const PlanResults results, int choose) {
  __shared__ TracebackLds sh;
  __shared__ FormStageChoice pick;
  extern __shared__ __align__(16) char staged[];
  if (fs.rec && !form_stage_picked(probs, fs, plan_stride, pick)) return;
  const ProblemDev pr = probs[fs.rec ? pick.at : (int)blockIdx.x];
  const int forced = fs.rec ? pick.S : d_levels ? d_levels[pr.q] : 0;
  if (pr.bits == 32) traceback_body<uint32_t, true>(pr, sh, forced, staged, results, choose != 0);
  else traceback_body<uint64_t, true>(pr, sh, forced, staged, results, choose != 0);
  plan_out(pr, plan_stride, d_stage_end + (int64_t)pr.q * plan_stride, d_replicas + (int64_t)pr.q * plan_stride, sh, fs, results);
}

// ---------------------------------------------------------------------------------------
// Whole search of a SMALL problem (N <= 128, i.e. at most two column chunks) in one workgroup and
// one launch: prefix sums, tables, every level, choice of the stage count.  Same arithmetic as the
// kernels above (the same build_unit / row_merge), but two consecutive levels of V
// live in LDS, so the waves of the workgroup fold their merges with LDS atomics and meet at
// workgroup barriers: no launch per level, no global atomics.  Every level is also copied to the
// V table in memory (plan recovery and export read it there).  Meant for searches at the
// paper's own scale (k = 32 blocks, D <= 32, Sec. IV-A) and for batches of them (the many
// form_stage_dp calls of Algorithm 2): one workgroup per search.
// ---------------------------------------------------------------------------------------
constexpr int kSmallMaxN = 128;
// Sixteen waves per search, eight where a lane's value array alone takes 64 registers or more (64
// devices, or 64-bit values from 32 devices on): with the 128 registers of sixteen waves those
// kernels spilled up to 1 600 registers per lane.
constexpr int kSmallWavesMax = 16;
template <typename VT, int DP> constexpr int small_waves() { return sizeof(VT) * DP >= 256 ? 8 : kSmallWavesMax; }

// Waves per SIMD the one-launch kernel is compiled for.  A batch of hundreds of searches wants TWO workgroups of
// sixteen waves on a compute unit, 64 registers.  The recomputing form on 32-bit values at 16 devices is held to them
// (70 left alone).  The forms at 8 devices, and the table form on 32-bit values at 16, get there without the plan
// recovery, which takes 10 to 25 registers and is for few searches: they have an instance without it (PLAN = false) and
// one with, which launches of up to a search to a compute unit take as well (100 searches of 40 blocks, 16 devices, send
// times 73 us a call, held to 64 registers 78).  (Both as one had 52 to 77 registers and one workgroup to a compute
// unit: 2000 searches of 17 blocks at 8 devices 179 us a call instead of 159, 1000 of 100 blocks 242 instead of 204,
// with send times 520 instead of 392, at 16 devices 743 instead of 673.)
template <typename VT, int DP, bool DIRECT> constexpr bool small_plan_apart() { return DP == 8 || (DP == 16 && sizeof(VT) == 4 && !DIRECT); }
template <typename VT, int DP, bool DIRECT, bool PLAN> constexpr int small_waves_per_simd() {
  return !PLAN || (DIRECT && sizeof(VT) == 4 && DP == 16) ? 8 : small_waves<VT, DP>() / 4;
}

template <typename VT, int DP, bool DIRECT, bool PLAN>
__global__ __launch_bounds__((64 * small_waves<VT, DP>())) __attribute__((amdgpu_waves_per_eu((small_waves_per_simd<VT, DP, DIRECT, PLAN>()))))
void solve_small_kernel(
    const ProblemDev *src, ProblemDev *probs, int64_t *d_opt, int32_t *d_n_stages, int64_t *d_est,
    int32_t *d_status, const ProblemDev one, int use_one, int plan_stride, const PlanResults results) {
  __shared__ __align__(8) uint32_t desc[sizeof(ProblemDev) / 4];
  const ProblemDev pr = fetch_problem(src + blockIdx.x, probs + blockIdx.x, true, desc, one, use_one);
  constexpr VT INF = Lim<VT>::inf;
  constexpr int LS = DP + 1;  // row stride of a level in LDS: lanes (= columns) hit different banks
  constexpr int kSmallWaves = small_waves<VT, DP>();
  constexpr int NT = 64 * kSmallWaves;
  __shared__ int64_t sT[kSmallMaxN + 1], sP[kSmallMaxN + 1], sA[kSmallMaxN + 1], sC[kSmallMaxN + 1];
  __shared__ unsigned long long s_max_cut;
  // levels of V in LDS: the one being read and the one being folded into; the recomputing form keeps
  // a third, cleared while a level runs, so that a level costs one workgroup barrier instead of two
  constexpr int kLevelBufs = DIRECT ? 3 : 2;
  __shared__ VT levels[kLevelBufs * (kSmallMaxN + 1) * LS];
  __shared__ VT s_top[64];
  __shared__ int s_flags, s_wlo[2];
  __shared__ Chosen s_chosen;
  // DIRECT: the stage times are recomputed from the prefix sums in LDS (as the recomputing level
  // kernel does), and the stages that fit are listed in LDS, row by row: no table is written and the levels
  // read nothing from memory.  A word is { row, last block << 8, smallest r that fits << 16 }.
  constexpr int kPairs = kSmallMaxN * (kSmallMaxN + 1) / 2 + 64;
  __shared__ uint32_t s_word[DIRECT ? kPairs : 1];
  __shared__ uint32_t s_end[DIRECT ? kSmallMaxN : 1], s_at[DIRECT ? kSmallMaxN + 1 : 1];
  __shared__ uint64_t s_z[DIRECT ? kSmallMaxN + 1 : 1];
  __shared__ int s_sum[2];
  const int N = pr.N, D = pr.D, nch = pr.nch, S_eff = pr.S_eff;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // (a chain shorter than the longest one has room for more levels: for all of them, if it is short enough)
  const int per_level = (N + 1) * LS;
  const int bufs = DIRECT ? min(max(S_eff, kLevelBufs), kLevelBufs * (kSmallMaxN + 1) * LS / per_level) : kLevelBufs;
  auto level = [&](int s) -> VT * { return levels + (s - 1) % bufs * per_level; };
  // (inside the levels: what is formed from it is formed there again and takes no register for the whole loop)
  auto opaque = [](int x) -> int {
    if constexpr (!PLAN) asm volatile("" : "+v"(x));
    return x;
  };

  // ---- prefix sums and validation (as setup_kernel) ----
  if (tid == 0) {
    s_flags = 0; s_wlo[0] = kNoRow; s_wlo[1] = kNoRow; s_max_cut = 0ull; sC[0] = 0;
    if (pr.o) pr.C[0] = 0;
  }
  int myflags = 0;
  __syncthreads();
  if (tid < N && pr.o) {  // per-cut send time (as setup_kernel)
    const uint64_t c = cut_time(pr.o[tid], pr.bw, myflags);
    sC[tid + 1] = (tid + 1 < N) ? (int64_t)c : 0;
    pr.C[tid + 1] = sC[tid + 1];  // plan recovery values the stages from the prefix sums in memory
    if (tid + 1 < N && c) atomicMax(&s_max_cut, (unsigned long long)c);
  }
  // A wave per array, two blocks per lane, so that the sums need no barrier (a scan over the workgroup had
  // fourteen; whole call, 16 blocks: 26.1 -> 24.8 us, the outer driver at 32 blocks: 102.2 -> 98.8 us).
  if (wave < 3) {
    const int64_t *in = wave == 0 ? pr.t : wave == 1 ? pr.p : pr.a;
    int64_t *out = wave == 0 ? pr.T : wave == 1 ? pr.P : pr.A;
    int64_t *sout = wave == 0 ? sT : wave == 1 ? sP : sA;
    uint64_t u[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      int64_t v = 2 * lane + k < N ? in[2 * lane + k] : 0;
      if (v < 0) { myflags |= 1; v = 0; }
      u[k] = (uint64_t)v;
      if (u[k] >= kSumLimit) { myflags |= 2; u[k] = kSumLimit; }
    }
    uint64_t sum = u[0] + u[1];  // of the lanes up to this one; every sum saturates at kSumLimit
    sum = sum > kSumLimit ? kSumLimit : sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint64_t below = (uint64_t)__shfl_up((unsigned long long)sum, off);
      if (lane >= off) sum += below;
      sum = sum > kSumLimit ? kSumLimit : sum;
    }
    uint64_t before = (uint64_t)__shfl_up((unsigned long long)sum, 1);
    if (lane == 0) before = 0;
    const uint64_t mid = before + u[0] > kSumLimit ? kSumLimit : before + u[0];
    if (sum >= kSumLimit) myflags |= 2;  // (the largest of the lane's sums; beyond block N it stays the last one)
    if (2 * lane < N) { sout[2 * lane + 1] = (int64_t)mid; out[2 * lane + 1] = (int64_t)mid; }
    if (2 * lane + 1 < N) { sout[2 * lane + 2] = (int64_t)sum; out[2 * lane + 2] = (int64_t)sum; }
  }
  if (tid == 0) { sT[0] = sP[0] = sA[0] = 0; pr.T[0] = pr.P[0] = pr.A[0] = 0; }
  if (myflags) atomicOr(&s_flags, myflags);
  // level 1 buffer: "no plan" everywhere, padding columns 0
  for (int e = tid; e < (N + 1) * LS; e += NT) level(1)[e] = ((e % LS) < D) ? INF : (VT)0;
  if constexpr (DIRECT)  // level 2's buffer as well
    for (int e = tid; e < (N + 1) * LS; e += NT) level(2)[e] = ((e % LS) < D) ? INF : (VT)0;
  __syncthreads();
  int st = RANNC_DP_PROBLEM_OK;
  if (s_flags & 1) st = RANNC_DP_PROBLEM_NEGATIVE_INPUT;
  else if (s_flags & 2) st = RANNC_DP_PROBLEM_SUM_OVERFLOW;
  else if ((uint64_t)sT[N] + s_max_cut > (uint64_t)pr.time_limit) st = RANNC_DP_PROBLEM_TIME_TOO_LARGE;
  if (tid == 0) *pr.status = st;

  if constexpr (DIRECT) {
    // Where every row's stages begin in the list: ends[] (pass_entries; a thread per row, on the sums Z as in
    // prepare_kernel where they cannot wrap) and their running sum.  In any case at most N (N + 1) / 2 stages: the
    // ends lie between the row and N.
    const uint64_t M = (uint64_t)pr.M;
    const bool small = (uint64_t)sP[N] < (1ull << 55) && (uint64_t)sA[N] < (1ull << 60);
    if (small && tid <= N) s_z[tid] = (uint64_t)D * (uint64_t)sP[tid] + (uint64_t)sA[tid];
    // (below 64 blocks the first wave holds every row and meets no other wave here)
    if (N < 64) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    else lds_barrier();
    if (64 * wave < N) {
      const int i = min(tid, N - 1);
      int end;
      if (small) {
        const uint64_t DM = __umul64hi(M, (uint64_t)D) ? ~0ull : M * (uint64_t)D, Zi = s_z[i];
        end = prepare_end(i, N, [&](int j) { return s_z[j] - Zi <= DM; });
      } else {
        const uint64_t Pi = (uint64_t)sP[i], Ai = (uint64_t)sA[i];
        end = prepare_end(i, N, [&](int j) { return fits_at((uint64_t)sP[j] - Pi, (uint64_t)sA[j] - Ai, M, D); });
      }
      if (tid < N) s_end[tid] = (uint32_t)end;
      int run = tid < N ? end - tid : 0;
      const int mine = run;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int x = __shfl_up(run, o);
        if (lane >= o) run += x;
      }
      if (tid < N) s_at[tid] = (uint32_t)(run - mine);
      if (N < 64) {
        if (tid == 63) s_at[N] = (uint32_t)run;
      } else if (lane == 63) {
        s_sum[wave] = run;
      }
    }
    lds_barrier();
    if (N >= 64) {
      if (tid >= 64 && tid < N) s_at[tid] += (uint32_t)s_sum[0];
      if (tid == 0) s_at[N] = (uint32_t)(s_sum[0] + (N > 64 ? s_sum[1] : 0));
      lds_barrier();
    }
  }

  // ---- tables (as build_kernel): rows 0..min(63,N-1) of chunk 0, then rows 0..N-1 of chunk 1 ----
  const int R0 = min(64, N), RT = R0 + (nch > 1 ? N : 0);
  for (int f = wave; f < RT; f += kSmallWaves) {
    const int c = f >= R0, i = c ? f - R0 : f;
    if constexpr (DIRECT) {
      if ((int)s_end[i] <= max(i, 64 * c) && i != 0) {  // no stage of the unit fits
        const int64_t u = unit_index(nch, i, c);
        pr.rmin[u * 64 + lane] = 255;
        if (lane == 0) pr.ufit[u] = 0;
        continue;
      }
    }
    UnitStages<VT> stage;
    const bool fits = build_unit<VT, DP>(pr, sT, sP, sA, pr.o ? sC : nullptr, i, c, lane, level(1), LS, 0, nullptr, !DIRECT, &stage);
    if (fits && lane == 0) atomicMin(&s_wlo[c], i);
    if constexpr (DIRECT) {
      const int jj = 64 * c + lane;
      if (jj >= i && jj < (int)s_end[i])
        s_word[s_at[i] + jj - i] = (uint32_t)i | (uint32_t)(jj + 1) << 8 | (uint32_t)(stage.fits ? stage.rmin : 255) << 16;
    }
  }
  [[maybe_unused]] int passes = 0;
  if constexpr (DIRECT) {
    const int all = s_at[N];
    passes = (all + 63) >> 6;
    if (tid < 64 && all + tid < 64 * passes) s_word[all + tid] = 255u << 16;  // (fits nowhere)
  }
  __syncthreads();
  if (tid < nch) pr.wlo[tid] = s_wlo[tid];
  const int64_t lvl = (int64_t)(N + 1) * DP;
  VT RANNC_GLOBAL *Vg = gptr((VT *)pr.V);
  const VT RANNC_GLOBAL *cost = gptr((const VT *)pr.cost);
  const uint8_t RANNC_GLOBAL *rmin = gptr((const uint8_t *)pr.rmin);
  // level 1 to memory
  for (int e = tid; e < (N + 1) * DP; e += NT) Vg[e] = level(1)[(e / DP) * LS + (e % DP)];
  if (tid == 0) s_top[0] = level(1)[N * LS + D - 1];

  // ---- levels 2..S_eff ----
  [[maybe_unused]] DirectConsts<DP> kc;
  if constexpr (DIRECT) direct_consts_init(kc);
  for (int s = 2; s <= S_eff; ++s) {
    const VT *prev = level(s - 1);
    VT *cur = level(s);
    const int rl = D - s + 1;
    if constexpr (!DIRECT) {
      for (int e = tid; e < (N + 1) * LS; e += NT) cur[e] = ((e % LS) < D) ? INF : (VT)0;
      lds_barrier();  // LDS only: the copy of the previous level to memory stays in flight
    }
    if constexpr (DIRECT) {
      // One pass of a wave = 64 stages of the list, one per lane, whatever rows they come from: every lane
      // reads its own a[] row from LDS and folds its own column in.  (With the triangle of a chunk as pairs of
      // rows, stages that do not fit among them, 32 blocks took nine passes a level; the outer driver's
      // searches of that size hold two passes of stages that fit.)
      for (int f = wave; f < passes; f += kSmallWaves) {
        const uint32_t word = s_word[64 * f + opaque(lane)];
        const int row = (int)(word & 255u), j = (int)(word >> 8) & 255, rmn = (int)(word >> 16);
        // some (s-1)-stage plan covers blocks 1..row
        const bool act = rmn <= rl && row >= s - 1 && prev[row * LS + D - 1] != INF;
        if (__ballot(act) == 0ull) continue;
        const VT tij = (VT)(sT[j] - sT[row]);
#define RANNC_ROW(HH)                                                                                \
  {                                                                                                  \
    constexpr int H = (HH) <= DP ? (HH) : DP;                                                        \
    const int sig = merge_shift(s, DP, H);                                                           \
    VT x[H];                                                                                         \
    _Pragma("unroll") for (int t = 0; t < H; ++t) x[t] = prev[row * LS + sig + t];                   \
    row_merge_direct<VT, H>(x, tij, rmn, act, kc);                                                   \
    if (act) {                                                                                       \
      /* no test per entry: columns D.. hold 0 and keep it, column DP (t + 1 + sig <= DP) is padding */ \
      VT *dst = cur + j * LS + 1 + sig;                                                              \
      _Pragma("unroll") for (int t = 0; t < H; ++t) atomicMin(&dst[t], x[t]);                        \
    }                                                                                                \
  }
        if (rl <= 8) RANNC_ROW(8)
        else if (rl <= 16) RANNC_ROW(16)
        else if (rl <= 24) RANNC_ROW(24)
        else RANNC_ROW(32)
#undef RANNC_ROW
      }
    } else {
      for (int f = wave; f < RT; f += kSmallWaves) {
        const int c = f >= R0, i = c ? f - R0 : f;
        if (i < s - 1 || i < s_wlo[c] || 64 * c + 64 < s) continue;
        if (prev[i * LS + D - 1] == INF) continue;  // no (s-1)-stage plan covers blocks 1..i
        const int jj = 64 * c + lane;
        const int64_t u = unit_index(nch, i, c);
        int rmn = 255;
        if (jj >= i && jj < N) rmn = rmin[u * 64 + lane];
        const bool act = rmn <= rl;
        if (__ballot(act) == 0ull) continue;
        const int col = act ? lane : __ffsll((long long)__ballot(act)) - 1;
        const VT RANNC_GLOBAL *unit = cost + u * 64 * D + col;
        const VT off = act ? (VT)0 : INF;
#define RANNC_ROW(K)                                                                                  \
  case K:                                                                                             \
    if constexpr (8 * K <= DP) {                                                                      \
      constexpr int H = 8 * K;                                                                        \
      const int sig = merge_shift(s, DP, H);                                                          \
      VT x[H];                                                                                        \
      row_merge<VT, H, const VT *>(x, unit, prev + i * LS + sig, off, rl);                            \
      /* (no test per entry, as above; folding INF in is a no-op) */                                  \
      if (act && jj + 1 >= s) {                                                                       \
        VT *dst = cur + (jj + 1) * LS + 1 + sig;                                                      \
        _Pragma("unroll") for (int t = 0; t < H; ++t) atomicMin(&dst[t], x[t]);                       \
      }                                                                                               \
    }                                                                                                 \
    break;
        switch ((rl + 7) >> 3) {
          RANNC_ROW(1) RANNC_ROW(2) RANNC_ROW(3) RANNC_ROW(4)
          RANNC_ROW(5) RANNC_ROW(6) RANNC_ROW(7) RANNC_ROW(8)
          default: break;
        }
#undef RANNC_ROW
      }
    }
    if constexpr (DIRECT) {
      // The next level's buffer held level s-2: its last readers were the passes of level s-1, which
      // the barrier before this level's passes closed, and its copy to memory was issued by these
      // same threads before their passes of level s-1.
      if (s < S_eff) {
        VT *next = level(s + 1);
        for (int e = opaque(tid); e < (N + 1) * LS; e += NT) next[e] = ((e % LS) < D) ? INF : (VT)0;
      }
    }
    lds_barrier();
    VT RANNC_GLOBAL *Vs = Vg + (int64_t)(s - 1) * lvl;
    for (int e = opaque(tid); e < (N + 1) * DP; e += NT) Vs[e] = cur[(e / DP) * LS + (e % DP)];
    if (tid == 0) s_top[s - 1] = cur[N * LS + D - 1];
  }
  __syncthreads();

  // ---- choice of the stage count (as select_kernel) ----
  if (wave == 0) {
    int64_t v = INT64_MAX;
    if (st == 0 && lane < S_eff) {
      const VT u = s_top[lane];
      v = (u == INF) ? INT64_MAX : (int64_t)u;
    }
    const Chosen chosen = select_finish(pr, v, st, d_opt, d_n_stages, d_est, d_status);
    if (tid == 0) s_chosen = chosen;
  }
  if constexpr (!PLAN) return;
  if (!results.d_stage_end) return;
  if constexpr (DIRECT) asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 2, 2), 0" ::);  // (direct_consts_init)
  // ---- plan recovery, where the caller wants it from this launch: out of LDS, but for levels that had to make room
  // and the tables' own bytes ----
  __shared__ TracebackLds sh;
  if (wave == 0) {
    if (lane == 0) { sh.chosen = s_chosen; sh.ns = s_chosen.status == 0 ? s_chosen.n_stages : 0; }
    if (lane < 3) sh.key[lane] = 0xFFFFFFFFu;
  }
  __syncthreads();
  if (sh.ns > 0) {
    struct Common {
      const int64_t *T, *C;
      const int *wlo;
      const uint8_t *rmin;
      const uint32_t *word, *at, *end;
      int nch;
      __device__ __forceinline__ int64_t sum(int i) const { return T[i]; }
      __device__ __forceinline__ uint64_t send(int j) const { return C ? (uint64_t)C[j] : 0ull; }
      __device__ __forceinline__ int first(int j) const { return min(wlo[(j - 1) >> 6], j); }
      __device__ __forceinline__ int least(int i, int j) const {
        if constexpr (DIRECT) return j <= (int)end[i] ? (int)(word[at[i] + j - 1 - i] >> 16) : 255;
        else return (int)rmin[unit_index(nch, i, (j - 1) >> 6) * 64 + ((j - 1) & 63)];
      }
    };
    const Common common = {sT, pr.o ? sC : nullptr, s_wlo, pr.rmin, s_word, s_at, s_end, nch};
    if (DIRECT && bufs >= S_eff) {
      struct InLds : Common {
        const VT *levels;
        int per_level;
        __device__ __forceinline__ const VT *row(int s, int i) const { return levels + (s - 1) * per_level + i * LS; }
      };
      traceback_walk<VT>(InLds{common, levels, per_level}, N, D, sh.ns, sh);
    } else {
      struct InMemory : Common {
        const VT RANNC_GLOBAL *V;
        int64_t lvl;
        __device__ __forceinline__ const VT RANNC_GLOBAL *row(int s, int i) const { return V + (int64_t)(s - 1) * lvl + (int64_t)i * DP; }
      };
      traceback_walk<VT>(InMemory{common, Vg, lvl}, N, D, sh.ns, sh);
    }
  }
  const int64_t q = (int64_t)pr.q * plan_stride;
  plan_out(pr, plan_stride, results.d_stage_end + q, results.d_replicas + q, sh, FormStageIn{}, results);
}

// ---------------------------------------------------------------------------------------
// Table export in the layout-independent form of the public header (parity and inspection).
// ---------------------------------------------------------------------------------------
template <typename VT>
__global__ __launch_bounds__(256) void export_kernel(const ProblemDev *__restrict__ prob, int which,
                                                     void *__restrict__ dst) {
  const ProblemDev &pr = *prob;
  const int N = pr.N, D = pr.D, DP = pr.DP, nch = pr.nch;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  constexpr VT INF = Lim<VT>::inf;
  const bool bad = *pr.status != 0;
  if (which == RANNC_DP_TABLE_COST || which == RANNC_DP_TABLE_FIT || which == RANNC_DP_TABLE_COST_BWD) {
    const VT *ctab = (const VT *)(which == RANNC_DP_TABLE_COST_BWD ? pr.costb : pr.cost);
    const int64_t total = (int64_t)N * (N + 1) / 2 * D;
    for (int64_t e = t0; e < total; e += stride) {
      const int r = (int)(e % D) + 1;
      const int64_t pair = e / D;  // j(j-1)/2 + i
      int j = (int)((1.0 + sqrt(1.0 + 8.0 * (double)pair)) * 0.5);
      while ((int64_t)j * (j - 1) / 2 > pair) --j;
      while ((int64_t)(j + 1) * j / 2 <= pair) ++j;
      const int i = (int)(pair - (int64_t)j * (j - 1) / 2);
      const int jj = j - 1;
      const int64_t u = unit_index(nch, i, jj >> 6);
      if (which == RANNC_DP_TABLE_FIT) {
        ((uint8_t *)dst)[e] = bad ? 0 : (uint8_t)(r >= (int)pr.rmin[u * 64 + (jj & 63)]);
      } else {
        const bool fit = !bad && r >= (int)pr.rmin[u * 64 + (jj & 63)];
        const VT v = fit ? ctab[(u * D + (r - 1)) * 64 + (jj & 63)] : INF;
        ((int64_t *)dst)[e] = (v == INF) ? INT64_MAX : (int64_t)v;
      }
    }
  } else if (which == RANNC_DP_TABLE_V || which == RANNC_DP_TABLE_MAX_FWD || which == RANNC_DP_TABLE_MAX_BWD) {
    const VT *vtab = (const VT *)(which == RANNC_DP_TABLE_V ? pr.V : which == RANNC_DP_TABLE_MAX_FWD ? pr.VF : pr.VB);
    const int64_t per = (int64_t)(N + 1) * (D + 1);
    const int64_t total = (int64_t)(pr.S_eff + 1) * per;
    const int64_t lvl = (int64_t)(N + 1) * DP;
    for (int64_t e = t0; e < total; e += stride) {
      const int s = (int)(e / per);
      const int j = (int)((e % per) / (D + 1));
      const int d = (int)(e % (D + 1));
      int64_t v = INT64_MAX;
      if (s == 0) v = (j == 0 && d == 0) ? 0 : INT64_MAX;
      else if (d >= 1 && !bad) {
        const VT u = vtab[(int64_t)(s - 1) * lvl + (int64_t)j * DP + d - 1];
        v = (u == INF) ? INT64_MAX : (int64_t)u;
      }
      ((int64_t *)dst)[e] = v;
    }
  }
}

// argmin export helpers: whole table to -1, then level 1 (the single stage 1..j on d devices
// has predecessor (0,0)); levels >= 2 come from level_scan_kernel.
template <typename VT>
__global__ __launch_bounds__(256) void arg_init_kernel(const ProblemDev *__restrict__ prob,
                                                       int32_t *__restrict__ arg) {
  const ProblemDev &pr = *prob;
  const int N = pr.N, D = pr.D, DP = pr.DP;
  const int64_t per = (int64_t)(N + 1) * (D + 1);
  const int64_t total = (int64_t)(pr.S_eff + 1) * per;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const bool bad = *pr.status != 0;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += stride) {
    const int s = (int)(e / per);
    const int j = (int)((e % per) / (D + 1));
    const int d = (int)(e % (D + 1));
    int32_t v = -1;
    if (s == 1 && j >= 1 && d >= 1 && !bad) {
      if (((const VT *)pr.V)[(int64_t)j * DP + d - 1] != Lim<VT>::inf) v = 0;
    }
    arg[e] = v;
  }
}

// ---------------------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------------------
hipError_t launch_setup(const ProblemDev *src, ProblemDev *probs, int Q, int rows_per_item, int max_items, int slots,
                        bool paired, int max_rows, const ProblemDev *host_one, hipStream_t st) {
  const int fill = Q >= 256 ? 4 : Q >= 16 ? 16 : 128;  // workgroups that fill a search's V
  for (int q0 = 0; q0 < Q; q0 += 65535) {
    const int nq = min(65535, Q - q0);
    hipLaunchKernelGGL(setup_kernel, dim3(1 + fill, nq), dim3(kSetupThreads), 0, st, src + q0, probs + q0, rows_per_item,
                       max_items, Q, slots, paired ? 1 : 0, max_rows, host_one ? *host_one : ProblemDev{}, host_one ? 1 : 0);
  }
  return hipGetLastError();
}

int merge_rows_per_item(int rows_per_wave) {
  if (rows_per_wave <= 0) return -1;  // chosen on the device
  return kMergeWaves * (rows_per_wave <= 1 ? 1 : rows_per_wave <= 2 ? 2 : rows_per_wave <= 4 ? 4 : rows_per_wave <= 8 ? 8 : rows_per_wave <= 12 ? 12 : 16);
}

constexpr int kBuildRowsFitOnly = 8;  // rows per wave when only the fits-in-memory part is built ...
constexpr int kBuildFewWaves = 1024;  // ... by at least this many waves

template <typename VT, int DP>
static void build_go(const ProblemDev *p, const LaunchShape &sh, int parts, hipStream_t st) {
  // (a small launch is a wave's latency: one row each while that leaves compute units without a workgroup)
  const int64_t waves8 = (int64_t)sh.nprob * sh.max_nch * ((sh.max_N + kBuildRowsFitOnly - 1) / kBuildRowsFitOnly);
  const int rows = (parts & 2) || waves8 < kBuildFewWaves ? 1 : kBuildRowsFitOnly;
  const int per_group = kBuildWaves * rows;
  for (int q0 = 0; q0 < sh.nprob; q0 += 65535) {
    const int nq = min(65535, sh.nprob - q0);
    const int groups = (sh.max_N + per_group - 1) / per_group, many = nq > 1;
    const dim3 grid = many ? dim3(nq, groups, sh.max_nch) : dim3(sh.max_nch, groups, 1), block(64 * kBuildWaves);
    if (rows == 1) hipLaunchKernelGGL((build_kernel<VT, DP, 1>), grid, block, 0, st, p + q0, parts, many);
    else hipLaunchKernelGGL((build_kernel<VT, DP, kBuildRowsFitOnly>), grid, block, 0, st, p + q0, parts, many);
  }
}

hipError_t launch_build(const ProblemDev *p, const LaunchShape &sh, int bits, int DP, int parts, hipStream_t st) {
  if (sh.max_N > 65535) return hipErrorInvalidValue;
#define GO(B, T)                                                   \
  if (bits == B) {                                                 \
    if (DP == 8) build_go<T, 8>(p, sh, parts, st);                 \
    else if (DP == 16) build_go<T, 16>(p, sh, parts, st);          \
    else if (DP == 32) build_go<T, 32>(p, sh, parts, st);          \
    else build_go<T, 64>(p, sh, parts, st);                        \
  }
  GO(32, uint32_t)
  GO(64, uint64_t)
#undef GO
  return hipGetLastError();
}

hipError_t launch_build_passes(const ProblemDev *p, const LaunchShape &sh, int bits, int DP, hipStream_t st) {
  if (sh.max_N > 65535) return hipErrorInvalidValue;
  for (int q0 = 0; q0 < sh.nprob; q0 += 65535) {
    const int nq = min(65535, sh.nprob - q0);
    // waves to a row: as many as leave some 32 thousand, and a wave at most 64 units
    const int64_t rows = (int64_t)sh.max_N * nq;
    const int parts = max((sh.max_nch + 63) / 64, (int)std::min<int64_t>(sh.max_nch / 4, 32768 / rows));
    const int groups = (int)(((int64_t)sh.max_N * parts + kBuildWaves - 1) / kBuildWaves);
    const int per = kPassBuildThreads / DP, first = min((sh.max_N + per) / per, max(1, 1024 / nq));  // of level 1
    const dim3 grid((unsigned)(groups + first), (unsigned)nq);
    if (bits == 32) hipLaunchKernelGGL((build_passes_kernel<uint32_t>), grid, dim3(kPassBuildThreads), 0, st, p + q0, groups, parts);
    else hipLaunchKernelGGL((build_passes_kernel<uint64_t>), grid, dim3(kPassBuildThreads), 0, st, p + q0, groups, parts);
  }
  return hipGetLastError();
}

bool can_prepare(const LaunchShape &sh) { return sh.max_N <= kSetupLdsN; }


template <typename VT, int DP, bool TIMES>
static hipError_t prepare_go(const ProblemDev *src, ProblemDev *probs, const LaunchShape &sh, PrepareIn in, size_t lds, int fill,
                             const ProblemDev *host_one, hipStream_t st) {
  const ProblemDev one = host_one ? *host_one : ProblemDev{};
  for (int q0 = 0; q0 < sh.nprob; q0 += 65535) {
    const dim3 grid(in.groups + fill, min(65535, sh.nprob - q0));
    if (sh.nprob == 1)
      hipLaunchKernelGGL((prepare_kernel<VT, DP, TIMES, 1024>), grid, dim3(1024), lds, st, src + q0, probs + q0, in, one, host_one ? 1 : 0);
    else
      hipLaunchKernelGGL((prepare_kernel<VT, DP, TIMES, 256>), grid, dim3(256), lds, st, src + q0, probs + q0, in, one, host_one ? 1 : 0);
  }
  return hipGetLastError();
}

hipError_t launch_prepare(const ProblemDev *src, ProblemDev *probs, const LaunchShape &sh, int bits, int DP, int parts,
                          int rows_per_item, int max_items, int slots, bool paired, int max_rows, bool split, bool comm,
                          const ProblemDev *host_one, hipStream_t st) {
  if (!can_prepare(sh)) return hipErrorInvalidValue;
  PrepareIn in;
  in.rows = rows_per_item; in.max_items = max_items; in.batch = sh.nprob; in.slots = slots;
  in.paired = paired ? 1 : 0; in.max_rows = max_rows;
  // Workgroups that build: four waves to a row of a lone search, whole rows where there are many searches and
  // every further workgroup would only form the sums once more.
  const bool many = sh.nprob > 1;
  in.parts = many ? 1 : 4;
  in.groups = many ? max(1, min((sh.max_N + 3) / 4, 1280 / sh.nprob)) : max(1, (sh.max_N * in.parts + 15) / 16);
  const int fill = many ? (sh.nprob >= 256 ? 4 : 16) : 32;  // workgroups that fill a search's V
  static_assert((kSetupLdsN + 1) * 8 * 6 + (2 * kSetupLdsN + 1) * 4 <= 60 * 1024, "dynamic LDS that need not be asked for");
  const size_t lds = (size_t)(sh.max_N + 1) * 8 * (4 + (split ? 1 : 0) + (comm ? 1 : 0)) + (size_t)(2 * sh.max_N + 1) * 4;
#define GO(B, T)                                                                                            \
  if (bits == B) {                                                                                          \
    if (!(parts & 2)) return prepare_go<T, 8, false>(src, probs, sh, in, lds, fill, host_one, st);          \
    if (DP == 8) return prepare_go<T, 8, true>(src, probs, sh, in, lds, fill, host_one, st);                \
    if (DP == 16) return prepare_go<T, 16, true>(src, probs, sh, in, lds, fill, host_one, st);              \
    if (DP == 32) return prepare_go<T, 32, true>(src, probs, sh, in, lds, fill, host_one, st);              \
    return prepare_go<T, 64, true>(src, probs, sh, in, lds, fill, host_one, st);                            \
  }
  GO(32, uint32_t)
  GO(64, uint64_t)
#undef GO
  return hipErrorInvalidValue;
}

template <typename VT, int HMAX, bool DIRECT>
static void merge_go(const ProblemDev *p, const LaunchShape &sh, int s, int items, const ProblemDev *host_one,
                     hipStream_t st) {
  if constexpr (HMAX >= 32) {
    if (host_one && sh.nprob == 1) {
      hipLaunchKernelGGL((level_merge_one_kernel<VT, HMAX, DIRECT>), dim3((unsigned)items, 1, 1), dim3(64 * kMergeWaves),
                         0, st, *host_one, s);
      return;
    }
  }
  for (int q0 = 0; q0 < sh.nprob; q0 += 65535) {
    const int nq = min(65535, sh.nprob - q0);
    // (the table form keeps the items of a search together: workgroups that run at the same time
    // then read neighbouring units of few tables instead of one unit each of hundreds of tables,
    // which measured 10 % slower on config 5)
    if (DIRECT && nq > 1 && items <= 65535)
      hipLaunchKernelGGL((level_merge_kernel<VT, HMAX, DIRECT>), dim3(nq, 1, (unsigned)items), dim3(64 * kMergeWaves), 0,
                         st, p + q0, s, 0);
    else
      hipLaunchKernelGGL((level_merge_kernel<VT, HMAX, DIRECT>), dim3((unsigned)items, 1, nq), dim3(64 * kMergeWaves), 0,
                         st, p + q0, s, 1);
  }
}

hipError_t launch_level_merge(const ProblemDev *p, const LaunchShape &sh, int bits, int s, bool recompute,
                              int items, const ProblemDev *host_one, hipStream_t st) {
  const int need = sh.max_D - s + 1;  // widest merge of the launch
#define GO(B, T, X)                                                                       \
  if (bits == B && recompute == X) {                                                      \
    if (need <= 8) merge_go<T, 8, X>(p, sh, s, items, host_one, st);                      \
    else if (need <= 16) merge_go<T, 16, X>(p, sh, s, items, host_one, st);               \
    else if (need <= 32) merge_go<T, 32, X>(p, sh, s, items, host_one, st);               \
    else if (need <= 48) merge_go<T, 48, X>(p, sh, s, items, host_one, st);               \
    else merge_go<T, 64, X>(p, sh, s, items, host_one, st);                               \
  }
  GO(32, uint32_t, false)
  GO(32, uint32_t, true)
  GO(64, uint64_t, false)
  GO(64, uint64_t, true)
#undef GO
  return hipGetLastError();
}

int small_max_blocks() { return kSmallMaxN; }
// the one-launch kernel can recompute the stage times up to the 32-device class (beyond it the
// reciprocals and the merge do not fit the 128 registers of its sixteen waves): 32-bit values, or
// 64-bit values where the caller's bound on a search's total time keeps every stage time in the
// range the double-precision quotient is exact for
bool can_recompute_times(int bits, int64_t max_total_time) { return bits == 32 || max_total_time <= kDirectWideMaxTime; }
bool small_can_recompute(int bits, int DP, int64_t max_total_time) {
  return DP <= 32 && can_recompute_times(bits, max_total_time);
}

hipError_t launch_solve_small(const ProblemDev *src, ProblemDev *p, int Q, int bits, int DP, bool direct, int64_t *d_opt,
                              int32_t *d_n_stages, int64_t *d_est, int32_t *d_status, const ProblemDev *host_one,
                              int plan_stride, const PlanResults *results, int cus, hipStream_t st) {
  const ProblemDev one = host_one ? *host_one : ProblemDev{};
  const PlanResults plan = results ? *results : PlanResults{};
  if (direct && DP > 32) return hipErrorInvalidValue;
#define GO(B, T, W, X)                                                                                           \
  if (bits == B && DP == W && direct == X) {                                                                     \
    constexpr bool apart = small_plan_apart<T, W, X>();                                                          \
    auto *kernel = solve_small_kernel<T, W, X, true>;                                                            \
    if (apart && !results && Q > cus) kernel = solve_small_kernel<T, W, X, !apart>;                              \
    hipLaunchKernelGGL(kernel, dim3(Q), dim3(64 * small_waves<T, W>()), 0, st, src, p, d_opt, d_n_stages, d_est, \
                       d_status, one, host_one ? 1 : 0, plan_stride, plan);                                      \
  }
  GO(32, uint32_t, 8, false) GO(32, uint32_t, 16, false) GO(32, uint32_t, 32, false) GO(32, uint32_t, 64, false)
  GO(64, uint64_t, 8, false) GO(64, uint64_t, 16, false) GO(64, uint64_t, 32, false) GO(64, uint64_t, 64, false)
  GO(32, uint32_t, 8, true) GO(32, uint32_t, 16, true) GO(32, uint32_t, 32, true)
  GO(64, uint64_t, 8, true) GO(64, uint64_t, 16, true) GO(64, uint64_t, 32, true)
#undef GO
  return hipGetLastError();
}

hipError_t launch_level_scan(const ProblemDev *p, const LaunchShape &sh, int bits, int s, int write_v,
                             int32_t *arg_i, int32_t *arg_d, hipStream_t st) {
  for (int q0 = 0; q0 < sh.nprob; q0 += 65535) {
    const int nq = min(65535, sh.nprob - q0);
    const dim3 grid(sh.max_nch, sh.max_D, nq);
    if (bits == 32)
      hipLaunchKernelGGL((level_scan_kernel<uint32_t>), grid, dim3(64), 0, st, p + q0, s, write_v, arg_i,
                         arg_d);
    else
      hipLaunchKernelGGL((level_scan_kernel<uint64_t>), grid, dim3(64), 0, st, p + q0, s, write_v, arg_i,
                         arg_d);
  }
  return hipGetLastError();
}

hipError_t launch_select(const ProblemDev *p, int Q, int64_t *d_opt, int32_t *d_n_stages,
                         int64_t *d_est, int32_t *d_status, hipStream_t st) {
  hipLaunchKernelGGL(select_kernel, dim3(Q), dim3(64), 0, st, p, d_opt, d_n_stages, d_est, d_status);
  return hipGetLastError();
}

int64_t traceback_lds_bytes(int N, int DP, int S_eff, int bits) {
  const int nch = (N + 63) / 64;
  const int64_t nT = (((int64_t)(N + 1) * 8 + 31) / 32) * 32;
  return (int64_t)S_eff * (N + 1) * DP * (bits / 8) + 2 * nT + (((int64_t)nch * 4 + 31) / 32) * 32 +
         units_before(nch, N) * 64;
}

hipError_t launch_traceback(const ProblemDev *p, int Q, int plan_stride, int32_t *d_stage_end,
                            int32_t *d_replicas, const int32_t *d_levels, int64_t lds_bytes,
                            const FormStageIn *form_stage, const PlanResults *results, bool choose, hipStream_t st) {
  const PlanResults none = {};
  const PlanResults &r = results ? *results : none;
  const FormStageIn no_choice = {};
  const FormStageIn &f = form_stage ? *form_stage : no_choice;
  if (form_stage) Q = 1;
  if (lds_bytes > 0) {
    // more than the default 64 KiB of dynamic LDS has to be asked for
    static std::atomic<uint64_t> asked{0};
    const hipError_t attr = allow_lds(asked, (const void *)traceback_lds_kernel, kTracebackLdsMax);
    if (attr != hipSuccess) return attr;
    if (lds_bytes > kTracebackLdsMax) return hipErrorInvalidValue;
    hipLaunchKernelGGL(traceback_lds_kernel, dim3(Q), dim3(kTracebackThreads), (size_t)lds_bytes, st, p, plan_stride,
                       d_stage_end, d_replicas, d_levels, f, r, choose ? 1 : 0);
  } else {
    hipLaunchKernelGGL(traceback_kernel, dim3(Q), dim3(kTracebackThreads), 0, st, p, plan_stride, d_stage_end,
                       d_replicas, d_levels, f, r, choose ? 1 : 0);
  }
  return hipGetLastError();
}

// V[s][N][D] for s = 1..S_eff of every problem (INT64_MAX: no plan of exactly s stages, or s
// beyond S_eff, or bad inputs): Algorithm 1's answer for each exact stage count.
__global__ __launch_bounds__(64) void level_values_kernel(const ProblemDev *__restrict__ probs, int stride,
                                                          int64_t *__restrict__ out) {
  const ProblemDev &pr = probs[blockIdx.x];
  const bool bad = *pr.status != 0;
  const int64_t lvl = (int64_t)(pr.N + 1) * pr.DP;
  const int64_t cell = (int64_t)pr.N * pr.DP + pr.D - 1;
  for (int k = threadIdx.x; k < stride; k += 64) {
    int64_t v = INT64_MAX;
    if (!bad && k < pr.S_eff) {
      if (pr.bits == 32) {
        const uint32_t u = ((const uint32_t *)pr.V)[k * lvl + cell];
        v = (u == Lim<uint32_t>::inf) ? INT64_MAX : (int64_t)u;
      } else {
        const uint64_t u = ((const uint64_t *)pr.V)[k * lvl + cell];
        v = (u == Lim<uint64_t>::inf) ? INT64_MAX : (int64_t)u;
      }
    }
    out[(int64_t)pr.q * stride + k] = v;
  }
}

hipError_t launch_level_values(const ProblemDev *p, int Q, int stride, int64_t *d_out, hipStream_t st) {
  hipLaunchKernelGGL(level_values_kernel, dim3(Q), dim3(64), 0, st, p, stride, d_out);
  return hipGetLastError();
}

hipError_t launch_export(const ProblemDev *p, int which, int bits, void *d_dst, hipStream_t st) {
  const dim3 grid(1024), block(256);
  if (which != RANNC_DP_TABLE_ARG_I && which != RANNC_DP_TABLE_ARG_D) {
    if (bits == 32) hipLaunchKernelGGL((export_kernel<uint32_t>), grid, block, 0, st, p, which, d_dst);
    else hipLaunchKernelGGL((export_kernel<uint64_t>), grid, block, 0, st, p, which, d_dst);
  } else {
    if (bits == 32) hipLaunchKernelGGL((arg_init_kernel<uint32_t>), grid, block, 0, st, p, (int32_t *)d_dst);
    else hipLaunchKernelGGL((arg_init_kernel<uint64_t>), grid, block, 0, st, p, (int32_t *)d_dst);
  }
  return hipGetLastError();
}

}  // namespace rannc
