// cc_device.h -- device-side data layout and helpers of the C4 / ClusterWild!
// round loop (arXiv 1507.05086, Algorithm 2) on gfx950.
//
// Memory layout of a run (all in HBM, sized for one graph of n vertices and
// nnz stored adjacency entries):
//   rank   int32[n]   position of each vertex in pi (rank = order^-1)
//   lab    int32[n]   clusterID: rank of the vertex's center, INF while unclustered
//   ub     int32[n]   remaining-degree bound: an upper bound while Delta is
//                     large, the exact remaining degree once the run switches
//   unc    uint32[n/32] one bit per vertex, set while it is unclustered (8 MB at
//                     2^26 vertices: gathers stay in L2 / the Infinity Cache)
//   state  uint8[n]   ACTIVE / CENTER / NONCENTER marks of the current round
//   flag   uint8[n]   per-round scratch mark (blocked / waiting / conflict)
//   work lists: active set, centers, newly clustered, rescans; each a vertex
//   array plus the exclusive prefix of the row weights max(deg, 1), so that
//   adjacency passes can hand out equal numbers of entries to every workgroup.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace ccd {

constexpr int BS = 256;             // threads per workgroup (4 wave64s)
constexpr int WAVES = BS / 64;
constexpr int IPT = 4;              // adjacency items per thread per tile
constexpr int TW = BS * IPT;        // adjacency items per tile
constexpr int SIPT = 4;            // pi positions per thread in the active-set scan (2 / 4 / 8: R-MAT 26 53.3 / 51.7 / 52.5 ms)
constexpr int SEL_BS = 512;         // threads of an active-set scan workgroup
constexpr int TSEL = SEL_BS * SIPT; // pi positions per scan tile
constexpr int32_t INF = 0x7fffffff;

enum : uint8_t { UNCL = 0, ACTIVE = 1, CENTER = 2, NONCENTER = 3, ORDER_SEEN = 4 };
constexpr int DSW = 64;            // bounds below this never need a bucket entry
constexpr int LVL_MIN = 6;         // log2(DSW): lowest bucket level of the bound buckets
constexpr int NLVL = 32;           // bucket levels (level = floor(log2(ub)))
constexpr int DITER = 3;           // band passes of the lazy Delta search per round
constexpr int SWL = 128;           // a band floor below this switches to exact degrees
constexpr int HLDS = 256;          // degree-histogram bins kept per workgroup in LDS
// pass j rescans candidates with bound >= ceil(BAND_j * T_j)
__host__ __device__ inline float band_factor(int pass) { return pass == 0 ? 0.7f : (pass == 1 ? 0.3f : 0.05f); }
enum : int { ALGO_C4 = 0, ALGO_CW = 1 };
enum : int { POL_FIXED = 0, POL_LEARNED = 1, POL_TRACE = 2, POL_BINOMIAL = 3 };
enum : int { ERR_NONE = 0, ERR_PERM = 5, ERR_NO_PROGRESS = 8, ERR_OVERFLOW = 11, ERR_LABEL = 12, ERR_INJECTED = 13 };
enum : int { PHASE_LAZY = 0, PHASE_EXACT = 1 };
// The part of the current round from which the round kernels have to run it:
// nothing (k_team takes the round), all of it, or what k_team has left.
enum : int { ST_TEAM = 0, ST_SELECT = 1, ST_ELECT = 2, ST_CLASSIFY = 3, ST_DELTA = 4 };

// A list is packed in one 64-bit counter: (total weight << 31) | count, so a
// single atomic reserves both a slot range and its weight range, and the
// stored weight offsets come out sorted in slot order.
__host__ __device__ inline unsigned long long pk(int64_t work, int64_t cnt) {
  return ((unsigned long long)work << 31) | (unsigned long long)cnt;
}
__host__ __device__ inline int64_t pk_cnt(unsigned long long p) { return (int64_t)(p & 0x7fffffffULL); }
__host__ __device__ inline int64_t pk_work(unsigned long long p) { return (int64_t)(p >> 31); }

struct RoundRec {  // mirrors cc_round_record
  int64_t n_i, delta_i, b_i, r_i, centers, claimed, conflicts;
  double eps_used;
  int64_t t_ns;  // raw wall-clock ticks here; the host converts
};

// The fields a round kernel reads before it starts its work, at the front of
// Ctrl and in the layout of CtrlHead, so one wide load brings them all (a
// chain of dependent scalar loads of these fields was most of the 4-5 us an
// idle kernel cost).
struct CtrlHead {
  int done;                  // the run is finished (or failed)
  int16_t phase;             // PHASE_LAZY (upper bounds) or PHASE_EXACT (exact degrees)
  int8_t stage;              // ST_*: where the round kernels take up the round
  int8_t pass;               // lazy Delta search: passes that are behind
  unsigned int n_blocked;    // C4: blocked active vertices of this round
  unsigned int n_cedges;     // C4: conflict edges listed this round
  long long delta;           // Delta_i of the current round
  long long b;               // active-set size of the current round
  long long cursor;          // first pi position not yet passed
  long long n_rem;           // unclustered vertices
  int d_max[DITER];          // lazy Delta search: largest exact degree found by each band pass
  unsigned int tile_counter; // active-set scan tiles taken this round
  unsigned long long a_pack, c_pack, n_pack, p_pack;  // active / center / newly / peel lists
  unsigned long long r_pack[DITER];  // per band pass, the rescan list
  unsigned long long x_pack;  // rows of degree >= DSW recounted when switching to exact degrees
};

struct Ctrl {
  // ---- the head (same layout as CtrlHead) ----
  int done;
  int16_t phase;
  int8_t stage, pass;
  unsigned int n_blocked, n_cedges;
  long long delta;
  long long b;
  long long cursor;
  long long n_rem;
  int d_max[DITER];
  unsigned int tile_counter;
  unsigned long long a_pack, c_pack, n_pack, p_pack;
  unsigned long long r_pack[DITER];
  unsigned long long x_pack;
  // ---- carried across rounds ----
  long long round;         // rounds finished
  long long n_start;       // n_i of the current round
  long long r_last;        // rank of the last active vertex
  int error;
  int has_round;           // a round has been run since the start
  int fallback;            // learned policy fell back to the fixed rule
  int select_done;         // per round: the active set is complete
  double eps_used;         // eps behind b
  float feat_conf, feat_claim, feat_eps;  // previous-round features for the learned policy
  float rate;              // entries walked per active vertex in the last round
  int slots;               // round slots (the round kernels, k_team if there is one) the device has finished
  long long t_start;       // wall clock at round start
  unsigned long long conflicts;  // per round: ClusterWild! conflict marks counted by k_clear
  unsigned long long x_low[64];  // adjacency entries of the lower-degree rows recounted at the switch (spread)
  // bound buckets: entries per level (capacity fixed per graph)
  unsigned int lvl_cnt[NLVL];
  // run totals
  unsigned long long sum_elect, sum_claim, sum_rescan, sum_peel, sum_blocked, sum_atomics;
  // per-round statistics spread over 64 slots (slot = workgroup mod 64): one
  // address taken by every workgroup would serialise their atomics
  unsigned long long spread_atom[64], spread_conf[64];
  // active vertices of this round settled by the selection itself (no
  // unclustered neighbour: a center that claims nobody), spread the same way
  unsigned long long spread_lone[64];
};
static_assert(sizeof(CtrlHead) == 128, "the head is one 128-byte line");
static_assert(offsetof(Ctrl, done) == offsetof(CtrlHead, done) && offsetof(Ctrl, phase) == offsetof(CtrlHead, phase) &&
                  offsetof(Ctrl, stage) == offsetof(CtrlHead, stage) && offsetof(Ctrl, pass) == offsetof(CtrlHead, pass) &&
                  offsetof(Ctrl, n_blocked) == offsetof(CtrlHead, n_blocked) &&
                  offsetof(Ctrl, n_cedges) == offsetof(CtrlHead, n_cedges) &&
                  offsetof(Ctrl, delta) == offsetof(CtrlHead, delta) && offsetof(Ctrl, b) == offsetof(CtrlHead, b) &&
                  offsetof(Ctrl, cursor) == offsetof(CtrlHead, cursor) &&
                  offsetof(Ctrl, n_rem) == offsetof(CtrlHead, n_rem) &&
                  offsetof(Ctrl, d_max) == offsetof(CtrlHead, d_max) &&
                  offsetof(Ctrl, tile_counter) == offsetof(CtrlHead, tile_counter) &&
                  offsetof(Ctrl, a_pack) == offsetof(CtrlHead, a_pack) &&
                  offsetof(Ctrl, c_pack) == offsetof(CtrlHead, c_pack) &&
                  offsetof(Ctrl, n_pack) == offsetof(CtrlHead, n_pack) &&
                  offsetof(Ctrl, p_pack) == offsetof(CtrlHead, p_pack) &&
                  offsetof(Ctrl, r_pack) == offsetof(CtrlHead, r_pack) &&
                  offsetof(Ctrl, x_pack) == offsetof(CtrlHead, x_pack),
              "Ctrl starts with CtrlHead's layout");

// The head as the kernel starts: eight independent 16-byte scalar loads
// issued together (the values were written by earlier kernels of the
// stream).  The empty asm takes every loaded value, so the compiler can
// neither split the head into loads made one after another behind each
// test nor sink them past the early exits.
__device__ inline CtrlHead ctrl_head(const Ctrl *c) {
  const uint4 *p = reinterpret_cast<const uint4 *>(c);
  uint4 q[8];
#pragma unroll
  for (int i = 0; i < 8; i++) q[i] = p[i];
#pragma unroll
  for (int i = 0; i < 8; i++) asm volatile("" ::"s"(q[i].x), "s"(q[i].y), "s"(q[i].z), "s"(q[i].w));
  CtrlHead h;
  __builtin_memcpy(&h, q, sizeof(h));
  return h;
}

// A listed vertex's row: start of its adjacency in col, its degree and its
// rank in pi.  Carried along the active and center lists so the passes over
// those rows never look the offsets or the rank up again.
struct RowInfo {
  int64_t start;
  int32_t deg;
  int32_t rank;
};

// What k_team takes (one XCD, an eighth of the device).  A round with more
// positions to pass, or more to walk, is a matter of throughput and runs on
// the whole device; so does the rest of a round whose Delta candidates or
// level entries turn out longer.  A round costs 15 - 45 us on a team and 55 -
// 90 us as kernels while it is short.  Measured (median call, team limits
// varied): TEAM_ITEMS 2^17 / 2^18: power law 2 M ClusterWild! 6.1 / 5.7 ms,
// R-MAT 22 C4 7.50 / 7.31, under the learned policy 3.29 / 3.47 ms, R-MAT 23 C4
// 11.1 / 10.9 ms; with slots of 13 to 16 kernels, TEAM_ITEMS 2^19: 5.6, -,
// 3.83, 11.0 (2^18: 5.5, -, 3.73, 11.1), TEAM_WORK 2^20 / 2^22: R-MAT 23 C4 11.1
// / 11.8 ms, TEAM_POS 2^16 / 2^18 / 2^20: R-MAT 22 C4 9.1 / 7.65 / 7.65 ms,
// learned 3.8 / 3.7 / 4.0 ms.  Graphs above TEAM_MAX_N vertices stay with the
// kernels: R-MAT 23 C4 11.1 -> 10.9 ms with a team, R-MAT 22 9.8 -> 7.3, but
// R-MAT 24 14.1 -> 14.2 and R-MAT 26 (C4 + ClusterWild!) 56.6 -> 61 ms.  The line
// is not right for every run below it: with 2^21 instead of 2^23 R-MAT 22 under
// the learned policy takes 3.16 ms (3.47) and C4 on power law 4 M 5.65 (5.91),
// since most of their rounds are wide, and a slot for a single round costs more
// than a quarter of a graph of four.
constexpr int64_t TEAM_MAX_N = int64_t(1) << 23;
constexpr long long TEAM_POS = 1 << 18;     // positions of pi to pass
constexpr long long TEAM_ITEMS = 1 << 18;   // entries that claims and peeling are expected to walk
constexpr long long TEAM_WORK = 1 << 20;    // entries of a Delta pass's candidates
constexpr long long TEAM_SCAN = 1 << 18;    // entries of the bound levels to look through
// Entries of the listed active rows (over TLONG each, or more rows than fit the
// LDS) at which the round is left to the device after all: TEAM_ITEMS goes by
// the mean, and the active may be hubs.  2000 rows of 10 K entries at once: C4
// 2.9 ms on the team, 0.67 so; a star of 2 M, the hub first: 0.95, 0.44.  2^17 to
// 2^21 are alike there and on R-MAT 20, power law 500 K and 3 M (within 1 %).
constexpr int TEAM_ACTIVE = 1 << 19;
// A round's positions go to the workgroups 64 at a time, so that a short round
// keeps most of them out of its counts.  What an active vertex claims stays
// with its workgroup, though, so where more entries than this are expected
// the positions are dealt singly.  ClusterWild! on ER 5 K of degree 300 (seven
// active, 130 K entries a round) 1.80 -> 0.96 ms, R-MAT 16 in its own order 2.11
// -> 1.46; 2 K / 8 K / 32 K: ER 5 K 0.95 / 0.96 / 1.00, R-MAT 16 1.47 / 1.48 / 1.80.
constexpr long long TEAM_SPREAD = 8192;
// A graph of at most this many vertices and stored entries runs whole in one
// workgroup (SOLO): C4 on 517 vertices and 14 K entries takes 256 us so, 356
// us on 8 workgroups and 377 us on 32; ClusterWild! on 5 K and 60 K, 467, 446
// and 468 us.
constexpr int64_t TEAM_SOLO = 48 * 1024;
// Up to this many stored entries a run keeps exact degrees from the start
// (no Delta passes, no switch).  On a power-law graph of 4 M entries that
// costs more than it saves: 8.9 against 2.2 ms.
constexpr int64_t TEAM_EXACT = 1 << 17;

// k_team: workgroups, and what one of its rounds counts (four in turn).
constexpr int TEAM_NT = 512;       // threads of a workgroup
constexpr int TEAM_MAX = 32;       // workgroups: the compute units of one XCD
struct TeamSlot {
  unsigned long long a_pack, c_pack, r_pack[DITER];  // long active rows / promoted / rescan lists
  unsigned long long listed;  // active vertices with a row (low half), settled alone (high half)
  unsigned long long claimed; // newly claimed (low half), entries walked by claims and peeling (high half)
  long long r_last;
  int d_max[DITER];
  int err;
  unsigned n_cedges, n_blocked, conflicts;
};
struct TeamCtl {  // zero when k_team starts
  unsigned pick, reg, size;    // the XCD (id + 1), registrations (top bit: closed), members
  unsigned arrive, gen, abort; // the barrier
  unsigned tcnt[2][64];        // unclustered positions found by each workgroup
  TeamSlot slot[4];
};

struct Ws {
  // graph: the full renumbered rows are col[off[v] .. rend[v]) (rend = off +
  // 1).  The switch to exact degrees writes compacted rows, xcol[off[v] ..
  // xend[v]), holding only the neighbours then unclustered, at the start of
  // each row's original slot; every round after the switch walks those.
  const int64_t *off;
  const int64_t *rend;
  const int32_t *col;
  int32_t *xcol;        // compacted rows (col-sized; written at the switch)
  int64_t *xend;        // their ends (n)
  int64_t n;
  int64_t max_deg;
  int64_t low_start;        // internal ids from here on have degree < DSW ...
  int64_t iso_start;        // ... and from here on degree 0 (they sort last)
  // run input
  const int32_t *order;     // pi in internal ids (written by k_check_order)
  int32_t *iorder;          // the same buffer, writable
  const int32_t *order_in;  // the caller's pi (input ids)
  const int32_t *perm;      // input id -> internal id
  const int32_t *iperm;     // internal id -> input id
  int order_mapped;         // pi was mapped and checked by the bucketed passes: no marks in state
  // per-vertex arrays
  int32_t *rank, *lab, *ub;
  uint32_t *unc;
  uint8_t *state, *flag;
  // lists
  int32_t *alist, *clist, *nlist, *blist, *rlist, *xlist, *plist;
  int64_t *awork, *cwork, *rwork, *xwork, *pwork;
  RowInfo *ainfo, *cinfo;  // row info of alist / clist entries
  unsigned long long *racc;  // rescan accumulators (items covered << 32 | count), DITER * rcap
  int64_t rcap;         // capacity of one pass's rescan list
  int2 *cedge;
  int64_t cedge_cap;
  // C4's blocked vertices (k_resolve): the blocked index of a vertex (by
  // vertex id), and per blocked index its undecided earlier blocked
  // neighbours, its decision, the range of its later blocked neighbours in
  // bradj, and the queue of decided indices
  int32_t *bpos, *bpend, *bdec, *bdep, *bq, *bradj;
  unsigned long long *tstat;
  int64_t tstat_cap;
  // bound buckets
  int32_t *lvl;         // entries of all levels
  const int64_t *lvl_off;  // [NLVL+1] start of each level in lvl (device)
  const int64_t *lvl_first;  // [NLVL] a level's first internal id (ids are grouped by level), and
  const unsigned *lvl_cnt0;  // [NLVL] its vertices, at the start of a run (levels from LVL_MIN on)
  int *hist;            // exact phase: vertices per remaining degree, [max_deg + 1]
  Ctrl *ctrl;
  RoundRec *trace;
  int64_t trace_cap;
  // epsilon policy
  int policy;
  int algo;
  int64_t eps_q;        // per-call eps in millionths
  double eps;
  const int64_t *sched; // TRACE: B_i schedule; BINOMIAL: pi positions per round (device)
  int64_t sched_len;
  int64_t bin_period;   // BINOMIAL: rounds between two halvings of Delta-hat
  const float *mlp;     // LEARNED: 6-64-1 weights (device)
  float eps_min, eps_max;
  int64_t max_rounds;   // > 0: stop after this many rounds (partial run)
  int64_t fault_round;  // > 0: test hook, the loop reports a device error after this round
  TeamCtl *team;        // null: the round kernels run every round
  int team_n;           // workgroups of k_team (1: it runs whole runs by itself)
  int solo;             // team_n == 1: k_team also sets the run up and writes the labels
  int32_t *labels_out;  // solo: where they go
  int start_exact;      // the run starts with exact degrees (xcol / xend are the full rows)
  // progress word in pinned host memory, written by k_close at the end of
  // every round slot: slots finished (bits 0..31), done (32), exact phase
  // (33), error (34); by k_team where there is one, which also says whether it
  // has run a round itself (35)
  unsigned long long *progress;
};

constexpr int PROGRESS_DONE = 32, PROGRESS_EXACT = 33, PROGRESS_ERROR = 34, PROGRESS_RAN = 35;

__host__ __device__ inline int level_of(int64_t x) {  // floor(log2(x)), x >= 1
  return 63 - __builtin_clzll((unsigned long long)x);
}

// ------------------------------------------------------------- atomics ----

template <class T>
__device__ inline T ld_rlx(T *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Relaxed device-scope atomic store: coherent across the XCDs like any
// device-scope atomic, without the release's write-back of the whole L2.
template <class T>
__device__ inline void st_rlx(T *p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ inline T add_rlx(T *p, T v) {
  return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline void set_error(Ctrl *c, int code) { atomicCAS(&c->error, 0, code); }

__device__ inline int lane_id() { return (int)(threadIdx.x & 63); }
__device__ inline int wave_id() { return (int)(threadIdx.x >> 6); }
__device__ inline unsigned long long lanemask_lt() {
  const int l = lane_id();
  return l == 0 ? 0ull : (~0ull >> (64 - l));
}

// Wave64 scans and reductions by data-parallel moves inside the vector unit:
// a step takes a few cycles, where a shuffle goes through the LDS unit and
// takes about sixty.  Every lane of the wave takes part.
template <int CTRL, int ROWS>
__device__ inline int dpp_mov(int old, int x) {
  return __builtin_amdgcn_update_dpp(old, x, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS>
__device__ inline int dpp_add(int x) {
  return x + dpp_mov<CTRL, ROWS>(0, x);
}
template <int CTRL, int ROWS>
__device__ inline int64_t dpp_add(int64_t x) {
  const unsigned lo = (unsigned)dpp_mov<CTRL, ROWS>(0, (int)x), hi = (unsigned)dpp_mov<CTRL, ROWS>(0, (int)(x >> 32));
  return x + (int64_t)((unsigned long long)hi << 32 | lo);
}
// Inclusive scan.
template <class T>
__device__ inline T wave_incl_scan(T x) {
  static_assert(sizeof(T) == 4 || sizeof(T) == 8, "32 or 64 bits");
  x = dpp_add<0x111, 0xf>(x);  // row_shr:1, 2, 4, 8 within rows of 16 lanes
  x = dpp_add<0x112, 0xf>(x);
  x = dpp_add<0x114, 0xf>(x);
  x = dpp_add<0x118, 0xf>(x);
  x = dpp_add<0x142, 0xa>(x);  // row_bcast:15 into rows 1 and 3
  x = dpp_add<0x143, 0xc>(x);  // row_bcast:31 into rows 2 and 3
  return x;
}
__device__ inline int lane_value(int x, int lane) { return __builtin_amdgcn_readlane(x, lane); }
__device__ inline int64_t lane_value(int64_t x, int lane) {
  return (int64_t)((unsigned long long)(unsigned)lane_value((int)(x >> 32), lane) << 32 | (unsigned)lane_value((int)x, lane));
}
template <class T>
__device__ inline T wave_sum(T x) {
  return lane_value(wave_incl_scan(x), 63);
}
// Inclusive prefix maximum, and the maximum, of values >= 0.
__device__ inline int wave_incl_max(int x) {
  x = max(x, dpp_mov<0x111, 0xf>(0, x));
  x = max(x, dpp_mov<0x112, 0xf>(0, x));
  x = max(x, dpp_mov<0x114, 0xf>(0, x));
  x = max(x, dpp_mov<0x118, 0xf>(0, x));
  x = max(x, dpp_mov<0x142, 0xa>(0, x));
  x = max(x, dpp_mov<0x143, 0xc>(0, x));
  return x;
}
__device__ inline int wave_max(int x) { return lane_value(wave_incl_max(x), 63); }
// x of a lane whose number is the same in the whole wave.
template <class T>
__device__ inline T from_lane(T x, int lane) {
  return lane_value(x, __builtin_amdgcn_readfirstlane(lane));
}

// Workgroup exclusive scan of 32- or 64-bit values for NT threads; *total receives
// the sum.  Uses `sh` (NT/64 + 1 slots of shared memory); two barriers.
template <int NT = BS, class T = int64_t>
__device__ inline T wg_excl_scan(T x, T *total, T *sh) {
  constexpr int NW = NT / 64;
  const T inc = wave_incl_scan(x);
  if (lane_id() == 63) sh[wave_id()] = inc;
  __syncthreads();
  T base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < NW; w++) {
    if (w < wave_id()) base += sh[w];
    tot += sh[w];
  }
  __syncthreads();
  *total = tot;
  return base + inc - x;
}

// Appends the calling lanes' vertices (pred true) and their row info to a
// packed list, one atomic per wave (weight = max(deg, 1)).
__device__ inline void wave_append_info(bool pred, int32_t v, RowInfo ri, unsigned long long *packc, int32_t *list,
                                        int64_t *work, RowInfo *info) {
  const unsigned long long m = __ballot(pred);
  if (m == 0) return;
  const int64_t w = pred ? (ri.deg > 0 ? ri.deg : 1) : 0;
  const int64_t winc = wave_incl_scan(w);
  const int64_t wtot = lane_value(winc, 63);
  const int leader = __ffsll((long long)m) - 1;
  unsigned long long base = 0;
  if (lane_id() == leader) base = atomicAdd(packc, pk(wtot, __popcll(m)));
  base = (unsigned long long)from_lane((int64_t)base, leader);
  if (pred) {
    const int64_t slot = pk_cnt(base) + __popcll(m & lanemask_lt());
    list[slot] = v;
    work[slot] = pk_work(base) + winc - w;
    info[slot] = ri;
  }
}


// Largest i in [0, cnt) with work[i] <= s (work[0] = 0 <= s): a 64-ary search
// by one wave, about log64(cnt) dependent loads.
__device__ inline int64_t wave_find_entry(const int64_t *work, int64_t cnt, int64_t s) {
  int64_t lo = 0, hi = cnt;
  while (hi - lo > 1) {
    const int64_t step = (hi - lo + 63) / 64;
    const int64_t idx = lo + (int64_t)lane_id() * step;
    const bool pred = idx < hi && work[idx] <= s;
    const unsigned long long m = __ballot(pred);
    const int k = __popcll(m);  // lanes 0..k-1 hold true (work is sorted)
    lo = lo + (int64_t)(k - 1) * step;
    hi = min(hi, lo + step);
  }
  return lo;
}

__device__ inline bool unc_bit(const uint32_t *unc, int32_t v) { return (unc[v >> 5] >> (v & 31)) & 1u; }

}  // namespace ccd

namespace ccd {

// Workgroup-staged appends to a packed list: threads push (vertex, weight)
// into LDS; a flush reserves the whole batch with one atomic on the list
// counter and writes it out with coalesced stores.  Same-address device
// atomics serialise, so this keeps them to one per flush instead of one per
// wave and item group.
template <int CAP>
struct StageBuf {
  int32_t id[CAP];
  int32_t wt[CAP];
  int cnt;
  unsigned long long base;
  int64_t sh[WAVES + 1];
};

// Staging buffer of bare ids for a list nobody walks edge-balanced: one
// atomic reservation per flush, no weights and no work prefix.
template <int CAP>
struct IdBuf {
  int32_t id[CAP];
  int cnt;
  unsigned long long base;
};

template <int CAP>
__device__ inline void id_init(IdBuf<CAP> &b) {
  if (threadIdx.x == 0) b.cnt = 0;
  __syncthreads();
}

template <int CAP>
__device__ inline void id_push(IdBuf<CAP> &b, int32_t v) {
  b.id[atomicAdd(&b.cnt, 1)] = v;
}

// Collective: every thread of the workgroup calls it.
template <int CAP>
__device__ inline void id_flush(IdBuf<CAP> &b, unsigned long long *packc, int32_t *list) {
  __syncthreads();
  const int cnt = b.cnt;
  if (cnt == 0) return;
  if (threadIdx.x == 0) b.base = atomicAdd(packc, pk(0, cnt));
  __syncthreads();
  const int64_t slot0 = pk_cnt(b.base);
  for (int i = threadIdx.x; i < cnt; i += BS) list[slot0 + i] = b.id[i];
  __syncthreads();
  if (threadIdx.x == 0) b.cnt = 0;
  __syncthreads();
}

// Staging buffer whose entries also carry row info.
template <int CAP>
struct StageBufI : StageBuf<CAP> {
  RowInfo info[CAP];
};

template <int CAP>
__device__ inline void stage_push_info(StageBufI<CAP> &b, int32_t v, RowInfo ri) {
  const int p = atomicAdd(&b.cnt, 1);
  b.id[p] = v;
  b.wt[p] = ri.deg > 0 ? ri.deg : 1;
  b.info[p] = ri;
}

template <int CAP>
__device__ inline void stage_init(StageBuf<CAP> &b) {
  if (threadIdx.x == 0) b.cnt = 0;
  __syncthreads();
}

template <int CAP>
__device__ inline void stage_push(StageBuf<CAP> &b, int32_t v, int32_t weight) {
  const int p = atomicAdd(&b.cnt, 1);
  b.id[p] = v;
  b.wt[p] = weight;
}

// Whether the buffer holds more than a workgroup's worth.  Collective: every
// thread has the same answer before any of them pushes again.
template <int CAP>
__device__ inline bool staged_over(const StageBuf<CAP> &b) {
  __syncthreads();
  const int cnt = b.cnt;
  __syncthreads();
  return cnt > BS;
}

// Collective: every thread of the workgroup calls it.
template <int CAP>
__device__ inline void stage_flush(StageBuf<CAP> &b, unsigned long long *packc, int32_t *list, int64_t *work,
                                   unsigned long long *zero_acc = nullptr, RowInfo *info = nullptr,
                                   const RowInfo *staged = nullptr) {
  __syncthreads();
  const int cnt = b.cnt;
  if (cnt == 0) return;
  constexpr int PER = (CAP + BS - 1) / BS;
  const int i0 = threadIdx.x * PER;
  int64_t s = 0;
  for (int i = i0; i < i0 + PER && i < cnt; i++) s += b.wt[i];
  int64_t tot;
  int64_t pre = wg_excl_scan(s, &tot, b.sh);
  if (threadIdx.x == 0) b.base = atomicAdd(packc, pk(tot, cnt));
  __syncthreads();
  const int64_t slot0 = pk_cnt(b.base), w0 = pk_work(b.base);
  for (int i = i0; i < i0 + PER && i < cnt; i++) {
    work[slot0 + i] = w0 + pre;
    pre += b.wt[i];
  }
  for (int i = threadIdx.x; i < cnt; i += BS) {
    list[slot0 + i] = b.id[i];
    if (zero_acc) zero_acc[slot0 + i] = 0;
    if (info) info[slot0 + i] = staged[i];
  }
  __syncthreads();
  if (threadIdx.x == 0) b.cnt = 0;
  __syncthreads();
}

}  // namespace ccd
