// cc_team.hip -- many rounds of C4 / ClusterWild! (arXiv 1507.05086,
// Algorithm 2) in one launch, by the workgroups of one XCD.
//
// A round of a few thousand active vertices is bound by latency, not by
// work.  As a sequence of kernels each step pays its launch (about 1.6 us)
// and then a chain of accesses that the launch has made cold (the L2 does
// not keep other XCDs' writes, so each goes to the Infinity Cache or HBM).
// The compute units of one XCD share an L2: a barrier over their 32
// workgroups takes 1.1 - 1.7 us, and what one workgroup stores the others read
// back from that L2 in 0.1 - 0.2 us.  (Over all 8 XCDs the same barrier takes
// 4.2 us with 256 workgroups and 14 with the 1024 of a round kernel, and 30 and
// 117 with the fences that make one XCD's stores visible to the others.)  So
// the rounds whose lists are short enough for an eighth of the device run here,
// with two to five barriers a round and two more for each Delta pass, and the
// others on the whole device as kernels (cc_rounds.hip); next_stage() and its
// limits draw the line.
//
// Team.  The launch puts one workgroup on every compute unit.  The first to
// start picks its XCD; the workgroups of that XCD register until the wanted
// number is there or a time limit passes, then the team is closed and every
// other workgroup leaves.  Only registered workgroups, all running, wait for
// each other, so nothing is assumed about what else the device runs.  Every
// wait is bounded.
//
// Memory.  Data that changes within the launch is read with relaxed
// device-scope loads, which pass the compute unit's own cache and hit the
// shared L2, and written with plain stores or atomics, which reach that L2;
// each wave waits for its stores before a barrier.  Nothing needs the L2
// written back or invalidated.  The CSR, pi and the schedule do not change
// and are read plainly.
#include "cc_device.h"
#include "cc_launch.h"
#include "cc_round.h"

namespace ccd {

namespace {

constexpr int TNT = TEAM_NT;
constexpr int TNW = TNT / 64;
constexpr int TIPT = 4;            // adjacency items per thread per tile
constexpr int TTW = TNT * TIPT;    // adjacency items per tile
constexpr int TCLAIM = 2 * TTW;    // newly claimed vertices kept in LDS (a tile adds at most TTW)
constexpr int TROWS = 4096;        // active rows a workgroup keeps in LDS
constexpr int TLONG = 2048;        // longer rows are shared by the team
constexpr int TEDGE = 4096;        // conflict edges settled in LDS by one workgroup
constexpr int32_t UB_GONE = INT32_MIN / 2;  // degree word of a vertex that left (exact phase)
constexpr long long TEAM_WINDOW = 2000;       // registration window, wall clock ticks (100 MHz)
constexpr long long TEAM_LIMIT = 200000000;   // longest wait at a barrier: 2 s

struct Lds {
  int32_t lw[TTW + 1];   // item at which the tile's row j starts, relative to the tile
  int32_t lv[TTW + 1];   // its vertex
  int32_t loff[TTW + 1]; // where its adjacency starts in col, less lw
  int32_t lval[TTW + 1]; // its rank, or its count (rescan)
  int32_t cl[TCLAIM];    // newly claimed vertices; row lengths (rescan); blocked vertices' words (resolve)
  // this workgroup's active rows: vertex, first item, start in col less that, rank
  int32_t rv[TROWS], rw[TROWS], ro[TROWS], rr[TROWS];
  uint8_t rmark[TROWS];  // blocked (C4) or in conflict (ClusterWild!)
  int32_t pw[TNT];       // rows_of_wg: prefix of row lengths, ...
  int32_t poff[TNT];     // ... row starts less the prefix ...
  int32_t pval[TNT];     // ... and a value per row
  int hist[HLDS];
  int sh[4][TNW];
  int32_t s_ent;
  unsigned long long s_base;
  int32_t lbase[NLVL + 1];
  int ncl, ok, smax;
  unsigned n, me;
};

// The team as each of its workgroups sees it.
struct Team {
  TeamCtl *t;
  Ctrl *c;
  unsigned n, me;  // workgroups, and this one's index
  unsigned gen;    // barriers passed
};

template <class T>
__device__ inline T ld(const T *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Workgroup barrier that also orders this workgroup's global stores.
__device__ inline void wg_sync() {
  stores_done();
  __syncthreads();
}

__device__ inline void team_abort(const Team &tm) {
  set_error(tm.c, ERR_NO_PROGRESS);
  atomicExch(&tm.t->abort, 1u);
  atomicExch(&tm.c->done, 1);
}

// Barrier of the team; false when a wait has expired somewhere (every
// workgroup then leaves).
__device__ inline bool team_sync(Team &tm, Lds &L) {
  stores_done();
  __syncthreads();
  if (tm.n <= 1) return true;
  tm.gen++;
  if (threadIdx.x == 0) {
    int ok = 1;
    if (add_rlx(&tm.t->arrive, 1u) + 1 == tm.gen * tm.n) {
      st_rlx(&tm.t->gen, tm.gen);
    } else {
      const long long t0 = wall_clock64();
      for (unsigned spin = 1; (int)(ld_rlx(&tm.t->gen) - tm.gen) < 0; spin++) {
        if (spin % 256 == 0) {
          if (ld_rlx(&tm.t->abort)) {
            ok = 0;
            break;
          }
          if (wall_clock64() - t0 > TEAM_LIMIT) {
            team_abort(tm);
            ok = 0;
            break;
          }
        }
      }
    }
    L.ok = ok;
  }
  __syncthreads();
  return L.ok != 0;
}

// One XCD's workgroups become the team (see the top).  Returns false in a
// workgroup that is not part of it.
__device__ inline bool team_form(Team &tm, Lds &L, unsigned want) {
  if (threadIdx.x == 0) {
    L.n = 0;
    const unsigned xcc = __builtin_amdgcn_s_getreg((3 << 11) | 20) + 1;  // HW_REG_XCC_ID, 4 bits
    TeamCtl *t = tm.t;
    const unsigned old = atomicCAS(&t->pick, 0u, xcc);
    if (old == 0 || old == xcc) {
      const unsigned me = atomicAdd(&t->reg, 1u);
      if (!(me & 0x80000000u)) {
        L.me = me;
        const long long t0 = wall_clock64();
        if (me == 0) {  // closes the team
          while ((ld_rlx(&t->reg) & 0x7fffffffu) < want && wall_clock64() - t0 < TEAM_WINDOW) {
          }
          L.n = atomicOr(&t->reg, 0x80000000u);
          st_rlx(&t->size, L.n);
        } else {
          unsigned n = 0;
          while ((n = ld_rlx(&t->size)) == 0 && wall_clock64() - t0 < TEAM_LIMIT) {
          }
          L.n = n;
        }
      }
    }
  }
  __syncthreads();
  tm.n = L.n;
  tm.me = L.me;
  return tm.n > 0;
}

__device__ inline int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ inline unsigned long long uni(unsigned long long x) {
  return (unsigned long long)(unsigned)uni((int)(x >> 32)) << 32 | (unsigned)uni((int)x);
}
__device__ inline long long uni(long long x) { return (long long)uni((unsigned long long)x); }

// Exclusive scan over the workgroup, one barrier; `sh` may be used again
// after the next barrier.
__device__ inline int wg_scan(int x, int *tot, int *sh) {
  const int inc = wave_incl_scan(x), l = lane_id(), w = uni(wave_id());
  if (l == 63) sh[w] = inc;
  __syncthreads();
  int s = l < TNW ? sh[l] : 0;
  s = dpp_add<0x111, 0xf>(s);
  s = dpp_add<0x112, 0xf>(s);
  if (TNW > 4) s = dpp_add<0x114, 0xf>(s);
  if (TNW > 8) s = dpp_add<0x118, 0xf>(s);
  *tot = __builtin_amdgcn_readlane(s, TNW - 1);
  const int base = w > 0 ? __builtin_amdgcn_readlane(s, w - 1) : 0;
  return base + inc - x;
}
// Two at once.
__device__ inline void wg_scan2(int x, int y, int *px, int *py, int *tx, int *ty, int *sh, int *sh2) {
  const int ix = wave_incl_scan(x), iy = wave_incl_scan(y), l = lane_id(), w = uni(wave_id());
  if (l == 63) {
    sh[w] = ix;
    sh2[w] = iy;
  }
  __syncthreads();
  int s = l < TNW ? sh[l] : 0, t = l < TNW ? sh2[l] : 0;
  s = dpp_add<0x111, 0xf>(s);
  t = dpp_add<0x111, 0xf>(t);
  s = dpp_add<0x112, 0xf>(s);
  t = dpp_add<0x112, 0xf>(t);
  if (TNW > 4) {
    s = dpp_add<0x114, 0xf>(s);
    t = dpp_add<0x114, 0xf>(t);
  }
  if (TNW > 8) {
    s = dpp_add<0x118, 0xf>(s);
    t = dpp_add<0x118, 0xf>(t);
  }
  *tx = __builtin_amdgcn_readlane(s, TNW - 1);
  *ty = __builtin_amdgcn_readlane(t, TNW - 1);
  *px = (w > 0 ? __builtin_amdgcn_readlane(s, w - 1) : 0) + ix - x;
  *py = (w > 0 ? __builtin_amdgcn_readlane(t, w - 1) : 0) + iy - y;
}

// The low words of 64-bit offsets and prefixes: a team's graph has fewer
// than 2^31 stored entries.
__device__ inline int32_t lo32(const int64_t *p) { return *reinterpret_cast<const int32_t *>(p); }
__device__ inline int32_t ld_lo(const int64_t *p) { return ld(reinterpret_cast<const int32_t *>(p)); }

__device__ inline bool bit(const uint32_t *unc, int32_t v) { return (ld(&unc[v >> 5]) >> (v & 31)) & 1u; }

// wave_find_entry on a list written in this launch.
__device__ inline int find_entry(const int64_t *work, int cnt, int s) {
  int lo = 0, hi = cnt;
  while (hi - lo > 1) {
    const int step = (hi - lo + 63) / 64;
    const int idx = lo + lane_id() * step;
    const bool pred = idx < hi && ld_lo(&work[idx]) <= s;
    const int k = __popcll(__ballot(pred));
    lo = lo + (k - 1) * step;
    hi = lo + step < hi ? lo + step : hi;
  }
  return lo;
}

// last j < n with a[j] <= x (a sorted, a[0] <= x)
__device__ inline int last_le(const int32_t *a, int n, int32_t x) {
  int j = 0, step = 1;
  while (step * 2 < n) step *= 2;
  for (; step > 0; step >>= 1)
    if (j + step < n && a[j + step] <= x) j += step;
  return j;
}

struct Item {
  int ent[TIPT];    // row within the tile, -1: none
  int32_t u[TIPT];  // neighbour
  unsigned vert;    // bit k: the first item of its row
};

// A list (vertices and the exclusive prefix of their row lengths) is cut
// into equal shares of items, one per workgroup; a share is walked in tiles
// of TTW items.  Stages the rows that items [s, te) of the list touch (the
// first is entry ent0), finds this thread's items and loads their neighbours.
// With info, rows come from it and lval is the rank; else from off / end,
// lval is 0 and cl the row length.  Returns the number of rows.
template <bool INFO>
__device__ inline int tile_load(Lds &L, const int32_t *list, const int64_t *work, const RowInfo *info,
                                const int64_t *off, const int64_t *end, const int32_t *col, int cnt, int s, int te,
                                int ent0, Item &it) {
  int nrows = 0;
  for (;; nrows += TNT) {
    const int idx = ent0 + nrows + (int)threadIdx.x;
    bool in = false;
    if (idx < cnt && nrows + (int)threadIdx.x <= TTW) {
      const int32_t wk = ld_lo(&work[idx]);
      const int32_t v = ld(&list[idx]);
      int32_t start = 0, val = 0;
      if (INFO) {
        start = ld_lo(&info[idx].start);
        val = ld(&info[idx].rank);
      }
      if (wk < te) {
        in = true;
        const int j = nrows + threadIdx.x;
        if (!INFO) {
          start = lo32(&off[v]);
          L.cl[j] = lo32(&end[v]) - start;
        }
        L.lw[j] = wk - s;
        L.lv[j] = v;
        L.loff[j] = start - (wk - s);
        L.lval[j] = val;
      }
    }
    const int c = __syncthreads_count(in);
    if (c < TNT) {
      nrows += c;
      break;
    }
  }
  it.vert = 0;
  int32_t pos[TIPT];
#pragma unroll
  for (int k = 0; k < TIPT; k++) {
    const int x = k * TNT + (int)threadIdx.x;
    it.ent[k] = -1;
    it.u[k] = 0;
    pos[k] = 0;
    if (s + x < te) {
      const int j = last_le(L.lw, nrows, x);
      it.ent[k] = j;
      if (x == L.lw[j]) it.vert |= 1u << k;
      pos[k] = L.loff[j] + x;
    }
  }
#pragma unroll
  for (int k = 0; k < TIPT; k++)
    if (it.ent[k] >= 0) it.u[k] = col[pos[k]];
  return nrows;
}

// Walks the rows of entries 0 .. cnt-1 inside one workgroup, balanced over
// its items: row(i, start, len, val) describes entry i, f(u, val) takes a
// neighbour.
template <class R, class F>
__device__ inline void rows_of_wg(Lds &L, int cnt, const int32_t *col, R &&row, F &&f) {
  for (int i0 = 0; i0 < cnt; i0 += TNT) {
    int32_t start = 0, len = 0, val = 0;
    const int i = i0 + threadIdx.x;
    if (i < cnt) row(i, start, len, val);
    int tot;
    const int pre = wg_scan(len, &tot, L.sh[0]);
    L.pw[threadIdx.x] = pre;
    L.poff[threadIdx.x] = start - pre;
    L.pval[threadIdx.x] = val;
    __syncthreads();
    const int rows = cnt - i0 < TNT ? cnt - i0 : TNT;
    for (int e0 = 0; e0 < tot; e0 += TNT * TIPT) {
      int32_t u[TIPT], pv[TIPT];
#pragma unroll
      for (int k = 0; k < TIPT; k++) {
        const int e = e0 + k * TNT + (int)threadIdx.x;
        u[k] = -1;
        pv[k] = 0;
        if (e < tot) {
          const int j = last_le(L.pw, rows, e);
          u[k] = col[L.poff[j] + e];
          pv[k] = L.pval[j];
        }
      }
      f(u, pv);
    }
    __syncthreads();
  }
}

// This workgroup's share of `total` items.
__device__ inline void share_of(const Team &tm, int total, int *s0, int *s1) {
  unsigned per = ((unsigned)total + tm.n - 1) / tm.n;
  if (per < 256) per = 256;
  const unsigned long long a = (unsigned long long)tm.me * per, b = a + per;
  *s0 = a < (unsigned)total ? (int)a : total;
  *s1 = b < (unsigned)total ? (int)b : total;
}

// One workgroup settles the blocked vertices of a C4 round (rule 1: the
// greedy MIS of G[A] in pi order, restricted to them): a blocked vertex is a
// non-center once an earlier active neighbour is a center, and a center once
// all of them are non-centers.  The conflict edges stay in registers, the
// words of settle_edges are in the room of the newly claimed, of which there
// are none yet.  The promoted go to the center list; *work_in and *work_out
// get the row lengths of the promoted and of all blocked vertices.
__device__ inline void resolve_lds(const Ws &w, Lds &L, TeamSlot *sl, int nb, int ne, const int64_t *rend,
                                   int *work_in, int *work_out) {
  static_assert(TEDGE <= TCLAIM && TEDGE < RES_GONE, "a blocked vertex has an edge");
  int *word = L.cl;
  for (int i = threadIdx.x; i < nb; i += TNT) {
    w.bpos[ld(&w.blist[i])] = i;
    word[i] = 0;
  }
  wg_sync();
  constexpr int EPT = TEDGE / TNT;
  int ia[EPT], iu[EPT];
  unsigned open = 0;
#pragma unroll
  for (int k = 0; k < EPT; k++) {
    const int e = k * TNT + (int)threadIdx.x;
    ia[k] = 0;
    iu[k] = -1;
    if (e < ne) {
      const int32_t a = ld(&w.cedge[e].x), u = ld(&w.cedge[e].y);
      const uint8_t fu = ld(&w.flag[u]);
      ia[k] = ld(&w.bpos[a]);
      if (fu) iu[k] = ld(&w.bpos[u]);  // not blocked: a root, a center already
      open |= 1u << k;
      atomicAdd(&word[ia[k]], 1);
    }
  }
  __syncthreads();
  settle_edges<EPT>(word, open, [&](int k) { return ia[k]; }, [&](int k) { return iu[k]; });
  __syncthreads();
  int win = 0, wout = 0;
  for (int i = threadIdx.x; i < nb; i += TNT) {
    const int32_t a = ld(&w.blist[i]);
    const int32_t start = lo32(&w.off[a]), d = lo32(&rend[a]) - start;
    wout += d;
    const int decided = res_decision(word[i]);
    if (decided == 0) sl->err = ERR_NO_PROGRESS;
    if (decided == 1) {
      win += d;
      const int32_t rk = ld(&w.rank[a]);
      w.state[a] = CENTER;
      w.lab[a] = rk;
      const unsigned long long q = atomicAdd(&sl->c_pack, pk(d, 1));
      w.clist[pk_cnt(q)] = a;
      w.cwork[pk_cnt(q)] = pk_work(q);
      w.cinfo[pk_cnt(q)] = RowInfo{start, d, rk};
    } else {
      w.state[a] = NONCENTER;
    }
  }
  *work_in = win;
  *work_out = wout;
  __syncthreads();  // the words' room is the newly claimed's again
}

}  // namespace

namespace {

// The end of a round slot, told to the host.
__device__ inline void end_slot(const Ws &w, Ctrl *c, bool done, bool ran, bool error, int phase) {
  const int slots = c->slots + 1;
  c->slots = slots;
  if (!w.progress) return;
  __hip_atomic_store(w.progress, (unsigned long long)(unsigned)slots |
                                     (unsigned long long)done << PROGRESS_DONE |
                                     (unsigned long long)ran << PROGRESS_RAN |
                                     (unsigned long long)(phase == PHASE_EXACT) << PROGRESS_EXACT |
                                     (unsigned long long)error << PROGRESS_ERROR,
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// What k_check_order, k_init and the first k_close do, by one workgroup, for
// a run that keeps exact degrees from the start or none at all.  A rank
// exchanged twice is a repeated entry of pi; n in-range entries without one
// are a permutation.  Returns false when pi is none.
__device__ inline bool run_init(const Ws &w, Lds &L) {
  Ctrl *c = w.ctrl;
  const int n = (int)w.n, tid = threadIdx.x;
  for (int i = tid; i < (int)(sizeof(Ctrl) / 4); i += TNT) reinterpret_cast<int *>(c)[i] = 0;
  for (int i = tid; i < (int)(sizeof(TeamCtl) / 4); i += TNT) reinterpret_cast<int *>(w.team)[i] = 0;
  for (int i = tid; i < (int)w.max_deg + 2; i += TNT) w.hist[i] = 0;
  for (int i = tid; i < HLDS; i += TNT) L.hist[i] = 0;
  if (tid == 0) L.ok = 0;  // set by a thread that finds pi wrong
  for (int i = tid; i < (n + 31) / 32; i += TNT) w.unc[i] = n - i * 32 >= 32 ? 0xFFFFFFFFu : (1u << (n - i * 32)) - 1u;
  __syncthreads();
  for (int v = tid; v < n; v += TNT) {
    const int d = lo32(&w.off[v + 1]) - lo32(&w.off[v]);
    w.rank[v] = -1;
    w.lab[v] = INF;
    w.state[v] = UNCL;
    w.flag[v] = 0;
    w.ub[v] = d;
    if (w.start_exact) hist_add(L.hist, w.hist, d, 1);
  }
  wg_sync();
  if (w.start_exact)
    for (int i = tid; i < HLDS; i += TNT)
      if (L.hist[i]) atomicAdd(&w.hist[i], L.hist[i]);
  bool bad = false;
  for (int k = tid; k < n; k += TNT) {
    const int32_t v = w.order_in[k];
    if (v < 0 || v >= n) {
      bad = true;
      continue;
    }
    const int32_t vi = w.perm[v];
    w.iorder[k] = vi;
    bad |= atomicExch(&w.rank[vi], k) != -1;
  }
  if (bad) L.ok = 1;
  wg_sync();
  if (uni(L.ok)) {
    if (tid == 0) {
      c->error = ERR_PERM;
      c->done = 1;
      end_slot(w, c, true, false, true, PHASE_EXACT);
    }
    return false;
  }
  // round 0, by every wave alike; thread 0 writes it down
  const int phase = w.start_exact ? PHASE_EXACT : PHASE_LAZY;
  long long b = 0;
  double eps_used = 0.0;
  int fb = 0;
  next_batch(w, n, w.max_deg, 0, 0.f, 0.f, (float)w.eps, &b, &eps_used, &fb);
  if (tid == 0) {
    c->n_rem = c->n_start = n;
    c->delta = w.max_deg;
    c->b = b < n ? b : n;
    c->r_last = c->b - 1;  // (the practical schedule's; else set by the selection)
    c->eps_used = eps_used;
    c->feat_eps = (float)w.eps;
    c->fallback = fb;
    c->phase = (int16_t)phase;
    c->has_round = 1;
    c->t_start = (long long)wall_clock64();
  }
  wg_sync();
  return true;
}

// k_finalize by one workgroup: every label is looked at before the first is
// written, so a failing run leaves the caller's buffer alone.  The input id of
// a center comes from the workspace, not from order_in: the caller may have
// given one buffer as pi and as labels.
__device__ inline void run_labels(const Ws &w, Ctrl *c) {
  const int n = (int)w.n, tid = threadIdx.x;
  const bool bounded = w.max_rounds > 0;
  // the label of input id vin: >= -1, or -2: none
  auto label = [&](int vin) -> int32_t {
    const int32_t v = w.perm[vin];
    if (v >= w.iso_start && !bounded) return vin;
    const int32_t l = ld(&w.lab[v]);
    if (l == INF) {
      if (v < w.iso_start && !bit(w.unc, v)) return vin;
      return bounded ? -1 : -2;
    }
    return l < 0 || l >= n ? -2 : w.iperm[w.iorder[l]];
  };
  bool bad = false;
  for (int v = tid; v < n; v += TNT) bad |= label(v) == -2;
  if (__syncthreads_or(bad)) {
    if (tid == 0) c->error = ERR_LABEL;
    return;
  }
  for (int v = tid; v < n; v += TNT) w.labels_out[v] = label(v);
}

}  // namespace

// Runs rounds until the run is done or a round (or the rest of one) is for
// the whole device; leaves the state in Ctrl as the round kernels keep it.
// SOLO: one workgroup, which also sets the run up (run_init) and, when it is
// done, writes the labels: one launch for a small graph.
template <int ALGO, bool SOLO>
__global__ void __launch_bounds__(TNT) k_team(Ws w) {
  __shared__ Lds L;
  Ctrl *c = w.ctrl;
  Team tm{w.team, c, 0, 0, 0};
  if constexpr (SOLO) {
    tm.n = 1;
    if (!run_init(w, L)) return;
  } else {
    const CtrlHead h = ctrl_head(c);
    if (h.done) return;
    if (h.stage != ST_TEAM) {
      // the round is for the device (or a team of this launch has left it)
      if (blockIdx.x == 0 && threadIdx.x == 0 && ld(&w.team->reg) == 0) end_slot(w, c, false, false, false, h.phase);
      return;
    }
    if (!team_form(tm, L, (unsigned)w.team_n)) return;
  }
  constexpr bool c4 = ALGO == ALGO_C4;
  const bool binomial = w.policy == POL_BINOMIAL;
  const int tid = threadIdx.x;
  const bool lead = tm.me == 0 && tid == 0;
  // the round prepared by the kernel before this one
  long long n_rem = ld(&c->n_rem), delta = ld(&c->delta), B = ld(&c->b), cursor = ld(&c->cursor);
  long long round = ld(&c->round), r_last = ld(&c->r_last), t_start = ld(&c->t_start);
  double eps_used = c->eps_used;
  float fconf = c->feat_conf, fclaim = c->feat_claim, feps = c->feat_eps;
  int phase = ld(&c->phase);
  int fallback = 0;
  unsigned long long sum_rescan = 0, sum_blocked = 0, sum_atom = 0;
  long long sum_items = 0;    // items of this workgroup's rows
  long long sum_long = 0;     // of the long rows this wave has listed
  long long sum_claim_x = 0;  // this wave's: promoted less blocked rows
  int64_t atoms = 0;  // this thread's atomic updates
  int64_t peeled = 0; // this workgroup's (thread 0)
  const int64_t n = w.n;
  int step = 0;       // selection steps, for the parity of tcnt
  int stage = ST_TEAM;
  bool done = false;
  const bool bounded = w.max_rounds > 0;
  long long rounds = 0;  // run here
  float rate = ld(&c->rate);  // entries walked per active vertex, the round before
  for (unsigned rr = 0;; rr++) {
    TeamSlot *sl = &tm.t->slot[rr & 3];
    const bool exact = phase == PHASE_EXACT;
    const int64_t *rend = round_end(w, phase);
    const int32_t *col = round_col(w, phase);
    // ---- the active set: the next B unclustered vertices of pi (the
    // unclustered among the next B positions under the practical schedule)
    const long long sel_end = binomial ? (cursor + B < n ? cursor + B : n) : n;
    long long taken = 0, pos0 = cursor;
    int lone = 0;
    if (tid == 0) L.ncl = 0;
    const bool spread = (double)B * rate > (double)TEAM_SPREAD;
    for (int i = tid; i < HLDS; i += TNT) L.hist[i] = 0;
    int nrow = 0, nitem = 0, wlong = 0;  // rows kept here, their items; items of the long rows listed here
    while (pos0 < sel_end && (binomial || taken < B)) {
      long long need = sel_end - pos0;
      if (!binomial) {
        const double per = (double)(n - pos0) / (double)(n_rem - taken > 0 ? n_rem - taken : 1);
        const long long est = (long long)((double)(B - taken) * per * 1.0625) + 64;
        need = est < need ? est : need;
      }
      int chunk = need >= (long long)4 * TNT * tm.n ? 4 * TNT : ((int)need + (int)tm.n - 1) / (int)tm.n;
      if (!spread || chunk > 64) chunk = (chunk + 63) / 64 * 64;
      if (chunk > 4 * TNT) chunk = 4 * TNT;
      const int q = (chunk + TNT - 1) / TNT;
      int32_t vv[4], rs[4], dg[4];
      unsigned un = 0, lonely = 0;
      const int base = (int)pos0 + (int)tm.me * chunk + tid * q;
#pragma unroll
      for (int k = 0; k < 4; k++) {
        vv[k] = -1;
        if (k < q && tid * q + k < chunk && (long long)base + k < sel_end) vv[k] = w.order[base + k];
      }
#pragma unroll
      for (int k = 0; k < 4; k++) {
        rs[k] = 0;
        dg[k] = 0;
        if (vv[k] < 0) continue;
        if (vv[k] >= w.iso_start) {
          un |= 1u << k;
          lonely |= 1u << k;
        } else if (bit(w.unc, vv[k])) {
          un |= 1u << k;
        }
      }
      // the rows of the unclustered, in flight while the counts are exchanged
#pragma unroll
      for (int k = 0; k < 4; k++)
        if ((un & ~lonely) >> k & 1) {
          rs[k] = lo32(&w.off[vv[k]]);
          dg[k] = lo32(&rend[vv[k]]) - rs[k];
          if (exact && ld(&w.ub[vv[k]]) == 0) lonely |= 1u << k;
        }
      unsigned act = un;
      if (!binomial) {
        int tot;
        const int pre = wg_scan(__popc(un), &tot, L.sh[0]);
        int excl = 0, all = tot;
        if (tm.n > 1) {
          if (tid == 0) tm.t->tcnt[step & 1][tm.me] = (unsigned)tot;
          if (!team_sync(tm, L)) return;
          const int l = lane_id();
          const int x = l < (int)tm.n ? (int)ld(&tm.t->tcnt[step & 1][l]) : 0;
          const int inc = wave_incl_scan(x);
          all = __builtin_amdgcn_readlane(inc, 63);
          excl = tm.me > 0 ? __builtin_amdgcn_readlane(inc, tm.me - 1) : 0;
        }
        step++;
        long long r = taken + excl + pre;
        act = 0;
#pragma unroll
        for (int k = 0; k < 4; k++)
          if (un >> k & 1) {
            if (r < B) {
              act |= 1u << k;
              if (r == B - 1) sl->r_last = (long long)base + k;
            }
            r++;
          }
        taken += all;
      }
      // an active vertex with no unclustered neighbour is settled here
      // (k_select says why); the others keep their rows in LDS, or list
      // them for the team if they are long
      const unsigned lst = act & ~lonely;
      int wsum = 0, csum = 0;
#pragma unroll
      for (int k = 0; k < 4; k++) {
        if (lst >> k & 1 && dg[k] <= TLONG) {
          wsum += dg[k];
          csum++;
        }
        if ((act & lonely) >> k & 1) {
          lone++;
          if (vv[k] >= w.iso_start) {
            if (bounded) w.lab[vv[k]] = base + k;
          } else {
            atomicAnd(&w.unc[vv[k] >> 5], ~(1u << (vv[k] & 31)));
            atoms++;
          }
        }
      }
      int ctot, wtot, cpre, wpre;
      wg_scan2(csum, wsum, &cpre, &wpre, &ctot, &wtot, L.sh[1], L.sh[2]);
      int slot = nrow + cpre, item = nitem + wpre;
      const bool fits = nrow + ctot <= TROWS;  // or every row of this step is listed
#pragma unroll
      for (int k = 0; k < 4; k++)
        if (lst >> k & 1) {
          const int32_t v = vv[k], p = base + k;
          w.state[v] = ACTIVE;
          if (c4) w.rank[v] = p;
          else w.lab[v] = p;
          if (fits && dg[k] <= TLONG) {
            L.rv[slot] = v;
            L.rw[slot] = item;
            L.ro[slot] = rs[k] - item;
            L.rr[slot] = p;
            L.rmark[slot] = 0;
            slot++;
            item += dg[k];
          } else {
            const unsigned long long x = atomicAdd(&sl->a_pack, pk(dg[k], 1));
            w.alist[pk_cnt(x)] = v;
            w.awork[pk_cnt(x)] = pk_work(x);
            w.ainfo[pk_cnt(x)] = RowInfo{rs[k], dg[k], p};
            wlong += dg[k];
          }
        }
      if (fits) {
        nrow += ctot;
        nitem += wtot;
      }
      lone += __popc(lst) << 16;  // a step adds at most 4 of each
      pos0 += (long long)tm.n * chunk;
      // the next step scans in the same scratch (the count above parts the steps of the other rules)
      if (binomial && pos0 < sel_end) __syncthreads();
    }
    {
      int lt, wt, x, y;
      wg_scan2(lone & 0xFFFF, lone >> 16, &x, &y, &lt, &wt, L.sh[0], L.sh[3]);
      if (tid == 0 && (lt | wt))
        atomicAdd(&sl->listed, (unsigned long long)(unsigned)wt | (unsigned long long)(unsigned)lt << 32);
    }
    // the first tile of this workgroup's items, loaded while the team meets
    int32_t iu[TIPT];
    int ij[TIPT];
    auto own_items = [&](int i0) {
#pragma unroll
      for (int k = 0; k < TIPT; k++) {
        const int x = i0 + k * TNT + tid;
        ij[k] = -1;
        iu[k] = -1;
        if (x < nitem) {
          ij[k] = last_le(L.rw, nrow, x);
          iu[k] = col[L.ro[ij[k]] + x];
        }
      }
    };
    own_items(0);
    if (!team_sync(tm, L)) return;
    if (!binomial) r_last = uni(ld(&sl->r_last));
    const unsigned long long lp = uni(ld(&sl->listed)), ap = uni(ld(&sl->a_pack));
    const int na = (int)(lp & 0xFFFFFFFFull), lones = (int)(lp >> 32);
    const int nlong = (int)pk_cnt(ap), along = (int)pk_work(ap);
    // Lists every active row for the round kernels; false when a wait has expired.
    auto list_all = [&]() {
      if (tid == 0) L.s_base = nrow > 0 ? atomicAdd(&sl->a_pack, pk(nitem, nrow)) : 0;
      __syncthreads();
      const unsigned long long b0 = L.s_base;
      for (int i = tid; i < nrow; i += TNT) {
        const int d = (i + 1 < nrow ? L.rw[i + 1] : nitem) - L.rw[i];
        w.alist[pk_cnt(b0) + i] = L.rv[i];
        w.awork[pk_cnt(b0) + i] = pk_work(b0) + L.rw[i];
        w.ainfo[pk_cnt(b0) + i] = RowInfo{L.ro[i] + L.rw[i], d, L.rr[i]};
      }
      if (!team_sync(tm, L)) return false;
      if (lead) {
        c->a_pack = ld(&sl->a_pack);
        c->spread_lone[0] += (unsigned long long)lones;
      }
      return true;
    };
    if (!SOLO && along > TEAM_ACTIVE) {  // hubs: far more than the rate said
      if (!list_all()) return;
      stage = ST_ELECT;
      break;
    }
    // this workgroup's share of the long rows' items
    int s0, s1, first = 0;
    share_of(tm, along, &s0, &s1);
    if (s0 < s1) {
      if (tid < 64) {
        const int e = find_entry(w.awork, nlong, s0);
        if (tid == 0) L.s_ent = e;
      }
      __syncthreads();
      first = uni(L.s_ent);
    }
    Item it;
    int rows = 0;
    int nb = 0, ne = 0;
    int work_in = 0, work_out = 0;
    // ---- C4's election: active vertices with an earlier active neighbour
    if (c4) {
      // row a of rank rk sees neighbour u; true: a is blocked
      auto elect = [&](const int32_t *u, const int32_t *a, const int32_t *rk, bool *conf) {
        uint8_t su[TIPT];
#pragma unroll
        for (int k = 0; k < TIPT; k++) su[k] = u[k] >= 0 ? ld(&w.state[u[k]]) : (uint8_t)UNCL;
#pragma unroll
        for (int k = 0; k < TIPT; k++) {
          conf[k] = su[k] == ACTIVE && ld(&w.rank[u[k]]) < rk[k];
          const unsigned long long m = __ballot(conf[k]);
          if (m == 0) continue;
          if (conf[k]) {
            const unsigned b8 = 1u << (8 * (a[k] & 3));
            if (!(atomicOr((unsigned *)(w.flag + (a[k] & ~3)), b8) & b8))
              w.blist[atomicAdd(&sl->n_blocked, 1u)] = a[k];  // the first to see it blocked
          }
          const int leader = __ffsll((long long)m) - 1;
          unsigned b0 = 0;
          if (lane_id() == leader) b0 = atomicAdd(&sl->n_cedges, (unsigned)__popcll(m));
          b0 = __shfl(b0, leader, 64);
          const int64_t x = (int64_t)b0 + __popcll(m & lanemask_lt());
          if (conf[k] && x < w.cedge_cap) w.cedge[x] = make_int2(a[k], u[k]);
        }
      };
      for (int i0 = 0; i0 < nitem; i0 += TTW) {
        if (i0 > 0) own_items(i0);
        int32_t a[TIPT], rk[TIPT];
        bool conf[TIPT];
#pragma unroll
        for (int k = 0; k < TIPT; k++) {
          a[k] = ij[k] >= 0 ? L.rv[ij[k]] : 0;
          rk[k] = ij[k] >= 0 ? L.rr[ij[k]] : 0;
        }
        elect(iu, a, rk, conf);
#pragma unroll
        for (int k = 0; k < TIPT; k++)
          if (conf[k]) L.rmark[ij[k]] = 1;
      }
      int ent = first;
      for (int s = s0; s < s1; s += TTW) {
        const int te = s + TTW < s1 ? s + TTW : s1;
        rows = tile_load<true>(L, w.alist, w.awork, w.ainfo, nullptr, nullptr, col, nlong, s, te, ent, it);
        ent += rows - 1;
        int32_t u[TIPT], a[TIPT], rk[TIPT];
        bool conf[TIPT];
#pragma unroll
        for (int k = 0; k < TIPT; k++) {
          u[k] = it.ent[k] >= 0 ? it.u[k] : -1;
          a[k] = it.ent[k] >= 0 ? L.lv[it.ent[k]] : 0;
          rk[k] = it.ent[k] >= 0 ? L.lval[it.ent[k]] : 0;
        }
        elect(u, a, rk, conf);
        __syncthreads();  // the next tile takes the same LDS
      }
      if (!team_sync(tm, L)) return;
      ne = uni((int)ld(&sl->n_cedges));
      nb = uni((int)ld(&sl->n_blocked));
      if (ne > TEDGE) {  // settled by k_resolve
        if (!list_all()) return;
        if (lead) c->n_cedges = (unsigned)ne;
        stage = ST_CLASSIFY;
        break;
      }
      if (nb > 0 && tm.me == 0) resolve_lds(w, L, sl, nb, ne, rend, &work_in, &work_out);
    }
    sum_items += nitem;
    // ---- claims: a neighbour takes the lowest center rank.  An earlier
    // round's label is below this round's ranks, so the label alone says
    // whether a neighbour can still be claimed (a vertex that k_select or the
    // selection above settled has no unclustered neighbour), and the newly
    // clustered can leave while others still claim.  A root's own label may
    // still be unset, so a row that holds its own vertex must not list it.
    int conf_n = 0;
    auto claim = [&](const int32_t *u, const int32_t *rk, const bool *on, bool *broken, auto &&row) {
      int32_t cur[TIPT];
      uint8_t su[TIPT];
#pragma unroll
      for (int k = 0; k < TIPT; k++) {
        cur[k] = on[k] ? ld(&w.lab[u[k]]) : -1;
        if (!c4) su[k] = on[k] ? ld(&w.state[u[k]]) : (uint8_t)UNCL;
      }
#pragma unroll
      for (int k = 0; k < TIPT; k++) {
        broken[k] = false;
        if (!c4 && su[k] == ACTIVE) {  // ClusterWild! claims Gamma(c) \ A
          broken[k] = cur[k] < rk[k];  // rule 1 broken (lab = rank here)
        } else if (rk[k] < cur[k]) {
          atoms++;
          if (atomicMin(&w.lab[u[k]], rk[k]) == INF && u[k] != row(k)) L.cl[atomicAdd(&L.ncl, 1)] = u[k];  // newly claimed
        }
      }
    };
    // A vertex leaves: its bit goes, and in the exact phase it leaves the
    // degree histogram once (its word is exchanged for a value that later
    // decrements leave negative).
    auto leave = [&](int32_t v) {
      atomicAnd(&w.unc[v >> 5], ~(1u << (v & 31)));
      if (exact) hist_add(L.hist, w.hist, atomicExch(&w.ub[v], UB_GONE), -1);
    };
    // The claimed leave and, in the exact phase, take one degree from their
    // unclustered neighbours.  A neighbour that leaves in this same phase is
    // settled by the order of the two atomics on its word.
    int ncl_sum = 0;
    const int64_t peeled0 = peeled;
    auto drain = [&]() {  // every thread; L.ncl complete (after a barrier)
      const int ncl = uni(L.ncl);
      ncl_sum += ncl;
      if (!exact) {
        for (int i = tid; i < ncl; i += TNT) leave(L.cl[i]);
      } else {
        rows_of_wg(
            L, ncl, col,
            [&](int i, int32_t &start, int32_t &len, int32_t &) {
              const int32_t v = L.cl[i];
              start = lo32(&w.off[v]);
              len = lo32(&rend[v]) - start;
              leave(v);
              peeled += len;
            },
            [&](const int32_t *u, const int32_t *) {
              bool un[TIPT];
#pragma unroll
              for (int k = 0; k < TIPT; k++) un[k] = u[k] >= 0 && bit(w.unc, u[k]);
#pragma unroll
              for (int k = 0; k < TIPT; k++)
                if (un[k]) {
                  const int32_t old = atomicSub(&w.ub[u[k]], 1);
                  atoms++;
                  if (old > 0) {
                    hist_add(L.hist, w.hist, old, -1);
                    hist_add(L.hist, w.hist, old - 1, 1);
                  }
                }
            });
      }
      __syncthreads();
      if (tid == 0) L.ncl = 0;
      __syncthreads();
    };
    auto drain_if_full = [&]() {  // room for another tile
      __syncthreads();
      const int have = uni(L.ncl);
      __syncthreads();  // every wave has read it before any adds to it
      if (have > TTW) drain();
    };
    // long rows of a list, shared by the team
    auto claim_long = [&](const int32_t *list, const int64_t *work, const RowInfo *info, int cnt, bool check) {
      int ent = first;
      for (int s = s0; s < s1; s += TTW) {
        const int te = s + TTW < s1 ? s + TTW : s1;
        rows = tile_load<true>(L, list, work, info, nullptr, nullptr, col, cnt, s, te, ent, it);
        ent += rows - 1;
        if (check) {  // a blocked vertex claims only if it is promoted
          for (int j = tid; j < rows; j += TNT)
            if (ld(&w.flag[L.lv[j]])) L.lval[j] = -1;
          __syncthreads();
        }
        int32_t u[TIPT], rk[TIPT];
        bool on[TIPT], broken[TIPT];
#pragma unroll
        for (int k = 0; k < TIPT; k++) {
          u[k] = it.u[k];
          rk[k] = it.ent[k] >= 0 ? L.lval[it.ent[k]] : -1;
          on[k] = rk[k] >= 0;
          if (c4 && on[k] && (it.vert >> k & 1)) {  // a root (or promoted, as it is already)
            const int32_t a = L.lv[it.ent[k]];
            w.state[a] = CENTER;
            w.lab[a] = rk[k];
          }
        }
        claim(u, rk, on, broken, [&](int k) { return L.lv[it.ent[k]]; });
#pragma unroll
        for (int k = 0; k < TIPT; k++)
          if (broken[k]) {
            const int32_t a = L.lv[it.ent[k]];
            const unsigned b8 = 1u << (8 * (a & 3));
            if (!(atomicOr((unsigned *)(w.flag + (a & ~3)), b8) & b8)) conf_n++;
          }
        drain_if_full();
      }
    };
    for (int i0 = 0; i0 < nitem; i0 += TTW) {
      if (i0 > 0 || (c4 && nitem > TTW)) own_items(i0);
      int32_t rk[TIPT];
      bool on[TIPT], broken[TIPT];
#pragma unroll
      for (int k = 0; k < TIPT; k++) {
        on[k] = ij[k] >= 0 && !(c4 && L.rmark[ij[k]]);
        rk[k] = ij[k] >= 0 ? L.rr[ij[k]] : -1;
      }
      claim(iu, rk, on, broken, [&](int k) { return L.rv[ij[k]]; });
      if (!c4) {
#pragma unroll
        for (int k = 0; k < TIPT; k++)
          if (broken[k]) L.rmark[ij[k]] = 1;
      }
      if (nitem > TTW) drain_if_full();
    }
    // the active leave: every one of them is a center or will have been claimed
    for (int i = tid; i < nrow; i += TNT) {
      const int32_t v = L.rv[i];
      if (c4 && !L.rmark[i]) {  // a root
        w.state[v] = CENTER;
        w.lab[v] = L.rr[i];
      }
      leave(v);
    }
    for (int i = (int)tm.me * TNT + tid; i < nlong; i += (int)tm.n * TNT) leave(ld(&w.alist[i]));
    if (nlong > 0) claim_long(w.alist, w.awork, w.ainfo, nlong, c4 && nb > 0);
    __syncthreads();
    if (!c4)
      for (int i = tid; i < nrow; i += TNT) conf_n += L.rmark[i];
    drain();
    if (exact)
      for (int i = tid; i < HLDS; i += TNT) {
        const int x = L.hist[i];
        if (x) atomicAdd(&w.hist[i], x);
        L.hist[i] = 0;
      }
    auto count = [&]() {
      if (!c4) {
        int ct;
        (void)wg_scan(conf_n, &ct, L.sh[3]);
        if (tid == 0 && ct) atomicAdd(&sl->conflicts, (unsigned)ct);
      }
      int walked = nitem + (tm.me == 0 ? along : 0);
      if (exact) {
        int pt;
        (void)wg_scan((int)(peeled - peeled0), &pt, L.sh[0]);
        walked += pt;
      }
      if (tid == 0 && (ncl_sum | walked))
        atomicAdd(&sl->claimed, (unsigned long long)(unsigned)ncl_sum | (unsigned long long)(unsigned)walked << 32);
    };
    int promoted = 0;
    if (c4 && nb > 0) {
      if (!team_sync(tm, L)) return;  // the promoted are known
      const unsigned long long cp = uni(ld(&sl->c_pack));
      promoted = (int)pk_cnt(cp);
      if (tm.me == 0) {
        sum_claim_x += wave_sum(work_in) - wave_sum(work_out);
        for (int i = tid; i < nb; i += TNT) w.flag[ld(&w.blist[i])] = 0;
      }
      if (promoted > 0) {
        share_of(tm, (int)pk_work(cp), &s0, &s1);
        if (s0 < s1) {
          if (tid < 64) {
            const int e = find_entry(w.cwork, promoted, s0);
            if (tid == 0) L.s_ent = e;
          }
          __syncthreads();
          first = uni(L.s_ent);
        }
        claim_long(w.clist, w.cwork, w.cinfo, promoted, false);
        __syncthreads();
        drain();
        if (exact)
          for (int i = tid; i < HLDS; i += TNT) {
            const int x = L.hist[i];
            if (x) atomicAdd(&w.hist[i], x);
            L.hist[i] = 0;
          }
      }
    }
    count();
    if (nlong > 0) sum_long += wave_sum(wlong);
    // ---- the next Delta, lazy phase: band passes over stale bounds (dsearch)
    long long d_next = 0;
    bool to_device = false;
    if (!SOLO && !exact && !binomial) {
      int dm[DITER] = {0, 0, 0};
      struct {
        int phase;
        long long delta;
        int *d_max;
      } ds{PHASE_LAZY, delta, dm};
      DSearch sr = dsearch(&ds, 0);
      int pass = 0;
      for (; sr.pending; pass++) {
        // candidates: live entries with bound >= L
        const int kL = level_of(sr.L < DSW ? DSW : sr.L);
        __syncthreads();
        if (tid < 64) {
          int x = 0;
          if (tid < NLVL && tid >= kL) {
            const int cap = (int)(w.lvl_off[tid + 1] - w.lvl_off[tid]);
            x = (int)ld(&c->lvl_cnt[tid]);
            x = x < cap ? x : cap;
          }
          const int inc = wave_incl_scan(x);
          if (tid < NLVL) L.lbase[tid] = inc - x;
          if (tid == NLVL) L.lbase[NLVL] = inc;
        }
        __syncthreads();
        const int tot = uni(L.lbase[NLVL]);
        // entries are only ever added between the barriers that follow, so
        // every workgroup sees the same counts here
        if (tot > TEAM_SCAN) {
          to_device = true;
          break;
        }
        int32_t *rl = w.rlist + pass * w.rcap;
        int64_t *rw = w.rwork + pass * w.rcap;
        unsigned long long *ra = w.racc + pass * w.rcap;
        for (int i0 = (int)tm.me * TNT; i0 < tot; i0 += (int)tm.n * TNT) {
          const int i = i0 + tid;
          int32_t v = 0, d = 0;
          bool in = false;
          if (i < tot) {
            int k = kL;
            while (k < NLVL - 1 && i >= L.lbase[k + 1]) k++;
            v = ld(&w.lvl[w.lvl_off[k] + (i - L.lbase[k])]);
            const int32_t x = ld(&w.ub[v]);
            in = x >= sr.L && level_of(x) == k && bit(w.unc, v);
            if (in) d = lo32(&w.rend[v]) - lo32(&w.off[v]);
          }
          int ctot, wtot, cpre, wpre;
          wg_scan2(in ? 1 : 0, d, &cpre, &wpre, &ctot, &wtot, L.sh[1], L.sh[2]);
          if (ctot > 0) {
            if (tid == 0) L.s_base = atomicAdd(&sl->r_pack[pass], pk(wtot, ctot));
            __syncthreads();
            const int64_t slot = pk_cnt(L.s_base) + cpre;
            if (in && slot < w.rcap) {
              rl[slot] = v;
              rw[slot] = pk_work(L.s_base) + wpre;
              ra[slot] = 0;
            }
          }
          __syncthreads();
        }
        if (!team_sync(tm, L)) return;
        const unsigned long long rp = uni(ld(&sl->r_pack[pass]));
        const int rcnt = (int)(pk_cnt(rp) < w.rcap ? pk_cnt(rp) : w.rcap), rwk = (int)pk_work(rp);
        if (rwk > TEAM_WORK) {
          to_device = true;
          break;
        }
        sum_rescan += (unsigned long long)rwk;
        // their exact remaining degrees; new bounds move entries down the levels
        share_of(tm, rwk, &s0, &s1);
        if (tid == 0) L.smax = 0;
        if (s0 < s1) {
          if (tid < 64) {
            const int e = find_entry(rw, rcnt, s0);
            if (tid == 0) L.s_ent = e;
          }
          __syncthreads();
          int ent = uni(L.s_ent);
          for (int s = s0; s < s1; s += TTW) {
            const int te = s + TTW < s1 ? s + TTW : s1;
            rows = tile_load<false>(L, rl, rw, nullptr, w.off, w.rend, w.col, rcnt, s, te, ent, it);
            bool un[TIPT];
#pragma unroll
            for (int k = 0; k < TIPT; k++) un[k] = it.ent[k] >= 0 && bit(w.unc, it.u[k]);
#pragma unroll
            for (int k = 0; k < TIPT; k++)
              if (un[k]) atomicAdd(&L.lval[it.ent[k]], 1);
            __syncthreads();
            for (int j = tid; j < rows; j += TNT) {
              const int32_t v = L.lv[j], deg = L.cl[j];
              const int a = L.lw[j] > 0 ? L.lw[j] : 0;
              const int b = L.lw[j] + deg < te - s ? L.lw[j] + deg : te - s;
              int r = L.lval[j];
              // the row before a share's first can end where the share begins
              if (b > a && (b - a == deg || row_combine(ra, ent + j, r, b - a, deg, &r))) {
                const int32_t old = ld(&w.ub[v]);
                w.ub[v] = r;
                if (bit(w.unc, v)) atomicMax(&L.smax, r);
                const int kn = r >= DSW ? level_of(r) : -1;
                if (kn >= 0 && kn != level_of(old)) {
                  const int64_t p = atomicAdd(&c->lvl_cnt[kn], 1u);
                  if (p < w.lvl_off[kn + 1] - w.lvl_off[kn]) w.lvl[w.lvl_off[kn] + p] = v;
                  else sl->err = ERR_OVERFLOW;
                }
              }
            }
            ent += rows - 1;
            __syncthreads();
          }
        }
        __syncthreads();
        if (tid == 0 && L.smax > 0) atomicMax(&sl->d_max[pass], L.smax);
        if (!team_sync(tm, L)) return;
        dm[pass] = uni(ld(&sl->d_max[pass]));
        sr = dsearch(&ds, pass + 1);
      }
      if (!to_device && sr.switching) to_device = true;
      d_next = sr.delta;
      if (to_device) {
        if (lead) {  // the device goes on from this pass
          c->pass = (int8_t)pass;
#pragma unroll
          for (int j = 0; j < DITER; j++)
            if (j < pass) c->d_max[j] = dm[j];
        }
        // every workgroup's counts are in: the barrier of the first pass, or here
        if (!team_sync(tm, L)) return;
      }
    } else {
      if (!team_sync(tm, L)) return;
    }
    // ClusterWild!'s marks of this round, which nobody reads any more
    if (!c4) {
      for (int i = tid; i < nrow; i += TNT) w.state[L.rv[i]] = CENTER;
      for (int i = (int)tm.me * TNT + tid; i < nlong; i += (int)tm.n * TNT) {
        const int32_t v = ld(&w.alist[i]);
        w.state[v] = CENTER;
        w.flag[v] = 0;
      }
      // the next listing starts over in alist (the count exchange parts the two under the other rules)
      if (binomial && nlong > 0 && !team_sync(tm, L)) return;
    }
    const long long now = (long long)wall_clock64();
    const int err = uni(ld(&sl->err));
    const unsigned long long clp = uni(ld(&sl->claimed));
    const int claimed = (int)(clp & 0xFFFFFFFFull);
    const int conflicts = c4 ? nb : uni((int)ld(&sl->conflicts));
    const int listed = c4 ? na - nb + promoted : na;  // centers that were listed
    if (to_device) {  // k_candidates and what follows finish the round
      if (lead) {
        if (c4) c->c_pack = pk(0, listed);  // (their rows are counted here)
        else c->a_pack = pk(0, listed);
        c->n_pack = pk(0, claimed);
        c->n_blocked = (unsigned)nb;
        c->conflicts += c4 ? 0ull : (unsigned long long)conflicts;
        c->spread_lone[0] += (unsigned long long)lones;
      }
      stage = ST_DELTA;
      break;
    }
    // ---- close the round: every workgroup computes the same
    const long long newly = (long long)claimed + listed + lones;
    if (lead) {
      if (round < w.trace_cap) {
        RoundRec r;
        r.n_i = n_rem;
        r.delta_i = delta;
        r.b_i = B;
        r.r_i = r_last;
        r.centers = listed + lones;
        r.claimed = newly - listed - lones;
        r.conflicts = conflicts;
        r.eps_used = eps_used;
        r.t_ns = now - t_start;
        w.trace[round] = r;
      }
      sum_atom += (unsigned long long)(claimed + listed);
      sum_blocked += (unsigned long long)conflicts;
      // the slot after next is nobody's now
      TeamSlot *z = &tm.t->slot[(rr + 2) & 3];
      z->a_pack = z->c_pack = z->listed = z->claimed = 0;
      for (int j = 0; j < DITER; j++) {
        z->r_pack[j] = 0;
        z->d_max[j] = 0;
      }
      z->r_last = 0;
      z->n_cedges = z->n_blocked = z->conflicts = 0;
      z->err = 0;
    }
    fconf = B > 0 ? (float)conflicts / (float)B : 0.f;
    fclaim = n_rem > 0 ? (float)(newly - listed - lones) / (float)n_rem : 0.f;
    feps = (float)eps_used;
    cursor = r_last + 1;
    n_rem -= newly;
    round++;
    rounds++;
    int error = err;
    if (!error && !binomial && round > n + 1) error = ERR_NO_PROGRESS;
    if (!error && w.fault_round > 0 && round == w.fault_round) error = ERR_INJECTED;
    if (error && lead) set_error(c, error);
    done = n_rem <= 0 || error || (bounded && round >= w.max_rounds);
    if (!done && binomial && round >= w.sched_len) {
      if (lead) set_error(c, ERR_NO_PROGRESS);
      done = true;
    }
    if (binomial) {
      delta = delta_hat(w, round);
    } else if (!exact) {
      delta = d_next;
    } else if (!done) {
      long long found = 0;  // the highest non-empty bin
      for (long long top = delta < w.max_deg ? delta : w.max_deg; top >= 1 && !found; top -= 64) {
        const long long x = top - lane_id();
        const unsigned long long m = __ballot(x >= 1 && ld(&w.hist[x < 1 ? 1 : x]) > 0);
        if (m) found = top - (__ffsll((long long)m) - 1);
      }
      delta = found;
    } else {
      delta = 0;
    }
    if (done) break;
    rate = B > 0 ? (float)(unsigned)(clp >> 32) / (float)B : 0.f;
    int fb = 0;
    long long b = 0;
    next_batch(w, n_rem, delta, round, fconf, fclaim, feps, &b, &eps_used, &fb);
    if (fb) fallback = 1;
    if (binomial) {
      const long long left = n - cursor;
      if (b > left) b = left;
      r_last = cursor + b - 1;
    }
    B = b;
    t_start = now;
    if (!SOLO) {
      stage = next_stage(w, B, cursor, n_rem, rate);
      if (stage != ST_TEAM) break;
    }
  }
  // ---- leave the state where the round kernels and the host read it
  __syncthreads();
  const int64_t as = wave_sum(atoms), ps = wave_sum(peeled);
  if (lane_id() == 0) {
    if (as) atomicAdd(&c->sum_atomics, (unsigned long long)as);
    if (ps) atomicAdd(&c->sum_peel, (unsigned long long)ps);
    const long long walked = sum_long + (tid == 0 ? sum_items : 0);
    if (walked && c4) atomicAdd(&c->sum_elect, (unsigned long long)walked);
    if (walked + sum_claim_x) atomicAdd(&c->sum_claim, (unsigned long long)(walked + sum_claim_x));
  }
  if (lead) {
    c->n_rem = n_rem;
    c->n_start = n_rem;
    c->delta = delta;
    c->b = B;
    c->cursor = cursor;
    c->round = round;
    c->r_last = r_last;
    c->eps_used = eps_used;
    c->feat_conf = fconf;
    c->feat_claim = fclaim;
    c->feat_eps = feps;
    c->t_start = t_start;
    c->sum_rescan += sum_rescan;
    c->sum_blocked += sum_blocked;
    atomicAdd(&c->sum_atomics, sum_atom);
    if (fallback) c->fallback = 1;
    c->stage = (int8_t)(done ? ST_TEAM : stage);
    if (done) c->done = 1;
    if (!SOLO) end_slot(w, c, done, rounds > 0, false, phase);
  }
  if (SOLO) {
    wg_sync();
    const bool ok = done && ld(&c->error) == 0;
    if (ok) run_labels(w, c);
    wg_sync();
    if (tid == 0) end_slot(w, c, done, true, done && !ok, phase);
  }
}

RoundStep team_step(const Ws &w) {
  const bool c4 = w.algo == ALGO_C4;
  if (w.solo) return RoundStep{c4 ? k_team<ALGO_C4, true> : k_team<ALGO_CW, true>, 1, TNT};
  // one workgroup on every compute unit of the eight XCDs
  return RoundStep{c4 ? k_team<ALGO_C4, false> : k_team<ALGO_CW, false>, (unsigned)w.team_n * 8u, TNT};
}

hipError_t launch_team(const Ws &w, hipStream_t s) {
  const RoundStep t = team_step(w);
  hipLaunchKernelGGL(t.kernel, dim3(t.grid), dim3(t.block), 0, s, w);
  return hipGetLastError();
}

}  // namespace ccd
