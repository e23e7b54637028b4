// cc_rounds.hip -- the bulk-synchronous round loop of C4 and ClusterWild!
// (arXiv 1507.05086, Algorithm 2) as a fixed sequence of gfx950 kernels per
// round.  Kernel boundaries are the round's barriers (cheaper on this GPU than
// a software grid barrier); every kernel returns at once when its part of the
// round has nothing to do, so the host can queue rounds in groups and look at
// the done flag once per group.
//
//   select    next B_i unclustered vertices of pi (lazy deletion: a cursor
//             walks pi once); one pass with decoupled look-back
//   elect     C4: does an active vertex have an earlier-ranked active
//             neighbour?  (concurrency rule 1; edge-balanced)
//   classify  C4: roots become centers, the others are blocked
//   resolve   C4: one workgroup settles the blocked vertices over the conflict
//             edges (the greedy MIS of G[A] in pi order)
//   claim     every center claims its unclustered neighbours with atomicMin on
//             the center rank (concurrency rule 2, createCluster)
//   clear     the newly clustered leave the unclustered bitmap
//   candidates / degrees   lazy phase: a pass of the search for the next Delta
//             from stale upper bounds, which rescans only rows in a band below
//             the current Delta (a pass per slot); at the end of the phase,
//             the switch to exact degrees
//   peel      exact phase: neighbours of the newly clustered lose one
//             remaining degree each (degree histogram kept per workgroup)
//   close     one wave: round record, Delta_{i+1}, B_{i+1}, counters
//
// The paper deletes lazily (clustered vertices are skipped, the graph is never
// changed); here that extends to the remaining degrees: while Delta is large
// they are upper bounds refreshed only where the maximum could be, and the
// edge-by-edge peeling starts only when little of the graph is left.
#include "cc_device.h"
#include "cc_launch.h"
#include "cc_round.h"
#include "cc_walk.h"

namespace ccd {

// ------------------------------------------------------------------ init --

// pi moves to internal ids (one gather, written in pi order) and must be a
// permutation: n entries, each in range and none repeated.  Each entry marks
// its vertex in the (zeroed) state bytes with a plain store; n entries in
// range mark all n vertices exactly when none repeats, which k_init checks.
// pi is not inverted: the rank of a vertex is recorded when it becomes
// active, the only time anyone asks for it.
__global__ void __launch_bounds__(BS) k_check_order(Ws w) {
  const int64_t n = w.n;
  for (int64_t k = (int64_t)blockIdx.x * BS + threadIdx.x; k < n; k += (int64_t)gridDim.x * BS) {
    const int32_t v = w.order_in[k];
    if (v < 0 || (int64_t)v >= n) {
      set_error(w.ctrl, ERR_PERM);
      w.iorder[k] = 0;
    } else {
      const int32_t vi = w.perm[v];
      w.iorder[k] = vi;
      w.state[vi] = ORDER_SEEN;
    }
  }
}

// An isolated vertex (id >= iso_start) has no neighbour to read its state,
// flag or bound, and k_select settles it by its id alone, so only a partial
// run (whose k_finalize reads its label) and the direct check of pi (which
// reads its mark) visit those ids.
__global__ void __launch_bounds__(BS) k_init(Ws w) {
  const int64_t n = w.n;
  const int64_t end = (w.order_mapped && w.max_rounds == 0) ? w.iso_start : n;
  __shared__ int s_hist[HLDS];
  for (int i = threadIdx.x; i < HLDS; i += BS) s_hist[i] = 0;
  __syncthreads();
  for (int64_t v = (int64_t)blockIdx.x * BS + threadIdx.x; v < end; v += (int64_t)gridDim.x * BS) {
    if (!w.order_mapped && w.state[v] != ORDER_SEEN) set_error(w.ctrl, ERR_PERM);  // no entry of pi names v
    w.lab[v] = INF;
    if (v >= w.iso_start) continue;
    w.state[v] = UNCL;
    w.flag[v] = 0;
    w.ub[v] = (int32_t)(w.off[v + 1] - w.off[v]);
    if (w.start_exact) hist_add(s_hist, w.hist, w.ub[v], 1);
    if (v < w.low_start) {  // degree >= DSW: a bound bucket entry
      const int k = level_of(w.ub[v]);
      w.lvl[w.lvl_off[k] + (v - w.lvl_first[k])] = (int32_t)v;
    }
  }
  __syncthreads();
  if (w.start_exact)
    for (int i = threadIdx.x; i < HLDS; i += BS)
      if (s_hist[i]) atomicAdd(&w.hist[i], s_hist[i]);
  const int64_t nw = (n + 31) / 32;
  for (int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x; i < nw; i += (int64_t)gridDim.x * BS) {
    const int64_t rem = n - i * 32;
    w.unc[i] = rem >= 32 ? 0xFFFFFFFFu : ((1u << rem) - 1u);
  }
  Ctrl *c = w.ctrl;
  if (blockIdx.x == 0) {
    if (threadIdx.x < NLVL) c->lvl_cnt[threadIdx.x] = w.lvl_cnt0[threadIdx.x];
    if (threadIdx.x == 0) {
      c->n_rem = n;
      c->n_start = n;
      c->done = (n == 0);
      c->phase = w.start_exact ? PHASE_EXACT : PHASE_LAZY;
      c->feat_eps = (float)w.eps;
      // an active vertex claims a row of neighbours; with exact degrees, each of their rows is peeled
      const float deg = w.iso_start > 0 ? (float)w.off[n] / (float)w.iso_start : 0.f;
      c->rate = w.start_exact ? deg + deg * deg : deg;
    }
  }
}

// ------------------------------------------------------- remaining degrees --
// After the claims a round is in one of three states, and the same two kernels
// serve them: the lazy Delta search has a pass to run (dsearch), the run
// switches to exact degrees, or it keeps exact degrees and peels.  A slot
// runs one pass; where the search needs another, k_close leaves the round
// open and the next slot's earlier kernels return at once.  R-MAT 26 needs a
// second pass in 6 of 96 lazy rounds, a third in none, and switches once: as
// kernels of their own these returned idle in nearly every round, at 5 us
// each, and peeling too until the switch: 7 of a round's 13 launches and 36
// of its 95 us.

// Pass h.pass: the live entries with bound >= L, found in the levels level(L)
// .. top (a bound can be stale above the current Delta).  At the switch: the
// unclustered rows of degree >= DSW (their accumulators live in the
// active-list weights, free at this point of the round).
__global__ void __launch_bounds__(BS) k_candidates(Ws w) {
  Ctrl *c = w.ctrl;
  const CtrlHead h = ctrl_head(c);
  if (idle(h, ST_DELTA) || h.phase != PHASE_LAZY) return;
  const int pass = h.pass;
  const DSearch s = dsearch(&h, pass);
  constexpr int PER = 4;  // entries of a thread in flight: each is a chain of three dependent reads
  __shared__ StageBuf<(PER + 1) * BS> sb;
  __shared__ int64_t s_base[NLVL + 1];
  if (s.switching) {
    unsigned long long *xacc = (unsigned long long *)w.awork;
    stage_init(sb);
    const int64_t n = w.low_start;  // lower-degree rows are counted by id in count_exact
    const int64_t per = ((n + gridDim.x - 1) / gridDim.x + BS - 1) / BS * BS;
    const int64_t v0 = (int64_t)blockIdx.x * per, v1 = v0 + per < n ? v0 + per : n;
    for (int64_t vb = v0; vb < v1; vb += BS) {
      const int64_t v = vb + threadIdx.x;
      if (v < v1 && unc_bit(w.unc, (int32_t)v)) {
        const int64_t d = w.off[v + 1] - w.off[v];
        w.xend[v] = w.off[v];  // count_exact appends the row's unclustered neighbours
        if (d > 0) stage_push(sb, (int32_t)v, (int32_t)d);
      }
      if (vb + BS < v1 && staged_over(sb)) stage_flush(sb, &c->x_pack, w.xlist, w.xwork, xacc);
    }
    stage_flush(sb, &c->x_pack, w.xlist, w.xwork, xacc);
    return;
  }
  if (!s.pending) return;
  const int kL = level_of(s.L < DSW ? DSW : s.L);
  if (threadIdx.x < 64) {  // where each level's entries start among those of kL and above
    const int k = threadIdx.x;
    int64_t cnt = 0;
    if (k >= kL && k < NLVL) {
      const int64_t cap = w.lvl_off[k + 1] - w.lvl_off[k], have = c->lvl_cnt[k];
      cnt = have < cap ? have : cap;
    }
    const int64_t inc = wave_incl_scan(cnt);
    if (k < NLVL) s_base[k] = inc - cnt;
    if (k == NLVL) s_base[k] = inc;
  }
  stage_init(sb);
  const int64_t tot = s_base[NLVL];
  int32_t *list = w.rlist + pass * w.rcap;
  int64_t *work = w.rwork + pass * w.rcap;
  unsigned long long *acc = w.racc + pass * w.rcap;
  // a contiguous share of the entries per workgroup
  const int64_t per = ((tot + gridDim.x - 1) / gridDim.x + BS - 1) / BS * BS;
  const int64_t e0 = (int64_t)blockIdx.x * per, e1 = e0 + per < tot ? e0 + per : tot;
  for (int64_t i0 = e0; i0 < e1; i0 += PER * BS) {
    int32_t v[PER], x[PER];
    int lv[PER];
#pragma unroll
    for (int q = 0; q < PER; q++) {
      const int64_t i = i0 + q * BS + threadIdx.x;
      v[q] = -1;
      lv[q] = kL;
      if (i < e1) {
        while (lv[q] < NLVL - 1 && i >= s_base[lv[q] + 1]) lv[q]++;
        v[q] = w.lvl[w.lvl_off[lv[q]] + (i - s_base[lv[q]])];
      }
    }
#pragma unroll
    for (int q = 0; q < PER; q++) x[q] = v[q] >= 0 ? w.ub[v[q]] : 0;
#pragma unroll
    for (int q = 0; q < PER; q++)
      if (v[q] >= 0 && x[q] >= s.L && level_of(x[q]) == lv[q] && unc_bit(w.unc, v[q]))  // live entry, inside the band
        stage_push(sb, v[q], (int32_t)(w.rend[v[q]] - w.off[v[q]]));
    if (i0 + PER * BS < e1 && staged_over(sb)) stage_flush(sb, &c->r_pack[pass], list, work, acc);
  }
  stage_flush(sb, &c->r_pack[pass], list, work, acc);
}

struct RescanLds {
  int cnt[TW];
  int32_t mv[TW];
  int8_t mvk[TW];
  int mvn[NLVL], mvbase[NLVL];
  int mx, nmv;
};
struct ExactLds {
  int cnt[TW];
  int64_t base[TW];  // where this tile's share of its row j goes in xcol
  int hist[HLDS];
};
struct PeelLds {
  int hist[HLDS];
  unsigned atom;
};

// Exact remaining degrees of the pass's candidates; the new bounds move
// entries down the levels; the pass maximum goes to d_max.
__device__ __forceinline__ void rescan(const Ws &w, Ctrl *c, const CtrlHead &h, WalkLds &wl, RescanLds &L) {
  for (int i = threadIdx.x; i < TW; i += BS) L.cnt[i] = 0;
  if (threadIdx.x < NLVL) L.mvn[threadIdx.x] = 0;
  if (threadIdx.x == 0) {
    L.mx = 0;
    L.nmv = 0;
  }
  __syncthreads();
  const int pass = h.pass;
  unsigned long long rp = 0;
#pragma unroll
  for (int j = 0; j < DITER; j++) rp |= j == pass ? h.r_pack[j] : 0;  // (no index of a register array)
  const int64_t cnt = pk_cnt(rp) < w.rcap ? pk_cnt(rp) : w.rcap;
  unsigned long long *ra = w.racc + pass * w.rcap;
  auto finalize = [&](int32_t v, int r) {
    const int32_t old = w.ub[v];
    w.ub[v] = r;
    atomicMax(&L.mx, r);
    const int kn = r >= DSW ? level_of(r) : -1;
    if (kn >= 0 && kn != level_of(old)) {
      const int p = atomicAdd(&L.nmv, 1);
      L.mv[p] = v;
      L.mvk[p] = (int8_t)kn;
      atomicAdd(&L.mvn[kn], 1);
    }
  };
  lb_walk_in(
      wl, w.rlist + pass * w.rcap, w.rwork + pass * w.rcap, cnt, pk_work(rp), w.off, w.rend, w.col, nullptr, nullptr,
      [&](Items &it) {
#pragma unroll
        for (int k = 0; k < IPT; k++)
          if ((it.edge >> k & 1) && unc_bit(w.unc, it.u[k])) atomicAdd(&L.cnt[it.ent[k]], 1);
      },
      [&](int j, int64_t slot, int32_t v, int32_t deg, int64_t covered) {
        const int cj = L.cnt[j];
        L.cnt[j] = 0;
        int total = cj;
        if (covered == deg || row_combine(ra, slot, cj, covered, deg, &total)) finalize(v, total);
      },
      [&]() {
        // this tile's level moves: one reservation per level, then the writes
        __syncthreads();
        if (threadIdx.x < NLVL && L.mvn[threadIdx.x]) {
          const int k = threadIdx.x;
          L.mvbase[k] = (int)atomicAdd(&c->lvl_cnt[k], (unsigned)L.mvn[k]);
        }
        __syncthreads();
        const int nmv = L.nmv;
        for (int p = threadIdx.x; p < nmv; p += BS) {
          const int k = L.mvk[p];
          int q = 0;  // rank among this tile's earlier moves to the same level
          for (int x = 0; x < p; x++) q += (L.mvk[x] == k);
          const int64_t pos = (int64_t)L.mvbase[k] + q;
          if (pos < w.lvl_off[k + 1] - w.lvl_off[k]) w.lvl[w.lvl_off[k] + pos] = L.mv[p];
          else set_error(c, ERR_OVERFLOW);
        }
        __syncthreads();
        if (threadIdx.x < NLVL) L.mvn[threadIdx.x] = 0;
        if (threadIdx.x == 0) L.nmv = 0;
      });
  __syncthreads();
  if (threadIdx.x == 0 && L.mx > 0) atomicMax(&c->d_max[pass], L.mx);
}

// The switch: every unclustered vertex's unclustered neighbours are counted
// into ub and the histogram: the listed rows edge-balanced, the rows of
// degree below DSW (ids low_start .. iso_start, by falling level) one lane per
// row, so a wave's rows are of about one length and no search or barrier is
// needed.  The unclustered neighbours found are also written to the compacted
// rows (xcol, from the start of each row's slot; xend = where the row ends):
// every vertex the exact rounds walk is unclustered now, and its neighbours
// clustered before now can never count again.  A listed row's tiles reserve
// their shares of the slot with one atomic each, so its entries are in no
// particular order.
__device__ __forceinline__ void count_exact(const Ws &w, Ctrl *c, const CtrlHead &h, WalkLds &wl, ExactLds &L) {
  for (int i = threadIdx.x; i < TW; i += BS) L.cnt[i] = 0;
  for (int i = threadIdx.x; i < HLDS; i += BS) L.hist[i] = 0;
  __syncthreads();
  unsigned long long *xacc = (unsigned long long *)w.awork;
  const unsigned long long xp = h.x_pack;
  auto finalize = [&](int32_t v, int r) {
    w.ub[v] = r;
    if (r > 0 && r < HLDS) atomicAdd(&L.hist[r], 1);
    else if (r >= HLDS) atomicAdd(&w.hist[r], 1);
  };
  // this thread's unclustered neighbours in the current tile: the neighbour,
  // its row's slot in the tile, and its index in the tile's share of the row
  int32_t pu[IPT];
  int pj[IPT], pl[IPT];
  unsigned pending = 0;
  lb_walk_in(
      wl, w.xlist, w.xwork, pk_cnt(xp), pk_work(xp), w.off, w.off + 1, w.col, nullptr, nullptr,
      [&](Items &it) {
        pending = 0;
#pragma unroll
        for (int k = 0; k < IPT; k++)
          if ((it.edge >> k & 1) && unc_bit(w.unc, it.u[k])) {
            pu[k] = it.u[k];
            pj[k] = it.ent[k];
            pl[k] = atomicAdd(&L.cnt[it.ent[k]], 1);
            pending |= 1u << k;
          }
      },
      [&](int j, int64_t slot, int32_t v, int32_t deg, int64_t covered) {
        const int cj = L.cnt[j];
        L.cnt[j] = 0;
        L.base[j] = cj > 0 ? (int64_t)atomicAdd((unsigned long long *)&w.xend[v], (unsigned long long)cj) : 0;
        int total = cj;
        if (covered == deg || row_combine(xacc, slot, cj, covered, deg, &total)) finalize(v, total);
      },
      [&]() {
        __syncthreads();  // every row of the tile has its share reserved
#pragma unroll
        for (int k = 0; k < IPT; k++)
          if (pending >> k & 1) w.xcol[L.base[pj[k]] + pl[k]] = pu[k];
      });
  static_assert(DSW <= HLDS, "a lower-degree row's count fits the LDS histogram");
  int64_t scanned = 0;
  for (int64_t v = w.low_start + (int64_t)blockIdx.x * BS + threadIdx.x; v < w.iso_start;
       v += (int64_t)gridDim.x * BS) {
    if (!unc_bit(w.unc, (int32_t)v)) continue;
    const int64_t s0 = w.off[v];
    const int d = (int)(w.off[v + 1] - s0);
    int r = 0;
    for (int j = 0; j < d; j += 4) {
      int32_t u[4];
#pragma unroll
      for (int q = 0; q < 4; q++) u[q] = j + q < d ? w.col[s0 + j + q] : -1;
#pragma unroll
      for (int q = 0; q < 4; q++)
        if (u[q] >= 0 && unc_bit(w.unc, u[q])) w.xcol[s0 + r++] = u[q];
    }
    scanned += d;
    w.ub[v] = r;
    w.xend[v] = s0 + r;
    if (r > 0) atomicAdd(&L.hist[r], 1);
  }
  const int64_t wsc = wave_sum(scanned);
  if (lane_id() == 0 && wsc) atomicAdd(&c->x_low[(blockIdx.x * (BS / 64) + wave_id()) & 63], (unsigned long long)wsc);
  __syncthreads();
  for (int i = threadIdx.x; i < HLDS; i += BS)
    if (L.hist[i]) atomicAdd(&w.hist[i], L.hist[i]);
}

// Exact phase: every unclustered neighbour of a newly clustered vertex loses
// one remaining degree; the degree histogram follows (low bins per workgroup).
__device__ __forceinline__ void peel(const Ws &w, Ctrl *c, const CtrlHead &h, WalkLds &wl, PeelLds &L) {
  for (int i = threadIdx.x; i < HLDS; i += BS) L.hist[i] = 0;
  if (threadIdx.x == 0) L.atom = 0;
  __syncthreads();
  const unsigned long long pp = h.p_pack;
  lb_walk_in(wl, w.plist, w.pwork, pk_cnt(pp), pk_work(pp), w.off, round_end(w, h.phase), round_col(w, h.phase),
             nullptr, nullptr, [&](Items &it) {
#pragma unroll
    for (int k = 0; k < IPT; k++)
      if (it.vert >> k & 1) hist_add(L.hist, w.hist, w.ub[it.v[k]], -1);  // the vertex leaves
    bool un[IPT];
#pragma unroll
    for (int k = 0; k < IPT; k++) un[k] = (it.edge >> k & 1) && unc_bit(w.unc, it.u[k]);
    unsigned dec = 0;
#pragma unroll
    for (int k = 0; k < IPT; k++)
      if (un[k]) {
        const int32_t old = atomicSub(&w.ub[it.u[k]], 1);
        hist_add(L.hist, w.hist, old, -1);
        hist_add(L.hist, w.hist, old - 1, 1);
        dec++;
      }
    if (dec) atomicAdd(&L.atom, dec);
  });
  __syncthreads();
  for (int i = threadIdx.x; i < HLDS; i += BS)
    if (L.hist[i]) atomicAdd(&w.hist[i], L.hist[i]);
  if (threadIdx.x == 0 && L.atom) atomicAdd(&c->spread_atom[blockIdx.x & 63], (unsigned long long)L.atom);
}

__global__ void __launch_bounds__(BS) k_degrees(Ws w) {
  Ctrl *c = w.ctrl;
  const CtrlHead h = ctrl_head(c);
  __shared__ WalkLds wl;
  __shared__ union {
    RescanLds rescan;
    ExactLds exact;
    PeelLds peel;
  } L;
  if (h.phase == PHASE_EXACT) {
    if (!idle(h, ST_CLASSIFY)) peel(w, c, h, wl, L.peel);
    return;
  }
  if (idle(h, ST_DELTA)) return;
  const DSearch s = dsearch(&h, h.pass);
  if (s.pending) rescan(w, c, h, wl, L.rescan);
  else if (s.switching) count_exact(w, c, h, wl, L.exact);
}

// ------------------------------------------------------------- select -----
// Tile status word: bits 63..62 = 1 (aggregate) or 2 (inclusive prefix),
// bits 61..0 = value.  Tiles are handed out in order by an atomic counter, so
// a tile only ever waits for tiles that are already being processed.  The
// word carries its value with its flag, so it is read and written with
// relaxed device-scope atomics: nothing else needs ordering against it.  (A
// release or acquire at device scope would write back or invalidate the
// whole L2 of the XCD each time; the select_done flag is relaxed for the
// same reason, and r_last, written before it, is read after the kernel.)

// Decoupled look-back by one wave: lane l reads the status of tile j - l, so
// each step covers 64 predecessors; the walk stops at the nearest inclusive
// prefix.  Called by all 64 lanes of a wave; returns the exclusive prefix.
__device__ inline long long lookback(const Ws &w, unsigned t) {
  long long excl = 0;
  long long j = (long long)t - 1;
  unsigned spins = 0;
  const int l = lane_id();
  while (j >= 0) {
    const long long idx = j - l;
    const unsigned long long s = idx >= 0 ? ld_rlx(&w.tstat[idx]) : (2ull << 62);
    const unsigned flag = (unsigned)(s >> 62);
    const unsigned long long incl = __ballot(flag == 2);
    const unsigned long long notready = __ballot(flag == 0);
    const int first = incl ? __ffsll((long long)incl) - 1 : 64;  // nearest inclusive prefix
    const unsigned long long need = first < 63 ? ((2ull << first) - 1) : ~0ull;
    if (notready & need) {  // a nearer predecessor has not published yet
      if (++spins > (1u << 22)) {
        if (l == 0) set_error(w.ctrl, ERR_NO_PROGRESS);
        return excl;
      }
      __builtin_amdgcn_s_sleep(1);
      continue;
    }
    const long long val = (l <= first) ? (long long)(s & ((1ull << 62) - 1)) : 0;
    excl += wave_sum((int64_t)val);
    if (first < 64) break;
    j -= 64;
  }
  return excl;
}

// The positions of this thread's slots marked in `act` hold this round's
// active vertices (vv[k] at position base + k).  An active vertex with no
// unclustered neighbour (degree 0, or an exact remaining degree of 0) is a
// center that claims nobody and that no other active vertex can see: it is
// settled here and never listed.  Its label stays unset; k_finalize makes it
// its own center (an isolated vertex once the run is complete -- a partial
// run labels the isolated vertices it reaches -- or a vertex with its bit
// cleared and no label).  The others go to the active list with their row
// info.  Collective: every thread of the workgroup calls it.
__device__ inline void activate(const Ws &w, Ctrl *c, const int32_t vv[SIPT], unsigned act, int64_t base, bool exact,
                                const int64_t *rend,
                                int64_t *sh, unsigned long long *s_base) {
  int64_t wsum = 0;
  int cnt = 0, lone = 0;
  unsigned clears = 0;
  unsigned listed = 0;
  int32_t wt[SIPT];
  int64_t rs[SIPT];
#pragma unroll
  for (int k = 0; k < SIPT; k++) {
    wt[k] = 0;
    rs[k] = 0;
    if (act & (1u << k)) {
      const int32_t v = vv[k];
      if (v >= w.iso_start) {
        if (w.max_rounds > 0) w.lab[v] = (int32_t)(base + k);  // a partial run must tell it apart
        lone++;
      } else if (exact && w.ub[v] == 0) {
        atomicAnd(&w.unc[v >> 5], ~(1u << (v & 31)));
        lone++;
        clears++;
      } else {
        rs[k] = w.off[v];
        wt[k] = (int32_t)(rend[v] - rs[k]);
        listed |= 1u << k;
        cnt++;
        wsum += wt[k];
      }
    }
  }
  int64_t wtot, ctot;
  const int64_t wpre = wg_excl_scan<SEL_BS>(wsum, &wtot, sh);
  // listed count in the low half, settled count above (a tile holds fewer than 2^16 of both)
  int both;
  const int cpre = wg_excl_scan<SEL_BS>(cnt | lone << 16, &both, (int *)sh) & 0xFFFF;
  const int64_t ltot = both >> 16;
  ctot = both & 0xFFFF;
  if (threadIdx.x == 0 && ctot > 0) *s_base = atomicAdd(&c->a_pack, pk(wtot, ctot));
  if (threadIdx.x == 0 && ltot > 0) atomicAdd(&c->spread_lone[blockIdx.x & 63], (unsigned long long)ltot);
  const int64_t wc = wave_sum((int64_t)clears);  // every lane takes part in the sum
  if (lane_id() == 0 && wc) atomicAdd(&c->spread_atom[blockIdx.x & 63], (unsigned long long)wc);
  __syncthreads();
  if (ctot > 0) {
    int64_t slot = pk_cnt(*s_base) + cpre, wpos = pk_work(*s_base) + wpre;
#pragma unroll
    for (int k = 0; k < SIPT; k++) {
      if (listed & (1u << k)) {
        const int32_t v = vv[k];
        w.state[v] = ACTIVE;
        // the rank of an active vertex, as its neighbours will ask for it:
        // ClusterWild! keeps it as the label (every active vertex is a center)
        if (w.algo == ALGO_CW) w.lab[v] = (int32_t)(base + k);
        else w.rank[v] = (int32_t)(base + k);
        w.alist[slot] = v;
        w.awork[slot] = wpos;
        w.ainfo[slot] = RowInfo{rs[k], wt[k], (int32_t)(base + k)};
        slot++;
        wpos += wt[k];
      }
    }
  }
}

// An unclustered-or-isolated mask of this thread's slots from base on (an
// isolated vertex's bit is never cleared: only its own position, which the
// cursor passes once, asks whether it is clustered).
__device__ inline unsigned load_slots(const Ws &w, int64_t base, int64_t end, int32_t vv[SIPT]) {
  unsigned un = 0;
#pragma unroll
  for (int k = 0; k < SIPT; k++) {
    const int64_t p = base + k;
    vv[k] = p < end ? w.order[p] : 0;
  }
#pragma unroll
  for (int k = 0; k < SIPT; k++) {
    const int64_t p = base + k;
    if (p < end && (vv[k] >= w.iso_start || unc_bit(w.unc, vv[k]))) un |= 1u << k;
  }
  return un;
}

// The next B_i unclustered vertices of pi (Algorithm 2's active set).
__global__ void __launch_bounds__(SEL_BS) k_select(Ws w) {
  Ctrl *c = w.ctrl;
  const CtrlHead h = ctrl_head(c);
  if (idle(h, ST_SELECT)) return;
  __shared__ unsigned s_tile;
  __shared__ int s_stop;
  __shared__ long long s_excl;
  __shared__ int64_t sh[SEL_BS / 64 + 1];
  __shared__ unsigned long long s_base;
  const long long B = h.b, cur0 = h.cursor;
  const bool exact = h.phase == PHASE_EXACT;
  const int64_t n = w.n;
  // Workgroups this round can use: B_i unclustered are spread over the
  // positions ahead with density n_i / (n - cursor); extra groups would only
  // grab tiles past the end of the active set.
  const long long ahead = n - cur0, n_i = h.n_rem > 0 ? h.n_rem : 1;
  const long long need_pos = (long long)((double)B * (double)ahead / (double)n_i) + TSEL;
  if ((long long)blockIdx.x > need_pos / TSEL) return;
  for (bool first = true;; first = false) {
    if (threadIdx.x == 0) {  // (a first tile is taken without a look at the flag: one dependent read less)
      s_stop = first ? 0 : ld_rlx(&c->select_done);
      if (!s_stop) s_tile = atomicAdd(&c->tile_counter, 1u);
    }
    __syncthreads();
    if (s_stop) break;
    const unsigned t = s_tile;
    if ((int64_t)t >= w.tstat_cap) {  // cannot happen while B <= n_rem
      if (threadIdx.x == 0) set_error(c, ERR_OVERFLOW);
      break;
    }
    const int64_t base = cur0 + (int64_t)t * TSEL + (int64_t)threadIdx.x * SIPT;
    int32_t vv[SIPT];
    const unsigned un = load_slots(w, base, n, vv);
    int64_t agg;
    int found;
    const int mine = wg_excl_scan<SEL_BS>((int)__popc(un), &found, (int *)sh);
    agg = found;
    if (threadIdx.x < 64) {  // wave 0 publishes and looks back
      long long excl = 0;
      if (t == 0) {
        if (threadIdx.x == 0) st_rlx(&w.tstat[0], (2ull << 62) | (unsigned long long)agg);
      } else {
        if (threadIdx.x == 0) st_rlx(&w.tstat[t], (1ull << 62) | (unsigned long long)agg);
        excl = lookback(w, t);
        if (threadIdx.x == 0) st_rlx(&w.tstat[t], (2ull << 62) | (unsigned long long)(excl + agg));
      }
      if (threadIdx.x == 0) s_excl = excl;
    }
    __syncthreads();
    const long long excl = s_excl;
    // the first (B - excl) unclustered positions of this tile are active
    unsigned act = 0;
    long long r = excl + mine;
#pragma unroll
    for (int k = 0; k < SIPT; k++) {
      if (un & (1u << k)) {
        if (r < B) {
          act |= 1u << k;
          if (r == B - 1) {
            c->r_last = base + k;
            st_rlx(&c->select_done, 1);
          }
        }
        r++;
      }
    }
    activate(w, c, vv, act, base, exact, round_end(w, h.phase), sh, &s_base);
    if (excl + agg >= B) break;
    __syncthreads();
  }
}

// The practical schedule's active set: the unclustered vertices among the
// next B_i positions of pi (Binomial batches over the unprocessed suffix).
// No prefix count is needed, so tiles are dealt statically.
__global__ void __launch_bounds__(SEL_BS) k_select_range(Ws w) {
  Ctrl *c = w.ctrl;
  const CtrlHead h = ctrl_head(c);
  if (idle(h, ST_SELECT)) return;
  __shared__ int64_t sh[SEL_BS / 64 + 1];
  __shared__ unsigned long long s_base;
  const int64_t cur0 = h.cursor;
  const int64_t end = cur0 + h.b < w.n ? cur0 + h.b : w.n;
  for (int64_t t = blockIdx.x; cur0 + t * TSEL < end; t += gridDim.x) {
    const int64_t base = cur0 + t * TSEL + (int64_t)threadIdx.x * SIPT;
    int32_t vv[SIPT];
    const unsigned un = load_slots(w, base, end, vv);
    activate(w, c, vv, un, base, false, round_end(w, h.phase), sh, &s_base);
    __syncthreads();
  }
}

// -------------------------------------------------------------- elect -----

__global__ void __launch_bounds__(BS) k_elect(Ws w) {
  Ctrl *c = w.ctrl;
  const CtrlHead h = ctrl_head(c);
  if (idle(h, ST_ELECT)) return;
  const unsigned long long ap = h.a_pack;
  lb_walk(w.alist, w.awork, pk_cnt(ap), pk_work(ap), w.off, round_end(w, h.phase), round_col(w, h.phase), nullptr,
          w.ainfo, [&](Items &it) {
    uint8_t su[IPT];
#pragma unroll
    for (int k = 0; k < IPT; k++) su[k] = (it.edge >> k & 1) ? w.state[it.u[k]] : (uint8_t)UNCL;
#pragma unroll
    for (int k = 0; k < IPT; k++) {
      bool conf = false;
      // an ACTIVE mark is always this round's: C4 settles every active vertex
      if (su[k] == ACTIVE) conf = w.rank[it.u[k]] < it.val[k];  // earlier-ranked active neighbour
      if (conf) w.flag[it.v[k]] = 1;
      const unsigned long long m = __ballot(conf);
      if (m) {
        const int leader = __ffsll((long long)m) - 1;
        unsigned base = 0;
        if (lane_id() == leader) base = atomicAdd(&c->n_cedges, (unsigned)__popcll(m));
        base = __shfl(base, leader, 64);
        if (conf) {
          const int64_t slot = (int64_t)base + __popcll(m & lanemask_lt());
          if (slot < w.cedge_cap) w.cedge[slot] = make_int2(it.v[k], it.u[k]);  // else: rescan rows
        }
      }
    }
  });
}

// Roots (no earlier active neighbour) are centers at once; the rest wait.
__global__ void __launch_bounds__(BS) k_classify(Ws w) {
  Ctrl *c = w.ctrl;
  const CtrlHead h = ctrl_head(c);
  if (idle(h, ST_CLASSIFY)) return;
  __shared__ StageBufI<2 * BS> sb;
  stage_init(sb);
  const int64_t na = pk_cnt(h.a_pack);
  const int64_t per = ((na + gridDim.x - 1) / gridDim.x + BS - 1) / BS * BS;
  const int64_t a0 = (int64_t)blockIdx.x * per, a1 = a0 + per < na ? a0 + per : na;
  for (int64_t ib = a0; ib < a1; ib += BS) {
    const int64_t i = ib + threadIdx.x;
    int32_t a = 0;
    bool blocked = false;
    if (i < a1) {
      a = w.alist[i];
      blocked = w.flag[a] != 0;
      if (!blocked) {
        const RowInfo ri = w.ainfo[i];
        w.state[a] = CENTER;
        w.lab[a] = ri.rank;
        stage_push_info(sb, a, ri);
      }
    }
    const unsigned long long m = __ballot(blocked);  // blocked vertices are rare
    if (m) {
      const int leader = __ffsll((long long)m) - 1;
      unsigned base = 0;
      if (lane_id() == leader) base = atomicAdd(&c->n_blocked, (unsigned)__popcll(m));
      base = __shfl(base, leader, 64);
      if (blocked) w.blist[base + __popcll(m & lanemask_lt())] = a;
    }
    if (ib + BS < a1 && staged_over(sb)) stage_flush(sb, &c->c_pack, w.clist, w.cwork, nullptr, w.cinfo, sb.info);
  }
  stage_flush(sb, &c->c_pack, w.clist, w.cwork, nullptr, w.cinfo, sb.info);
}

// One workgroup settles the blocked vertices: the greedy MIS of G[A] in pi
// order restricted to them (rule 1).  A blocked vertex is a non-center as soon
// as an earlier active neighbour is a center, and a center once every earlier
// active neighbour is a non-center.
constexpr int RBS = 1024;

__device__ inline void mark_decided(Ws &w, int32_t i, unsigned *tail) {
  const unsigned q = atomicAdd(tail, 1u);
  w.bq[q] = i;
}

// The blocked vertices as decided (1: center): centers join the center list.
template <class F>
__device__ __forceinline__ void promote_decided(const Ws &w, Ctrl *c, int64_t nb, const int64_t *rend, F &&decided) {
  for (int64_t i0 = 0; i0 < nb; i0 += RBS) {
    const int64_t i = i0 + threadIdx.x;
    int32_t a = 0;
    bool promote = false;
    if (i < nb) {
      a = w.blist[i];
      const int d = decided(i);
      if (d == 1) promote = true;
      else w.state[a] = NONCENTER;
      if (d == 0) set_error(c, ERR_NO_PROGRESS);  // every blocked vertex is decided by now
    }
    RowInfo ri{0, 0, 0};
    if (promote) {
      ri = RowInfo{w.off[a], (int32_t)(rend[a] - w.off[a]), w.rank[a]};
      w.state[a] = CENTER;
      w.lab[a] = ri.rank;
    }
    wave_append_info(promote, a, ri, &c->c_pack, w.clist, w.cwork, w.cinfo);
  }
}

// Up to RES_EDGES conflict edges: every thread holds its share in registers
// (the blocked vertex and the earlier one it waits for as indices of the
// blocked list) and settles them on words in LDS (settle_edges), where the
// queue below pays a chain of six reads and atomics in the L2 per level.  R-MAT
// 22 under the learned policy 3.65 -> 3.52 ms, C4 7.64 -> 7.44 ms; a path of
// 100 K in its own order, whose rounds are one chain: 113 ms by the queue, 542
// with two barriers a level, 74 so.  The limit is what fits the LDS.
constexpr int RES_EPT = 32, RES_EDGES = RBS * RES_EPT;
__device__ void resolve_edges(const Ws &w, Ctrl *c, int nb, int ne, const int64_t *rend) {
  __shared__ int word[RES_EDGES];  // (a blocked vertex has an edge)
  const int tid = threadIdx.x;
  for (int i = tid; i < nb; i += RBS) {
    w.bpos[w.blist[i]] = i;
    word[i] = 0;
  }
  __syncthreads();
  unsigned ed[RES_EPT];  // vertex | (earlier one + 1, 0: a center) << 16
  unsigned open = 0;
  static_assert(RES_EDGES <= 1 << 15 && RES_EDGES < RES_GONE, "an index and a zero fit 16 bits");
  constexpr int CH = 8;  // in flight
#pragma unroll
  for (int k0 = 0; k0 < RES_EPT; k0 += CH) {
    if (k0 * RBS >= ne) break;
    int2 e[CH];
    int32_t ia[CH], iu[CH];
    uint8_t su[CH];
#pragma unroll
    for (int k = 0; k < CH; k++) {
      const int x = (k0 + k) * RBS + tid;
      e[k] = x < ne ? w.cedge[x] : make_int2(-1, -1);
    }
#pragma unroll
    for (int k = 0; k < CH; k++) {
      ia[k] = e[k].x >= 0 ? w.bpos[e[k].x] : 0;
      su[k] = e[k].x >= 0 ? w.state[e[k].y] : (uint8_t)CENTER;
      iu[k] = e[k].x >= 0 ? w.bpos[e[k].y] : 0;  // (not a position where y is a center)
    }
#pragma unroll
    for (int k = 0; k < CH; k++) {
      ed[k0 + k] = (unsigned)ia[k] | (su[k] == CENTER ? 0u : (unsigned)(iu[k] + 1) << 16);
      if (e[k].x < 0) continue;
      open |= 1u << (k0 + k);
      atomicAdd(&word[ia[k]], 1);
    }
  }
  __syncthreads();
  settle_edges<RES_EPT>(word, open, [&](int k) { return (int)(ed[k] & 0xFFFF); },
                        [&](int k) { return (int)(ed[k] >> 16) - 1; });
  __syncthreads();
  promote_decided(w, c, nb, rend, [&](int64_t i) { return res_decision(word[i]); });
}

// The conflict edges are listed: build the dependence graph among the blocked
// vertices (edge (a, u): a waits for u) and settle it from the vertices whose
// earlier neighbours are all decided, level by level.  Every blocked vertex
// enters the queue once, when it is decided, and then walks its later
// neighbours once: O(blocked + conflict edges) work, one barrier per level.
__device__ void resolve_listed(Ws &w, Ctrl *c, int64_t nb, int64_t ne, const int64_t *rend) {
  __shared__ unsigned s_tail;
  __shared__ int64_t sh[RBS / 64 + 1];
  __shared__ int64_t s_carry;
  const int64_t total_dep = ne;  // upper bound of the dependence edges
  if (threadIdx.x == 0) {
    s_tail = 0;
    s_carry = 0;
  }
  for (int64_t i = threadIdx.x; i < nb; i += RBS) {
    w.bpos[w.blist[i]] = (int32_t)i;
    w.bpend[i] = 0;
    w.bdec[i] = 0;
    w.bdep[i] = 0;
  }
  __syncthreads();
  // an earlier neighbour that is a center already (a root) decides a at
  // once; an earlier blocked one is a dependence
  for (int64_t e = threadIdx.x; e < ne; e += RBS) {
    const int2 ed = w.cedge[e];
    const int32_t ia = w.bpos[ed.x];
    if (w.state[ed.y] == CENTER) {
      w.bdec[ia] = 2;
    } else {
      atomicAdd(&w.bpend[ia], 1);
      atomicAdd(&w.bdep[w.bpos[ed.y]], 1);
    }
  }
  __syncthreads();
  // inclusive prefix of the dependents' counts: bdep[i] = end of i's range
  for (int64_t i0 = 0; i0 < nb; i0 += RBS) {
    const int64_t i = i0 + threadIdx.x;
    const int64_t x = i < nb ? w.bdep[i] : 0;
    int64_t tot;
    const int64_t pre = wg_excl_scan<RBS>(x, &tot, sh) + s_carry;
    if (i < nb) w.bdep[i] = (int32_t)(pre + x);
    __syncthreads();
    if (threadIdx.x == 0) s_carry += tot;
    __syncthreads();
  }
  if (s_carry > total_dep) {  // cannot happen: every dependence is a listed edge
    if (threadIdx.x == 0) set_error(c, ERR_OVERFLOW);
    return;
  }
  const int64_t ndep = s_carry;
  // fill from the ends down: afterwards bdep[i] = start of i's range
  for (int64_t e = threadIdx.x; e < ne; e += RBS) {
    const int2 ed = w.cedge[e];
    if (w.state[ed.y] != CENTER) {
      const int32_t slot = atomicSub(&w.bdep[w.bpos[ed.y]], 1) - 1;
      w.bradj[slot] = w.bpos[ed.x];
    }
  }
  __syncthreads();
  for (int64_t i = threadIdx.x; i < nb; i += RBS) {
    if (w.bdec[i] == 2) {
      mark_decided(w, (int32_t)i, &s_tail);
    } else if (w.bpend[i] == 0) {
      w.bdec[i] = 1;
      mark_decided(w, (int32_t)i, &s_tail);
    }
  }
  __syncthreads();
  int64_t h0 = 0;
  for (int64_t level = 0; level <= nb; level++) {
    const int64_t h1 = s_tail;  // the decided indices this level walks
    __syncthreads();            // every thread has read it before any appends
    if (h0 >= h1) break;
    for (int64_t q = h0 + threadIdx.x; q < h1; q += RBS) {
      const int32_t x = w.bq[q];
      const bool center = w.bdec[x] == 1;
      const int64_t d0 = w.bdep[x], d1 = x + 1 < nb ? w.bdep[x + 1] : ndep;
      for (int64_t d = d0; d < d1; d++) {
        const int32_t y = w.bradj[d];
        if (center) {
          if (atomicCAS(&w.bdec[y], 0, 2) == 0) mark_decided(w, y, &s_tail);
        } else if (atomicSub(&w.bpend[y], 1) == 1) {
          if (atomicCAS(&w.bdec[y], 0, 1) == 0) mark_decided(w, y, &s_tail);
        }
      }
    }
    __syncthreads();
    h0 = h1;
  }
  promote_decided(w, c, nb, rend, [&](int64_t i) { return w.bdec[i]; });
}

// Too many conflict edges to list: sweep the rows of the blocked vertices
// until nothing changes (every earlier-ranked unclustered neighbour of an
// active vertex is active).  Each sweep settles at least the lowest-ranked
// undecided vertex.
__device__ void resolve_rows(Ws &w, Ctrl *c, int64_t nb, const int64_t *rend, const int32_t *col) {
  __shared__ int s_any;
  for (int64_t iter = 0; iter <= nb; iter++) {
    if (threadIdx.x == 0) s_any = 0;
    __syncthreads();
    for (int64_t i0 = 0; i0 < nb; i0 += RBS) {
      const int64_t i = i0 + threadIdx.x;
      int32_t a = 0;
      bool promote = false;
      if (i < nb) {
        a = w.blist[i];
        if (w.state[a] == ACTIVE) {
          const int32_t ra = w.rank[a];
          bool center_before = false, undecided_before = false;
          for (int64_t e = w.off[a]; e < rend[a] && !center_before; e++) {
            const int32_t u = col[e];
            if (!unc_bit(w.unc, u)) continue;
            const uint8_t su = w.state[u];
            if ((su == CENTER || su == ACTIVE) && w.rank[u] < ra) {
              if (su == CENTER) center_before = true;
              else undecided_before = true;
            }
          }
          if (center_before) w.state[a] = NONCENTER;
          else if (!undecided_before) promote = true;
          else s_any = 1;
        }
      }
      RowInfo ri{0, 0, 0};
      if (promote) {
        ri = RowInfo{w.off[a], (int32_t)(rend[a] - w.off[a]), w.rank[a]};
        w.state[a] = CENTER;
        w.lab[a] = ri.rank;
      }
      wave_append_info(promote, a, ri, &c->c_pack, w.clist, w.cwork, w.cinfo);
    }
    __syncthreads();
    if (!s_any) break;
  }
}

__global__ void __launch_bounds__(RBS) k_resolve(Ws w) {
  Ctrl *c = w.ctrl;
  const CtrlHead h = ctrl_head(c);
  if (idle(h, ST_CLASSIFY)) return;
  const int64_t nb = h.n_blocked;
  if (nb == 0) return;
  const int64_t ne = h.n_cedges;
  if (ne <= RES_EDGES) resolve_edges(w, c, (int)nb, (int)ne, round_end(w, h.phase));
  else if (ne <= w.cedge_cap) resolve_listed(w, c, nb, ne, round_end(w, h.phase));
  else resolve_rows(w, c, nb, round_end(w, h.phase), round_col(w, h.phase));
  __syncthreads();
  for (int64_t i = threadIdx.x; i < nb; i += RBS) w.flag[w.blist[i]] = 0;
}

// -------------------------------------------------------------- claim -----

constexpr int CLAIM_CAP = 2 * TW;  // staged newly claimed vertices (a tile adds <= TW)

__global__ void __launch_bounds__(BS) k_claim(Ws w) {
  Ctrl *c = w.ctrl;
  const CtrlHead h = ctrl_head(c);
  if (idle(h, ST_CLASSIFY)) return;
  const bool c4 = w.algo == ALGO_C4;
  const unsigned long long lp = c4 ? h.c_pack : h.a_pack;
  const int32_t *list = c4 ? w.clist : w.alist;
  const int64_t *work = c4 ? w.cwork : w.awork;
  const RowInfo *info = c4 ? w.cinfo : w.ainfo;
  __shared__ unsigned s_atom;
  __shared__ IdBuf<CLAIM_CAP> sb;
  if (threadIdx.x == 0) s_atom = 0;
  id_init(sb);
  lb_walk(
      list, work, pk_cnt(lp), pk_work(lp), w.off, round_end(w, h.phase), round_col(w, h.phase), nullptr, info,
      [&](Items &it) {
        bool un[IPT];
#pragma unroll
        for (int k = 0; k < IPT; k++) un[k] = (it.edge >> k & 1) && unc_bit(w.unc, it.u[k]);
        bool elig[IPT];
        int32_t cur[IPT];
#pragma unroll
        for (int k = 0; k < IPT; k++) {
          elig[k] = un[k];
          if (!c4 && un[k] && w.state[it.u[k]] == ACTIVE) {  // ClusterWild! claims Gamma(c) \ A
            elig[k] = false;
            if (w.lab[it.u[k]] < it.val[k]) w.flag[it.v[k]] = 1;  // rule 1 broken (lab = rank here)
          }
          cur[k] = elig[k] ? w.lab[it.u[k]] : 0;  // stale reads are safe: labels only decrease
        }
        unsigned atom = 0;
#pragma unroll
        for (int k = 0; k < IPT; k++) {
          if (elig[k] && it.val[k] < cur[k]) {
            const int32_t old = atomicMin(&w.lab[it.u[k]], it.val[k]);
            atom++;
            if (old == INF) id_push(sb, it.u[k]);  // the newly claimed list
          }
        }
        if (atom) atomicAdd(&s_atom, atom);
      },
      NoEpilogue(),
      [&]() {
        __syncthreads();
        if (sb.cnt > CLAIM_CAP - TW) id_flush(sb, &c->n_pack, w.nlist);
      });
  id_flush(sb, &c->n_pack, w.nlist);
  if (threadIdx.x == 0 && s_atom) atomicAdd(&c->spread_atom[blockIdx.x & 63], (unsigned long long)s_atom);
}

// The newly clustered -- the listed centers (C4's center list, ClusterWild!'s
// active list) and the newly claimed -- leave the unclustered bitmap;
// ClusterWild! conflict marks are counted; the scan tiles of this round are
// forgotten.  In the exact phase the claimed vertices that still had
// unclustered neighbours go to the peel list.  Centers do not: every
// unclustered neighbour of a center is claimed in the same round (C4 claims
// all of them and no two centers are adjacent; ClusterWild!'s active
// neighbours are centers themselves), so a center's row has nobody left to
// peel; it only leaves the degree histogram.
__global__ void __launch_bounds__(BS) k_clear(Ws w) {
  Ctrl *c = w.ctrl;
  const CtrlHead h = ctrl_head(c);
  if (idle(h, ST_CLASSIFY)) return;
  __shared__ StageBuf<2 * BS> sp;
  __shared__ int s_hist[HLDS];
  for (int i = threadIdx.x; i < HLDS; i += BS) s_hist[i] = 0;
  stage_init(sp);
  const bool cw = w.algo == ALGO_CW, exact = h.phase == PHASE_EXACT;
  const int64_t *rend = round_end(w, h.phase);
  const int64_t nc = pk_cnt(cw ? h.a_pack : h.c_pack);
  const int32_t *centers = cw ? w.alist : w.clist;
  const int64_t nn = nc + pk_cnt(h.n_pack);
  unsigned conf = 0;
  const int64_t per = ((nn + gridDim.x - 1) / gridDim.x + BS - 1) / BS * BS;
  const int64_t i0 = (int64_t)blockIdx.x * per, i1 = i0 + per < nn ? i0 + per : nn;
  for (int64_t ib = i0; ib < i1; ib += BS) {
    const int64_t i = ib + threadIdx.x;
    if (i < i1) {
      const bool center = i < nc;
      const int32_t u = center ? centers[i] : w.nlist[i - nc];
      atomicAnd(&w.unc[u >> 5], ~(1u << (u & 31)));
      if (cw && center) {
        w.state[u] = CENTER;  // an ACTIVE mark is always this round's (k_team relies on it)
        if (w.flag[u]) {
          w.flag[u] = 0;
          conf++;
        }
      }
      if (exact) {
        const int32_t d = w.ub[u];
        if (center) hist_add(s_hist, w.hist, d, -1);
        else if (d > 0) stage_push(sp, u, (int32_t)(rend[u] - w.off[u]));
      }
    }
    if (ib + BS < i1 && staged_over(sp)) stage_flush(sp, &c->p_pack, w.plist, w.pwork);
  }
  stage_flush(sp, &c->p_pack, w.plist, w.pwork);
  const int64_t tiles = (int64_t)h.tile_counter + 1;
  for (int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x; t < tiles && t < w.tstat_cap;
       t += (int64_t)gridDim.x * BS)
    w.tstat[t] = 0;
  if (cw) {
    const int64_t s = wave_sum((int64_t)conf);
    if (lane_id() == 0 && s) atomicAdd(&c->spread_conf[blockIdx.x & 63], (unsigned long long)s);
  }
  if (exact) {
    __syncthreads();
    for (int i = threadIdx.x; i < HLDS; i += BS)
      if (s_hist[i]) atomicAdd(&w.hist[i], s_hist[i]);
  }
}

// Peeling alone, once the run keeps exact degrees for good.
__global__ void __launch_bounds__(BS) k_peel(Ws w) {
  Ctrl *c = w.ctrl;
  const CtrlHead h = ctrl_head(c);
  if (idle(h, ST_CLASSIFY) || h.phase != PHASE_EXACT) return;
  __shared__ WalkLds wl;
  __shared__ PeelLds L;
  peel(w, c, h, wl, L);
}

// -------------------------------------------------------------- close -----
// One wave: record the finished round, find Delta_{i+1}, size the next round.

__global__ void __launch_bounds__(64) k_close(Ws w) {
  Ctrl *c = w.ctrl;
  if (c->done) return;
  if (w.team) {  // the next k_team starts from zeroed counters, also where the round goes on: it ends the slot by them
    unsigned *t = reinterpret_cast<unsigned *>(w.team);
    for (int i = threadIdx.x; i < (int)(sizeof(TeamCtl) / sizeof(unsigned)); i += 64) t[i] = 0;
  }
  if (c->has_round && c->phase == PHASE_LAZY && w.policy != POL_BINOMIAL && !c->error) {
    const int pass = c->pass;  // run by this slot, unless it switched
    if (dsearch(c, pass).pending) {
      const DSearch s = dsearch(c, pass + 1);
      if (s.pending || s.switching) {  // the round goes on in the next slot
        if (threadIdx.x == 0) {
          c->pass = (int8_t)(pass + 1);
          c->stage = ST_DELTA;
          if (!w.team) {
            const int slots = c->slots + 1;
            c->slots = slots;
            if (w.progress)
              __hip_atomic_store(w.progress, (unsigned long long)(unsigned)slots, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_SYSTEM);
          }
        }
        return;
      }
    }
  }
  const long long now = (long long)wall_clock64();
  long long lone = 0;  // centers settled by k_select
  long long xlow = 0;  // entries of lower-degree rows recounted at the switch
  {  // fold the spread statistics of the round
    const int l = lane_id();
    const unsigned long long sa = (unsigned long long)wave_sum((int64_t)c->spread_atom[l]);
    const unsigned long long sc = (unsigned long long)wave_sum((int64_t)c->spread_conf[l]);
    lone = wave_sum((int64_t)c->spread_lone[l]);
    xlow = wave_sum((int64_t)c->x_low[l]);
    c->spread_atom[l] = 0;
    c->spread_conf[l] = 0;
    c->spread_lone[l] = 0;
    c->x_low[l] = 0;
    if (l == 0) {
      c->sum_atomics += sa;
      c->conflicts += sc;
    }
  }
  long long n_rem = 0, delta = 0, round = 0;
  int done = 0;
  float fconf = 0.f, fclaim = 0.f, feps = 0.f;
  long long prev_delta = 0;
  int slots = 0;
  if (threadIdx.x == 0) {
    prev_delta = c->has_round ? c->delta : w.max_deg;
    if (!w.team) {  // (k_team ends the slots where there is one)
      slots = c->has_round ? c->slots + 1 : 0;
      c->slots = slots;
    } else {
      slots = c->slots;
    }
    if (c->has_round) {
      const int phase_run = c->phase;  // phase the finished round ran in
      const bool c4 = w.algo == ALGO_C4;
      const long long listed = c4 ? pk_cnt(c->c_pack) : pk_cnt(c->a_pack);  // centers in a list
      const long long centers = listed + lone;
      const long long newly = pk_cnt(c->n_pack) + listed + lone;
      const long long conf = c4 ? (long long)c->n_blocked : (long long)c->conflicts;
      if (c->round < w.trace_cap) {
        RoundRec r;
        r.n_i = c->n_start;
        r.delta_i = c->delta;
        r.b_i = c->b;
        r.r_i = c->r_last;
        r.centers = centers;
        r.claimed = newly - centers;
        r.conflicts = conf;
        r.eps_used = c->eps_used;
        r.t_ns = now - c->t_start;
        w.trace[c->round] = r;
      }
      unsigned long long resc = pk_work(c->x_pack) + (unsigned long long)xlow;
      for (int j = 0; j < DITER; j++) resc += pk_work(c->r_pack[j]);
      c->sum_elect += c4 ? (unsigned long long)pk_work(c->a_pack) : 0ull;
      c->sum_claim += c4 ? (unsigned long long)pk_work(c->c_pack) : (unsigned long long)pk_work(c->a_pack);
      c->sum_rescan += resc;
      c->sum_peel += phase_run == PHASE_EXACT ? (unsigned long long)pk_work(c->p_pack) : 0ull;
      c->sum_atomics += (unsigned long long)(pk_cnt(c->n_pack) + listed);  // bitmap clears of the listed
      c->sum_blocked += (unsigned long long)conf;
      c->feat_conf = c->b > 0 ? (float)conf / (float)c->b : 0.f;
      c->feat_claim = c->n_start > 0 ? (float)(newly - centers) / (float)c->n_start : 0.f;
      c->feat_eps = (float)c->eps_used;
      c->rate = c->b > 0 ? (float)(pk_work(c->a_pack) + pk_work(c->p_pack)) / (float)c->b : 0.f;
      c->cursor = c->r_last + 1;
      c->n_rem = c->n_start - newly;
      c->round += 1;
      // every round of the fixed rule clusters a vertex; the practical
      // schedule can have empty rounds and is bounded by its length instead
      if (w.policy != POL_BINOMIAL && c->round > w.n + 1) set_error(c, ERR_NO_PROGRESS);
      if (w.fault_round > 0 && c->round == w.fault_round) set_error(c, ERR_INJECTED);
      long long d = 0;
      if (w.policy == POL_BINOMIAL) {
        d = delta_hat(w, c->round);  // Delta-hat_{i+1}: no remaining degree is kept
      } else if (phase_run == PHASE_LAZY) {  // Delta_{i+1} (lazy search, or the exact histogram below)
        const int pass = c->pass;
        DSearch s = dsearch(c, pass);
        if (s.pending) s = dsearch(c, pass + 1);  // the pass this slot ran
        if (s.switching) {
          c->phase = PHASE_EXACT;
          c->rate = 1e30f;  // peeling starts: its first round is measured on the whole device
        }
        else d = s.delta;
      }
      c->delta = d;
    } else {
      c->delta = w.max_deg;  // Delta_0 (= Delta-hat_0)
    }
    c->has_round = 1;
    c->a_pack = c->c_pack = c->n_pack = c->p_pack = 0;
    c->tile_counter = 0;
    c->select_done = 0;
    c->n_blocked = 0;
    c->n_cedges = 0;
    c->conflicts = 0;
    for (int j = 0; j < DITER; j++) {
      c->r_pack[j] = 0;
      c->d_max[j] = 0;
    }
    c->x_pack = 0;
    c->pass = 0;
    if (c->n_rem <= 0 || c->error || (w.max_rounds > 0 && c->round >= w.max_rounds)) c->done = 1;
    // the practical schedule ends by taking every remaining position, so it
    // cannot run out while vertices are left
    if (!c->done && w.policy == POL_BINOMIAL && c->round >= w.sched_len) {
      set_error(c, ERR_NO_PROGRESS);
      c->done = 1;
    }
    n_rem = c->n_rem;
    delta = c->delta;
    round = c->round;
    done = c->done;
    fconf = c->feat_conf;
    fclaim = c->feat_claim;
    feps = c->feat_eps;
  }
  // exact phase: Delta = highest non-empty histogram bin, at most Delta_i
  int exact = 0;
  long long dprev = 0;
  if (threadIdx.x == 0) {
    exact = c->phase == PHASE_EXACT && c->has_round && !c->done;
    dprev = prev_delta;
  }
  exact = __shfl(exact, 0, 64);
  dprev = __shfl(dprev, 0, 64);
  if (exact) {
    long long found = 0;
    for (long long top = (dprev < w.max_deg ? dprev : w.max_deg); top >= 1 && !found; top -= 64) {
      const long long x = top - lane_id();
      const bool nz = x >= 1 && w.hist[x] > 0;
      const unsigned long long m = __ballot(nz);
      if (m) found = top - (__ffsll((long long)m) - 1);
    }
    if (threadIdx.x == 0) {
      c->delta = found;
      delta = found;
    }
  }
  n_rem = __shfl(n_rem, 0, 64);
  delta = __shfl(delta, 0, 64);
  round = __shfl(round, 0, 64);
  done = __shfl(done, 0, 64);
  fconf = __shfl(fconf, 0, 64);
  fclaim = __shfl(fclaim, 0, 64);
  feps = __shfl(feps, 0, 64);
  if (!done) {
    long long b = 0;
    double eps_used = 0.0;
    int fb = 0;
    next_batch(w, n_rem, delta, round, fconf, fclaim, feps, &b, &eps_used, &fb);
    if (threadIdx.x == 0) {
      if (w.policy == POL_BINOMIAL) {  // positions: the last one taken is known now
        const long long left = w.n - c->cursor;
        if (b > left) b = left;
        c->r_last = c->cursor + b - 1;
      }
      c->b = b;
      c->eps_used = eps_used;
      if (fb) c->fallback = 1;
      c->n_start = n_rem;
      c->t_start = now;
      c->stage = (int8_t)next_stage(w, b, c->cursor, n_rem, c->rate);
    }
  }
  if (threadIdx.x == 0 && w.progress && (!w.team || done)) {
    const unsigned long long p = (unsigned long long)(unsigned)slots | (unsigned long long)(done != 0) << PROGRESS_DONE |
                                 (unsigned long long)(c->phase == PHASE_EXACT) << PROGRESS_EXACT |
                                 (unsigned long long)(c->error != 0) << PROGRESS_ERROR;
    // relaxed: the host acts on this word alone and reads the rest of the
    // state only after the stream has drained
    __hip_atomic_store(w.progress, p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// ----------------------------------------------------------- finalize -----

__global__ void __launch_bounds__(BS) k_finalize(Ws w, int32_t *labels) {
  const int64_t n = w.n;
  // by input id, so the labels are written in order; only the ids that are
  // not isolated look at their internal state
  for (int64_t vin = (int64_t)blockIdx.x * BS + threadIdx.x; vin < n; vin += (int64_t)gridDim.x * BS) {
    const int32_t v = w.perm[vin];
    if (v >= w.iso_start && w.max_rounds == 0) {  // a complete run settled every isolated vertex alone
      labels[vin] = (int32_t)vin;
      continue;
    }
    const int32_t l = w.lab[v];
    // no label: a center k_select settled (an isolated vertex -- a partial
    // run labels those it reached -- or a vertex whose bit it cleared), or
    // still unclustered
    const bool lone = l == INF && v < w.iso_start && !unc_bit(w.unc, v);
    if (lone) {
      labels[vin] = (int32_t)vin;
    } else if (l == INF && w.max_rounds > 0) {
      labels[vin] = -1;  // a partial run left v unclustered
    } else if (l < 0 || (int64_t)l >= n) {
      set_error(w.ctrl, ERR_LABEL);
      labels[vin] = -1;
    } else {
      labels[vin] = w.order_in[l];  // the input id at the center's position (a center's own)
    }
  }
}

// The labels of a run that has not failed reach the caller's device buffer; a
// failed run leaves it alone, with no host round trip in between.
__global__ void __launch_bounds__(BS) k_deliver(const int32_t *from, int32_t *to, int64_t n, const int *error) {
  if (*error) return;
  const int64_t q = (((uintptr_t)to | (uintptr_t)from) & 15) ? 0 : n / 4;  // whole 16-byte words, if both are aligned
  for (int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x; i < q; i += (int64_t)gridDim.x * BS)
    reinterpret_cast<int4 *>(to)[i] = reinterpret_cast<const int4 *>(from)[i];
  for (int64_t i = q * 4 + (int64_t)blockIdx.x * BS + threadIdx.x; i < n; i += (int64_t)gridDim.x * BS) to[i] = from[i];
}

// -------------------------------------------------------------- launch ----

static inline unsigned grid_for(int64_t items, unsigned cap) {
  int64_t g = (items + BS - 1) / BS;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (unsigned)g;
}

hipError_t launch_init(const Ws &w, hipStream_t s) {
  if (!w.order_mapped) hipLaunchKernelGGL(k_check_order, dim3(grid_for(w.n, 4096)), dim3(BS), 0, s, w);
  hipLaunchKernelGGL(k_init, dim3(grid_for(w.n, 4096)), dim3(BS), 0, s, w);
  hipLaunchKernelGGL(k_close, dim3(1), dim3(64), 0, s, w);
  return hipGetLastError();
}

int round_steps(const Ws &w, const LaunchShape &ls, RoundStep *out) {
  int k = 0;
  auto add = [&](void (*f)(Ws), unsigned grid, unsigned block) { out[k++] = RoundStep{f, grid, block}; };
  const bool binomial = w.policy == POL_BINOMIAL;
  add(binomial ? k_select_range : k_select, ls.select_grid, SEL_BS);
  if (w.algo == ALGO_C4) {
    add(k_elect, ls.edge_grid, BS);
    add(k_classify, ls.vertex_grid, BS);
    add(k_resolve, 1, RBS);
  }
  add(k_claim, ls.edge_grid, BS);
  add(k_clear, ls.vertex_grid, BS);
  if (!binomial) {  // Delta-hat needs no remaining degrees: no peel, no Delta search
    if (ls.exact_seen) {  // the run has switched to exact degrees for good
      add(k_peel, ls.edge_grid, BS);
    } else {
      add(k_candidates, ls.vertex_grid, BS);
      add(k_degrees, ls.edge_grid, BS);
    }
  }
  add(k_close, 1, 64);
  if (w.team) out[k++] = team_step(w);
  return k;
}

hipError_t launch_finalize(const Ws &w, int32_t *labels, hipStream_t s) {
  hipLaunchKernelGGL(k_finalize, dim3(grid_for(w.n, 4096)), dim3(BS), 0, s, w, labels);
  return hipGetLastError();
}

hipError_t launch_deliver(const int32_t *from, int32_t *to, int64_t n, const int *error, hipStream_t s) {
  hipLaunchKernelGGL(k_deliver, dim3(grid_for((n + 3) / 4, 4096)), dim3(BS), 0, s, from, to, n, error);
  return hipGetLastError();
}

}  // namespace ccd
