// cc_walk.h -- edge-balanced walk over the adjacency rows of a vertex list.
//
// A list (vertices + exclusive prefix of their row weights max(deg,1)) is cut
// into equal item ranges, one per workgroup, so a hub row of 10^6 entries is
// shared by many workgroups while thousands of short rows share one.  Inside
// a workgroup the items are processed in tiles of TW: the row weights of the
// tile's rows are staged in LDS (as 32-bit items from the tile's start) and
// each lane finds its row by binary search there (load-balanced search), then reads the adjacency entry with coalesced
// loads along the row.
#pragma once
#include <type_traits>

#include "cc_device.h"

namespace ccd {

// Items of one tile held by one thread.  Item k is an adjacency entry when
// bit k of `edge` is set (u[k] valid) and the first item of its row when bit
// k of `vert` is set (rows of degree 0 own exactly one such item).
struct Items {
  int ent[IPT];      // row index within the tile (LDS slot), -1 if no item
  int32_t v[IPT];    // row vertex
  int32_t u[IPT];    // neighbour (edge items)
  int32_t val[IPT];  // staged per-row value (e.g. rank or lab of v)
  int32_t deg[IPT];  // degree of v
  int64_t pos[IPT];  // position of the entry in col (edge items)
  unsigned edge, vert;
};

// last j < len with a[j] <= x (a sorted, a[0] <= x); one length for the workgroup
__device__ inline int lds_last_le(const int32_t *a, int len, int32_t x) {
  int j = 0, step = 1;
  while (step * 2 < len) step *= 2;
  for (; step > 0; step >>= 1)
    if (j + step < len && a[j + step] <= x) j += step;
  return j;
}

struct NoEpilogue {
  __device__ void operator()(int, int64_t, int32_t, int32_t, int64_t) const {}
};
struct NoPost {
  __device__ void operator()() const {}
};

// What a walk keeps in LDS.  A kernel that takes one of several walks hands
// the same one to each (lb_walk_in).
struct WalkLds {
  int32_t lw[TW + 1];    // first item of each row of the tile, from the tile's start (-1: before it)
  int32_t lv[TW];
  int64_t loff[TW];      // where item 0 of the tile would be in col, were it in the row
  int32_t ldeg[TW];
  int32_t lval[TW];
  int64_t ent;
  int nent, next;
};

// Calls f(Items&) once per tile in every thread of the workgroup (uniformly,
// so f may use wave-wide operations).  Row v is col[off[v] .. end[v]) (end =
// off + 1 for a plain CSR).  `vals` (may be null) is gathered per row into
// Items::val.  A null `list` means the rows 0..cnt-1 themselves.
// With `info` (per list entry), rows come from it and Items::val is the rank.
// After f, ep(j, slot, v, deg, covered) runs once for every row j the tile
// touched (slot = list index, covered = items of that row in this tile), so
// per-row partial results kept in LDS by f can be combined across tiles; then
// post() runs in every thread (it may use barriers).
template <class F, class E = NoEpilogue, class P = NoPost>
__device__ __forceinline__ void lb_walk_in(WalkLds &L, const int32_t *__restrict__ list, const int64_t *__restrict__ work, int64_t cnt,
                        int64_t total, const int64_t *__restrict__ off, const int64_t *__restrict__ end,
                        const int32_t *__restrict__ col,
                        const int32_t *__restrict__ vals, const RowInfo *__restrict__ info, F &&f, E &&ep = E(),
                        P &&post = P()) {
  int32_t *lw = L.lw, *lv = L.lv, *ldeg = L.ldeg, *lval = L.lval;
  int64_t *loff = L.loff;
  if (total <= 0 || cnt <= 0) return;
  const int64_t ntiles = (total + TW - 1) / TW;
  const int64_t nwg = ntiles < (int64_t)gridDim.x ? ntiles : (int64_t)gridDim.x;
  if ((int64_t)blockIdx.x >= nwg) return;
  const int64_t per = (ntiles + nwg - 1) / nwg;  // tiles per workgroup
  const int64_t s0 = (int64_t)blockIdx.x * per * TW;
  if (s0 >= total) return;
  const int64_t s1 = (s0 + per * TW) < total ? (s0 + per * TW) : total;
  if (threadIdx.x < 64) {
    const int64_t e = wave_find_entry(work, cnt, s0);
    if (threadIdx.x == 0) {
      L.ent = e;
      L.nent = 0;
      L.next = 0;
    }
  }
  __syncthreads();
  int64_t ent0 = L.ent;
  // the tile's window of row prefixes, held in registers so that the next
  // tile's window is in flight while this tile is processed
  constexpr int NPW = (TW + 1 + BS - 1) / BS;
  int64_t pw[NPW];
  auto load_window = [&](int64_t e0) {
#pragma unroll
    for (int q = 0; q < NPW; q++) {
      const int j = (int)threadIdx.x + q * BS;
      const int64_t idx = e0 + j;
      pw[q] = (j <= TW && idx < cnt) ? work[idx] : INT64_MAX;
    }
  };
  load_window(ent0);
  for (int64_t s = s0; s < s1; s += TW) {
    const int64_t send = (s + TW) < s1 ? (s + TW) : s1;
    // the window is sorted, so counting its entries below a bound is the
    // upper-bound search: rows touched by this tile, and where the next starts
    int w_rows = 0, w_next = 0;
#pragma unroll
    for (int q = 0; q < NPW; q++) {
      const int j = (int)threadIdx.x + q * BS;
      if (j <= TW) lw[j] = pw[q] < s ? -1 : pw[q] < s + TW ? (int32_t)(pw[q] - s) : TW;
      if (j < TW) loff[j] = s - pw[q];
      w_rows += __popcll(__ballot(j <= TW && pw[q] <= send - 1));
      w_next += __popcll(__ballot(j <= TW && pw[q] <= s + TW));
    }
    if (lane_id() == 0) {
      atomicAdd(&L.nent, w_rows);
      atomicAdd(&L.next, w_next);
    }
    __syncthreads();
    const int nent = L.nent;
    const int next = (s + TW < s1) ? L.next - 1 : 0;
    if (s + TW < s1) load_window(ent0 + next);  // the next tile's window
    for (int j = threadIdx.x; j < nent; j += BS) {
      const int32_t v = list ? list[ent0 + j] : (int32_t)(ent0 + j);
      lv[j] = v;
      if (info) {  // row info carried by the list: no offset or rank lookups
        const RowInfo ri = info[ent0 + j];
        loff[j] += ri.start;
        ldeg[j] = ri.deg;
        lval[j] = ri.rank;
      } else {
        const int64_t o = off[v];
        loff[j] += o;
        ldeg[j] = (int32_t)(end[v] - o);
        lval[j] = vals ? vals[v] : 0;
      }
    }
    __syncthreads();
    if (threadIdx.x == 0) {  // every thread has read them; the next tile counts afresh
      L.nent = 0;
      L.next = 0;
    }
    Items it;
    it.edge = 0;
    it.vert = 0;
    int64_t epos[IPT];
    const int items = (int)(send - s);
#pragma unroll
    for (int k = 0; k < IPT; k++) {
      const int x = k * BS + (int)threadIdx.x;
      it.v[k] = 0;
      it.u[k] = 0;
      it.val[k] = 0;
      it.deg[k] = 0;
      it.pos[k] = -1;
      it.ent[k] = -1;
      epos[k] = -1;
      if (x < items) {
        const int j = lds_last_le(lw, nent, x);
        it.ent[k] = j;
        it.v[k] = lv[j];
        it.val[k] = lval[j];
        it.deg[k] = ldeg[j];
        if (x == lw[j]) it.vert |= 1u << k;
        if (ldeg[j] > 0) {
          it.edge |= 1u << k;
          epos[k] = loff[j] + x;
          it.pos[k] = epos[k];
        }
      }
    }
#pragma unroll
    for (int k = 0; k < IPT; k++)
      if (epos[k] >= 0) it.u[k] = col[epos[k]];
    f(it);
    if constexpr (!std::is_same<typename std::decay<E>::type, NoEpilogue>::value) {
      __syncthreads();
      for (int j = threadIdx.x; j < nent; j += BS) {
        const int lo = lw[j] > 0 ? lw[j] : 0, hi = j + 1 < nent ? lw[j + 1] : items;
        ep(j, ent0 + j, lv[j], ldeg[j], (int64_t)(hi - lo));
      }
    }
    if constexpr (!std::is_same<typename std::decay<P>::type, NoPost>::value) post();
    ent0 += next;
    __syncthreads();
  }
}

template <class F, class E = NoEpilogue, class P = NoPost>
__device__ __forceinline__ void lb_walk(const int32_t *__restrict__ list, const int64_t *__restrict__ work, int64_t cnt,
                                        int64_t total, const int64_t *__restrict__ off, const int64_t *__restrict__ end,
                                        const int32_t *__restrict__ col, const int32_t *__restrict__ vals,
                                        const RowInfo *__restrict__ info, F &&f, E &&ep = E(), P &&post = P()) {
  __shared__ WalkLds lds;
  lb_walk_in(lds, list, work, cnt, total, off, end, col, vals, info, f, ep, post);
}

}  // namespace ccd
