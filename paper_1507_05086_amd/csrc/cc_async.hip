// cc_async.hip -- asynchronous C4 and ClusterWild! (arXiv 1507.05086,
// Algorithm 3: the round loop without its bulk synchronisation).
//
// Threads take the vertices of pi in order and never wait for a round to
// end.  On the GPU a wave takes the next 64 positions of pi (a chunk; lane l
// holds position 64 c + l) from a shared counter and settles them:
//
//   C4 (attemptCluster / isCenter): a vertex still unclustered when reached
//   is a center iff none of its earlier-ranked neighbours is one; an undecided
//   earlier neighbour is waited for.  The labels are KwikCluster's whatever the interleaving (C4 is
//   serializable).
//   ClusterWild! (createCluster): a vertex still unclustered when reached
//   becomes a center (compare-and-swap from "unclustered"), no waiting.  Its
//   labels depend on the interleaving.
//
// Centers then claim their neighbours with atomicMin on the center's rank
// (concurrency rule 2).  The label word of a vertex holds everything the
// waits need:
//   INF          not decided yet
//   -(rank + 1)  a center (rank = its position in pi); never changes again
//   INF - 1      a C4 vertex decided not to be a center, not yet claimed
//   r >= 0       claimed by the center of rank r (only ever decreases)
// and is read and written only with device-scope atomics, so a wave on one
// XCD sees another XCD's decisions.
//
// What bounds it.  Random gathers of ranks and labels, one memory line each
// where the arrays outgrow the caches, once the waits are short.  The waits
// were most of the time while a chunk's decisions were published together and
// a wave took 8 chunks per visit from the start: nearly every chunk has a
// neighbour in the chunk before it, so the chunks in flight finished one after
// the other.  Now a vertex is published when it is decided, a wave keeps the
// undecided neighbours of its 64 vertices and looks at those only (at the
// others of its own chunk in registers: a path of 100 K in its own order 119 ms
// with a read of the label for each, 11.7 so, 11.3 by whole chunks), and the
// runs of chunks grow with the position.  Whole calls: R-MAT 24 11.3
// -> 2.26 ms, R-MAT 26 13.9 -> 7.3, R-MAT 20 9.2 -> 0.42, power law 3 M 25.7 ->
// 0.81, ER 3 M 19.7 -> 0.75 ms.
//
// Progress: chunks are handed out in pi order (a run of consecutive chunks
// per visit to the counter, worked through in order), and a vertex waits
// only for earlier ones.  The earliest undecided vertex is in the chunk its
// wave is working on (that wave's earlier chunks are finished) or in the next
// one to be handed out, and it waits for nobody; its wave's loop never blocks
// on one of its other vertices.  A wave takes a new run only after finishing
// the last, so no resident-set assumption is needed.  Every wait is bounded
// (and stops when another wave has reported an error); every wave leaves when
// the counter passes the last chunk.
#include "cc_device.h"
#include "cc_launch.h"

namespace ccd {

constexpr int AS_BS = 256;  // 4 waves per workgroup, each on its own chunks
constexpr int AS_BIG = 2048;  // C4 centers with longer rows claim in a second, device-wide pass
// chunks a wave takes per visit to the shared counter (one device-scope
// atomic on one address serialises with every other wave's)
constexpr int AS_BATCH = 8;  // (4: R-MAT 26 8.2 ms when every run is as long, 16: 9.2, growing to 8: 7.4)
constexpr int32_t LAB_NONCENTER = INF - 1;
constexpr int AS_PAIRS = 512;  // undecided earlier neighbours a wave keeps
// Above this many vertices isCenter reads a neighbour's label before its rank
// (two arrays no longer stay in the 256 MB cache, and most neighbours, the
// hubs, are decided early): R-MAT 26 8.0 -> 7.35 ms a call, R-MAT 24 2.3 both
// ways, power law 4 M 1.12 -> 1.19 ms.
constexpr int64_t AS_LAB_FIRST = int64_t(1) << 25;
constexpr long long AS_LIMIT = 200000000;  // longest wait without a decision, wall clock ticks (100 MHz)

__device__ inline int32_t lab_load(const int32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A wave walks the rows of its lanes in two ways.  Rows of more than AS_LONG
// entries are streamed one after the other; the others (at most 64 * AS_LONG
// entries together) edge-balanced over the wave: entry e of the concatenated
// rows belongs to the first lane j whose inclusive prefix incl_j exceeds e
// (six steps of a lane-indexed binary search).  Either way AS_K entries per
// lane are in flight together (4 and 8 are alike; one makes a hub's row, met
// before anybody has claimed it, a chain of 6 K steps per 400 K entries).
constexpr int AS_LONG = 512;
constexpr int AS_K = 4;

__device__ inline int owner_lane(int incl, int e) {
  int j = 0;
#pragma unroll
  for (int step = 32; step >= 1; step >>= 1) {
    const int pj = __shfl(incl, j + step - 1, 64);
    if (pj <= e) j += step;
  }
  return j;
}

// f(u, j): AS_K neighbours of this lane (u[k] < 0: none) and the lanes whose
// rows they are in, for the rows [start, start + deg) of the lanes in `rows`;
// stop(mask) says whether the rows of those lanes need no further look.
// Every lane of the wave calls f each time.
template <class F, class S>
__device__ inline void wave_rows(const int32_t *col, unsigned long long rows, int64_t start, int32_t deg, F &&f, S &&stop) {
  const int lane = lane_id();
  int32_t u[AS_K];
  int jj[AS_K];
  const unsigned long long longs = __ballot((rows >> lane & 1) && deg > AS_LONG);
  const int sdeg = (rows >> lane & 1) && deg <= AS_LONG ? deg : 0;
  const int incl = wave_incl_scan(sdeg);
  const int total = __shfl(incl, 63, 64);
  const int64_t base = start - (incl - sdeg);  // of entry e of this lane's row: col[base + e]
  const unsigned long long shorts = rows & ~longs;
  for (int e0 = 0; e0 < total; e0 += 64 * AS_K) {
    if (stop(shorts)) break;
#pragma unroll
    for (int k = 0; k < AS_K; k++) {
      // lane-indexed shuffles run with the whole wave active
      const int e = e0 + 64 * k + lane;
      jj[k] = owner_lane(incl, e < total ? e : total - 1);
      const int64_t b = __shfl(base, jj[k], 64);
      u[k] = -1;
      if (e < total) u[k] = col[b + e];
    }
    f(u, jj);
  }
  for (unsigned long long m = longs; m; m &= m - 1) {
    const int j = __ffsll((long long)m) - 1;
    const int64_t s0 = __shfl(start, j, 64);
    const int32_t d = __shfl(deg, j, 64);
    for (int32_t e0 = 0; e0 < d; e0 += 64 * AS_K) {
      if (stop(1ull << j)) break;
#pragma unroll
      for (int k = 0; k < AS_K; k++) {
        const int32_t e = e0 + 64 * k + lane;
        jj[k] = j;
        u[k] = e < d ? col[s0 + e] : -1;
      }
      f(u, jj);
    }
  }
}

__device__ inline unsigned wave_or(unsigned x) {
  x |= dpp_mov<0x111, 0xf>(0, x);
  x |= dpp_mov<0x112, 0xf>(0, x);
  x |= dpp_mov<0x114, 0xf>(0, x);
  x |= dpp_mov<0x118, 0xf>(0, x);
  x |= dpp_mov<0x142, 0xf>(0, x);
  x |= dpp_mov<0x143, 0xf>(0, x);
  return lane_value((int)x, 63);
}
__device__ inline unsigned long long wave_or(unsigned long long x) {
  return (unsigned long long)wave_or((unsigned)(x >> 32)) << 32 | wave_or((unsigned)x);
}

// Next run of chunks of this wave (AS_BATCH of them; ramp: fewer while the
// run is young).  The vertices in flight are all met before anybody has
// claimed them, so C4 starts with one chunk per visit and a narrow window;
// later, when most positions are settled when reached, the counter (one
// device-scope atomic, serialised with every other wave's) would be the limit.
__device__ inline void next_run(Ctrl *c, int64_t nchunks, bool ramp, int64_t *chunk, int64_t *end) {
  long long run = AS_BATCH;
  if (ramp) {
    run = *end / (4 * (int64_t)gridDim.x * (AS_BS / 64)) + 1;
    if (run > AS_BATCH) run = AS_BATCH;
  }
  unsigned b = 0;
  if (lane_id() == 0) b = atomicAdd(&c->tile_counter, (unsigned)run);
  *chunk = (int64_t)__shfl(b, 0, 64);
  *end = *chunk + run < nchunks ? *chunk + run : nchunks;
}

template <int ALGO>
__global__ void __launch_bounds__(AS_BS) k_async(AsyncArgs a) {
  Ctrl *c = a.ctrl;
  const int lane = lane_id();
  __shared__ int32_t s_u[ALGO == ALGO_C4 ? AS_BS / 64 : 1][AS_PAIRS];
  __shared__ uint8_t s_j[ALGO == ALGO_C4 ? AS_BS / 64 : 1][AS_PAIRS];
  __shared__ unsigned s_dep[ALGO == ALGO_C4 ? AS_BS / 64 : 1][2][64];
  __shared__ int s_n[AS_BS / 64];
  const int64_t nchunks = (a.n + 63) / 64;
  unsigned long long walked = 0, claimed = 0, atoms = 0, waits = 0;
  int64_t chunk = 0, chunk_end = 0;  // the wave's current run of chunks
  const bool lab_first = a.n > AS_LAB_FIRST;
  for (;; chunk++) {
    if (chunk >= chunk_end) next_run(c, nchunks, ALGO == ALGO_C4, &chunk, &chunk_end);
    if (chunk >= nchunks) break;
    if (ld_rlx(&c->error)) break;
    const int64_t c0 = chunk * 64, p = c0 + lane;
    int32_t v = -1;
    if (p < a.n) v = a.order[p];
    // isolated vertices are their own clusters: k_async_finalize labels them
    const bool live = v >= 0 && v < a.iso_start;
    const bool pending = live && lab_load(&a.lab[v]) == INF;  // else claimed already: not a center
    int64_t start = 0;
    int32_t deg = 0;
    if (pending) {
      start = a.off[v];
      deg = (int32_t)(a.off[v + 1] - start);
    }
    // claims of the centers in a mask.  A C4 center with a long row is listed
    // and claims in k_async_big instead, spread over the whole device: a label
    // only decides whether its vertex is still unclustered when reached, and
    // a C4 vertex that should have been claimed already finds its earlier
    // center in isCenter anyway.  (ClusterWild! has no such check, so its
    // claims are never put off.)
    auto claim = [&](unsigned long long centers) {
      bool defer = false;
      if (ALGO == ALGO_C4 && (centers >> lane & 1) && deg > AS_BIG) {
        const unsigned slot = atomicAdd(&c->n_blocked, 1u);
        if ((int64_t)slot < a.big_cap) {
          a.big_v[slot] = v;
          a.big_p[slot] = (int32_t)p;
          defer = true;
        } else {
          set_error(c, ERR_OVERFLOW);  // cannot happen: a list slot per vertex
        }
      }
      wave_rows(
          a.col, __ballot((centers >> lane & 1) && !defer), start, deg,
          [&](const int32_t *u, const int *jj) {
            int32_t x[AS_K];
#pragma unroll
            for (int k = 0; k < AS_K; k++) x[k] = u[k] >= 0 ? a.lab[u[k]] : -1;
#pragma unroll
            for (int k = 0; k < AS_K; k++) {
              const int32_t pj = (int32_t)(c0 + jj[k]);
              claimed += u[k] >= 0;
              if (x[k] > pj) {  // stale reads are safe: a label only decreases
                // a hub met by many rows of the wave: the first has the lowest rank
                const bool again = u[k] == __builtin_amdgcn_readfirstlane(u[k]) &&
                                   lane != __builtin_amdgcn_readfirstlane(lane);
                if (!again) {
                  atomicMin(&a.lab[u[k]], pj);
                  atoms++;
                }
              }
            }
          },
          [](unsigned long long) { return false; });
    };
    if constexpr (ALGO == ALGO_CW) {
      // createCluster: a vertex still unclustered becomes a center
      bool won = false;
      if (pending) won = atomicCAS(&a.lab[v], INF, -(int32_t)p - 1) == INF;
      claim(__ballot(won));
    } else {
      // isCenter.  A pass over the rows finds the earlier-ranked neighbours:
      // a center decides its vertex at once, an undecided one is kept: as a
      // bit of the lane's `dep` if it is another of this chunk's vertices, whose
      // dependences are then followed in registers, else as a pair (neighbour,
      // lane); only the pairs are looked at again.  A vertex is published as
      // soon as it is decided, not with its chunk.
      int32_t *pu = s_u[wave_id()];
      uint8_t *pj = s_j[wave_id()];
      int *pn = &s_n[wave_id()];
      unsigned long long undecided = __ballot(pending);
      unsigned long long again = undecided;  // rows (still) to be walked: a pair did not fit
      unsigned long long toclaim = 0, own = 0;  // own: the chunk's centers
      unsigned long long dep = 0;               // earlier vertices of the chunk that this lane's waits for
      long long t0 = 0;
      unsigned(*pd)[64] = s_dep[wave_id()];
      pd[0][lane] = pd[1][lane] = 0;
      if (lane == 0) *pn = 0;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      while (undecided) {
        unsigned long long blocked = 0, waiting = 0;
        if (again) {
          unsigned long long skip = 0;  // lanes whose pairs do not all fit
          const unsigned long long rows = again;
          wave_rows(
              a.col, rows, start, deg,
              [&](const int32_t *u, const int *jj) {
                int32_t ru[AS_K], x[AS_K];
                unsigned long long found = 0, lost = 0;
#pragma unroll
                for (int k = 0; k < AS_K; k++) {
                  walked += u[k] >= 0;
                  // a plain load: a decision it sees is final, and a hub's label stays cached
                  x[k] = u[k] < 0 ? 0 : lab_first ? a.lab[u[k]] : INF;
                }
#pragma unroll
                for (int k = 0; k < AS_K; k++) ru[k] = x[k] == INF ? a.rank[u[k]] : -1;
#pragma unroll
                for (int k = 0; k < AS_K; k++) {
                  if (x[k] == INF) x[k] = ru[k] < c0 + jj[k] ? lab_load(&a.lab[u[k]]) : 0;
                  else if (x[k] < 0 && -x[k] - 1 > c0 + jj[k]) x[k] = 0;  // a later center
                }
#pragma unroll
                for (int k = 0; k < AS_K; k++) {
                  if (x[k] < 0) found |= 1ull << jj[k];  // a center
                  if (x[k] == INF && ru[k] >= c0) {
                    const int i = (int)(ru[k] - c0);
                    atomicOr(&pd[i >> 5][jj[k]], 1u << (i & 31));
                  } else if (x[k] == INF && !(blocked >> jj[k] & 1)) {
                    const int q = atomicAdd(pn, 1);
                    if (q < AS_PAIRS) {
                      pu[q] = u[k];
                      pj[q] = (uint8_t)jj[k];
                    } else {
                      lost |= 1ull << jj[k];
                    }
                  }
                }
                if (__ballot(found != 0)) blocked |= wave_or(found);
                if (__ballot(lost != 0)) skip |= wave_or(lost);
              },
              // until every vertex of these rows has an earlier center
              [&](unsigned long long rows) { return (blocked & rows) == rows; });
          again = skip & ~blocked;
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          __builtin_amdgcn_wave_barrier();
          dep = (unsigned long long)pd[1][lane] << 32 | pd[0][lane];
        }
        const int32_t mine = undecided >> lane & 1 ? lab_load(&a.lab[v]) : INF;
        // the pairs: decided ones go, the others close ranks
        const int np = *pn < AS_PAIRS ? *pn : AS_PAIRS;
        int out = 0;
        unsigned long long found = 0, wait = 0;
        for (int i0 = 0; i0 < np; i0 += 64) {
          const int i = i0 + lane;
          int32_t u = -1;
          int j = 0;
          if (i < np) {
            u = pu[i];
            j = pj[i];
          }
          bool keep = false;
          if (u >= 0 && (undecided & ~blocked) >> j & 1) {
            const int32_t x = lab_load(&a.lab[u]);
            if (x < 0) found |= 1ull << j;
            keep = x == INF;
          }
          if (keep) wait |= 1ull << j;
          const unsigned long long m = __ballot(keep);
          __builtin_amdgcn_wave_barrier();  // every lane has read its pair
          if (keep) {
            const int q = out + __popcll(m & lanemask_lt());
            pu[q] = u;
            pj[q] = (uint8_t)j;
          }
          out += __popcll(m);
          __builtin_amdgcn_wave_barrier();
        }
        if (lane == 0) *pn = out;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (np > 0) {
          blocked |= wave_or(found);
          waiting = wave_or(wait);
        }
        // a vertex claimed meanwhile has an earlier center too
        const bool taken = (undecided >> lane & 1) && mine != INF;
        blocked = (blocked | __ballot(taken)) & undecided;
        const unsigned long long held = waiting | again;
        unsigned long long no = 0, yes = 0, left = undecided;
        for (unsigned long long next = blocked;;) {  // what is settled settles others of the chunk, a level at a time
          next |= __ballot((dep & own) != 0) & left;
          const unsigned long long free = __ballot((dep & left) == 0) & left & ~(next | held);
          if ((next | free) == 0) break;
          no |= next;
          yes |= free;
          own |= free;
          left &= ~(next | free);
          next = 0;
        }
        if (yes >> lane & 1)
          __hip_atomic_store(&a.lab[v], -(int32_t)p - 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else if ((no >> lane & 1) && !taken)
          atomicMin(&a.lab[v], LAB_NONCENTER);
        undecided = left;
        again &= undecided;
        toclaim |= yes;
        if ((no | yes) == 0 || undecided == 0) {
          if (toclaim) {  // nothing more to decide for now
            claim(toclaim);
            toclaim = 0;
          } else if (undecided) {
            waits++;
            if (t0 == 0) t0 = wall_clock64();
            if ((waits & 255) == 0) {
              if (ld_rlx(&c->error)) break;
              if (wall_clock64() - t0 > AS_LIMIT) {
                set_error(c, ERR_NO_PROGRESS);
                break;
              }
            }
            __builtin_amdgcn_s_sleep(2);
          }
        } else {
          t0 = 0;
        }
      }
    }
  }
  const int64_t s0 = wave_sum((int64_t)walked), s1 = wave_sum((int64_t)claimed), s2 = wave_sum((int64_t)atoms),
                s3 = wave_sum((int64_t)waits);
  if (lane == 0) {
    const int slot = (blockIdx.x * (AS_BS / 64) + wave_id()) & 63;
    if (s0) atomicAdd(&c->spread_lone[slot], (unsigned long long)s0);
    if (s1) atomicAdd(&c->x_low[slot], (unsigned long long)s1);
    if (s2) atomicAdd(&c->spread_atom[slot], (unsigned long long)s2);
    if (s3) atomicAdd(&c->spread_conf[slot], (unsigned long long)s3);
  }
}

// The listed long-row claims: slice k of listed row i goes to workgroup
// (i + k) mod gridDim.x, so each row is spread over the device.
constexpr int AS_SLICE = 4096;

__global__ void __launch_bounds__(BS) k_async_big(AsyncArgs a) {
  Ctrl *c = a.ctrl;
  const int64_t nbig = c->n_blocked < a.big_cap ? (int64_t)c->n_blocked : a.big_cap;
  unsigned long long claimed = 0, atoms = 0;
  for (int64_t i = 0; i < nbig; i++) {
    const int32_t v = a.big_v[i], p = a.big_p[i];
    const int64_t start = a.off[v], deg = a.off[v + 1] - start;
    const int64_t nslices = (deg + AS_SLICE - 1) / AS_SLICE;
    for (int64_t k = ((int64_t)blockIdx.x - i % gridDim.x + gridDim.x) % gridDim.x; k < nslices; k += gridDim.x) {
      const int64_t e1 = (k + 1) * AS_SLICE < deg ? (k + 1) * AS_SLICE : deg;
      for (int64_t e = k * AS_SLICE + threadIdx.x; e < e1; e += BS) {
        const int32_t u = a.col[start + e];
        claimed++;
        if (a.lab[u] > p) {
          atomicMin(&a.lab[u], p);
          atoms++;
        }
      }
    }
  }
  const int64_t s1 = wave_sum((int64_t)claimed), s2 = wave_sum((int64_t)atoms);
  if (lane_id() == 0) {
    const int slot = (blockIdx.x * (BS / 64) + wave_id()) & 63;
    if (s1) atomicAdd(&c->x_low[slot], (unsigned long long)s1);
    if (s2) atomicAdd(&c->spread_atom[slot], (unsigned long long)s2);
  }
}

// pi in internal ids, each vertex's rank, and the permutation check: rank
// starts at -1 everywhere, and n entries in range that leave no vertex
// without a rank name every vertex once.
__global__ void __launch_bounds__(BS) k_async_order(AsyncArgs a, const int32_t *order_in, const int32_t *perm,
                                                    int32_t *iorder) {
  for (int64_t k = (int64_t)blockIdx.x * BS + threadIdx.x; k < a.n; k += (int64_t)gridDim.x * BS) {
    const int32_t v = order_in[k];
    if (v < 0 || (int64_t)v >= a.n) {
      set_error(a.ctrl, ERR_PERM);
      iorder[k] = -1;
    } else {
      const int32_t vi = perm[v];
      iorder[k] = vi;
      a.rank[vi] = (int32_t)k;
    }
  }
}

// check: the permutation check still to finish (after k_async_order; the
// bucketed mapping checks by itself)
__global__ void __launch_bounds__(BS) k_async_init(AsyncArgs a, int check) {
  for (int64_t v = (int64_t)blockIdx.x * BS + threadIdx.x; v < a.n; v += (int64_t)gridDim.x * BS) {
    if (check && a.rank[v] < 0) set_error(a.ctrl, ERR_PERM);  // no entry of pi names v
    a.lab[v] = INF;
  }
}

// Output labels by input id: a center's own id, a claimed vertex the id at
// its center's position; an isolated vertex is alone.
__global__ void __launch_bounds__(BS) k_async_finalize(AsyncArgs a, const int32_t *order_in, const int32_t *perm,
                                                       int32_t *labels) {
  for (int64_t vin = (int64_t)blockIdx.x * BS + threadIdx.x; vin < a.n; vin += (int64_t)gridDim.x * BS) {
    const int32_t v = perm[vin];
    if (v >= a.iso_start) {
      labels[vin] = (int32_t)vin;
      continue;
    }
    const int32_t l = a.lab[v];
    if (l < 0) {
      labels[vin] = (int32_t)vin;  // a center
    } else if (l >= LAB_NONCENTER || (int64_t)l >= a.n) {
      set_error(a.ctrl, ERR_LABEL);  // every vertex is settled when the kernel ends
      labels[vin] = -1;
    } else {
      labels[vin] = order_in[l];
    }
  }
}

static unsigned grid_n(int64_t n) {
  int64_t g = (n + BS - 1) / BS;
  if (g < 1) g = 1;
  if (g > 4096) g = 4096;
  return (unsigned)g;
}

hipError_t launch_async(const AsyncArgs &a, int algo, const int32_t *order_in, const int32_t *perm, int32_t *iorder,
                        int32_t *labels, int waves, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1,
                        const OrderMap *om) {
  hipError_t e;
  if (om) {
    if ((e = launch_order_map(*om, order_in, perm, a.n, iorder, a.ctrl, s, a.rank)) != hipSuccess) return e;
  } else {
    if ((e = hipMemsetAsync(a.rank, 0xFF, sizeof(int32_t) * (size_t)a.n, s)) != hipSuccess) return e;  // every rank -1
    hipLaunchKernelGGL(k_async_order, dim3(grid_n(a.n)), dim3(BS), 0, s, a, order_in, perm, iorder);
  }
  hipLaunchKernelGGL(k_async_init, dim3(grid_n(a.n)), dim3(BS), 0, s, a, om ? 0 : 1);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  auto kern = algo == ALGO_C4 ? k_async<ALGO_C4> : k_async<ALGO_CW>;
  int block = AS_BS, grid = 1;
  if (waves > 0 && waves < AS_BS / 64) {
    block = 64 * waves;
  } else if (waves > 0) {
    grid = (waves + AS_BS / 64 - 1) / (AS_BS / 64);
  } else {
    int dev = 0, cus = 0, per_cu = 0;
    if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
    if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, AS_BS, 0)) != hipSuccess) return e;
    grid = cus * (per_cu > 0 ? per_cu : 1);
    const int64_t need = ((a.n + 63) / 64 + AS_BS / 64 - 1) / (AS_BS / 64);
    if (need < grid) grid = (int)(need > 0 ? need : 1);
  }
  if (ev0 && (e = hipEventRecord(ev0, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(block), 0, s, a);
  if (algo == ALGO_C4) hipLaunchKernelGGL(k_async_big, dim3(1024), dim3(BS), 0, s, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (ev1 && (e = hipEventRecord(ev1, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_async_finalize, dim3(grid_n(a.n)), dim3(BS), 0, s, a, order_in, perm, labels);
  return hipGetLastError();
}

}  // namespace ccd
