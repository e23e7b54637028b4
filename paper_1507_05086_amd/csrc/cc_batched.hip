// cc_batched.hip -- C4 / ClusterWild! (arXiv 1507.05086, Algorithm 2) on a
// batch of small graphs in one persistent launch.
//
// A graph of a few thousand vertices fits in LDS, so the whole round loop of
// one graph runs inside one group of threads with its vertex state in LDS:
// a workgroup for large graphs, a single wave for small ones (several graphs
// per workgroup).  Groups take graphs from two queues (large first, most work
// first), so the launch is balanced by longest-processing-time order.
// Inside a graph the remaining degrees are kept exactly (LDS atomics are
// cheap), and the adjacency passes (election, claims, peeling) give each row
// to a few lanes (rows_pass).
#include "cc_device.h"
#include "cc_launch.h"
#include "cc_round.h"

namespace ccd {

enum : uint8_t { F_UNC = 1, F_ACT = 2, F_CEN = 4, F_NON = 8, F_BLK = 16, F_MC = 32, F_MU = 64 };

// Packed per-vertex word: clusterID (rank of the center, INF16 while
// unclustered) in the high half, remaining positive degree in the low half.
// Ranks and degrees of a batch member are below 2^15.
constexpr uint32_t INF16 = 0x7FFF;
__device__ inline uint32_t lw_pack(uint32_t lab, uint32_t deg) { return (lab << 16) | deg; }

// Barrier of a sub-group of nw waves inside a workgroup (sense reversal on a
// generation counter in LDS).  Every wave of a workgroup is resident, so the
// waiting lanes always see the last arrival.
struct SubBar {
  int count, gen;
};

__device__ __forceinline__ void sub_sync(SubBar *b, int nw) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  if (lane_id() == 0) {
    const int g = __hip_atomic_load(&b->gen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    const int arrived = __hip_atomic_fetch_add(&b->count, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (arrived == nw - 1) {
      __hip_atomic_store(&b->count, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      __hip_atomic_store(&b->gen, g + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    } else {
      while (__hip_atomic_load(&b->gen, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) == g)
        __builtin_amdgcn_s_sleep(1);
    }
  }
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// A group of G threads working on one graph: one wave (G = 64), a sub-group
// of G / 64 waves of a larger workgroup (SUB), or the whole workgroup.
template <int G, bool SUB = false>
struct Grp {
  static constexpr int size = G;
  int tid;      // 0 .. G-1
  int *sh;      // G/64 slots of scratch
  SubBar *bar;  // SUB only
  int wave0;    // first wave of the group in the workgroup
  __device__ __forceinline__ int wave() const { return G == 64 ? 0 : wave_id() - wave0; }
  __device__ __forceinline__ void sync() const {
    if (G == 64) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else if (SUB) {
      sub_sync(bar, G / 64);
    } else {
      __syncthreads();
    }
  }
  // exclusive scan; *tot = sum over the group
  __device__ __forceinline__ int scan(int x, int *tot) const {
    const int inc = wave_incl_scan(x);
    if (G == 64) {
      *tot = lane_value(inc, 63);
      return inc - x;
    }
    if (lane_id() == 63) sh[wave()] = inc;
    sync();
    int base = 0, t = 0;
#pragma unroll
    for (int w = 0; w < G / 64; w++) {
      const int y = sh[w];
      if (w < wave()) base += y;
      t += y;
    }
    sync();
    *tot = t;
    return base + inc - x;
  }
  // maximum of values >= 0
  __device__ __forceinline__ int max(int x) const {
    x = wave_max(x);
    if (G == 64) return x;
    if (lane_id() == 0) sh[wave()] = x;
    sync();
    int m = sh[0];
#pragma unroll
    for (int i = 1; i < G / 64; i++) m = sh[i] > m ? sh[i] : m;
    sync();
    return m;
  }
  __device__ __forceinline__ bool any(bool p) const { return max(p ? 1 : 0) != 0; }
};

struct BStats {
  unsigned long long elect, claim, peel, atom;
};

struct BatchArgs {
  const int64_t *off;      // global offsets (rows of all graphs)
  const int32_t *col;      // local ids
  const int64_t *vtx_ptr;  // [num_graphs + 1]
  const int32_t *order;    // per graph local permutation (concatenated)
  int32_t *labels;         // out: local center ids
  const int32_t *queue;    // graph ids, large-graph queue first, each part most work first
  int32_t n_big;           // queue[0, n_big): one graph per workgroup
  int32_t n_quad;          // queue[n_big, n_big + n_quad): one per 4-wave sub-group; rest: one per wave
  int32_t num_graphs;
  int32_t cap_big, cap_quad, cap_wave;  // LDS vertex capacity of a workgroup / sub-group / wave slot
  unsigned *heads;         // [3] queue heads
  int32_t *rounds;         // out: rounds per graph
  unsigned long long *stat;  // [4]: elect, claim, peel entries, atomics
  int *err;
  int algo;
  int64_t eps_q;
  int64_t nnz;             // entries of col
};

// LDS slot of capacity N vertices (21 bytes per vertex plus a few words):
//   row    start and end of each row in the graph's cols
//   lw     packed clusterID | remaining degree
//   ctr    list counter
//   fl     flag byte, padded to whole words (word atomics touch 4 flags)
//   rank   pi^-1 (int16)
//   ordl   pi, position -> vertex (int16)
//   alist  active vertices; compacted in place to the centers
//   nlist  undecided actives during the election, then the newly clustered
struct Slot {
  int2 *row;
  uint32_t *lw;
  int *ctr;
  uint8_t *fl;
  int16_t *rank, *ordl, *alist, *nlist;
  __host__ __device__ static size_t bytes(int N) {
    return (((size_t)N * 20 + 12 + (((size_t)N + 3) & ~(size_t)3)) + 15) / 16 * 16;
  }
  __device__ void carve(uint8_t *p, int N) {  // p: a multiple of 16
    row = (int2 *)p;
    lw = (uint32_t *)(row + N);
    ctr = (int *)(lw + N);
    fl = (uint8_t *)(ctr + 1);
    rank = (int16_t *)(fl + ((N + 3) & ~3));
    ordl = rank + N;
    alist = ordl + N;
    nlist = alist + N;
  }
};

// Four consecutive columns; rows start at any 4-byte address.
struct __attribute__((packed, aligned(4))) Cols4 {
  int32_t u[4];
};

// How the rows of a graph are walked: W = 1 << lg lanes share a row, four
// consecutive entries of it per lane and step.
struct Walk {
  const int32_t *col0;  // the graph's columns
  int last4;            // entries from here on (of col0) cannot be read four at a time: the array ends
  bool wide;            // four can be read at all
  int lg;
  int most;             // entries from which a row is walked by the whole group
  bool longs;           // some row has as many
};
constexpr int LONG = 256, SEG = 512;  // a long row is dealt to the waves by segments

// Pass over the rows of list[0..cnt): act(v, val(v), u) for every entry u of
// row v whose flags pass test(flags of u); returns this lane's share of the
// entries walked.  The kernel is bound by instruction issue (81 % of the
// cycles had one, at 4 waves a SIMD), so a row goes to a few lanes that read
// four or eight whole entries each: no prefix over the list and no search for
// an entry's row, which took most of the 58 vector instructions per 64
// entries that an edge-balanced walk had.  Rows far longer than the others
// are walked by the whole group, so a hub does not leave it idle.  Planted
// blocks, edge-balanced / this: 4096 graphs C4 1.22 / 0.86 ms, ClusterWild!
// 0.96 / 0.73, 301 graphs 0.38 / 0.23; two rows of a sub-wave at once, their
// ends tested entry by entry, took 1.34 and 0.34.  Stars, one row each that
// counts, are what it costs: 95 -> 105 us for 16 of 5000 vertices.
template <class GR, class Val, class Test, class Act>
__device__ __forceinline__ unsigned rows_pass(const GR &g, const int16_t *list, int cnt, const Slot &s, const Walk &k,
                                              Val &&val, Test &&test, Act &&act) {
  constexpr int NW = GR::size / 64;
  const int lane = lane_id();
  const int w = NW == 1 ? 0 : g.wave();
  const int32_t *col0 = k.col0;
  unsigned walked = 0;
  if (k.longs) {
    int turn = w;  // the wave whose segment comes first moves on from row to row
    for (int i0 = 0; i0 < cnt; i0 += 64) {
      int v = 0;
      bool lg = false;
      if (i0 + lane < cnt) {
        v = list[i0 + lane];
        lg = s.row[v].y - s.row[v].x >= k.most;
      }
      for (unsigned long long m = __ballot(lg); m; m &= m - 1) {
        const int a = __builtin_amdgcn_readlane(v, __ffsll((long long)m) - 1);
        const int2 r = s.row[a];
        const int d = r.y - r.x, x = val(a);
        const int32_t *cp = col0 + r.x;
        for (int e = (turn++ & (NW - 1)) * SEG; e < d; e += NW * SEG) {
          int32_t u[8];
          if (e + SEG <= d) {
            const Cols4 q0 = *reinterpret_cast<const Cols4 *>(cp + e + 4 * lane);
            const Cols4 q1 = *reinterpret_cast<const Cols4 *>(cp + e + SEG / 2 + 4 * lane);
#pragma unroll
            for (int j = 0; j < 4; j++) {
              u[j] = q0.u[j];
              u[4 + j] = q1.u[j];
            }
          } else {
#pragma unroll
            for (int j = 0; j < 8; j++) u[j] = e + 64 * j + lane < d ? cp[e + 64 * j + lane] : -1;
          }
          uint8_t f[8];
#pragma unroll
          for (int j = 0; j < 8; j++) f[j] = s.fl[u[j] < 0 ? 0 : u[j]];
#pragma unroll
          for (int j = 0; j < 8; j++)
            if (u[j] >= 0 && test(f[j])) act(a, x, u[j]);
        }
        if (w == 0 && lane == 0) walked += (unsigned)d;
      }
    }
  }
  int lg = k.lg;  // more lanes a row where the list has fewer rows than the group has places for
  while (lg < 6 && cnt <= (NW << (5 - lg))) lg++;
  const int gl = lane & ((1 << lg) - 1), rows = NW << (6 - lg), step = 4 << lg;
  for (int i = (w << (6 - lg)) + (lane >> lg); i < cnt; i += rows) {
    const int v = list[i], x = val(v);
    const int2 r = s.row[v];
    const int r0 = r.x, r1 = r.y;
    if (r1 - r0 >= k.most) continue;  // walked above
    if (gl == 0) walked += (unsigned)(r1 - r0);
    for (int b = r0 + 4 * gl; b < r1;) {
      if (__all(b + step + 4 <= r1)) {  // eight whole entries in every lane that is still at it
        const Cols4 q0 = *reinterpret_cast<const Cols4 *>(col0 + b), q1 = *reinterpret_cast<const Cols4 *>(col0 + b + step);
        uint8_t f[8];
#pragma unroll
        for (int j = 0; j < 4; j++) {
          f[j] = s.fl[q0.u[j]];
          f[4 + j] = s.fl[q1.u[j]];
        }
#pragma unroll
        for (int j = 0; j < 8; j++)
          if (test(f[j])) act(v, x, j < 4 ? q0.u[j & 3] : q1.u[j & 3]);
        b += 2 * step;
        continue;
      }
      // the row's last four may end behind it, and at the array's end they
      // start before the lane's own first
      int32_t u[4];
      bool in[4];
      if (k.wide) {
        const int at = b < k.last4 ? b : k.last4;
        const Cols4 q = *reinterpret_cast<const Cols4 *>(col0 + at);
#pragma unroll
        for (int j = 0; j < 4; j++) {
          u[j] = q.u[j];
          in[j] = at + j >= b && at + j < r1;
        }
      } else {
#pragma unroll
        for (int j = 0; j < 4; j++) {
          in[j] = b + j < r1;
          u[j] = in[j] ? col0[b + j] : 0;
        }
      }
      uint8_t f[4];
#pragma unroll
      for (int j = 0; j < 4; j++) f[j] = s.fl[in[j] ? u[j] : 0];
#pragma unroll
      for (int j = 0; j < 4; j++)
        if (in[j] && test(f[j])) act(v, x, u[j]);
      b += step;
    }
  }
  g.sync();
  return walked;
}

// Inlined into the kernel so that every Slot pointer is known to address LDS
// (an out-of-line call would turn them into generic pointers).
template <class GR>
__device__ __forceinline__ void solve_graph(const GR &g, const BatchArgs &a, int gi, int cap, Slot &s, BStats &st) {
  constexpr int G = GR::size;
  const int64_t v0 = a.vtx_ptr[gi];
  const int n = (int)(a.vtx_ptr[gi + 1] - v0);
  if (n > cap) {  // the host sizes the slots; never taken
    if (g.tid == 0) atomicCAS(a.err, 0, ERR_OVERFLOW);
    return;
  }
  const int64_t *off = a.off + v0;
  const int64_t obase = off[0];
  const int32_t *col0 = a.col + obase;
  const int32_t *ord = a.order + v0;
  const bool c4 = a.algo == ALGO_C4;
  // init: row starts, packed words, pi in LDS; rank = pi^-1 with a permutation check
  for (int v = g.tid; v < n; v += G) {
    const int64_t o = off[v], e = off[v + 1];
    s.row[v] = make_int2((int32_t)(o - obase), (int32_t)(e - obase));
    s.lw[v] = lw_pack(INF16, (uint32_t)(e - o));
    s.fl[v] = F_UNC;
    s.rank[v] = -1;
  }
  g.sync();
  bool bad = false;
  for (int k = g.tid; k < n; k += G) {
    const int32_t v = ord[k];
    s.ordl[k] = (int16_t)v;
    if (v < 0 || v >= n) bad = true;
    else s.rank[v] = (int16_t)k;
  }
  g.sync();
  for (int v = g.tid; v < n; v += G) {
    const int r = s.rank[v];
    if (r < 0 || s.ordl[r] != v) bad = true;
  }
  if (g.any(bad)) {
    if (g.tid == 0) atomicCAS(a.err, 0, ERR_PERM);
    return;
  }
  // lanes of a row, by the mean length (a step takes four entries of a lane,
  // then eight).  At most 8 / 16 / 32 / 64 lanes: planted blocks of 4096
  // graphs 0.85 / 0.87 / 1.00 ms / -, 301 0.226 / 0.242 / 0.245; at most 4:
  // 0.89 and 0.229
  const int64_t tail = a.nnz - 4 - obase;
  const int mean = n > 0 ? s.row[n - 1].y / n : 0;
  Walk walk{col0, (int)(tail < 0x7fffffff ? tail : 0x7fffffff), a.nnz >= 4, mean <= 2 ? 0 : mean <= 24 ? 1 : mean <= 48 ? 2 : 3,
            8 * mean > LONG ? 8 * mean : LONG, false};
  int n_rem = n, cur = 0, rounds = 0;
  while (n_rem > 0 && rounds <= n) {
    // Delta over the unclustered vertices
    int m = 0;
    for (int v = g.tid; v < n; v += G) {
      const int d = (int)(s.lw[v] & 0xFFFFu);
      if ((s.fl[v] & F_UNC) && d > m) m = d;
    }
    const long long delta = g.max(m);
    if (rounds == 0) walk.longs = delta >= walk.most;
    const int B = (int)fixed_batch(a.eps_q, n_rem, delta);
    // active set: the next B unclustered vertices of pi from the cursor
    int na = 0;
    while (na < B && cur < n) {
      const int p = cur + g.tid;
      int32_t v = 0;
      bool un = false;
      if (p < n) {
        v = s.ordl[p];
        un = (s.fl[v] & F_UNC) != 0;
      }
      int tot;
      const int pre = g.scan(un ? 1 : 0, &tot);
      if (un && na + pre < B) {
        s.alist[na + pre] = (int16_t)v;
        s.fl[v] |= F_ACT;
      }
      // position of the B-th unclustered vertex, if in this chunk
      const int last = g.max((un && na + pre == B - 1) ? p + 1 : 0);
      if (last > 0) {
        cur = last;
        na = B;
      } else {
        cur += G;
        na += tot;
      }
    }
    g.sync();
    // centers
    int nc = 0;
    if (c4) {
      // blocked: an earlier-ranked active neighbour
      const auto rank_of = [&](int v) { return (int)s.rank[v]; };
      const auto active = [](uint8_t f) { return (f & F_ACT) != 0; };
      st.elect += rows_pass(g, s.alist, B, s, walk, rank_of, active, [&](int av, int r, int32_t u) {
        if (s.rank[u] < r) s.fl[av] |= F_BLK;
      });
      for (int i = g.tid; i < B; i += G) {
        const int32_t av = s.alist[i];
        if (!(s.fl[av] & F_BLK)) s.fl[av] |= F_CEN;
      }
      g.sync();
      // fixed point over the blocked vertices: a vertex becomes a center once
      // no earlier active neighbour is a center or undecided, and a
      // non-center once an earlier active neighbour is a center
      for (int it = 0; it <= B; it++) {
        int nb = 0;
        for (int i0 = 0; i0 < B; i0 += G) {
          const int i = i0 + g.tid;
          bool und = false;
          if (i < B) {
            const int32_t av = s.alist[i];
            und = !(s.fl[av] & (F_CEN | F_NON));
          }
          int tot;
          const int pre = g.scan(und ? 1 : 0, &tot);
          if (und) s.nlist[nb + pre] = s.alist[i];
          nb += tot;
        }
        g.sync();
        if (nb == 0) break;
        st.elect += rows_pass(g, s.nlist, nb, s, walk, rank_of, active, [&](int av, int r, int32_t u) {
          if (s.rank[u] < r) {
            const uint8_t fu = s.fl[u];
            const unsigned bit = (fu & F_CEN) ? (unsigned)F_MC : ((fu & F_NON) ? 0u : (unsigned)F_MU);
            if (bit) atomicOr((unsigned *)(s.fl + (av & ~3)), bit << (8 * (av & 3)));
          }
        });
        for (int i = g.tid; i < nb; i += G) {
          const int32_t av = s.nlist[i];
          const uint8_t f = s.fl[av];
          uint8_t nf = (uint8_t)(f & ~(F_MC | F_MU));
          if (f & F_MC) nf |= F_NON;
          else if (!(f & F_MU)) nf |= F_CEN;
          s.fl[av] = nf;
        }
        g.sync();
      }
      // compact the centers to the front of alist, in place: every write
      // lands at or before the chunk whose entries are already read
      for (int i0 = 0; i0 < B; i0 += G) {
        const int i = i0 + g.tid;
        bool cen = false;
        int16_t av = 0;
        if (i < B) {
          av = s.alist[i];
          cen = (s.fl[av] & F_CEN) != 0;
        }
        int tot;
        const int pre = g.scan(cen ? 1 : 0, &tot);
        if (cen) s.alist[nc + pre] = av;
        nc += tot;
      }
    } else {
      for (int i = g.tid; i < B; i += G) s.fl[s.alist[i]] |= F_CEN;
      nc = B;
    }
    g.sync();
    // claims: lowest-rank adjacent center wins; newly = centers + first claims
    int *nn_ptr = s.ctr;
    if (g.tid == 0) *nn_ptr = 0;
    g.sync();
    for (int i = g.tid; i < nc; i += G) {
      const int32_t cv = s.alist[i];
      s.lw[cv] = lw_pack((uint32_t)s.rank[cv], 0);
      s.nlist[atomicAdd(nn_ptr, 1)] = (int16_t)cv;
    }
    g.sync();
    // ClusterWild! claims Gamma(c) \ A
    const uint8_t unfit = c4 ? F_CEN : F_CEN | F_ACT;
    st.claim += rows_pass(
        g, s.alist, nc, s, walk, [&](int v) { return (int)s.rank[v]; },
        [&](uint8_t f) { return (f & (F_UNC | unfit)) == F_UNC; },
        [&](int, int r, int32_t u) {
          const uint32_t rc = (uint32_t)r;
          if (rc < (s.lw[u] >> 16)) {
            const uint32_t old = atomicMin(&s.lw[u], lw_pack(rc, 0xFFFFu));
            st.atom++;
            if ((old >> 16) == INF16) s.nlist[atomicAdd(nn_ptr, 1)] = (int16_t)u;
          }
        });
    const int nn = *nn_ptr;
    // the newly clustered leave; the unclustered neighbours of the claimed
    // ones lose one degree.  Centers (nlist[0, nc)) have none left: every
    // unclustered neighbour of a center was claimed this round.
    for (int i = g.tid; i < nn; i += G) s.fl[s.nlist[i]] = 0;
    g.sync();
    st.peel += rows_pass(
        g, s.nlist + nc, nn - nc, s, walk, [](int) { return 0; }, [](uint8_t f) { return (f & F_UNC) != 0; },
        [&](int, int, int32_t u) {
          atomicSub(&s.lw[u], 1u);
          st.atom++;
        });
    n_rem -= nn;
    rounds++;
    g.sync();
  }
  for (int v = g.tid; v < n; v += G) {
    const uint32_t l = s.lw[v] >> 16;
    a.labels[v0 + v] = l < (uint32_t)n ? (int32_t)s.ordl[l] : -1;
    if (l >= (uint32_t)n) atomicCAS(a.err, 0, ERR_LABEL);
  }
  if (g.tid == 0) a.rounds[gi] = rounds;
  if (n_rem > 0 && g.tid == 0) atomicCAS(a.err, 0, ERR_NO_PROGRESS);
}

constexpr int QG = 256;  // threads of a sub-group (4 waves)

template <int T>
__global__ void __launch_bounds__(T) k_batched(BatchArgs a) {
  extern __shared__ __align__(16) uint8_t lds[];
  BStats st{0, 0, 0, 0};
  constexpr int NQ = T / QG > 0 ? T / QG : 1;
  __shared__ int s_gi[NQ];
  __shared__ int sh[T / 64];
  __shared__ int shq[NQ][QG / 64];
  __shared__ SubBar sbar[NQ];
  if (threadIdx.x < NQ) sbar[threadIdx.x] = SubBar{0, 0};
  __syncthreads();
  // phase 1: large graphs, one per workgroup
  Grp<T> gw{(int)threadIdx.x, sh, nullptr, 0};
  Slot sl;
  sl.carve(lds, a.cap_big);
  for (;;) {
    if (threadIdx.x == 0) {
      const unsigned q = atomicAdd(&a.heads[0], 1u);
      s_gi[0] = (int)q < a.n_big ? a.queue[q] : -1;
    }
    __syncthreads();
    const int gi = s_gi[0];
    __syncthreads();
    if (gi < 0) break;
    solve_graph(gw, a, gi, a.cap_big, sl, st);
    __syncthreads();
  }
  // phase 2: mid-size graphs, one per sub-group of 4 waves (workgroups of 512+)
  if (T > QG && a.n_quad > 0) {
    const int sg = (int)threadIdx.x / QG;
    Grp<QG, true> gq{(int)threadIdx.x % QG, shq[sg], &sbar[sg], sg * (QG / 64)};
    Slot sq;
    sq.carve(lds + (size_t)sg * Slot::bytes(a.cap_quad), a.cap_quad);
    for (;;) {
      if (gq.tid == 0) {
        const unsigned q = atomicAdd(&a.heads[2], 1u);
        s_gi[sg] = (int)q < a.n_quad ? a.queue[a.n_big + q] : -1;
      }
      gq.sync();
      const int gi = s_gi[sg];
      gq.sync();
      if (gi < 0) break;
      solve_graph(gq, a, gi, a.cap_quad, sq, st);
      gq.sync();
    }
    __syncthreads();
  }
  // phase 3: small graphs, one per wave
  Grp<64> gv{lane_id(), nullptr, nullptr, 0};
  Slot sv;
  sv.carve(lds + (size_t)wave_id() * Slot::bytes(a.cap_wave), a.cap_wave);
  const int n0 = a.n_big + a.n_quad, nsmall = a.num_graphs - n0;
  for (;;) {
    int q = 0;
    if (lane_id() == 0) q = (int)atomicAdd(&a.heads[1], 1u);
    q = __shfl(q, 0, 64);
    if (q >= nsmall) break;
    solve_graph(gv, a, a.queue[n0 + q], a.cap_wave, sv, st);
  }
  // statistics: one reduction per workgroup, one atomic per counter
  __syncthreads();
  unsigned long long v4[4] = {st.elect, st.claim, st.peel, st.atom};
  __shared__ unsigned long long s_stat[4];
  if (threadIdx.x < 4) s_stat[threadIdx.x] = 0;
  __syncthreads();
  for (int k = 0; k < 4; k++) {
    const int64_t t = wave_sum((int64_t)v4[k]);
    if (lane_id() == 0 && t) atomicAdd(&s_stat[k], (unsigned long long)t);
  }
  __syncthreads();
  if (threadIdx.x < 4 && s_stat[threadIdx.x]) atomicAdd(&a.stat[threadIdx.x], s_stat[threadIdx.x]);
}

// Kernels with more than 64 KB of dynamic LDS must say so before launch.
static hipError_t allow_lds(int block, size_t lds) {
  const void *k = block == 256 ? (const void *)k_batched<256>
                  : block == 512 ? (const void *)k_batched<512> : (const void *)k_batched<1024>;
  return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

hipError_t launch_batched(const BatchLaunch &bl, hipStream_t s) {
  BatchArgs a{bl.off, bl.col, bl.vtx_ptr, bl.order, bl.labels, bl.queue, bl.n_big, bl.n_quad, bl.num_graphs,
              bl.cap_big, bl.cap_quad, bl.cap_wave, bl.heads, bl.rounds, bl.stat, bl.err, bl.algo, bl.eps_q, bl.nnz};
  const size_t lds = batched_lds_bytes(bl.block, bl.cap_big, bl.cap_quad, bl.cap_wave);
  hipError_t e = allow_lds(bl.block, lds);
  if (e != hipSuccess) return e;
  if (bl.block == 256) hipLaunchKernelGGL(k_batched<256>, dim3(bl.grid), dim3(256), lds, s, a);
  else if (bl.block == 512) hipLaunchKernelGGL(k_batched<512>, dim3(bl.grid), dim3(512), lds, s, a);
  else hipLaunchKernelGGL(k_batched<1024>, dim3(bl.grid), dim3(1024), lds, s, a);
  return hipGetLastError();
}

size_t batched_lds_bytes(int block, int cap_big, int cap_quad, int cap_wave) {
  const size_t a = Slot::bytes(cap_big), b = (size_t)(block / 64) * Slot::bytes(cap_wave);
  const size_t q = block > QG ? (size_t)(block / QG) * Slot::bytes(cap_quad) : 0;
  const size_t m = a > b ? a : b;
  return m > q ? m : q;
}

hipError_t batched_max_grid(int block, size_t lds, int *grid) {
  int occ = 0;
  hipError_t e = allow_lds(block, lds);
  if (e != hipSuccess) return e;
  if (block == 256) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, (const void *)k_batched<256>, 256, lds);
  else if (block == 512) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, (const void *)k_batched<512>, 512, lds);
  else e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, (const void *)k_batched<1024>, 1024, lds);
  if (e != hipSuccess) return e;
  int dev = 0, cus = 0;
  e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  *grid = occ * cus;
  return e;
}

}  // namespace ccd
