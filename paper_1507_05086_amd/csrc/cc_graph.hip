// cc_graph.hip -- graph set-up (row weights, input checks) and the
// disagreement cost of a clustering (the objective of Section 2 of
// arXiv 1507.05086):
//   cost = sum_k C(s_k, 2) + m - 2 m_in
// counted per graph of a batch.  Both passes over the adjacency use the
// edge-balanced walk, so hub rows do not serialise on one wave.
#include "cc_device.h"
#include "cc_launch.h"
#include "cc_walk.h"

namespace ccd {

// ------------------------------------------------------ prefix of weights --
// wall[v] = sum_{x<v} max(deg(x), 1): the "all rows" list of the walk.

constexpr int SCAN_T = 4;  // items per thread in the block scan

__global__ void __launch_bounds__(BS) k_wscan_local(const int64_t *off, int64_t n, int64_t *wall,
                                                    int64_t *blocksum) {
  __shared__ int64_t sh[WAVES + 1];
  const int64_t base = ((int64_t)blockIdx.x * BS + threadIdx.x) * SCAN_T;
  int64_t x[SCAN_T], s = 0;
#pragma unroll
  for (int k = 0; k < SCAN_T; k++) {
    const int64_t v = base + k;
    x[k] = 0;
    if (v < n) {
      const int64_t d = off[v + 1] - off[v];
      x[k] = d > 0 ? d : 1;
    }
    s += x[k];
  }
  int64_t tot;
  int64_t pre = wg_excl_scan(s, &tot, sh);
#pragma unroll
  for (int k = 0; k < SCAN_T; k++) {
    const int64_t v = base + k;
    if (v < n) wall[v] = pre;
    pre += x[k];
  }
  if (threadIdx.x == 0) blocksum[blockIdx.x] = tot;
}

// One workgroup: exclusive scan of the block sums in place; total -> *out.
__global__ void __launch_bounds__(BS) k_wscan_blocks(int64_t *blocksum, int64_t nb, int64_t *out) {
  __shared__ int64_t sh[WAVES + 1];
  int64_t carry = 0;
  for (int64_t i0 = 0; i0 < nb; i0 += BS) {
    const int64_t i = i0 + threadIdx.x;
    const int64_t x = i < nb ? blocksum[i] : 0;
    int64_t tot;
    const int64_t pre = wg_excl_scan(x, &tot, sh);
    if (i < nb) blocksum[i] = carry + pre;
    carry += tot;
  }
  if (threadIdx.x == 0) *out = carry;
}

__global__ void __launch_bounds__(BS) k_wscan_add(int64_t *wall, int64_t n, const int64_t *blocksum,
                                                  const int64_t *total) {
  const int64_t base = ((int64_t)blockIdx.x * BS + threadIdx.x) * SCAN_T;
  const int64_t add = blocksum[blockIdx.x];
#pragma unroll
  for (int k = 0; k < SCAN_T; k++) {
    const int64_t v = base + k;
    if (v < n) wall[v] += add;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) wall[n] = *total;
}

hipError_t launch_row_weights(const int64_t *off, int64_t n, int64_t *wall, int64_t *blocksum,
                              hipStream_t s) {
  const int64_t per = (int64_t)BS * SCAN_T;
  const int64_t nb = (n + per - 1) / per;
  if (nb == 0) {
    return hipMemsetAsync(wall, 0, sizeof(int64_t), s);
  }
  hipLaunchKernelGGL(k_wscan_local, dim3((unsigned)nb), dim3(BS), 0, s, off, n, wall, blocksum);
  hipLaunchKernelGGL(k_wscan_blocks, dim3(1), dim3(BS), 0, s, blocksum, nb, blocksum + nb);
  hipLaunchKernelGGL(k_wscan_add, dim3((unsigned)nb), dim3(BS), 0, s, wall, n, blocksum, blocksum + nb);
  return hipGetLastError();
}

// ---------------------------------------------------------------- checks --

// A column outside its graph outranks every other finding (the others may be
// its consequences); then the smallest code wins.
__device__ inline void report(int *err, int code) { atomicMin(err, ((code == 10 ? 0 : 1) << 8) | code); }

// Every entry: its column's range and, validating, self-loops, the order in
// its row, and its mirror entry by binary search.  Validate == 1 searches for
// one entry of each pair only, the one in the longer row, so the search is
// in the shorter one; the entries of both kinds are counted (*above: searched
// minus not searched).  Rows without repeats, every searched entry mirrored
// and equal counts make the mirror map one-to-one and onto, so the graph is
// symmetric.  Anything else found is reported as CHECK_AGAIN, and validate
// == 2 (every entry searched) names it.  Power law 1 M, 40 M entries, dependent
// reads of the search: 4.1 ms with every entry searched, 2.0 ms with
// half of them and those in the shorter row, 1.5 ms where an equal entry ends
// the search (2.4 ms by quarters: fewer steps but more reads).
// Without validation (a kernel of its own: the searches' registers cost the
// range check 3 of 10 ms on R-MAT 26) only the range is checked.
template <bool VALIDATE>
__global__ void __launch_bounds__(BS) k_check(CheckArgs a) {
  long long above = 0;
  lb_walk(nullptr, a.wall, a.n, a.wall[a.n], a.off, a.off + 1, a.col, nullptr, nullptr, [&](Items &it) {
    int32_t x[IPT];                      // x[k] >= 0: look for it in a row, whose
    int64_t lo[IPT], hi[IPT], end[IPT];  // entries from lo on are not smaller
#pragma unroll
    for (int k = 0; k < IPT; k++) {
      lo[k] = hi[k] = end[k] = 0;
      x[k] = -1;
      if (!(it.edge >> k & 1)) continue;
      const int32_t v = it.v[k], u = it.u[k];
      int64_t base = 0, ng = a.n;
      if (a.gid) {
        const int32_t g = a.gid[v];
        base = a.vtx_ptr[g];
        ng = a.vtx_ptr[g + 1] - base;
      }
      if (u < 0 || (int64_t)u >= ng) {
        report(a.err, 10);  // CC_ERR_OUT_OF_RANGE
        continue;
      }
      if (!VALIDATE) continue;
      const int32_t vl = (int32_t)(v - base);
      const int64_t e = it.pos[k];
      const bool loop = u == vl, disorder = e + 1 < a.off[v + 1] && a.col[e + 1] <= u;
      if (a.validate == 2) {
        if (loop) report(a.err, 3);      // CC_ERR_SELF_LOOP
        if (disorder) report(a.err, 4);  // CC_ERR_DUPLICATE_EDGE
      } else if (loop || disorder) {
        atomicMin(a.err, CHECK_AGAIN);
      }
      const int64_t r0 = a.off[base + u], r1 = a.off[base + u + 1];
      const int64_t du = r1 - r0, dv = it.deg[k];
      const bool search = a.validate == 2 || du < dv || (du == dv && u < vl);
      above += search ? 1 : -1;
      if (search) {
        lo[k] = r0;
        hi[k] = end[k] = r1;
        x[k] = vl;
      }
    }
    if (!VALIDATE) return;
    // the searches of this thread's entries step together
    bool more = true;
    while (more) {
      more = false;
      int32_t c[IPT];
#pragma unroll
      for (int k = 0; k < IPT; k++)
        if (lo[k] < hi[k]) c[k] = a.col[lo[k] + ((hi[k] - lo[k]) >> 1)];
#pragma unroll
      for (int k = 0; k < IPT; k++)
        if (lo[k] < hi[k]) {
          const int64_t mid = lo[k] + ((hi[k] - lo[k]) >> 1);
          if (c[k] == x[k] && a.validate == 1) {  // found (on a row out of order validate 2 asks for the first entry not below)
            x[k] = -1;
            hi[k] = lo[k];
          } else if (c[k] < x[k]) {
            lo[k] = mid + 1;
          } else {
            hi[k] = mid;
          }
          more |= lo[k] < hi[k];
        }
    }
#pragma unroll
    for (int k = 0; k < IPT; k++)
      if (x[k] >= 0 && !(lo[k] < end[k] && a.col[lo[k]] == x[k])) {
        if (a.validate == 2) report(a.err, 2);  // CC_ERR_NOT_SYMMETRIC
        else atomicMin(a.err, CHECK_AGAIN);
      }
  });
  if (VALIDATE && a.validate == 1) {
    const int64_t t = wave_sum((int64_t)above);
    if (lane_id() == 0 && t) atomicAdd(a.above, (unsigned long long)t);
  }
}

__global__ void __launch_bounds__(64) k_check_counts(CheckArgs a) {
  if (threadIdx.x == 0 && *a.above) atomicMin(a.err, CHECK_AGAIN);
}

__global__ void __launch_bounds__(BS) k_offsets_check(const int64_t *off, int64_t n, int64_t *out) {
  bool bad = false;
  for (int64_t v = (int64_t)blockIdx.x * BS + threadIdx.x; v < n; v += (int64_t)gridDim.x * BS) bad |= off[v + 1] < off[v];
  if (bad) out[2] = 1;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    out[0] = off[n];
    if (off[0] != 0) out[1] = 1;
  }
}

__global__ void __launch_bounds__(BS) k_gather64(const int64_t *off, const int64_t *at, int64_t count, int64_t *out) {
  for (int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x; i < count; i += (int64_t)gridDim.x * BS) out[i] = off[at[i]];
}

static unsigned blocks_for(int64_t n, int64_t most) {
  const int64_t g = (n + BS - 1) / BS;
  return (unsigned)(g < 1 ? 1 : g < most ? g : most);
}

hipError_t launch_offsets_check(const int64_t *off, int64_t n, int64_t *out, hipStream_t s) {
  const hipError_t e = hipMemsetAsync(out, 0, 3 * sizeof(int64_t), s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_offsets_check, dim3(blocks_for(n, 2048)), dim3(BS), 0, s, off, n, out);
  return hipGetLastError();
}

hipError_t launch_gather64(const int64_t *off, const int64_t *at, int64_t count, int64_t *out, hipStream_t s) {
  hipLaunchKernelGGL(k_gather64, dim3(blocks_for(count, 1024)), dim3(BS), 0, s, off, at, count, out);
  return hipGetLastError();
}

__global__ void k_gid(const int64_t *vtx_ptr, int32_t num_graphs, int32_t *gid) {
  for (int32_t g = blockIdx.x; g < num_graphs; g += gridDim.x)
    for (int64_t v = vtx_ptr[g] + threadIdx.x; v < vtx_ptr[g + 1]; v += blockDim.x) gid[v] = g;
}

hipError_t launch_graph_check(const CheckArgs &a, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  hipLaunchKernelGGL(a.validate ? k_check<true> : k_check<false>, dim3(4096), dim3(BS), 0, s, a);
  if (a.validate == 1) hipLaunchKernelGGL(k_check_counts, dim3(1), dim3(64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_graph_setup(const CheckArgs &a, int32_t num_graphs, int32_t *gid, int64_t *wall, int64_t *blocksum,
                              hipStream_t s) {
  const hipError_t e = launch_row_weights(a.off, a.n, wall, blocksum, s);
  if (e != hipSuccess) return e;
  if (gid) hipLaunchKernelGGL(k_gid, dim3(num_graphs < 4096 ? num_graphs : 4096), dim3(BS), 0, s, a.vtx_ptr,
                              num_graphs, gid);
  return launch_graph_check(a, s);
}

// ----------------------------------------------------------- renumbering --
// Internal vertex ids group the vertices by degree level floor(log2 deg),
// highest level first and isolated vertices last.  A neighbour scan touches
// a vertex about as often as its degree, so the per-vertex state it reads
// most (that of the hubs) sits in a few contiguous lines that stay cached.
// Within a level the order is whatever the atomics give: no result depends
// on internal ids (labels and every record are mapped back or id-free).
constexpr int RBINS = RELABEL_BINS;
__device__ inline int relabel_bin(int64_t d) { return d > 0 ? NLVL - 1 - level_of(d) : NLVL; }

// count[0, RBINS): vertices per bin; count[2 RBINS]: the largest degree.
__global__ void __launch_bounds__(BS) k_relabel_count(const int64_t *off, int64_t n, unsigned *count) {
  __shared__ unsigned s_cnt[RBINS];
  __shared__ int s_max;
  if (threadIdx.x < RBINS) s_cnt[threadIdx.x] = 0;
  if (threadIdx.x == 0) s_max = 0;
  __syncthreads();
  int mx = 0;
  for (int64_t v = (int64_t)blockIdx.x * BS + threadIdx.x; v < n; v += (int64_t)gridDim.x * BS) {
    const int64_t d = off[v + 1] - off[v];
    mx = (int)d > mx ? (int)d : mx;
    atomicAdd(&s_cnt[relabel_bin(d)], 1u);
  }
  mx = wave_max(mx);
  if (lane_id() == 0) atomicMax(&s_max, mx);
  __syncthreads();
  if (threadIdx.x == 0 && s_max) atomicMax(&count[2 * RBINS], (unsigned)s_max);
  if (threadIdx.x < RBINS && s_cnt[threadIdx.x]) atomicAdd(&count[threadIdx.x], s_cnt[threadIdx.x]);
}

// Each workgroup takes a contiguous chunk, reserves its range in every bin
// with one atomic, then places its vertices.
__global__ void __launch_bounds__(BS) k_relabel_assign(const int64_t *off, int64_t n, const int64_t *bin_off,
                                                       unsigned *cursor, int32_t *perm, int32_t *iperm) {
  __shared__ unsigned s_cnt[RBINS], s_base[RBINS];
  const int64_t per = (n + gridDim.x - 1) / gridDim.x;
  const int64_t v0 = (int64_t)blockIdx.x * per, v1 = v0 + per < n ? v0 + per : n;
  if (threadIdx.x < RBINS) s_cnt[threadIdx.x] = 0;
  __syncthreads();
  for (int64_t v = v0 + threadIdx.x; v < v1; v += BS) atomicAdd(&s_cnt[relabel_bin(off[v + 1] - off[v])], 1u);
  __syncthreads();
  if (threadIdx.x < RBINS) {
    s_base[threadIdx.x] = s_cnt[threadIdx.x] ? atomicAdd(&cursor[threadIdx.x], s_cnt[threadIdx.x]) : 0u;
    s_cnt[threadIdx.x] = 0;
  }
  __syncthreads();
  for (int64_t v = v0 + threadIdx.x; v < v1; v += BS) {
    const int b = relabel_bin(off[v + 1] - off[v]);
    const int64_t p = bin_off[b] + s_base[b] + atomicAdd(&s_cnt[b], 1u);
    perm[v] = (int32_t)p;
    iperm[p] = (int32_t)v;
  }
}

// rdeg[i] = degree of internal vertex i (its original row's length)
__global__ void __launch_bounds__(BS) k_relabel_degrees(const int64_t *off, int64_t n, const int32_t *iperm,
                                                        int64_t *rdeg) {
  for (int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x; i < n; i += (int64_t)gridDim.x * BS) {
    const int32_t v = iperm[i];
    rdeg[i] = off[v + 1] - off[v];
  }
}

// Exclusive scan of rdeg into roff (block partial sums, then their scan, then add).
__global__ void __launch_bounds__(BS) k_plain_scan_local(const int64_t *x_in, int64_t n, int64_t *out,
                                                         int64_t *blocksum) {
  __shared__ int64_t sh[WAVES + 1];
  const int64_t base = ((int64_t)blockIdx.x * BS + threadIdx.x) * SCAN_T;
  int64_t x[SCAN_T], s = 0;
#pragma unroll
  for (int k = 0; k < SCAN_T; k++) {
    x[k] = base + k < n ? x_in[base + k] : 0;
    s += x[k];
  }
  int64_t tot;
  int64_t pre = wg_excl_scan(s, &tot, sh);
#pragma unroll
  for (int k = 0; k < SCAN_T; k++) {
    if (base + k < n) out[base + k] = pre;
    pre += x[k];
  }
  if (threadIdx.x == 0) blocksum[blockIdx.x] = tot;
}

// rcol[roff[perm[v]] + j] = perm[col[off[v] + j]], edge-balanced over the input rows.
__global__ void __launch_bounds__(BS) k_relabel_cols(const int64_t *off, const int32_t *col, const int64_t *wall,
                                                     int64_t n, const int32_t *perm, const int64_t *roff,
                                                     int32_t *rcol) {
  lb_walk(nullptr, wall, n, wall[n], off, off + 1, col, perm, nullptr, [&](Items &it) {
#pragma unroll
    for (int k = 0; k < IPT; k++) {
      if (!(it.edge >> k & 1)) continue;
      const int64_t local = it.pos[k] - off[it.v[k]];
      rcol[roff[it.val[k]] + local] = perm[it.u[k]];
    }
  });
}

hipError_t launch_relabel(const int64_t *off, const int32_t *col, const int64_t *wall, int64_t n, unsigned *count,
                          int64_t *bin_off_dev, int32_t *perm, int32_t *iperm, int64_t *rdeg, int64_t *roff,
                          int64_t *blocksum, int32_t *rcol, unsigned *bins, int64_t *max_deg, hipStream_t s) {
  for (int b = 0; b < RBINS; b++) bins[b] = 0;
  *max_deg = 0;
  if (n == 0) return hipMemsetAsync(roff, 0, sizeof(int64_t), s);
  const unsigned g = blocks_for(n, 4096);
  hipError_t e = hipMemsetAsync(count, 0, sizeof(unsigned) * (2 * RBINS + 1), s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_relabel_count, dim3(g), dim3(BS), 0, s, off, n, count);
  unsigned hc[2 * RBINS + 1];
  e = hipMemcpyAsync(hc, count, sizeof(hc), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return e;
  *max_deg = hc[2 * RBINS];
  int64_t hb[RBINS], acc = 0;
  for (int b = 0; b < RBINS; b++) {
    bins[b] = hc[b];
    hb[b] = acc;
    acc += hc[b];
  }
  e = hipMemcpyAsync(bin_off_dev, hb, sizeof(hb), hipMemcpyHostToDevice, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_relabel_assign, dim3(g), dim3(BS), 0, s, off, n, bin_off_dev, count + RBINS, perm, iperm);
  hipLaunchKernelGGL(k_relabel_degrees, dim3(g), dim3(BS), 0, s, off, n, iperm, rdeg);
  const int64_t per = (int64_t)BS * SCAN_T;
  const int64_t nb = (n + per - 1) / per;
  hipLaunchKernelGGL(k_plain_scan_local, dim3((unsigned)nb), dim3(BS), 0, s, rdeg, n, roff, blocksum);
  hipLaunchKernelGGL(k_wscan_blocks, dim3(1), dim3(BS), 0, s, blocksum, nb, blocksum + nb);
  hipLaunchKernelGGL(k_wscan_add, dim3((unsigned)nb), dim3(BS), 0, s, roff, n, blocksum, blocksum + nb);
  hipLaunchKernelGGL(k_relabel_cols, dim3(4096), dim3(BS), 0, s, off, col, wall, n, perm, roff, rcol);
  return hipGetLastError();
}

// ------------------------------------------------------------------ cost --

struct CostArgs {
  const int64_t *off;
  const int32_t *col;
  const int64_t *wall;
  int64_t n;
  const int64_t *vtx_ptr;
  const int32_t *gid;
  const int32_t *labels;
  int32_t *size;     // [n] cluster sizes, indexed by graph base + label
  long long *acc;    // [2 * num_graphs]: pairs inside clusters, same-label adjacency entries
  int *err;
};

// Per-lane running sums flushed when the graph changes; the whole workgroup
// adds once when every lane ends on the same graph.
__device__ inline void flush_acc(long long *acc, int slot, int g, long long x) {
  __shared__ int s_g, s_mixed;
  __shared__ long long s_sum;
  if (threadIdx.x == 0) {
    s_g = g;
    s_mixed = 0;
    s_sum = 0;
  }
  __syncthreads();
  if (g != s_g) s_mixed = 1;
  __syncthreads();
  if (s_mixed) {
    if (x) atomicAdd((unsigned long long *)&acc[2 * g + slot], (unsigned long long)x);
  } else {
    const int64_t ws = wave_sum((int64_t)x);
    if (lane_id() == 0 && ws) atomicAdd((unsigned long long *)&s_sum, (unsigned long long)ws);
    __syncthreads();
    if (threadIdx.x == 0 && s_sum) atomicAdd((unsigned long long *)&acc[2 * g + slot], (unsigned long long)s_sum);
  }
}

__global__ void __launch_bounds__(BS) k_cost_sizes(CostArgs a) {
  for (int64_t v = (int64_t)blockIdx.x * BS + threadIdx.x; v < a.n; v += (int64_t)gridDim.x * BS) {
    int64_t base = 0, ng = a.n;
    if (a.gid) {
      const int32_t g = a.gid[v];
      base = a.vtx_ptr[g];
      ng = a.vtx_ptr[g + 1] - base;
    }
    const int32_t l = a.labels[v];
    if (l < 0 || (int64_t)l >= ng) {
      report(a.err, 1);  // CC_ERR_INVALID_ARG: label outside its graph
      continue;
    }
    atomicAdd(&a.size[base + l], 1);
  }
}

__global__ void __launch_bounds__(BS) k_cost_same(CostArgs a) {
  int g_cur = -1;
  long long run = 0;
  lb_walk(nullptr, a.wall, a.n, a.wall[a.n], a.off, a.off + 1, a.col, a.labels, nullptr, [&](Items &it) {
#pragma unroll
    for (int k = 0; k < IPT; k++) {
      if (!(it.edge >> k & 1)) continue;
      int g = 0;
      int64_t base = 0;
      if (a.gid) {
        g = a.gid[it.v[k]];
        base = a.vtx_ptr[g];
      }
      if (g != g_cur) {
        if (g_cur >= 0 && run) atomicAdd((unsigned long long *)&a.acc[2 * g_cur + 1], (unsigned long long)run);
        g_cur = g;
        run = 0;
      }
      if (a.labels[base + it.u[k]] == it.val[k]) run++;
    }
  });
  flush_acc(a.acc, 1, g_cur < 0 ? 0 : g_cur, run);
}

// A single graph is scored on its renumbered rows.  Every edge is stored
// twice, and the entry whose neighbour has the lower internal id is the one
// to look at: ids fall with the degree level, so the gathers (one per edge
// instead of two) land mostly on the hubs' labels, which stay cached.  A row's
// own vertex (unvalidated rows may hold it) is one entry and counts as one.
__global__ void __launch_bounds__(BS) k_cost_labels(CostArgs a, const int32_t *iperm, int32_t *lab) {
  for (int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x; i < a.n; i += (int64_t)gridDim.x * BS) {
    const int32_t l = a.labels[iperm[i]];
    lab[i] = l;
    if (l < 0 || (int64_t)l >= a.n) report(a.err, 1);  // CC_ERR_INVALID_ARG: label outside its graph
    else atomicAdd(&a.size[l], 1);
  }
}

// The rows are consecutive and none is empty, so an entry's place in col says
// where it is without its row: a workgroup loads a tile of columns while it
// finds the rows the tile holds, four entries (16 bytes) per thread and load.
// What bounds it is the chain of a tile (offsets, LDS search, label gather),
// so a tile takes little LDS and there are many workgroups, each on a few
// tiles in a row (hub rows and short ones take very different times).  R-MAT
// 24 (0.5 G entries), whole call: 8.4 ms by label gathers on the input rows,
// 3.05 ms on these rows with the general walk, 2.80 / 2.33 / 2.04 / 1.94 ms
// here with 2 K / 4 K / 8 K / 16 K workgroups (2.90 with CE_K = 4 and 2 K);
// power law 2 M, 80 M entries: 0.51 ms, then 0.41 / 0.45 / 0.43 / 0.48.
constexpr int CE_K = 2;                  // 16-byte loads per thread and tile
constexpr int CE_TILE = BS * 4 * CE_K;

__global__ void __launch_bounds__(BS) k_cost_edges(CostArgs a, const int32_t *lab, int64_t rows) {
  __shared__ int32_t lw[CE_TILE + 1];  // first entry of the tile's row j, from the tile's start (-1: before it)
  __shared__ int32_t ll[CE_TILE];      // its label
  __shared__ int64_t s_row;
  const int64_t nnz = a.off[rows];
  const int64_t ntiles = (nnz + CE_TILE - 1) / CE_TILE;
  const int64_t per = (ntiles + gridDim.x - 1) / gridDim.x;
  const int64_t t0 = (int64_t)blockIdx.x * per, t1 = t0 + per < ntiles ? t0 + per : ntiles;
  if (t0 >= t1) return;
  if (threadIdx.x < 64) {
    const int64_t r = wave_find_entry(a.off, rows, t0 * CE_TILE);
    if (threadIdx.x == 0) s_row = r;
  }
  __syncthreads();
  int64_t row0 = s_row;  // the row that holds the tile's first entry
  long long run = 0, loops = 0;
  for (int64_t t = t0; t < t1; t++) {
    const int64_t s = t * CE_TILE;
    const int items = (int)(nnz - s < CE_TILE ? nnz - s : CE_TILE);
    int32_t u[CE_K][4];
#pragma unroll
    for (int k = 0; k < CE_K; k++) {
      const int x = (k * BS + (int)threadIdx.x) * 4;
      if (x + 3 < items) {  // (a.col + s is 16-byte aligned: s is a multiple of the tile)
        const int4 q = *reinterpret_cast<const int4 *>(a.col + s + x);
        u[k][0] = q.x;
        u[k][1] = q.y;
        u[k][2] = q.z;
        u[k][3] = q.w;
      } else {
#pragma unroll
        for (int y = 0; y < 4; y++) u[k][y] = x + y < items ? a.col[s + x + y] : 0x7fffffff;
      }
    }
    int nrow = 0;  // rows that start before the tile's end
    for (;;) {
      const int64_t r = row0 + nrow + threadIdx.x;
      int64_t o = INT64_MAX;
      int32_t l = 0;
      if (r < rows && nrow + (int)threadIdx.x < CE_TILE) {
        o = a.off[r];
        l = lab[r];
      }
      const bool in = o < s + items;
      if (in) {
        lw[nrow + threadIdx.x] = o < s ? -1 : (int32_t)(o - s);
        ll[nrow + threadIdx.x] = l;
      }
      const int c = __syncthreads_count(in);
      nrow += c;
      if (c < BS) break;
    }
#pragma unroll
    for (int k = 0; k < CE_K; k++) {
      const int x = (k * BS + (int)threadIdx.x) * 4;
      int j = lds_last_le(lw, nrow, x < items ? x : items - 1);  // (behind the end: no rows to step over)
      int32_t g[4], m[4];
#pragma unroll
      for (int y = 0; y < 4; y++) {
        while (j + 1 < nrow && lw[j + 1] <= x + y) j++;
        const int32_t v = (int32_t)row0 + j;
        g[y] = u[k][y] < v ? lab[u[k][y]] : -1;
        loops += u[k][y] == v;
        m[y] = ll[j];
      }
#pragma unroll
      for (int y = 0; y < 4; y++) run += g[y] >= 0 && g[y] == m[y];
    }
    // the next tile starts in the last row, or at the start of the one after
    row0 += nrow - 1;
    if (row0 + 1 < rows && a.off[row0 + 1] == s + CE_TILE) row0++;
    __syncthreads();
  }
  flush_acc(a.acc, 1, 0, 2 * run + loops);
}

constexpr int PAIR_T = 64;  // consecutive label slots per thread

__global__ void __launch_bounds__(BS) k_cost_pairs(CostArgs a) {
  int g_cur = -1;
  long long run = 0;
  const int64_t stride = (int64_t)gridDim.x * BS * PAIR_T;
  for (int64_t r0 = ((int64_t)blockIdx.x * BS + threadIdx.x) * PAIR_T; r0 < a.n; r0 += stride) {
    for (int64_t r = r0; r < r0 + PAIR_T && r < a.n; r++) {
      const int g = a.gid ? a.gid[r] : 0;
      if (g != g_cur) {
        if (g_cur >= 0 && run) atomicAdd((unsigned long long *)&a.acc[2 * g_cur], (unsigned long long)run);
        g_cur = g;
        run = 0;
      }
      const long long s = a.size[r];
      run += s * (s - 1) / 2;
    }
  }
  flush_acc(a.acc, 0, g_cur < 0 ? 0 : g_cur, run);
}

hipError_t launch_cost(const CostGraph &g, const int32_t *labels, int32_t *size, int32_t *lab, long long *acc, int *err,
                       hipStream_t s) {
  const int64_t n = g.n;
  hipError_t e = hipMemsetAsync(size, 0, sizeof(int32_t) * (size_t)(n > 0 ? n : 1), s);
  if (e == hipSuccess) e = hipMemsetAsync(acc, 0, sizeof(long long) * 2 * (size_t)g.num_graphs, s);
  if (e != hipSuccess || n == 0) return e;
  const bool single = g.iperm != nullptr;
  CostArgs a{single ? g.roff : g.off, single ? g.rcol : g.col, g.wall, n, g.vtx_ptr, g.gid, labels, size, acc, err};
  const unsigned gv = (unsigned)((n + BS - 1) / BS < 4096 ? (n + BS - 1) / BS : 4096);
  if (single) {
    hipLaunchKernelGGL(k_cost_labels, dim3(gv), dim3(BS), 0, s, a, g.iperm, lab);
    if (g.iso_start > 0) {
      const int64_t w = g.nnz / (8 * CE_TILE) + 1;  // workgroups of about eight tiles
      hipLaunchKernelGGL(k_cost_edges, dim3((unsigned)(w < 2048 ? 2048 : w < 16384 ? w : 16384)), dim3(BS), 0, s, a, lab,
                         g.iso_start);
    }
  } else {
    hipLaunchKernelGGL(k_cost_sizes, dim3(gv), dim3(BS), 0, s, a);
    hipLaunchKernelGGL(k_cost_same, dim3(4096), dim3(BS), 0, s, a);
  }
  const int64_t pg = (n + (int64_t)BS * PAIR_T - 1) / ((int64_t)BS * PAIR_T);
  hipLaunchKernelGGL(k_cost_pairs, dim3((unsigned)(pg < 2048 ? pg : 2048)), dim3(BS), 0, s, a);
  return hipGetLastError();
}

}  // namespace ccd
