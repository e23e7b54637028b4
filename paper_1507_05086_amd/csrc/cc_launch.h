// cc_launch.h -- host-side entry points of the kernels (C++ linkage, internal).
#pragma once
#include <hip/hip_runtime.h>

#include "cc_device.h"

namespace ccd {

struct LaunchShape {
  unsigned select_grid;  // workgroups of the active-set scan
  unsigned edge_grid;    // workgroups of the edge-balanced passes
  unsigned vertex_grid;  // workgroups of per-vertex list passes
  int exact_seen;        // the host saw the run switch to exact degrees
};

hipError_t launch_init(const Ws &w, hipStream_t s);
// The kernels of one round, in order; each takes the run's Ws.
struct RoundStep {
  void (*kernel)(Ws);
  unsigned grid, block;
};
constexpr int ROUND_STEPS = 12;  // at most
int round_steps(const Ws &w, const LaunchShape &ls, RoundStep *out);
RoundStep team_step(const Ws &w);
// Rounds on one XCD (cc_team.hip) until one is for the whole device; w.team set.
hipError_t launch_team(const Ws &w, hipStream_t s);
hipError_t launch_finalize(const Ws &w, int32_t *labels, hipStream_t s);
// Copies n labels (device memory, any alignment) unless *error is set.
hipError_t launch_deliver(const int32_t *from, int32_t *to, int64_t n, const int *error, hipStream_t s);

// Offsets of a graph on the device: out[0] = offsets[n], out[1] != 0 if they
// do not start at 0, out[2] != 0 if they decrease somewhere.
hipError_t launch_offsets_check(const int64_t *off, int64_t n, int64_t *out, hipStream_t s);
// out[i] = off[at[i]], i < count.
hipError_t launch_gather64(const int64_t *off, const int64_t *at, int64_t count, int64_t *out, hipStream_t s);

// Graph set-up: row-weight prefix wall[n+1] (the "all rows" list of the
// edge-balanced walk), per-row graph ids (batches), column-range check and,
// with validate, the symmetry / self-loop / duplicate checks.  *err receives
// the smallest failing cc_status code (it must hold 0x7fffffff beforehand),
// or CHECK_AGAIN when the checks of `validate` == 1 cannot tell which: then
// launch_graph_check with 2 finds it.  above: zeroed scratch word.
constexpr int CHECK_AGAIN = (1 << 8) | 0xFF;
struct CheckArgs {
  const int64_t *off;
  const int32_t *col;
  const int64_t *wall;
  int64_t n;
  const int64_t *vtx_ptr;  // device, or null
  const int32_t *gid;      // device per-row graph id, or null
  int validate;
  int *err;                // (priority << 8 | cc_status code) of the worst failure, 0x7fffffff = none
  unsigned long long *above;
};
hipError_t launch_graph_setup(const CheckArgs &a, int32_t num_graphs, int32_t *gid, int64_t *wall, int64_t *blocksum,
                              hipStream_t s);
hipError_t launch_graph_check(const CheckArgs &a, hipStream_t s);

// Batched C4 / ClusterWild!: one persistent launch over many small graphs.
struct BatchLaunch {
  const int64_t *off;
  const int32_t *col;
  const int64_t *vtx_ptr;
  const int32_t *order;
  int32_t *labels;
  const int32_t *queue;
  int32_t n_big, n_quad, num_graphs, cap_big, cap_quad, cap_wave;
  unsigned *heads;
  int32_t *rounds;
  unsigned long long *stat;
  int *err;
  int algo;
  int64_t eps_q;
  int block, grid;
  int64_t nnz;
};
hipError_t launch_batched(const BatchLaunch &bl, hipStream_t s);
size_t batched_lds_bytes(int block, int cap_big, int cap_quad, int cap_wave);
hipError_t batched_max_grid(int block, size_t lds, int *grid);

// Internal renumbering of a single graph (hubs first): perm (input id ->
// internal id), iperm, and the renumbered CSR roff / rcol.  count: 2 x
// RELABEL_BINS + 1 unsigned scratch, bin_off: RELABEL_BINS int64, rdeg: n
// int64, blocksum: n / (4 BS) + 2 int64.  On the host: vertices per bin (bin
// b < NLVL: degree level NLVL - 1 - b; the last: degree 0) and the largest
// degree; the ids of a bin follow those of the bins before it.
constexpr int RELABEL_BINS = NLVL + 1;
hipError_t launch_relabel(const int64_t *off, const int32_t *col, const int64_t *wall, int64_t n, unsigned *count,
                          int64_t *bin_off_dev, int32_t *perm, int32_t *iperm, int64_t *rdeg, int64_t *roff,
                          int64_t *blocksum, int32_t *rcol, unsigned *bins, int64_t *max_deg, hipStream_t s);

// pi mapped into internal ids and checked as a permutation, in bucketed
// passes (cc_order.hip) for OM_MIN_N < n <= OM_MAX_BUCKETS * OM_SIZE; other
// sizes gather directly.  Bucket kb of positions and bucket vb of ids hold
// OM_SIZE each.  The scratch (order_map_bytes(n), one device allocation) is
// laid out by order_map_layout.  A failed check sets ERR_PERM in ctrl.
constexpr int OM_SHIFT = 15;
constexpr int64_t OM_SIZE = int64_t(1) << OM_SHIFT;
constexpr int OM_MAX_BUCKETS = 2048;
constexpr int64_t OM_MIN_N = int64_t(1) << 22;
struct OrderMap {
  int nk, nv;               // position buckets, id buckets
  int nkt, nvt;             // 64-bucket tiles of each
  unsigned *cnt;            // [nk][nv] entries of kb in vb; then where (kb, vb) starts in ent, by row
  unsigned *pt;             // [nv][nk] where (kb, vb) starts in ent, by column
  unsigned *qt;             // [nv][nk] where (kb, vb) starts in pent, by column
  unsigned *csum, *rsum;    // [nkt][nv] column and [nvt][nk] row sums of 64 x 64 tiles
  unsigned *vstart;         // [nv + 1] start of each id bucket in ent
  unsigned *ent;            // [n] k low bits | (id low bits << OM_SHIFT), by id bucket, then kb
  unsigned long long *pent; // [n] (internal id << OM_SHIFT) | k low bits, by position bucket
};
bool order_map_applies(int64_t n);
size_t order_map_bytes(int64_t n);
OrderMap order_map_layout(int64_t n, void *base);
// rank (optional): also rank[iorder[k]] = k, the inverse of pi in internal ids.
hipError_t launch_order_map(const OrderMap &m, const int32_t *order_in, const int32_t *perm, int64_t n,
                            int32_t *iorder, Ctrl *ctrl, hipStream_t s, int32_t *rank = nullptr);

// Asynchronous C4 / ClusterWild! (Algorithm 3): one persistent launch, no
// rounds.  rank and lab are workspace arrays of n; order is pi in internal
// ids (written by the launch from order_in through perm into iorder).
struct AsyncArgs {
  const int64_t *off;
  const int32_t *col;
  int64_t n;
  int64_t iso_start;
  const int32_t *order;
  int32_t *rank;
  int32_t *lab;
  Ctrl *ctrl;
  int32_t *big_v, *big_p;  // C4 centers whose claims are spread over the device (vertex, rank)
  int64_t big_cap;
};
// waves > 0 limits the launch to that many waves (1: pi strictly in order,
// 64 positions at a time); 0 fills the device.  ev0 / ev1 (optional) bracket
// the asynchronous kernel itself.
// om: the bucketed mapping of pi when it applies to this n, else nullptr.
hipError_t launch_async(const AsyncArgs &a, int algo, const int32_t *order_in, const int32_t *perm, int32_t *iorder,
                        int32_t *labels, int waves, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1,
                        const OrderMap *om);

// Learned-policy network: inference over a batch, one training step.
int mlp_grad_blocks(int n);
// The current device's static partial-row buffer (no allocation): its
// device address and how many rows it holds.
hipError_t mlp_scratch(float **ptr, int *rows);
hipError_t launch_mlp_forward(const float *p, const float *x, int n, float *y, hipStream_t s);
hipError_t launch_mlp_train_step(float *p, float *m, float *v, const float *x, const float *t, int n, long long step,
                                 float lr, float *partial, int nblk, float *grad, float *loss, hipStream_t s);

// Disagreement cost per graph: acc[2g] = pairs inside clusters, acc[2g+1] =
// same-label adjacency entries (2 m_in).  A single graph (iperm set) is
// scored on its renumbered rows, of which iso_start have entries; size and
// lab are scratch [n].
struct CostGraph {
  const int64_t *off;
  const int32_t *col;
  const int64_t *wall;
  int64_t n;
  const int64_t *vtx_ptr;
  const int32_t *gid;
  int32_t num_graphs;
  const int64_t *roff;
  const int32_t *rcol, *iperm;
  int64_t iso_start, nnz;
};
hipError_t launch_cost(const CostGraph &g, const int32_t *labels, int32_t *size, int32_t *lab, long long *acc, int *err,
                       hipStream_t s);

}  // namespace ccd
