// cc_round.h -- the parts of a round that its kernels share: batch sizes,
// the lazy Delta search's state, the rows a phase walks, the degree histogram.
#pragma once
#include "cc_device.h"

namespace ccd {

// Who runs the round just sized; rate: entries walked per active vertex in
// the round before.
__device__ inline int next_stage(const Ws &w, long long b, long long cursor, long long n_rem, float rate) {
  if (!w.team) return ST_SELECT;
  if (w.team_n <= 1) return ST_TEAM;
  const double ahead = (double)(w.n - cursor);
  const double pos = w.policy == POL_BINOMIAL ? (double)b : (double)b * ahead / (double)(n_rem > 0 ? n_rem : 1);
  return pos <= (double)TEAM_POS && (double)b * rate <= (double)TEAM_ITEMS ? ST_TEAM : ST_SELECT;
}

// Whether a round kernel of stage `mine` has anything to do.
__device__ inline bool idle(const CtrlHead &h, int mine) {
  return h.done || (unsigned)(h.stage - 1) >= (unsigned)mine;
}

// Per-row partial counts of rows split across tiles: one 64-bit atomic adds
// (items covered << 32 | count); the contributor that completes the row
// (covered == degree) owns the total.
__device__ inline bool row_combine(unsigned long long *acc, int64_t slot, int cnt, int64_t covered, int32_t deg,
                                   int *total) {
  const unsigned long long add = ((unsigned long long)covered << 32) | (unsigned)cnt;
  const unsigned long long tot = atomicAdd(&acc[slot], add) + add;
  if ((int64_t)(tot >> 32) != (int64_t)deg) return false;
  *total = (int)(tot & 0xFFFFFFFFu);
  return true;
}

// The rows a round walks: the full rows until the run switches to exact
// degrees, the rows the switch compacted after it (the phase is read at the
// start of each kernel and changes only at the end of a round, in k_close).
__device__ inline const int64_t *round_end(const Ws &w, int phase) { return phase == PHASE_EXACT ? w.xend : w.rend; }
__device__ inline const int32_t *round_col(const Ws &w, int phase) { return phase == PHASE_EXACT ? w.xcol : w.col; }

__device__ inline void hist_add(int *s_hist, int *g_hist, int d, int x) {
  if (d <= 0) return;
  if (d < HLDS) atomicAdd(&s_hist[d], x);
  else atomicAdd(&g_hist[d], x);
}

// --------------------------------------------- settling the blocked ------
// The blocked vertices of a C4 round in one workgroup's LDS.  A vertex's word
// counts its earlier active neighbours that are not settled as non-centers:
// 0 makes it a center, and an earlier center sets RES_NON in it (what the
// other neighbours take off afterwards leaves it above RES_GONE).  Every
// thread looks at its edges until each has met its earlier end settled; the
// edges run from later to earlier ranks and every wave of the workgroup is
// running, so some edge always can be, and no barrier is needed between one
// level of the dependence and the next.  (The looks are bounded all the same;
// a word that is neither then says so.)
constexpr int RES_NON = 1 << 30, RES_GONE = 1 << 29;
constexpr int RES_LOOKS = 1 << 24;

__device__ inline int res_word(const int *word, int i) {
  return __hip_atomic_load(&word[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// `open`: this thread's edges, bit k the edge from blocked vertex a(k) to the
// earlier u(k) (below 0: a center); the words hold the counts.  Collective for
// a wave, which looks at eight edges per lane together and stays with them
// while they settle: neighbours in a chain are often listed next to each other.
template <int EPT, class A, class U>
__device__ __forceinline__ void settle_edges(int *word, unsigned open, A &&a, U &&u) {
  constexpr int CH = 8;
  for (int look = 0; __any(open) && look < RES_LOOKS; look++) {
#pragma unroll
    for (int k0 = 0; k0 < EPT; k0 += CH) {
      unsigned now = open >> k0 & 0xFF, settled = now;
      while (__any(now) && __any(settled)) {
        settled = 0;
        int wu[CH];
#pragma unroll
        for (int k = 0; k < CH; k++) wu[k] = (now >> k & 1) == 0 ? 1 : u(k0 + k) < 0 ? 0 : res_word(word, u(k0 + k));
#pragma unroll
        for (int k = 0; k < CH; k++)
          if (now >> k & 1) {
            if (wu[k] == 0) atomicOr(&word[a(k0 + k)], RES_NON);
            else if (wu[k] >= RES_GONE) atomicSub(&word[a(k0 + k)], 1);
            else continue;
            settled |= 1u << k;
          }
        now &= ~settled;
      }
      open = (open & ~(0xFFu << k0)) | now << k0;
    }
  }
}

// After a barrier: 1 a center, 2 a non-center, 0 unsettled.
__device__ inline int res_decision(int word) { return word == 0 ? 1 : word >= RES_GONE ? 2 : 0; }

// ------------------------------------------------------------ policy ------

__device__ inline long long fixed_batch(long long eps_q, long long n_rem, long long delta) {
  if (delta <= 0) return n_rem;
  // ceil(num / den): num < 2^62 and den >= 10^6, so the quotient stays below
  // 2^43, its double estimate is off by less than one, and two comparisons
  // make it exact (a 64-bit division is a few hundred instructions)
  const long long num = eps_q * n_rem, den = 1000000LL * delta;
  long long b = (long long)((double)num / (double)den);
  if (b * den < num) b++;
  if ((b - 1) * den >= num) b--;
  if (b < 1) b = 1;
  if (b > n_rem) b = n_rem;
  return b;
}

// Learned policy: eps = clamp(exp(w2 . relu(W1 x + b1) + b2)).  A whole wave;
// lane j computes hidden unit j.  Returns false on a non-finite output.
__device__ inline bool mlp_eps(const Ws &w, const float x[6], float *eps_out) {
  const float *W1 = w.mlp, *b1 = w.mlp + 64 * 6, *w2 = b1 + 64, *b2 = w2 + 64;
  const int j = lane_id();
  float h = b1[j];
#pragma unroll
  for (int k = 0; k < 6; k++) h = fmaf(W1[j * 6 + k], x[k], h);
  h = h > 0.f ? h : 0.f;
  float y = w2[j] * h;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) y += __shfl_xor(y, d, 64);
  // a lane's product may be fused into its first sum, so the lanes' sums can
  // differ in the last place: the first lane's is the wave's
  y = __shfl(y, 0, 64) + b2[0];
  if (!isfinite(y)) return false;
  float e = expf(y);
  e = fminf(fmaxf(e, w.eps_min), w.eps_max);
  *eps_out = e;
  return isfinite(e);
}

// Delta-hat of round i under the practical schedule: Delta_0 halved every
// bin_period rounds (rounded down, as the trace records it).
__device__ inline long long delta_hat(const Ws &w, long long round) {
  const long long h = round / w.bin_period;
  return h >= 63 ? 0 : (long long)w.max_deg >> h;
}

// Sizes the next round; called by all lanes of a wave with the same values.
__device__ inline void next_batch(const Ws &w, long long n_rem, long long delta, long long round, float fconf,
                           float fclaim, float feps, long long *b_out, double *eps_out, int *fallback) {
  long long b = 0;
  double eps_used = w.eps;
  bool have = false;
  if (w.policy == POL_BINOMIAL) {  // round < sched_len: checked by the caller
    b = w.sched[round];
    eps_used = w.eps;
    have = true;
  } else if (w.policy == POL_TRACE && round < w.sched_len) {
    b = w.sched[round];
    if (b > n_rem) b = n_rem;
    eps_used = delta > 0 ? (double)b * (double)delta / (double)n_rem : 0.0;
    have = true;
  } else if (w.policy == POL_LEARNED) {
    float x[6] = {logf((float)n_rem), logf((float)(delta > 1 ? delta : 1)), fconf, fclaim, feps, (float)round};
    float e = 0.f;
    if (mlp_eps(w, x, &e)) {
      const long long q = (long long)((double)e * 1e6 + 0.5);
      b = fixed_batch(q > 0 ? q : 1, n_rem, delta);
      eps_used = (double)e;
      have = true;
    } else {
      *fallback = 1;
    }
  }
  if (!have) b = fixed_batch(w.eps_q, n_rem, delta);
  *b_out = b;
  *eps_out = eps_used;
}

// ------------------------------------------------- lazy Delta search -----
// Pass j rescans every candidate whose bound is >= L_j = ceil(f_j * T_j)
// (T_0 = Delta_i; f = 0.7, 0.3, 0.05).  Every other vertex has a bound below
// L_j, so if the largest exact degree found is >= L_j it is Delta_{i+1};
// otherwise T_{j+1} = L_j - 1.  When a band floor would fall below SWL, or all
// passes fail, the run switches to exact remaining degrees.

struct DSearch {
  int pending;      // 1 while the search still needs the next pass
  int switching;    // 1 when the run moves to exact degrees
  long long delta;  // resolved Delta (when neither pending nor switching)
  long long T, L;   // bounds of the pending pass
};

__device__ inline long long band_floor(int pass, long long T) {
  return (long long)ceilf(band_factor(pass) * (float)T);
}

// State of the search after `done` passes (every thread computes the same);
// C is Ctrl or a CtrlHead snapshot of it.
template <class C>
__device__ inline DSearch dsearch(const C *c, int done) {
  DSearch s{0, 0, -1, 0, 0};
  if (c->phase != PHASE_LAZY) return s;
  long long T = c->delta;
#pragma unroll
  for (int j = 0; j < DITER; j++) {  // (a fixed count, so that no index of d_max is one of a register array)
    if (j >= done) break;
    const long long L = band_floor(j, T);
    if (L < SWL) {  // pass j never ran: the search switched before it
      s.switching = 1;
      return s;
    }
    const long long M = c->d_max[j];
    if (M >= L) {
      s.delta = M;
      return s;
    }
    T = L - 1;
  }
  if (done >= DITER || band_floor(done, T) < SWL) {
    s.switching = 1;
    return s;
  }
  s.pending = 1;
  s.T = T;
  s.L = band_floor(done, T);
  return s;
}


}  // namespace ccd
