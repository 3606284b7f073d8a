// nf_decide.h - what the kernels that reduce pass 1's partial statistics and
// decide a bucket's route share (k_slotsum and k_decide, k_small2).
#pragma once

#include "nf_device.h"

namespace nf {

// The wavefront's |g| sum of one worker as an XSum: in exact mode from the
// lanes' (s, c) pairs, otherwise the plain wavefront sum with no error kept.
template <bool EXACT>
__device__ __forceinline__ XSum lane_sum(double s, double c, uint32_t nz) {
  if constexpr (EXACT) return wave_xsum(xlane(s, c, nz));
  return XSum{wave_sum(s), 0.0, 0.0};
}

// p += q for partial statistics; in exact mode the |g| sums as XSums, else
// as plain FP64 sums (their error parts stay 0).
template <bool EXACT>
__device__ __forceinline__ void part_add(Partial& p, const Partial& q) {
  if constexpr (EXACT) {
    const XSum x = xcombine(XSum{p.sabs, p.sabs_c, p.sabs_b}, XSum{q.sabs, q.sabs_c, q.sabs_b});
    p.sabs = x.s;
    p.sabs_c = x.c;
    p.sabs_b = x.b;
  } else {
    p.sabs += q.sabs;
  }
  p.ssq += q.ssq;
  p.nonfinite += q.nonfinite;
}

// Exact mode: a worker whose rounding the bound could not certify is summed
// again from its gradients, exactly (rare: it takes a total within the bound
// of a rounding midpoint).  Returns how many were; every thread calls, and
// st is complete for all of them on return.
__device__ __forceinline__ uint32_t resum_exact(nf_worker_stats* st, const uint8_t* redo, const DecideArgs& a,
                                                int64_t base, int64_t nbe, unsigned long long* hist) {
  uint32_t resummed = 0;
  for (int w = 0; w < a.W; ++w) {
    if (!redo[w]) continue;  // block-uniform
    const double e = exact_abs_sum(a.g + (int64_t)w * a.wstride, a.mask, base, nbe, hist);
    if (threadIdx.x == 0) st[w].sum_abs_elig = e;
    ++resummed;
  }
  __syncthreads();
  return resummed;
}

struct DecideScratch {
  double med;
  double qterm[256];  // |g| sum / n_E per worker (the scale's terms)
};

// The decision of one bucket from its statistics st (LDS), by a block of at
// least 256 threads; thread 0 writes *dec.  The per-worker facts of the
// route rules, thread t for worker t (W <= 255): finite sums of squares
// counted by a block vote, the lower median by rank, the scale's terms |g|
// sum / n_E divided in parallel and added in worker order by one thread (as
// the host's decision adds them), and the reason flags by block votes.
// (With one thread scanning the workers the decision of two 255-worker
// buckets took 88 us; this way, 49 us.)
__device__ __forceinline__ void decide_block(const nf_worker_stats* st, int W, int64_t nbe, int64_t ne,
                                             const nf_route_policy& pol, uint32_t resummed, DecideScratch& scr,
                                             nf_route_decision* dec) {
  const int t = threadIdx.x;
  const bool mine = t < W;
  const double ssq = mine ? st[t].sum_sq : 0.0;
  const double sab = mine ? st[t].sum_abs_elig : 0.0;
  const bool fin = mine && finite64(ssq);
  if (t == 0) scr.med = 0.0;
  const int kfin = __syncthreads_count(fin);
  if (fin && ssq_rank(st, W, t) == (kfin - 1) / 2) scr.med = ssq;
  if (mine) scr.qterm[t] = ne > 0 ? sab / (double)ne : 0.0;
  const int nonf = __syncthreads_or(mine && st[t].nonfinite != 0);
  const int zero = __syncthreads_or(mine && sab == 0.0);
  const int spike = __syncthreads_or(kfin >= 2 && fin && ssq > spike_threshold(pol, scr.med));
  if (t == 0) {
    float scale = 0.0f;
    if (ne > 0) {
      double acc = 0.0;
#pragma unroll 4
      for (int w = 0; w < W; ++w) acc += scr.qterm[w];
      scale = (float)(acc / (double)W);
    }
    nf_route_decision d;
    decide_finish(nbe, ne, pol, nonf != 0, zero != 0, spike != 0, scale, &d);
    d.resummed = resummed;
    *dec = d;
  }
}

// decide_block by one wavefront, lane w for worker w (W <= 64): no barriers,
// the workers' values exchanged by scalar reads.  The same bits.
__device__ __forceinline__ void decide_wave(const nf_worker_stats* st, int W, int64_t nbe, int64_t ne,
                                            const nf_route_policy& pol, uint32_t resummed,
                                            nf_route_decision* dec) {
  const int t = threadIdx.x & 63;
  const bool mine = t < W;
  const double ssq = mine ? st[t].sum_sq : 0.0;
  const double sab = mine ? st[t].sum_abs_elig : 0.0;
  const bool fin = mine && finite64(ssq);
  const uint64_t fins = __ballot(fin);
  const int kfin = __popcll(fins);
  const double q = mine && ne > 0 ? sab / (double)ne : 0.0;
  int rank = 0;
  double acc = 0.0;
  for (int u = 0; u < W; ++u) {
    const double x = lane_value(ssq, u);
    if ((fins >> u) & 1ull) rank += (x < ssq || (x == ssq && u < t)) ? 1 : 0;
    acc += lane_value(q, u);
  }
  const uint64_t at = __ballot(fin && rank == (kfin - 1) / 2);
  const double med = at ? lane_value(ssq, __builtin_ctzll(at)) : 0.0;
  const bool nonf = __ballot(mine && st[t].nonfinite != 0) != 0;
  const bool zero = __ballot(mine && sab == 0.0) != 0;
  const bool spike = __ballot(kfin >= 2 && fin && ssq > spike_threshold(pol, med)) != 0;
  if (t == 0) {
    nf_route_decision d;
    decide_finish(nbe, ne, pol, nonf, zero, spike, ne > 0 ? (float)(acc / (double)W) : 0.0f, &d);
    d.resummed = resummed;
    *dec = d;
  }
}

}  // namespace nf
