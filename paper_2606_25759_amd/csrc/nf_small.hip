// nf_small.hip - decision and read side of a small problem in one launch
// (k_small2, gfx950): every block reduces its bucket's partials and decides
// the route itself, then counts and decodes, packs and counts the G-Ternary
// planes, or adds the workers in FP32.  Its write side is k_rows
// (nf_rows.hip).
//
// A small problem is one whose time is latency, not bandwidth: a few hundred
// chunks at most, one per compute unit (small_problem, nf_internal.h).
// Its gradients stay in the caches, so reading an element twice costs
// little, while every dependent step (a launch, a block barrier, a first
// fetch of an instruction line) costs a microsecond.
#include <hip/hip_ext.h>

#include "nf_decide.h"
#include "nf_device.h"

namespace nf {

// --------------------------------------------------- decision and read side
//
// Grid (blocks, buckets); four wavefronts a block.  Every block of a bucket
// repeats the bucket's decision from the partials (at most kSmallPartials of
// them, in the caches), in the same order, so all reach the same bits; block
// 0 stores it.  A launch of its own for the decision took 7 us on 8 x 70,001
// elements; repeated here it adds 2 to 3.
//
// G-Binary, route L: a wavefront takes 256 elements, lane l the elements 4l
// .. 4l + 3: one byte of every worker's row holds its nibble, which a
// multiply spreads over four count bytes, so no LDS transposes and sixteen
// times the wavefronts of k_pass2.  G-Ternary, route L: a wavefront takes one
// word, lane l element l: the gated ballots are the planes' words, and the
// lane's own bits its counts.  Route F: FP32 sums of the eligible elements.
template <bool TERNARY>
__global__ __launch_bounds__(kThreads2) void k_small2(Small2Args a) {
  constexpr bool EXACT = TERNARY;
  __shared__ nf_worker_stats st[kSmallWorkers];
  __shared__ unsigned long long hist[256];
  __shared__ nf_route_decision dec;
  __shared__ uint64_t ne_s;
  __shared__ uint8_t redo[kSmallWorkers];
  __shared__ float tab[2 * kSmallWorkers + 1];
  __shared__ float th[kSmallWorkers];
  const DecideArgs& d = a.d;
  const int b = blockIdx.y;
  const int W = d.W;
  const int t = threadIdx.x;
  const int lane = t & 63;
  const int v = __builtin_amdgcn_readfirstlane(t >> 6);
  int64_t base, nbe, chunk0;
  bucket_span(b, d.btab, d.n_total, d.bucket_n, d.slots, base, nbe, chunk0);
  const uint32_t chunk = (uint32_t)(d.tile * d.G);  // elements; a small problem has fewer than 2^24
  const int used = (int)(((uint32_t)nbe + chunk - 1) / chunk);
  const Partial* P = d.part + chunk0 * W;
  const int64_t step = (int64_t)gridDim.x * (kThreads2 / 64);
  const int64_t first = (int64_t)blockIdx.x * (kThreads2 / 64) + v;
  // G-Binary: four counts from element i0 of the bucket on, one a byte
  const uint8_t* rows = reinterpret_cast<const uint8_t*>(a.bits + base / 64);
  const int64_t rstride = a.bstride * 8;
  const int sh = 4 * (lane & 1);
  auto count = [&](int64_t i0) {
    const uint8_t* p = rows + i0 / 8;
    uint32_t cw4 = 0;
    auto spread = [&](uint32_t byte) { return (((byte >> sh) & 15u) * 0x00204081u) & 0x01010101u; };
    int w = 0;
#pragma unroll 1
    for (; w + 8 <= W; w += 8, p += 8 * rstride) {
      uint32_t x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = p[u * rstride];
#pragma unroll
      for (int u = 0; u < 8; ++u) cw4 += spread(x[u]);
    }
#pragma unroll 1
    for (; w < W; ++w, p += rstride) cw4 += spread(*p);
    return cw4;
  };
  // The first step's counts do not wait for the decision: their loads are in
  // flight with the partials'.
  uint32_t cw_first = 0;
  if (!TERNARY && 256 * first + 4 * lane < nbe) cw_first = count(256 * first + 4 * lane);
  // `wide` lanes a worker (at most 64), thread t for worker t / wide: every
  // wide-th slot, then the group's sum in its last lane.
  int wide = 64;
  while (wide * W > kThreads2) wide /= 2;
  {
    const int w = t / wide, j = t & (wide - 1);
    Partial r;
    r.sabs = r.sabs_c = r.sabs_b = r.ssq = 0.0;
    r.nonfinite = 0;
    if (w < W) {
#pragma unroll 4
      for (int k = j; k < used; k += wide) part_add<EXACT>(r, P[(int64_t)k * W + w]);
    }
    XSum x{r.sabs, r.sabs_c, r.sabs_b};
    double s2 = r.ssq;
    uint32_t nf = (uint32_t)r.nonfinite;  // at most the bucket's length, below 2^32
    group_steps(wide, [&](auto step) {
      if (EXACT) x = xstep(step, x);
      else x.s += step.of(x.s);
      s2 += step.of(s2);
      nf += step.of(nf);
    });
    if (w < W && j == wide - 1) {
      double s1;
      const bool certified = xround(x, s1);
      st[w].nonfinite = nf;
      st[w].sum_abs_elig = s1;
      st[w].sum_sq = s2;
      redo[w] = EXACT && !certified;
    }
  }
  if (v == 3) {
    uint32_t s = 0;
    for (int k = lane; k < used; k += 64) s += (uint32_t)d.part_ne[chunk0 + k];
    s = wave_sum_u32(s);
    if (lane == 0) ne_s = s;
  }
  __syncthreads();
  uint32_t resummed = 0;
  if (EXACT) resummed = resum_exact(st, redo, d, base, nbe, hist);
  if (v == 0) decide_wave(st, W, nbe, (int64_t)ne_s, d.pol, resummed, &dec);
  __syncthreads();
  if (blockIdx.x == 0) {
    if (t < W) d.stats[(int64_t)b * W + t] = st[t];
    if (t == 0) d.dec[b] = dec;
  }
  const int route = dec.route;
  if (route == NF_ROUTE_PLAIN || a.decide_only) return;

  if (route == NF_ROUTE_FALLBACK) {
    for (int64_t k = first; 64 * k < nbe; k += step) {
      const uint64_t m = uniform64(d.mask[base / 64 + k]) & low_bits(nbe - 64 * k);
      if ((m >> lane) & 1ull) {
        const int64_t e = base + 64 * k + lane;
        const float s = worker_sum(d.g[e], d.g + e + d.wstride, d.wstride, W - 1);
        a.out[e] = a.mean ? s / (float)W : s;
      }
    }
    return;
  }

  const float scale = dec.scale;
  if constexpr (!TERNARY) {
    if (t <= W) tab[t] = scale * decode_q(t, W, a.decode_mode);
    __syncthreads();
    const bool c4 = a.counts && ((reinterpret_cast<uintptr_t>(a.counts + base) & 3) == 0);
    const bool o16 = (reinterpret_cast<uintptr_t>(a.out + base) & 15) == 0;
    const uint8_t* mrow = reinterpret_cast<const uint8_t*>(d.mask + base / 64);
    for (int64_t k = first; 256 * k < nbe; k += step) {
      const int64_t i0 = 256 * k + 4 * lane;  // my first element in the bucket
      if (i0 >= nbe) continue;
      const uint32_t cw4 = k == first ? cw_first : count(i0);
      const uint32_t mnib = (mrow[i0 / 8] >> sh) & 15u;
      const int cnt = nbe - i0 < 4 ? (int)(nbe - i0) : 4;
      if (cnt == 4 && c4) {
        *reinterpret_cast<uint32_t*>(a.counts + base + i0) = cw4;
      } else if (a.counts) {
        for (int e = 0; e < cnt; ++e) a.counts[base + i0 + e] = (uint8_t)(cw4 >> (8 * e));
      }
      if (cnt == 4 && o16 && mnib == 15u) {
        const f32x4 y = {tab[cw4 & 255u], tab[(cw4 >> 8) & 255u], tab[(cw4 >> 16) & 255u], tab[cw4 >> 24]};
        *reinterpret_cast<f32x4*>(a.out + base + i0) = y;
      } else {
        for (int e = 0; e < cnt; ++e)
          if ((mnib >> e) & 1u) a.out[base + i0 + e] = tab[(cw4 >> (8 * e)) & 255u];
      }
    }
  } else {
    for (int i = t; i <= 2 * W; i += kThreads2) tab[i] = scale * decode_qt(i - W, W, a.decode_mode);
    if (t < W) th[t] = ternary_threshold(st[t], dec.n_eligible, a.tau);
    __syncthreads();
    uint64_t* pbits = a.bits + base / 64;
    uint64_t* nbits = pbits + (int64_t)W * a.bstride;
    for (int64_t k = first; 64 * k < nbe; k += step) {
      const int64_t left = nbe - 64 * k;
      const uint64_t m = uniform64(d.mask[base / 64 + k]) & low_bits(left);
      const bool live = lane < left;
      const int64_t e = base + 64 * k + lane;
      const float* p = d.g + (live ? e : base + nbe - 1);
      int cp = 0, cn = 0;
      // the planes' words of worker l, gathered in lane l
      uint64_t pw = 0, nw = 0;
#pragma unroll 1
      for (int i0 = 0; i0 < W; i0 += 8) {
        float x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = p[(int64_t)(i0 + u < W ? i0 + u : W - 1) * d.wstride];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int i = i0 + u;
          const uint64_t mi = i < W ? m : 0;
          const bool keep = !(__builtin_fabsf(x[u]) < th[i < W ? i : 0]);  // gated to 0 below the threshold
          const uint64_t pb = __ballot(keep && x[u] > 0.0f) & mi;
          const uint64_t nb = __ballot(keep && x[u] < 0.0f) & mi;
          pw = lane == i ? pb : pw;
          nw = lane == i ? nb : nw;
          cp = (int)add_lane_bit((uint32_t)cp, pb);
          cn = (int)add_lane_bit((uint32_t)cn, nb);
        }
      }
      if (lane < W) {
        pbits[(int64_t)lane * a.bstride + k] = pw;
        nbits[(int64_t)lane * a.bstride + k] = nw;
      }
      if (live) {
        if (a.counts) {
          a.counts[e] = (uint8_t)cp;
          a.counts[d.n_total + e] = (uint8_t)cn;
        }
        if ((m >> lane) & 1ull) a.out[e] = tab[cp - cn + W];
      }
    }
  }
}

// --------------------------------------------------------------- launchers

hipError_t launch_small2(const Geometry& geo, const Small2Args& a, hipStream_t s) {
  // A step of a wavefront is 256 elements (G-Binary) or 64; one or two
  // blocks per compute unit, so that the repeated decision stays small.
  int64_t blocks = ceil_div(geo.max_len, (a.ternary ? 64 : 256) * (kThreads2 / 64));
  const int64_t cap = ceil_div(a.ternary ? 1024 : 512, geo.nb);
  if (blocks > cap) blocks = cap;
  if (blocks < 1 || a.decide_only) blocks = 1;
  const dim3 grid((unsigned)blocks, (unsigned)geo.nb);
  if (a.ternary)
    hipLaunchKernelGGL(k_small2<true>, grid, dim3(kThreads2), 0, s, a);
  else
    hipLaunchKernelGGL(k_small2<false>, grid, dim3(kThreads2), 0, s, a);
  return hipGetLastError();
}

}  // namespace nf
