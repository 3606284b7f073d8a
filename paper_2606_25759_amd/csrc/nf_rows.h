// nf_rows.h - a chunk of pass 1 by rows (k_rows, which takes every chunk of the
// problems that rows_problem names).
#pragma once

#include "nf_decide.h"
#include "nf_device.h"

namespace nf {

__device__ __forceinline__ void put_partial(Partial& p, const XSum& x, double ssq, uint64_t nonfinite) {
  p.sabs = x.s;
  p.sabs_c = x.c;
  p.sabs_b = x.b;
  p.ssq = ssq;
  p.nonfinite = nonfinite;
}

// An item is one worker's words (64 elements each) of the chunk, or every
// parts-th eight of them; the 16 wavefronts take the items in turn.  Lane l
// loads element 64k + l of word k, so every load instruction reads 256
// contiguous bytes and the ballot of "g > 0" over the wavefront is exactly
// bitmap word k.  Health accumulates per lane in FP64 and lives for one item,
// so any number of workers takes the same registers (at most 64: eight
// wavefronts per SIMD).  The sign words wait in LDS, [wavefront] or
// [worker][item_words], and leave as whole rows (stored as 64-byte pieces among the reads, a step over
// 12 GB of 16 workers took 2.84 ms, so 2.56).  Then the words with an
// FP32-routed element are read again and their workers added in order: no
// LDS stage, and no barrier between the wavefronts but one at the end.
// red and red_ne: LDS for kItems partials and kWaves counts.

template <bool PACK, bool TERN, bool SMALL, bool CACHED>
__device__ __forceinline__ void chunk_by_rows(const Pass1Args& a, int64_t q, int b, int64_t e0, int len, uint64_t* lds,
                                              Partial* red, uint32_t* red_ne) {
  constexpr bool EXACT = !PACK;
  constexpr int NW = kBatch;
  const int v = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wavefront index, uniform
  const int lane = threadIdx.x & 63;
  const int nwc = (len + 63) / 64;
  const uint64_t* mrow = a.mask + e0 / 64;
  const float* g0 = a.g + e0;
  const int W = a.W;
  const int parts = a.parts;
  // FP32 sums at a position: an earlier row group's running sum comes first;
  // the mean divides by all workers after the last group.
  auto sum_last = [&](float s) { return a.mean && a.rfin ? s / (float)a.wtot : s; };
  // G-Ternary: no planes in a bucket that falls back (see Window); waited for
  // once the first gradients are on their way.
  float ahead = 0.0f;
  if (TERN) ahead = load_ahead(a.win0 + (int64_t)b * a.wtot);
  // Worker w's sign words, whole in LDS, to memory by one wavefront.
  auto put_row = [&](int w, const uint64_t* words) {
    if (TERN && ahead != 0.0f) return;
    uint64_t* to = a.bits + (int64_t)w * a.bstride + e0 / 64;
    for (int i = lane; i < nwc; i += 64) to[i] = words[i];
    if (TERN) {
      to = a.nbits + (int64_t)w * a.bstride + e0 / 64;
      for (int i = lane; i < nwc; i += 64) to[i] = words[a.item_words + i];
    }
  };
  constexpr int ROWS = TERN ? 2 : 1;  // LDS rows per worker: sign words, or both planes'


  for (int it = v; it < W * parts; it += kWaves) {
    int w = it, part = 0;
    while (w >= W) {
      w -= W;
      ++part;
    }
    const float* row = g0 + (int64_t)w * a.wstride;
    uint64_t* words = lds + (parts == 1 ? v : w) * ROWS * a.item_words;
    Window wd{0.0f, 0.0f};
    if (TERN) wd = load_window(a.win, (int64_t)b * a.wtot + w);
    double sabs = 0.0, sabc = 0.0, ssq = 0.0;
    uint32_t snz = 0, uml = ~0u;
    bool tw = false;
    uint64_t nonf = 0;
    uint32_t ne = 0;
    // Eight words from word k on: signs, and their terms into the lane's
    // health.  mv: lanes 0 .. 7 hold their mask words (the lanes above, if
    // nothing else, the same again).
    auto examine = [&](int k, const float (&x)[NW], uint64_t mv) {
      double s1 = 0.0, s2 = 0.0;
      uint32_t umt = ~0u, el8 = 0;
      uint64_t bb[NW], nb[NW];
      const bool skip = TERN && __builtin_amdgcn_readfirstlane((int)(ahead != 0.0f)) != 0;
#pragma unroll
      for (int u = 0; u < NW; ++u) {
        const uint64_t m = ((uint64_t)__builtin_amdgcn_readlane((uint32_t)(mv >> 32), u) << 32) |
                           (uint32_t)__builtin_amdgcn_readlane((uint32_t)mv, u);
        if (PACK) bb[u] = __ballot(x[u] > 0.0f) & m;
        if (TERN && !skip) tern_words(x[u], wd.lo, wd.hi, m, bb[u], nb[u]);
        const bool el = __builtin_amdgcn_inverse_ballot_w64(m);
        const double d = (double)x[u];
        s2 = __builtin_fma(d, d, s2);
        s1 += el ? __builtin_fabs(d) : 0.0;
        if constexpr (EXACT) {
          umt = term_umin(umt, el ? x[u] : 0.0f);
          el8 |= (uint32_t)el << u;
        }
      }
      if constexpr (EXACT) tile_into_lane<NW>(sabs, sabc, snz, uml, tw, s1, umt, row + 64 * k + lane, el8);
      if constexpr (!EXACT) sabs += s1;
      ssq += s2;
      if (__ballot(!finite64(s2))) {
#pragma unroll
        for (int u = 0; u < NW; ++u) nonf += __popcll(__ballot(!finite32(x[u])));
        if (TERN && lane == 0 && a.ratio >= 0.0f) set_ahead(a.win0 + (int64_t)b * a.wtot);
      }
      if (w == 0 && lane < NW) ne += __popcll(mv);
      if (PACK || (TERN && !skip)) {
        uint32_t lo, hi;
        lanes_from_ballots<NW>(bb, lo, hi);
        if (lane < NW) words[k + lane] = ((uint64_t)hi << 32) | lo;
        if (TERN) {
          lanes_from_ballots<NW>(nb, lo, hi);
          if (lane < NW) words[a.item_words + k + lane] = ((uint64_t)hi << 32) | lo;
        }
      }
    };
    // Words k .. k + 7 and, in lanes 0 .. 7, their mask words.  In the chunk's
    // last, partial eight, lanes past its end read its last element, and
    // clip drops it.
    auto load = [&](int k, float (&x)[NW], uint64_t& mv) {
      const float* p = row + 64 * k + lane;
      if (64 * (k + NW) <= len) {
        mv = mrow[k + (lane & (NW - 1))];
#pragma unroll
        for (int u = 0; u < NW; ++u) x[u] = CACHED ? p[64 * u] : __builtin_nontemporal_load(p + 64 * u);
      } else {
        mv = 0;
        if (lane < NW && k + lane < nwc) mv = mrow[k + lane] & low_bits(len - 64 * (k + lane));
#pragma unroll
        for (int u = 0; u < NW; ++u) {
          const int e = 64 * (k + u) + lane;
          x[u] = row[e < len ? e : len - 1];
        }
      }
    };
    auto clip = [&](int k, float (&x)[NW]) {
      if (64 * (k + NW) > len) {
#pragma unroll
        for (int u = 0; u < NW; ++u) x[u] = 64 * (k + u) + lane < len ? x[u] : 0.0f;
      }
    };
    // The next eight are in flight while eight are examined (SMALL: an item
    // has one or two, and the shorter code counts for more).
    const int dk = parts * NW;
    float x[NW];
    uint64_t mv;
    if constexpr (SMALL) {
#pragma unroll 1
      for (int k = part * NW; k < nwc; k += dk) {
        load(k, x, mv);
        clip(k, x);
        examine(k, x, mv);
      }
    } else {
      float xn[NW];
      uint64_t mvn;
      int k = part * NW;
      if (k < nwc) load(k, xn, mvn);
#pragma unroll 1
      for (; k < nwc; k += dk) {
#pragma unroll
        for (int u = 0; u < NW; ++u) x[u] = xn[u];
        mv = mvn;
        clip(k, x);
        if (k + dk < nwc) load(k + dk, xn, mvn);
        examine(k, x, mv);
      }
    }
    if ((PACK || TERN) && parts == 1) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      put_row(w, words);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    const XSum x1 = lane_sum<EXACT>(sabs, sabc, snz);
    const double s2 = wave_sum(ssq);
    const uint32_t nes = w == 0 ? wave_sum_u32(ne) : 0u;
    if (lane == 0) {
      if (parts == 1) {
        put_partial(a.part[q * a.wtot + w], x1, s2, nonf);
        if (w == 0) a.part_ne[q] = nes;
      } else {
        put_partial(red[it], x1, s2, nonf);
        if (w == 0) red_ne[part] = nes;
      }
    }
  }

  // FP32 sums, workers in order, at the words with a routed element (or at
  // every word).
  if (a.sums != kSumsNone) {
#pragma unroll 1
    for (int k = v; k < nwc; k += kWaves) {
      const uint64_t live = low_bits(len - 64 * k);
      const uint64_t pick = (a.sums == kSumsAll ? ~0ull : ~uniform64(mrow[k])) & live;
      if (!pick) continue;
      if (__builtin_amdgcn_inverse_ballot_w64(pick)) {
        float* to = a.out + e0 + 64 * k + lane;
        const float* p = g0 + 64 * k + lane;
        const float s = a.racc ? *to + *p : *p;
        *to = sum_last(worker_sum(s, p + a.wstride, a.wstride, W - 1));
      }
    }
  }

  if (parts > 1) {
    __syncthreads();
    if (PACK || TERN)
      for (int w = v; w < W; w += kWaves) put_row(w, lds + w * ROWS * a.item_words);
    const int w = threadIdx.x;
    if (w < W) {
      Partial p = red[w];
      for (int k = 1; k < parts; ++k) part_add<EXACT>(p, red[k * W + w]);
      a.part[q * a.wtot + w] = p;
    }
    if (w == 0) {
      uint64_t s = 0;
      for (int k = 0; k < parts; ++k) s += red_ne[k];
      a.part_ne[q] = s;
    }
  }
}

}  // namespace nf
