// nf_ternary.hip - G-Ternary write side and count/decode (§2.2; gfx950).
//
//   k_tsample a sample of every bucket and worker
//   k_twindow the window around each worker's threshold by which pass 1 packs
//             the planes as it reads
//   k_tsettle the elements that the window left open, read again
//   k_tpack   both planes per worker from given thresholds, laid out as
//             pass 1's chunks: in a second read of the gradients, or from
//             given thresholds (nf_pack_ternary)
//   k_tpass2  pass 2's bit-sliced counter over the positive and the negative
//             planes, decoded from their difference
#include <hip/hip_ext.h>

#include "nf_device.h"

namespace nf {

// ------------------------------------------------------- threshold windows
//
// The mean |g| of a sample of a worker's eligible elements in a bucket, at
// most `most` words, one from each of as many stretches of the bucket (so that
// every parameter's scale is met), at a place of its own in each.  The
// threshold is tau times the whole bucket's mean; with S1 and S2 the sample's
// sums of |g| and g*g, a mean over independent elements is off by less than
// sqrt(S2) / S1 of itself (one deviation; for normal values 1.25 / sqrt(m),
// and truly 0.75 / sqrt(m)), and the window is two of these wide on either
// side: about 0.5% of theta for 262,144 elements, which leaves 0.3% of normally
// distributed elements open.  A threshold outside its window costs a second
// read of that worker's rows, not a result.
//
// Block (worker, bucket, part): every np-th kSampleBlock of the sampled words,
// to a slot of pass 1's partials that pass 1 has yet to write (sabs S1, ssq S2,
// sabs_c the elements, nonfinite whether there is any).  A block is a chain of
// scattered reads: with one per worker and bucket, 8 workers of 1.5 GB took
// 106 us, 64 of 8 GB 86.
__global__ __launch_bounds__(kThreads1) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_tsample(TernArgs a, Partial* sample, int most) {
  __shared__ double r1[kWaves], r2[kWaves];
  __shared__ uint32_t rn[kWaves], rbad[kWaves];
  const int w = blockIdx.x, b = blockIdx.y;
  const int v = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  int64_t base, nbe, chunk0;
  bucket_span(b, a.btab, a.n_total, a.bucket_n, a.slots, base, nbe, chunk0);
  const int np = sample_parts(nbe, most, a.chunk);
  if ((int)blockIdx.z >= np) return;  // whole block
  const float* row = a.g + (int64_t)w * a.wstride + base;
  const int64_t nw = (nbe + 63) / 64;
  const int64_t ns = sample_words(nw, most);
  double s1 = 0.0, s2 = 0.0;
  uint32_t n = 0;
  bool bad = false;
  constexpr int NL = kSampleBlock / kWaves;  // words of a wavefront, all in flight
#pragma unroll 1
  for (int64_t j0 = (int64_t)blockIdx.z * kSampleBlock + v * NL; j0 < ns; j0 += np * kSampleBlock) {
    // this lane's sampled word, from stretch j of ns, and its mask word
    const int64_t j = j0 + (lane & (NL - 1));
    const bool some = lane < NL && j < ns;
    const int64_t k = j < ns ? (j * nw + (int64_t)((uint32_t)j * 2654435761u >> 8) % nw) / ns : 0;
    const uint64_t m = some ? a.mask[base / 64 + k] & low_bits(nbe - 64 * k) : 0;
    float x[NL];
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const int64_t e = 64 * (int64_t)__builtin_amdgcn_readlane((int)k, u) + lane;
      x[u] = row[e < nbe ? e : nbe - 1];
    }
    n += (uint32_t)__popcll(m);
    float f1 = 0.0f, f2 = 0.0f;  // FP32 will do for the window (all in FP64 took half the kernel's time)
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const uint64_t mu = ((uint64_t)__builtin_amdgcn_readlane((uint32_t)(m >> 32), u) << 32) |
                          (uint32_t)__builtin_amdgcn_readlane((uint32_t)m, u);
      const bool fin = finite32(x[u]);
      bad |= !fin;
      const float d = __builtin_amdgcn_inverse_ballot_w64(mu) && fin ? x[u] : 0.0f;
      f1 += __builtin_fabsf(d);
      f2 = __builtin_fmaf(d, d, f2);
    }
    s1 += (double)f1;
    s2 += (double)f2;
  }
  s1 = wave_sum(s1);
  s2 = wave_sum(s2);
  n = wave_sum_u32(n);
  if (lane == 0) {
    r1[v] = s1;
    r2[v] = s2;
    rn[v] = n;
  }
  if (const uint64_t any = __ballot(bad); lane == 0) rbad[v] = any != 0;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t1 = 0.0, t2 = 0.0, tn = 0.0;
    uint32_t some_bad = 0;
    for (int i = 0; i < kWaves; ++i) {
      some_bad |= rbad[i];
      t1 += r1[i];
      t2 += r2[i];
      tn += (double)rn[i];
    }
    Partial p;
    p.sabs = t1;
    p.ssq = t2;
    p.nonfinite = some_bad;
    p.sabs_c = tn;
    p.sabs_b = 0.0;
    sample[(chunk0 + blockIdx.z) * a.W + w] = p;
  }
}

// The windows of a bucket, a thread a worker, and whether the sample foretells
// the fallback (see Window).  A launch of its own, so that pass 1 knows from
// its first chunk on.
__global__ __launch_bounds__(256) void k_twindow(TernArgs a, const Partial* sample, nf_worker_stats* win, int most,
                                                 float ratio) {
  __shared__ float power[256];
  const int b = blockIdx.x, w = threadIdx.x;
  int64_t base, nbe, chunk0;
  bucket_span(b, a.btab, a.n_total, a.bucket_n, a.slots, base, nbe, chunk0);
  const int64_t nw = (nbe + 63) / 64;
  const int np = sample_parts(nbe, most, a.chunk);
  float* f = reinterpret_cast<float*>(win + (int64_t)b * a.W + w);
  if (w < a.W) {
    double t1 = 0.0, t2 = 0.0, tn = 0.0;
    uint64_t some_bad = 0;
#pragma unroll 8
    for (int p = 0; p < np; ++p) {
      const Partial q = sample[(chunk0 + p) * a.W + w];
      t1 += q.sabs;
      t2 += q.ssq;
      tn += q.sabs_c;
      some_bad |= q.nonfinite;
    }
    // a point where the sample says too little: the worker is read again
    double theta = 0.0, eps = 0.0;
    if (t1 > 0.0) {
      theta = (double)a.tau * (t1 / tn);
      eps = sample_words(nw, most) == nw ? 1e-5 : 2.0 * sqrt(t2) / t1;
      if (!(eps < 0.25)) eps = 0.0;
    }
    power[w] = t1 > 0.0 && !some_bad ? (float)(t2 / tn) : -1.0f;
    f[0] = (float)(theta * (1.0 - eps));
    f[1] = (float)(theta * (1.0 + eps));
    f[2] = power[w];
    f[3] = 0.0f;
  }
  __syncthreads();
  if (w >= 64 || ratio < 0.0f) return;
  // one wavefront
  uint32_t most_power = 0;  // as bits: from 0 on they are ordered alike
  bool bad = false;
#pragma unroll 1
  for (int i = w; i < a.W; i += 64) {
    const uint32_t u = __float_as_uint(power[i]);
    bad |= power[i] < 0.0f;
    most_power = power[i] >= 0.0f && u > most_power ? u : most_power;
  }
  group_steps(64, [&](auto step) {
    const uint32_t y = step.of(most_power);
    most_power = y > most_power ? y : most_power;
  });
  const float top = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)most_power, 63));
  // the largest above `ratio` times the lower median: more than half of the
  // workers are that far below it
  int below = 0;
#pragma unroll 1
  for (int i0 = 0; i0 < a.W; i0 += 64) {
    const int i = i0 + w;
    below += __popcll(__ballot(i < a.W && ratio * power[i < a.W ? i : 0] < top));
  }
  const bool ahead = __ballot(bad) != 0 || below > (a.W - 1) / 2;
  if (ahead && w == 0) f[3] = 1.0f;
}

// ---------------------------------------------------------------- G-Ternary
//
// Pack (write side), laid out as pass 1: a block takes one chunk (G tiles of
// one bucket) and wavefront v serves worker group v % WG and element group
// v / WG; lane l loads element 64k + l of word k, so the ballots of
// "eligible, not gated, g > 0" and "eligible, not gated, g < 0" are the
// two planes' words.  The next tile's loads (and mask words) are in flight
// while one tile is examined.  The chunk's words of both planes stay in LDS
// and leave at its end as coalesced rows; launches of pass 1's epochs
// bring the plane stores of a launch together, as in pass 1.
template <int WPW>
__global__ __launch_bounds__(kThreads1) __attribute__((amdgpu_waves_per_eu(WPW <= 2 ? 8 : 4, WPW <= 2 ? 8 : 4))) void k_tpack(
    TernArgs a, int64_t q0) {
  constexpr int NW = pass1_words(WPW);
  constexpr int NX = WPW * NW;
  extern __shared__ __align__(16) unsigned char smem[];
  const int64_t q = q0 + blockIdx.x;  // this block's chunk
  if (q >= a.total_chunks) return;     // whole block
  int b;
  int64_t c, base, nbe, chunk0;
  chunk_home(q, a.btab, a.cbucket, a.nb, a.chunks_full, b, c);
  if (a.dec && a.dec[b].route != NF_ROUTE_LOWBIT) return;  // whole block: no planes
  bucket_span(b, a.btab, a.n_total, a.bucket_n, 0, base, nbe, chunk0);
  const int v = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wavefront index, uniform
  const int lane = threadIdx.x & 63;
  const int wg = v % a.wg;
  const int eg = v / a.wg;
  const bool active = eg < a.eg;
  const int T = a.T;
  const int tile = a.eg * T;
  const int64_t ntiles = (nbe + tile - 1) / tile;
  const int64_t tb = c * a.G;
  const int64_t te = (tb + a.G < ntiles) ? tb + a.G : ntiles;
  const int64_t te_full = (te * tile <= nbe) ? te : te - 1;  // tiles [tb, te_full) are full
  const int cw = a.G * a.eg * NW;                             // words per worker row and chunk
  // This launch's rows: workers wbase .. wbase + R - 1; w below is a row of
  // the group, and the planes of the group's rows start at pbits (positive)
  // and nbits (negative).
  const int R = a.rows;
  const float* g = a.g + (int64_t)a.wbase * a.wstride;
  uint64_t* pbits = a.bits + (int64_t)a.wbase * a.bstride;
  uint64_t* nbits = a.bits + (int64_t)(a.W + a.wbase) * a.bstride;
  uint64_t* ppos = reinterpret_cast<uint64_t*>(smem);
  uint64_t* pneg = ppos + (size_t)R * cw;

  float th[WPW];
  const float* rp[WPW];
#pragma unroll
  for (int j = 0; j < WPW; ++j) {
    const int w = wg + j * a.wg;
    const int wl = w < R ? w : wg;
    th[j] = a.dec ? ternary_threshold(a.stats[(int64_t)b * a.W + a.wbase + wl], a.dec[b].n_eligible, a.tau)
                  : a.theta[a.wbase + wl];
    rp[j] = g + (int64_t)wl * a.wstride + base + (int64_t)eg * T + lane;
  }
  const uint64_t* mbase = a.mask + base / 64 + (int64_t)eg * (T / 64);
  // The first NW words of the bucket's first tile (full whenever any tile of
  // this chunk is): read by loads whose values are not needed.
  const float* dp = g + (int64_t)wg * a.wstride + base + lane;
  const uint64_t* dm = a.mask + base / 64;

  bool chunk_all = false, chunk_any = true;  // set below, after the first tile's loads are out

  // Loads of a full tile (or, for an idle wavefront or a tile past the full
  // ones, of the bucket's first words).
  auto issue_data = [&](int64_t tt, float (&X)[NX]) {
    const bool ok = active && tt < te_full;
    const int64_t o = tt * tile;
#pragma unroll
    for (int j = 0; j < WPW; ++j) {
      const float* row = ok ? rp[j] + o : dp;
#pragma unroll
      for (int k = 0; k < NW; ++k) X[j * NW + k] = __builtin_nontemporal_load(row + 64 * k);
    }
  };
  auto issue_mask = [&](int64_t tt, uint64_t (&M)[NW]) {
    const bool ok = active && tt < te_full;
    const int64_t o = tt * tile;
    if (chunk_all) {
      // every element of the chunk eligible: no mask words to load
#pragma unroll
      for (int k = 0; k < NW; ++k) M[k] = ~0ull;
      return;
    }
    const uint64_t* mrow = ok ? mbase + o / 64 : dm;
#pragma unroll
    for (int k = 0; k < NW; ++k) M[k] = uniform64(mrow[k]);
  };
  auto issue = [&](int64_t tt, float (&X)[NX], uint64_t (&M)[NW]) {
    issue_data(tt, X);
    issue_mask(tt, M);
  };
  auto body = [&](int64_t t, const float (&X)[NX], const uint64_t (&M)[NW]) {
    const int ti = (int)(t - tb);
#pragma unroll
    for (int j = 0; j < WPW; ++j) {
      const int w = wg + j * a.wg;
      if (j > 0 && w >= R) continue;
      uint64_t pb[NW], nb[NW];
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        const float x = X[j * NW + k];
        const bool keep = !(__builtin_fabsf(x) < th[j]);  // gated to 0 below the threshold
        pb[k] = __ballot(keep && x > 0.0f) & M[k];
        nb[k] = __ballot(keep && x < 0.0f) & M[k];
      }
      uint32_t lo, hi;
      const int at = w * cw + (ti * a.eg + eg) * NW + lane;
      lanes_from_ballots<NW>(pb, lo, hi);
      if (lane < NW) ppos[at] = ((uint64_t)hi << 32) | lo;
      lanes_from_ballots<NW>(nb, lo, hi);
      if (lane < NW) pneg[at] = ((uint64_t)hi << 32) | lo;
    }
  };
  auto consume = [&](const float (&X)[NX]) {
#pragma unroll
    for (int k = 0; k < NX; ++k) asm volatile("" ::"v"(X[k]));
  };

  float xa[NX], xb[NX];
  uint64_t ma[NW], mb[NW];
  if (te_full > tb) issue_data(tb, xa);
  // Whether every element of the chunk is eligible (then the tiles need no
  // mask words), and whether any is: a chunk with none is not read.
  {
    const int64_t cn = ((te * tile < nbe) ? te * tile : nbe) - tb * tile;  // elements of the chunk
    const int nwc = cn > 0 ? (int)((cn + 63) / 64) : 0;
    const uint64_t* cm = a.mask + (base + tb * tile) / 64;
    int any = 0, notall = cn % 64 != 0;  // a ragged chunk keeps its mask loads
    for (int i = threadIdx.x; i < nwc; i += kThreads1) {
      const uint64_t m = cm[i] & (i == nwc - 1 ? low_bits(cn - 64 * (int64_t)i) : ~0ull);
      any |= m != 0ull;
      notall |= m != ~0ull;
    }
    chunk_any = __syncthreads_or(any);
    chunk_all = !__syncthreads_or(notall);
  }

  // A chunk with no eligible element: both planes are zero and nothing more
  // is read (mask bits past the bucket's end do not count).
  if (!chunk_any) {
    if (te_full > tb) consume(xa);
    {
      const int64_t cn = ((te * tile < nbe) ? te * tile : nbe) - tb * tile;
      const int nwc = cn > 0 ? (int)((cn + 63) / 64) : 0;
      const int64_t gz = (base + tb * tile) / 64;
      for (int i = threadIdx.x; i < R * nwc; i += kThreads1) {
        const int w = i / nwc;
        const int o = i - w * nwc;
        pbits[(int64_t)w * a.bstride + gz + o] = 0ull;
        nbits[(int64_t)w * a.bstride + gz + o] = 0ull;
      }
      return;
    }
  }
  if (te_full > tb) issue_mask(tb, ma);
  int64_t t = tb;
  if (te_full > tb) {
    // Pairs of full tiles with the next one in flight, then the odd one.
    for (int64_t p = (te_full - tb) >> 1; p > 0; --p, t += 2) {
      issue(t + 1, xb, mb);
      if (active) body(t, xa, ma);
      issue(t + 2, xa, ma);
      if (active) body(t + 1, xb, mb);
    }
    if ((te_full - tb) & 1) {
      if (active) body(t, xa, ma);
      ++t;
    } else {
      consume(xa);
    }
  }
  if (t < te && active) {
    // The bucket's last, partial tile: loads and mask bits stop at its end.
    const int64_t e0 = t * tile + (int64_t)eg * T;
    const int64_t c64 = nbe - e0;
    const int cnt = (int)(c64 < 0 ? 0 : (c64 > T ? T : c64));
#pragma unroll
    for (int j = 0; j < WPW; ++j)
#pragma unroll
      for (int k = 0; k < NW; ++k)
        xb[j * NW + k] = (64 * k + lane < cnt) ? __builtin_nontemporal_load(rp[j] + t * tile + 64 * k) : 0.0f;
#pragma unroll
    for (int k = 0; k < NW; ++k)
      mb[k] = 64 * k < cnt ? uniform64(mbase[t * (tile / 64) + k] & low_bits(cnt - 64 * k)) : 0ull;
    body(t, xb, mb);
  }

  // The chunk's words of both planes, row by row.
  const int64_t e_beg = tb * tile;
  const int64_t e_end = (te * tile < nbe) ? te * tile : nbe;
  const int valid = te > tb ? (int)((e_end - e_beg + 63) / 64) : 0;
  const int64_t gw0 = (base + e_beg) / 64;
  if (a.eg == 1) {
    // each worker's words were written by its own wavefront only
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int j = 0; j < WPW; ++j) {
      const int w = wg + j * a.wg;
      if (w >= R || !active) break;  // 9 to 15 workers: a wavefront without one
      for (int o = lane; o < valid; o += 64) {
        pbits[(int64_t)w * a.bstride + gw0 + o] = ppos[w * cw + o];
        nbits[(int64_t)w * a.bstride + gw0 + o] = pneg[w * cw + o];
      }
    }
    return;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < R * valid; i += kThreads1) {
    const int w = i / valid;
    const int o = i - w * valid;
    pbits[(int64_t)w * a.bstride + gw0 + o] = ppos[w * cw + o];
    nbits[(int64_t)w * a.bstride + gw0 + o] = pneg[w * cw + o];
  }
}

// --------------------------------------------------------- open elements
//
// Block (words, bucket, worker) of a bucket routed L: a wavefront takes 256
// words of one worker, lane l words l, 64 + l, ...  An element that stands in
// both planes (pass 1's window left it open) is read again and keeps or loses
// its bits by the threshold.  What bounds it are single reads all over the
// gradients, each some microseconds away: the wavefront first lists its open
// elements in LDS (some 80 of 16,384), then reads them all at once, a lane
// an element.  (Lane by lane, a bit of each of its words a round, 25 MiB of 8
// workers took 39 us.)  The rows of a worker whose threshold missed its
// window are read whole and packed anew.
constexpr int kOpenList = 512;  // open elements listed at a time

__global__ __launch_bounds__(kThreads2) void k_tsettle(TernArgs a) {
  constexpr int NU = 4;
  __shared__ uint64_t pw[kThreads2 / 64][64 * NU], nv[kThreads2 / 64][64 * NU];
  __shared__ uint16_t list[kThreads2 / 64][kOpenList];
  const int b = blockIdx.y, w = blockIdx.z;
  if (a.dec[b].route != NF_ROUTE_LOWBIT) return;  // whole block
  int64_t base, nbe, chunk0;
  bucket_span(b, a.btab, a.n_total, a.bucket_n, a.slots, base, nbe, chunk0);
  const int v = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int64_t nw = (nbe + 63) / 64;
  const int64_t k0 = ((int64_t)blockIdx.x * (kThreads2 / 64) + v) * 64 * NU;
  if (k0 >= nw) return;  // whole wavefront
  uint64_t* prow = a.bits + (int64_t)w * a.bstride + base / 64;
  uint64_t* nrow = prow + (int64_t)a.W * a.bstride;
  const float* row = a.g + (int64_t)w * a.wstride + base;
  const float th = ternary_threshold(a.stats[(int64_t)b * a.W + w], a.dec[b].n_eligible, a.tau);
  if (a.part[chunk0 * a.W + w].sabs_b == 0.0) {
    uint64_t open[NU];
    uint32_t dirty = 0;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int64_t k = k0 + 64 * u + lane;
      const uint64_t p = k < nw ? prow[k] : 0ull;
      const uint64_t n = k < nw ? nrow[k] : 0ull;
      pw[v][64 * u + lane] = p;
      nv[v][64 * u + lane] = n;
      open[u] = p & n;
      dirty |= (open[u] != 0 ? 1u : 0u) << u;
    }
    if (!__any(dirty != 0)) return;
    while (true) {
      // list the open elements, as many as fit: lane l's after lane l - 1's
      int cnt = 0;
#pragma unroll
      for (int u = 0; u < NU; ++u) cnt += __popcll(open[u]);
      int at = cnt;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(at, d, 64);
        if (lane >= d) at += y;
      }
      const int total = __builtin_amdgcn_readlane(at, 63);
      if (total == 0) break;
      at -= cnt;
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        while (open[u] != 0 && at < kOpenList) {
          list[v][at++] = (uint16_t)((64 * u + lane) * 64 + __builtin_ctzll(open[u]));
          open[u] &= open[u] - 1;
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const int listed = total < kOpenList ? total : kOpenList;
      for (int i = lane; i < listed; i += 2 * 64) {
        const bool two = i + 64 < listed;
        const uint32_t e0 = list[v][i], e1 = list[v][two ? i + 64 : i];
        const float x0 = __builtin_nontemporal_load(row + 64 * k0 + e0);
        const float x1 = __builtin_nontemporal_load(row + 64 * k0 + e1);
        auto settle = [&](uint32_t e, float x) {
          const uint64_t others = ~(1ull << (e & 63));
          const bool keep = !(__builtin_fabsf(x) < th);
          if (!(keep && x > 0.0f)) atomicAnd((unsigned long long*)&pw[v][e >> 6], others);
          if (!(keep && x < 0.0f)) atomicAnd((unsigned long long*)&nv[v][e >> 6], others);
        };
        settle(e0, x0);
        if (two) settle(e1, x1);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
#pragma unroll
    for (int u = 0; u < NU; ++u)
      if ((dirty >> u) & 1u) {
        prow[k0 + 64 * u + lane] = pw[v][64 * u + lane];
        nrow[k0 + 64 * u + lane] = nv[v][64 * u + lane];
      }
    return;
  }
  const uint64_t* mrow = a.mask + base / 64;
#pragma unroll 1
  for (int64_t k1 = k0; k1 < k0 + 64 * NU && k1 < nw; k1 += 64) {
    const int64_t left = nbe - 64 * k1;  // elements from word k1 on
    const bool valid = k1 + lane < nw;
    const uint64_t mw = valid ? mrow[k1 + lane] & low_bits(left - 64 * lane) : 0ull;
    uint64_t p = 0, n = 0;
#pragma unroll 1
    for (int k = 0; k < 64 && 64 * k < left; k += 8) {
      float x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int64_t e = 64 * (k + i) + lane;
        x[i] = row[64 * k1 + (e < left ? e : left - 1)];
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint64_t m = ((uint64_t)__builtin_amdgcn_readlane((uint32_t)(mw >> 32), k + i) << 32) |
                           (uint32_t)__builtin_amdgcn_readlane((uint32_t)mw, k + i);
        const bool keep = !(__builtin_fabsf(x[i]) < th);
        const uint64_t pb = __ballot(keep && x[i] > 0.0f) & m, nb = __ballot(keep && x[i] < 0.0f) & m;
        p = lane == k + i ? pb : p;
        n = lane == k + i ? nb : n;
      }
    }
    if (valid) {
      prow[k1 + lane] = p;
      nrow[k1 + lane] = n;
    }
  }
}

// Count and decode (read side), as pass 2 with two counters: lane l counts
// word k0 + l of the positive rows and of the negative rows; the planes of
// both go through LDS so that each lane decodes four consecutive elements
// (one nibble per plane, spread into four count bytes by a multiply) from
// the difference of the two counts, d = c+ - c-, through a table of
// fl32(scale * q[d]).
constexpr int kRecT = 20;  // dwords per (word, half): 8 + 8 plane halves, mask half, pad

__global__ __launch_bounds__(kThreads2) void k_tpass2(TernArgs a) {
  __shared__ float tab[2 * 255 + 1];
  __shared__ __align__(16) uint32_t rec[4][64 * 2 * kRecT];
  const int b = blockIdx.y;
  float scale = 0.0f;
  if (a.dec) {
    if (a.dec[b].route != NF_ROUTE_LOWBIT) return;  // whole block
    scale = a.dec[b].scale;
  } else if (a.out) {
    scale = *a.scale;
  }
  if (a.out) {
    for (int d = threadIdx.x; d <= 2 * a.W; d += kThreads2) tab[d] = scale * decode_qt(d - a.W, a.W, a.decode_mode);
    __syncthreads();
  }
  int64_t base, nbe, chunk0;
  bucket_span(b, a.btab, a.n_total, a.bucket_n, a.slots, base, nbe, chunk0);
  const int64_t nwords = (nbe + 63) / 64;
  const int64_t wbase = base / 64;
  const int v = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wavefront index, uniform
  const int lane = threadIdx.x & 63;
  int nplanes = 1;
  while ((1 << nplanes) <= a.W) ++nplanes;  // counts 0..W need nplanes bits
  uint32_t* my = rec[v];
  const bool c4 = a.cpos && a.cneg && ((reinterpret_cast<uintptr_t>(a.cpos + base) & 3) == 0) &&
                  ((reinterpret_cast<uintptr_t>(a.cneg + base) & 3) == 0);
  const bool o16 = a.out && ((reinterpret_cast<uintptr_t>(a.out + base) & 15) == 0);

  for (int64_t ch = (int64_t)blockIdx.x * 4 + v; ch * 64 < nwords; ch += (int64_t)a.bpb2 * 4) {
    const int64_t k0 = ch * 64;
    const int nk = (int)((nwords - k0) < 64 ? (nwords - k0) : 64);
    const bool valid = lane < nk;
    uint64_t P[8], N[8];
    count_column(a.bits + wbase + k0 + lane, a.bstride, a.W, valid, nplanes, P);
    count_column(a.bits + (int64_t)a.W * a.bstride + wbase + k0 + lane, a.bstride, a.W, valid, nplanes, N);
    const uint64_t mw = (valid && a.mask) ? a.mask[wbase + k0 + lane] : 0ull;
    uint4* r0 = reinterpret_cast<uint4*>(my + (lane * 2) * kRecT);
    uint4* r1 = reinterpret_cast<uint4*>(my + (lane * 2 + 1) * kRecT);
    r0[0] = make_uint4((uint32_t)P[0], (uint32_t)P[1], (uint32_t)P[2], (uint32_t)P[3]);
    r0[1] = make_uint4((uint32_t)P[4], (uint32_t)P[5], (uint32_t)P[6], (uint32_t)P[7]);
    r0[2] = make_uint4((uint32_t)N[0], (uint32_t)N[1], (uint32_t)N[2], (uint32_t)N[3]);
    r0[3] = make_uint4((uint32_t)N[4], (uint32_t)N[5], (uint32_t)N[6], (uint32_t)N[7]);
    r0[4] = make_uint4((uint32_t)mw, 0u, 0u, 0u);
    r1[0] = make_uint4((uint32_t)(P[0] >> 32), (uint32_t)(P[1] >> 32), (uint32_t)(P[2] >> 32), (uint32_t)(P[3] >> 32));
    r1[1] = make_uint4((uint32_t)(P[4] >> 32), (uint32_t)(P[5] >> 32), (uint32_t)(P[6] >> 32), (uint32_t)(P[7] >> 32));
    r1[2] = make_uint4((uint32_t)(N[0] >> 32), (uint32_t)(N[1] >> 32), (uint32_t)(N[2] >> 32), (uint32_t)(N[3] >> 32));
    r1[3] = make_uint4((uint32_t)(N[4] >> 32), (uint32_t)(N[5] >> 32), (uint32_t)(N[6] >> 32), (uint32_t)(N[7] >> 32));
    r1[4] = make_uint4((uint32_t)(mw >> 32), 0u, 0u, 0u);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (int grp = 0; grp * 4 < nk; ++grp) {
      const int kk = grp * 4 + (lane >> 4);
      const int shn = 4 * (lane & 7);
      const uint4* r = reinterpret_cast<const uint4*>(my + (kk * 2 + ((lane >> 3) & 1)) * kRecT);
      const uint4 p03 = r[0];
      const uint4 p47 = r[1];
      const uint4 n03 = r[2];
      const uint4 n47 = r[3];
      const uint32_t mnib = (r[4].x >> shn) & 15u;
      auto spread = [&](uint32_t plane) { return (((plane >> shn) & 15u) * 0x00204081u) & 0x01010101u; };
      uint32_t cp4 = spread(p03.x) | (spread(p03.y) << 1) | (spread(p03.z) << 2) | (spread(p03.w) << 3);
      uint32_t cn4 = spread(n03.x) | (spread(n03.y) << 1) | (spread(n03.z) << 2) | (spread(n03.w) << 3);
      if (nplanes > 4) {
        cp4 |= (spread(p47.x) << 4) | (spread(p47.y) << 5) | (spread(p47.z) << 6) | (spread(p47.w) << 7);
        cn4 |= (spread(n47.x) << 4) | (spread(n47.y) << 5) | (spread(n47.z) << 6) | (spread(n47.w) << 7);
      }
      const int64_t i0 = (k0 + grp * 4) * 64 + 4 * lane;  // first of my four elements in the bucket
      if (kk >= nk || i0 >= nbe) continue;
      auto value = [&](int e) {
        return tab[(int)((cp4 >> (8 * e)) & 255u) - (int)((cn4 >> (8 * e)) & 255u) + a.W];
      };
      if (i0 + 3 < nbe) {
        if (c4) {
          __builtin_nontemporal_store(cp4, reinterpret_cast<uint32_t*>(a.cpos + base + i0));
          __builtin_nontemporal_store(cn4, reinterpret_cast<uint32_t*>(a.cneg + base + i0));
        } else if (a.cpos && a.cneg) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            a.cpos[base + i0 + e] = (uint8_t)(cp4 >> (8 * e));
            a.cneg[base + i0 + e] = (uint8_t)(cn4 >> (8 * e));
          }
        }
        if (a.out) {
          if (o16 && mnib == 15u) {
            const f32x4 y = {value(0), value(1), value(2), value(3)};
            __builtin_nontemporal_store(y, reinterpret_cast<f32x4*>(a.out + base + i0));
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if ((mnib >> e) & 1u) a.out[base + i0 + e] = value(e);
          }
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (i0 + e < nbe) {
            if (a.cpos && a.cneg) {
              a.cpos[base + i0 + e] = (uint8_t)(cp4 >> (8 * e));
              a.cneg[base + i0 + e] = (uint8_t)(cn4 >> (8 * e));
            }
            if (a.out && ((mnib >> e) & 1u)) a.out[base + i0 + e] = value(e);
          }
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// --------------------------------------------------------------- launchers

hipError_t launch_ternary_pack(const Geometry& geo, const TernArgs& a0, hipStream_t s) {
  TernArgs a = a0;
  a.chunks_full = geo.chunks_full;
  a.total_chunks = geo.total_chunks;
  a.nb = (int32_t)geo.nb;
  a.wg = geo.wg;
  a.eg = geo.eg;
  a.T = geo.T;
  a.G = geo.G;
  // Both planes of a chunk: 2 * R * G * EG * (T / 64) words, at most 64 KiB.
  const size_t smem = 2 * (size_t)geo.rows * geo.G * geo.eg * pass1_words(geo.wpw) * sizeof(uint64_t);
  if (smem > 65536) return hipErrorInvalidValue;
  // No chunk or row group shares state with another, so every launch after
  // the first may start while the one before drains.
  const int64_t epoch = one_launch_epoch(geo.total_chunks);  // chunks share no state here
  for (int grp = 0; grp < geo.ngroups; ++grp) {
    row_group(geo, grp, &a.wbase, &a.rows);
    // every wavefront's first worker (wg < geo.wg) must be a row of the group
    if (a.rows < geo.wg || a.rows > geo.rows) return hipErrorInvalidValue;
    for (int64_t q0 = 0; q0 < geo.total_chunks; q0 += epoch) {
      const int64_t left = geo.total_chunks - q0;
      const dim3 grid((unsigned)(left < epoch ? left : epoch));
      const uint32_t fl = (q0 > 0 || grp > 0) ? hipExtAnyOrderLaunch : 0u;
      switch (geo.wpw) {
        case 1: hipExtLaunchKernelGGL((k_tpack<1>), grid, dim3(kThreads1), smem, s, nullptr, nullptr, fl, a, q0); break;
        case 2: hipExtLaunchKernelGGL((k_tpack<2>), grid, dim3(kThreads1), smem, s, nullptr, nullptr, fl, a, q0); break;
        case 4: hipExtLaunchKernelGGL((k_tpack<4>), grid, dim3(kThreads1), smem, s, nullptr, nullptr, fl, a, q0); break;
        default: return hipErrorInvalidValue;
      }
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

hipError_t launch_ternary_window(const Geometry& geo, const TernArgs& a0, Partial* sample, nf_worker_stats* win,
                                 float ratio, hipStream_t s) {
  TernArgs a = a0;
  a.chunk = geo.tile * geo.G;
  const int most = geo.nb * geo.W >= 128 ? kSampleWords : kSampleWords / 4;
  const dim3 grid((unsigned)geo.W, (unsigned)geo.nb, (unsigned)sample_parts(geo.max_len, most, a.chunk));
  hipLaunchKernelGGL(k_tsample, grid, dim3(kThreads1), 0, s, a, sample, most);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_twindow, dim3((unsigned)geo.nb), dim3(256), 0, s, a, sample, win, most, ratio);
  return hipGetLastError();
}

hipError_t launch_ternary_settle(const Geometry& geo, const TernArgs& a, hipStream_t s) {
  const int64_t blocks = ceil_div((geo.max_len + 63) / 64, 4 * kThreads2);
  hipLaunchKernelGGL(k_tsettle, dim3((unsigned)blocks, (unsigned)geo.nb, (unsigned)geo.W), dim3(kThreads2), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_ternary_reduce(const Geometry& geo, const TernArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_tpass2, dim3((unsigned)geo.bpb2, (unsigned)geo.nb), dim3(kThreads2), 0, s, a);
  return hipGetLastError();
}

}  // namespace nf
