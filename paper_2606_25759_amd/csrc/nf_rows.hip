// nf_rows.hip - pass 1 by rows (k_rows, gfx950): small problems, and those
// whose chunks k_pass1 would take by its slower loops (rows_problem).  8 KiB
// of code a variant: k_pass1's four unrolled loops are 34, of which a block of
// one or two tiles runs every line once (on a bucket of 8 x 70,001 elements,
// 11 of its 17 us between the first loads and the last store, on one tile).
#include <hip/hip_ext.h>

#include "nf_rows.h"

namespace nf {

// A block takes chunk q0 + blockIdx.x, all its rows.
template <bool PACK, bool TERN, bool SMALL, bool CACHED>
__global__ __launch_bounds__(kThreads1) __attribute__((amdgpu_waves_per_eu(PACK ? 8 : 4, 8))) void k_rows(
    Pass1Args a, int64_t q0) {
  extern __shared__ uint64_t lds[];  // sign words: see chunk_by_rows
  __shared__ Partial red[kItems];
  __shared__ uint32_t red_ne[kWaves];
  const int64_t q = q0 + blockIdx.x;  // this block's chunk, and its partials' slot
  int b;
  int64_t c, base, nbe, chunk0;
  chunk_home(q, a.btab, a.cbucket, a.nb, a.chunks_full, b, c);
  bucket_span(b, a.btab, a.n_total, a.bucket_n, a.slots, base, nbe, chunk0);
  const int64_t ch = (int64_t)a.G * a.eg * a.T;  // elements of a whole chunk
  const int64_t e0 = base + c * ch;
  const int len = (int)(nbe - c * ch < ch ? nbe - c * ch : ch);  // >= 1
  chunk_by_rows<PACK, TERN, SMALL, CACHED>(a, q, b, e0, len, lds, red, red_ne);
}

hipError_t launch_rows(const Geometry& geo, const Pass1Args& a0, hipStream_t s) {
  const bool small = small_problem(geo);
  const bool cached = small || gradient_bytes(geo) <= kCachedBytes;
  const bool tern = a0.nbits != nullptr, pack = a0.bits && !tern;
  const auto kernel =
      tern ? k_rows<false, true, false, false>  // above kOneReadBytes
      : pack ? (small ? k_rows<true, false, true, true> : cached ? k_rows<true, false, false, true> : k_rows<true, false, false, false>)
             : (small ? k_rows<false, false, true, true> : cached ? k_rows<false, false, false, true> : k_rows<false, false, false, false>);
  Pass1Args a = a0;
  a.wtot = geo.W;
  a.item_words = (int)(ceil_div((int64_t)geo.G * geo.tile / 64, kBatch) * kBatch);
  // Up to 64 workers a block takes all rows of its chunk, and the launches
  // (two above 32 workers) are shares of the chunks; above, a launch takes a
  // row group of every chunk, in order where the FP32 sums go from one
  // group to the next.
  const bool by_group = !small && geo.W > kRowGroup;
  const int launches = (int)pass1_launches(geo, tern ? 2 : pack);
  for (int i = 0; i < launches; ++i) {
    int wb = 0, rows = geo.W;
    int64_t q0 = 0, q1 = geo.total_chunks;
    if (by_group) {
      row_group(geo, i, &wb, &rows);
    } else {
      q0 = geo.total_chunks * i / launches;
      q1 = geo.total_chunks * (i + 1) / launches;
      if (q1 == q0) continue;
    }
    a.W = rows;
    a.racc = wb > 0;
    a.rfin = wb + rows == geo.W;
    a.g = a0.g + (int64_t)wb * a0.wstride;
    if (a0.bits) a.bits = a0.bits + (int64_t)wb * a0.bstride;
    if (tern) {
      a.nbits = a0.nbits + (int64_t)wb * a0.bstride;
      a.win = a0.win + wb;
    }
    a.part = a0.part + wb;
    a.parts = pass1_parts(rows, a.item_words / kBatch);
    // sign words: a row for each wavefront, or (several items a worker) for
    // each worker
    const size_t lds =
        (size_t)((pack ? 1 : tern ? 2 : 0) * (a.parts == 1 ? kWaves : rows)) * a.item_words * sizeof(uint64_t);
    if (lds > 65536 - kItems * sizeof(Partial) - 1024) {
      // above 64 KiB of LDS a kernel must opt in (gfx950 has 160 KiB per CU)
      const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
    }
    const bool ordered = i == 0 || (by_group && a.sums != kSumsNone);
    hipExtLaunchKernelGGL(kernel, dim3((unsigned)(q1 - q0)), dim3(kThreads1), lds, s, nullptr, nullptr,
                          ordered ? 0u : (uint32_t)hipExtAnyOrderLaunch, a, q0);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace nf
