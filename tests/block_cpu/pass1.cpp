// k_pass1 with the G-Ternary planes, one block at a time on the CPU
// (hip/hip_runtime.h here), while the bucket's fallback flag turns between
// the wavefronts' loads.  PASS1_KERNELS: nf_pass1.hip's kernels, prepared by
// test_pass1_block.py.
#include PASS1_KERNELS

namespace nf {
unsigned char smem[160 << 10];
}

// g [W][n], mask and bits [2W] rows of n / 64 words, windows and flag in
// stats [W]; the flag reads 0 in wavefronts before `turn` and 1 from there
// on.  Runs the bucket's chunks, a row group after another; part [chunks][W],
// part_ne [chunks].
// Returns 0, or 1 with the fault in msg.
extern "C" int pass1_planes(const float* g, const uint64_t* mask, int W, int64_t n, int G, int turn, uint64_t* bits,
                            float* out, void* part, uint64_t* part_ne, void* stats, char* msg) {
  const nf::Geometry geo = nf::geometry_core(W);
  if (geo.wpw == 2) return 2;
  nf::Pass1Args a;
  memset(&a, 0, sizeof a);
  const int64_t words = (n + 63) / 64, chunk = (int64_t)G * geo.tile;
  a.g = g;
  a.wstride = n;
  a.mask = mask;
  a.bits = bits;
  a.nbits = bits + W * words;
  a.bstride = words;
  a.out = out;
  a.part = (nf::Partial*)part;
  a.part_ne = part_ne;
  a.n_total = a.bucket_n = n;
  a.chunks_full = a.total_chunks = a.slots = (n + chunk - 1) / chunk;
  a.nb = 1;
  a.wtot = W;
  a.wg = geo.wg;
  a.eg = geo.eg;
  a.T = geo.T;
  a.G = G;
  a.sums = nf::kSumsRouted;
  a.win = a.win0 = (nf_worker_stats*)stats;
  a.ratio = 32.0f;
  cpu::on_load = [&](const float*, int wavefront) { return wavefront >= turn ? 1.0f : 0.0f; };
  const nf::Pass1Args a0 = a;
  for (int grp = 0; grp < geo.ngroups; ++grp) {
    int wb;
    nf::row_group(geo, grp, &wb, &a.W);
    a.racc = grp > 0;
    a.rfin = grp == geo.ngroups - 1;
    a.g = a0.g + wb * n;
    a.bits = a0.bits + wb * words;
    a.nbits = a0.nbits + wb * words;
    a.win = a0.win + wb;
    a.part = a0.part + wb;
    for (int64_t q = 0; q < a.total_chunks; ++q) {
      const std::string fault = cpu::run(nf::kThreads1, (unsigned)q, [&] {
        if (geo.wpw == 1)
          nf::k_pass1<1, false, true>(a.g, a.mask, a.bits, a.out, a.part, a.part_ne, a, 0);
        else
          nf::k_pass1<4, false, true>(a.g, a.mask, a.bits, a.out, a.part, a.part_ne, a, 0);
      });
      if (!fault.empty()) {
        snprintf(msg, 200, "row group %d, chunk %lld: %s", grp, (long long)q, fault.c_str());
        return 1;
      }
    }
  }
  return 0;
}
