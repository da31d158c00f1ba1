// Which output tile and which part of the reduction a workgroup of a GEMM launch takes.
#pragma once
#include "common.h"

namespace il {

// `local`: the workgroup's index within its problem, `tiles`: output tiles of the problem.  Workgroups that
// land on one XCD (index mod 8) take neighbouring tiles of the same part: XCD x gets as many consecutive places as it has
// workgroups, also where eight does not divide the count.  (Left in launch order, such a count had eight neighbours fetch
// their operand panels into eight L2s: 832 x 31992 x 768, 500 tiles of 256 x 256, 79.6 -> 71.9 us, 1600 x 2304 x 768, 234 of
// 128 x 128, 13.5 -> 12.2 us; the bf16 step of 1600 tokens at d = 768 4.80 -> 4.50 ms.)  Returns the tile; sets the reduction
// range [k0, k1) and points g.C at the part's output.
__device__ inline int my_tile(GemmArgs &g, int local, int tiles, int &k0, int &k1) {
  const int splits = g.splits > 1 ? g.splits : 1, total = tiles * splits;
  const int xcd = local & 7;
  local = xcd * (total >> 3) + min(xcd, total & 7) + (local >> 3);
  k0 = 0;
  k1 = g.K;
  if (splits > 1) {
    const int part = local / tiles;
    local -= part * tiles;
    k0 = part * g.k_per;
    k1 = min(g.K, k0 + g.k_per);
    g.C = (float *)g.C + (size_t)part * g.M * g.N;
  }
  return local;
}
// every part starts inside K, on a multiple of the K step
inline bool split_ok(const GemmArgs &g) {
  return g.splits < 2 || (g.epi == EPI_STORE_F32 && g.ldc == g.N && g.k_per > 0 && g.k_per % 64 == 0 &&
                          (long long)(g.splits - 1) * g.k_per < g.K);
}

}  // namespace il
