// Which problem, which output tile and which part of the reduction a workgroup of a GEMM launch takes.
#pragma once
#include <cstring>

#include "common.h"

namespace il {

// The problems of one launch, passed by value.  Only the weight gradients go several to a launch; all others are launched
// with room for one, whose fields are read at fixed places by the first instructions.  (With room for eight the host wrote
// 1.4 KB of arguments per launch, 4.3 us against 3.3, and a workgroup read the count, then its problem, before it could start.)
template <int MAX>
struct Problems {
  static constexpr int kRoom = MAX;
  int count;
  int tile_end[MAX];  // exclusive prefix of tile counts
  GemmArgs p[MAX];
};
template <>
struct Problems<1> {
  static constexpr int kRoom = 1;
  GemmArgs p[1];
};
// The problem of this workgroup (uniform) and that problem's first workgroup.
template <int MAX>
__device__ inline GemmArgs my_problem(const Problems<MAX> &b, int &first) {
  first = 0;
  if constexpr (MAX == 1) {
    return b.p[0];
  } else {
    int prob = 0;
    for (int i = 0; i < b.count - 1; ++i)
      if ((int)blockIdx.x >= b.tile_end[i]) { prob = i + 1; first = b.tile_end[i]; }
    return b.p[prob];
  }
}
// go(the launch's problems, its workgroups); tiles(p): the workgroups of problem p.
template <bool SEVERAL, typename T, typename F>
hipError_t with_problems(const GemmArgs *list, int count, T &&tiles, F &&go) {
  if (count == 1) {
    Problems<1> one;
    one.p[0] = list[0];
    return go(one, tiles(list[0]));
  }
  if constexpr (SEVERAL) {
    Problems<kMaxBatch> b;
    memset(&b, 0, sizeof(b));
    b.count = count;
    int end = 0;
    for (int i = 0; i < count; ++i) {
      b.p[i] = list[i];
      b.tile_end[i] = end += tiles(list[i]);
    }
    return go(b, end);
  } else {
    return hipErrorInvalidValue;
  }
}

// The tile of a workgroup: `local` is its index within its problem, tiles_m x tiles_n the problem's output tiles.
// Workgroups that land on one XCD (index mod 8) take neighbouring tiles of the same part: XCD x gets as many consecutive
// places as it has workgroups, also where eight does not divide the count.  (Left in launch order, such a count had eight
// neighbours fetch their operand panels into eight L2s: 832 x 31992 x 768, 500 tiles of 256 x 256, 79.6 -> 71.9 us,
// 1600 x 2304 x 768, 234 of 128 x 128, 13.5 -> 12.2 us; the bf16 step of 1600 tokens at d = 768 4.80 -> 4.50 ms.)  Sets the
// reduction range [k0, k1) and points g.C at the part's output.
struct MyTile { int m, n, k0, k1; };
__device__ inline MyTile my_tile(GemmArgs &g, int local, int tiles_m, int tiles_n) {
  const int tiles = tiles_m * tiles_n, splits = g.splits > 1 ? g.splits : 1, total = tiles * splits;
  const int xcd = local & 7;
  local = xcd * (total >> 3) + min(xcd, total & 7) + (local >> 3);
  MyTile t{0, 0, 0, g.K};
  if (splits > 1) {
    const int part = local / tiles;
    local -= part * tiles;
    t.k0 = part * g.k_per;
    t.k1 = min(g.K, t.k0 + g.k_per);
    g.C = (float *)g.C + (size_t)part * g.M * g.N;
  }
  constexpr int GM = 8;  // rows of tiles that are taken column by column
  const int per_group = GM * tiles_n, first_m = local / per_group * GM, rows = min(tiles_m - first_m, GM);
  t.m = first_m + local % per_group % rows;
  t.n = local % per_group / rows;
  return t;
}
// every part starts inside K, on a multiple of the K step
inline bool split_ok(const GemmArgs &g) {
  return g.splits < 2 || (g.epi == EPI_STORE_F32 && g.ldc == g.N && g.k_per > 0 && g.k_per % 64 == 0 &&
                          (long long)(g.splits - 1) * g.k_per < g.K);
}

}  // namespace il
