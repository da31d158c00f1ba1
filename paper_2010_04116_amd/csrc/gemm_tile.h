// Which problem, which output tile and which part of the reduction a workgroup of a GEMM launch takes.
#pragma once
#include <algorithm>
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
// Output tiles of a problem (m x n of them) and their edges.
struct TileGrid { int m, n, bm, bn; };

// Where the `at`-th of a problem's tiles lies.
struct TilePlace { int m, n; };
__host__ __device__ inline TilePlace tile_place(int at, int tiles_m, int tiles_n) {
  constexpr int GM = 8;  // rows of tiles that are taken column by column
  const int per_group = GM * tiles_n, first_m = at / per_group * GM, left = tiles_m - first_m, rows = left < GM ? left : GM;
  return {first_m + at % per_group % rows, at % per_group / rows};
}
// The place in that order of the workgroup `local` of `total`.  Workgroups land on XCD `local` mod 8.  in_turn: in launch
// order; otherwise XCD x gets as many consecutive places as it has workgroups, also where eight does not divide the count.
__host__ __device__ inline int tile_turn(int local, int total, bool in_turn) {
  const int xcd = local & 7, rest = total & 7, run = xcd * (total >> 3) + (xcd < rest ? xcd : rest) + (local >> 3);
  return in_turn ? local : run;
}
// Which of the two, where eight does not divide the number of tiles: the one for which the XCDs' L2s fetch fewer operand
// rows and columns.  In launch order XCD x has every eighth row of tiles and all columns; with consecutive places it has
// neighbouring rows and columns, but two neighbours on both sides of a group of eight rows' end.  So launch order is for tall
// outputs of few columns, us, in turn and consecutive: 1768 x 296 x 3064 12.8 and 16.6, 5168 x 280 x 4872 40.0 and 47.5, 3112 x 728 x 4104
// 46.0 and 54.1, 2136 x 280 x 1872 9.2 and 11.5; but 272 x 1184 x 2968 17.6 and 11.4, 832 x 1960 x 1920 21.4 and 16.8, 832 x 31992 x 768
// 79.6 and 71.9, 1600 x 2304 x 768 13.5 and 12.2, 3984 x 184 x 2568 (each XCD one group) 15.3 and 11.5.  Of 890 products whose tiles
// eight does not divide, consecutive places alone took up to 31 % longer than launch order; by this count the worst takes 15 %.
// Consecutive stay parts along K, which were within 5 % of launch order everywhere, sums of less than 1024, for which the two are
// as fast (70 such products: median 0.995, 5 % either way, one 10 %), and what a twentieth of the operands would decide.
inline bool tiles_in_turn(const TileGrid &t, int K, int splits) {
  const int total = t.m * t.n;
  if (splits > 1 || K < 1024 || t.m < 9 || (total & 7) == 0) return false;
  const int groups = t.m >> 3, left = t.m & 7, of_left = (left * t.n + 7) / 8;
  // rows of the last, incomplete group that every eighth of its tiles meets, no more than these are
  const int left_rows = std::min(left == 0 ? 0 : left == 4 ? 1 : (left & 1) ? left : left / 2, of_left);
  const long turn = 8l * ((groups + left_rows) * t.bm + t.n * t.bn);
  long run = 0;
  for (int x = 0, at = 0; x < 8; ++x) {
    const int end = at + (total >> 3) + (x < (total & 7));
    if (end == at) continue;
    const int group = 8 * t.n, g0 = at / group, g1 = (end - 1) / group, rows0 = std::min(8, t.m - 8 * g0), rows1 = std::min(8, t.m - 8 * g1);
    const int c0 = at % group / rows0, c1 = (end - 1) % group / rows1;  // first column of the first group, last of the last
    const int cols = g1 == g0 ? c1 - c0 + 1 : g1 == g0 + 1 ? std::min(t.n, t.n - c0 + c1 + 1) : t.n;
    const int rows = g1 == g0 ? std::min(rows0, end - at)
                              : std::min(rows0, group * (g0 + 1) - at) + 8 * (g1 - g0 - 1) + std::min(rows1, end - group * g1);
    run += rows * t.bm + cols * t.bn;
    at = end;
  }
  return turn + turn / 20 < run;
}

// go(the launch's problems, its workgroups); grid(p): the tiles of problem p.
template <bool SEVERAL, typename T, typename F>
hipError_t with_problems(const GemmArgs *list, int count, T &&grid, F &&go) {
  auto take = [&](GemmArgs &p, const GemmArgs &from) {
    p = from;
    const TileGrid t = grid(from);
    if (tiles_in_turn(t, from.K, from.splits)) p.splits = kInTurn;
    return t.m * t.n * std::max(from.splits, 1);
  };
  if (count == 1) {
    Problems<1> one;
    const int tiles = take(one.p[0], list[0]);
    return go(one, tiles);
  }
  if constexpr (SEVERAL) {
    Problems<kMaxBatch> b;
    memset(&b, 0, sizeof(b));
    b.count = count;
    int end = 0;
    for (int i = 0; i < count; ++i) b.tile_end[i] = end += take(b.p[i], list[i]);
    return go(b, end);
  } else {
    return hipErrorInvalidValue;
  }
}

// The tile of a workgroup: `local` is its index within its problem, tiles_m x tiles_n the problem's output tiles.  Sets the
// reduction range [k0, k1) and points g.C at the part's output.
struct MyTile { int m, n, k0, k1; };
__device__ inline MyTile my_tile(GemmArgs &g, int local, int tiles_m, int tiles_n) {
  const int tiles = tiles_m * tiles_n, splits = g.splits > 1 ? g.splits : 1;
  local = tile_turn(local, tiles * splits, g.splits == kInTurn);
  MyTile t{0, 0, 0, g.K};
  if (splits > 1) {
    const int part = local / tiles;
    local -= part * tiles;
    t.k0 = part * g.k_per;
    t.k1 = min(g.K, t.k0 + g.k_per);
    g.C = (float *)g.C + (size_t)part * g.M * g.N;
  }
  const TilePlace at = tile_place(local, tiles_m, tiles_n);
  t.m = at.m;
  t.n = at.n;
  return t;
}
// every part starts inside K, on a multiple of the K step
inline bool split_ok(const GemmArgs &g) {
  return g.splits < 2 || (g.epi == EPI_STORE_F32 && g.ldc == g.N && g.k_per > 0 && g.k_per % 64 == 0 &&
                          (long long)(g.splits - 1) * g.k_per < g.K);
}

}  // namespace il
