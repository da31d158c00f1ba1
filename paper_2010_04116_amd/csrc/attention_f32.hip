// Causal attention with fp32 products: the path of fp32 runs, and of bf16 runs with narrow heads (16 and 32),
// where probabilities and their gradients stay fp32.  v_mfma_f32_16x16x4_f32 on fp32 values staged in
// LDS (bf16 inputs are widened on the way in), fp32 softmax; nothing is rounded below the inputs' and
// outputs' own type.
//
// A wavefront owns 16 queries (forward, dQ) or 16 keys (dK, dV).  Where there are enough of them a workgroup is four
// such neighbours, which share tiles of the other axis in LDS: a T = 256, 64-head problem then is one wavefront per
// SIMD, and the longest one 16 k matrix cycles.  In small grids it is four or eight wavefronts that share 16 queries
// (keys) and divide up the other axis (the second half of this file).  (One thread per row, as this file's predecessor
// had it, left most lanes' loads serial: forward + backward of a block took 1.5 ms at 8 x 256 tokens, 8 heads of 64.)
//
// Layout of a product: lane l holds matrix row (A) or column (B) l & 15 and k = l >> 4; of the result
// column l & 15, rows 4 (l >> 4) + 0..3.  Scores are computed with the streamed axis as rows, so a lane
// owns one query (key) and its four registers are four consecutive streamed rows: k step r of the second
// product takes register r as its B operand and streamed row 4 (l >> 4) + r as its A operand, and
// probabilities never leave the registers.
//
// A query sees the keys up to its own and nothing else: 16-row blocks without a visible pair are not computed,
// and a masked score is -inf, never a finite number that a visible score can lie below.  In the one 16x16 block
// on the diagonal a matrix product multiplies every streamed row into every owned column, so there a row that is
// not finite reaches columns it is masked for (0 x NaN).  A wavefront whose sums come out other than finite
// therefore adds them up again pair by pair, over the visible pairs only: nothing in the loop pays for it (a
// check of that block's operands cost 5 % at widths up to 64 and 25 % at 128, by its registers).
#include <type_traits>

#include "common.h"

namespace il {
namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f4;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr int kOwn = 64;  // queries / keys per workgroup, 16 per wavefront

__device__ inline f4 get4(const float *p) { return *reinterpret_cast<const f4 *>(p); }
__device__ inline f4 get4(const bf16_t *p) {
  const uint2 q = *reinterpret_cast<const uint2 *>(p);
  return f4{bf16_to_f32((bf16_t)(q.x & 0xFFFF)), bf16_to_f32((bf16_t)(q.x >> 16)), bf16_to_f32((bf16_t)(q.y & 0xFFFF)),
            bf16_to_f32((bf16_t)(q.y >> 16))};
}
__device__ inline void put4(float *p, f4 v) { *reinterpret_cast<f4 *>(p) = v; }
__device__ inline void put4(bf16_t *p, f4 v) {
  *reinterpret_cast<uint2 *>(p) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
}
__device__ inline f4 mma(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ inline float sum_groups(float v) {  // over the four lanes that hold a column
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}

// ROWS x DH fp32 values in LDS, filled by 256 threads through registers.  16-byte chunk c of row r sits at
// c ^ (r >> S) & (CPR - 1): the 16 rows of a vector read start in 16 different places of the 256-byte bank
// span, whatever the row length.
template <int ROWS, int DH>
struct Tile {
  static constexpr int CPR = DH / 4, NLD = ROWS * CPR / 256, S = CPR >= 16 ? 0 : (CPR == 8 ? 1 : 2);
  static constexpr int MASK = (CPR < 16 ? CPR : 16) - 1, FLOATS = ROWS * DH;
  static_assert(NLD >= 1 && ROWS * CPR % 256 == 0, "a tile divides over the threads");
  f4 reg[NLD];
  __device__ static inline int at(int r, int c) { return r * DH + ((c ^ ((r >> S) & MASK)) << 2); }
  // rows [row0, row0 + ROWS) of a matrix with `ld` elements per row; rows >= end read as zero
  template <typename T>
  __device__ inline void fetch(const T *base, size_t ld, int row0, int end, int t) {
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int p = i * 256 + t, r = row0 + p / CPR;
      reg[i] = r < end ? get4(base + (size_t)r * ld + (p % CPR) * 4) : f4{0.f, 0.f, 0.f, 0.f};
    }
  }
  __device__ inline void put(float *lds, int t) const {
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int p = i * 256 + t;
      *reinterpret_cast<f4 *>(lds + at(p / CPR, p % CPR)) = reg[i];
    }
  }
  // rows r0 + (lane & 15), columns 16 s + 4 (lane >> 4) + 0..3
  __device__ static inline f4 rows(const float *lds, int r0, int s, int lane) {
    return *reinterpret_cast<const f4 *>(lds + at(r0 + (lane & 15), 4 * s + (lane >> 4)));
  }
  // row r0 + 4 (lane >> 4) + r, column 16 dt + (lane & 15)
  __device__ static inline float cols(const float *lds, int r0, int r, int dt, int lane) {
    return lds[at(r0 + 4 * (lane >> 4) + r, 4 * dt + ((lane & 15) >> 2)) + (lane & 3)];
  }
};

template <typename T, int DH>
__device__ inline void load_own(f4 (&f)[DH / 16], const T *row, bool in, int lane) {
#pragma unroll
  for (int s = 0; s < DH / 16; ++s) f[s] = in ? get4(row + 16 * s + 4 * (lane >> 4)) : f4{0.f, 0.f, 0.f, 0.f};
}
template <int DH>
__device__ inline void zero(f4 (&f)[DH / 16]) {
#pragma unroll
  for (int s = 0; s < DH / 16; ++s) f[s] = f4{0.f, 0.f, 0.f, 0.f};
}
template <typename T, int DH>
__device__ inline void store_own(T *row, const f4 (&f)[DH / 16], float scale, int lane) {
#pragma unroll
  for (int s = 0; s < DH / 16; ++s) put4(row + 16 * s + 4 * (lane >> 4), f[s] * scale);
}

// What exponentials are taken relative to while the maximum so far is m: scores of -inf weigh nothing.
__device__ inline float base_of(float m) { return m == -INFINITY ? 0.f : m; }

// acc[dh][column] += sum over the 16 streamed rows of w[row][column] X[row][dh], in the layout above (w[r]: row
// 4 (lane >> 4) + r).
template <typename TL, int DH>
__device__ inline void add_block(f4 (&acc)[DH / 16], const float *lds, int r0, const f4 &w, int lane) {
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int dt = 0; dt < DH / 16; ++dt) acc[dt] = mma(TL::cols(lds, r0, r, dt, lane), w[r], acc[dt]);
}
// ... and pair by pair, for the wavefronts that redo their sums: own . X of a streamed row, acc += w X.
template <typename T, int DH>
__device__ inline float dot_row(const f4 (&own)[DH / 16], const T *X, int lane) {
  float s = 0.f;
#pragma unroll
  for (int e4 = 0; e4 < DH / 16; ++e4) {
    const f4 x = get4(X + 16 * e4 + 4 * (lane >> 4));
#pragma unroll
    for (int e = 0; e < 4; ++e) s = fmaf(own[e4][e], x[e], s);
  }
  return sum_groups(s);
}
template <typename T, int DH>
__device__ inline void add_row(f4 (&acc)[DH / 16], float w, const T *X, int lane) {
#pragma unroll
  for (int dt = 0; dt < DH / 16; ++dt) acc[dt] += get4(X + 16 * dt + 4 * (lane >> 4)) * w;
}
template <int DH>
__device__ inline bool all_finite(const f4 (&acc)[DH / 16]) {  // (uniform over the wavefront)
  bool ok = true;
#pragma unroll
  for (int dt = 0; dt < DH / 16; ++dt)
#pragma unroll
    for (int e = 0; e < 4; ++e) ok = ok && __builtin_isfinite(acc[dt][e]);
  return __ballot(!ok) == 0;
}

// Streamed rows per LDS tile: two stages of two tiles stay within 64 KB.
constexpr int tile_rows(int dh) { return dh >= 128 ? 32 : 64; }

// grid (ceil(T/64), B*H); the longest query tiles start first
template <typename T, int DH>
__global__ __launch_bounds__(256) void attn_fwd_f32(const T *__restrict__ qkv, int Tn, int H, T *__restrict__ o,
                                                    float *__restrict__ lse) {
  constexpr int R = tile_rows(DH), NB = R / 16;
  typedef Tile<R, DH> TL;
  __shared__ __attribute__((aligned(16))) float sm[2][2][TL::FLOATS];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), kk = lane >> 4;
  const int b = blockIdx.y / H, h = blockIdx.y % H, d = H * DH;
  const size_t ld = 3 * (size_t)d;
  const T *base = qkv + (size_t)b * Tn * ld + h * DH;
  const int q0 = (gridDim.x - 1 - blockIdx.x) * kOwn, qw = q0 + 16 * wave, q = qw + (lane & 15);
  const int nt = (min(Tn, q0 + kOwn) + R - 1) / R;
  f4 qf[DH / 16], acc[DH / 16];
  load_own<T, DH>(qf, base + (size_t)q * ld, q < Tn, lane);
  zero<DH>(acc);
  float m = -INFINITY, l = 0.f;
  const float sc = rsqrtf((float)DH) * kLog2e;
  TL tk, tv;
  tk.fetch(base + d, ld, 0, Tn, t);
  tv.fetch(base + 2 * d, ld, 0, Tn, t);
  for (int it = 0; it < nt; ++it) {
    float *sk = sm[it & 1][0], *sv = sm[it & 1][1];
    tk.put(sk, t);
    tv.put(sv, t);
    __syncthreads();  // (the other stage was last read before the previous barrier but one)
    if (it + 1 < nt) {
      tk.fetch(base + d, ld, (it + 1) * R, Tn, t);
      tv.fetch(base + 2 * d, ld, (it + 1) * R, Tn, t);
    }
    const int kv0 = it * R;
    if (kv0 > qw + 15) continue;
    const int live = min(NB, (qw + 15 - kv0) / 16 + 1);  // blocks that some query of the wavefront sees (uniform)
    f4 s[NB];
    float mx = -INFINITY;
#pragma unroll
    for (int a = 0; a < NB; ++a) {
      if (a >= live) break;
      s[a] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int e4 = 0; e4 < DH / 16; ++e4) {
        const f4 kf = TL::rows(sk, 16 * a, e4, lane);
#pragma unroll
        for (int e = 0; e < 4; ++e) s[a] = mma(kf[e], qf[e4][e], s[a]);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int kv = kv0 + 16 * a + 4 * kk + r;
        s[a][r] = kv > q || kv >= Tn ? -INFINITY : s[a][r] * sc;
        mx = fmaxf(mx, s[a][r]);
      }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mn = fmaxf(m, mx), at = base_of(mn), alpha = __builtin_amdgcn_exp2f(m - at);
    m = mn;
    l *= alpha;
#pragma unroll
    for (int i = 0; i < DH / 16; ++i) acc[i] *= alpha;
#pragma unroll
    for (int a = 0; a < NB; ++a) {
      if (a >= live) break;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[a][r] = __builtin_amdgcn_exp2f(s[a][r] - at);
        l += s[a][r];
      }
      add_block<TL, DH>(acc, sv, 16 * a, s[a], lane);
    }
  }
  if (!all_finite<DH>(acc)) {
    zero<DH>(acc);
    for (int u = 0; u < min(Tn, qw + 16); ++u) {
      const T *row = base + u * ld;
      const float p = __builtin_amdgcn_exp2f(dot_row<T, DH>(qf, row + d, lane) * sc - base_of(m));
      if (u <= q) add_row<T, DH>(acc, p, row + 2 * d, lane);
    }
  }
  l = sum_groups(l);
  if (q < Tn) {
    store_own<T, DH>(o + ((size_t)b * Tn + q) * d + h * DH, acc, 1.f / l, lane);
    if (kk == 0) lse[((size_t)b * H + h) * Tn + q] = (m + log2f(l)) * kLn2;
  }
}

// dQ, and dsum[s][b][h][t] = sum_i dO O for the dK/dV kernel; grid (ceil(T/64), B*H, streams)
template <typename T, int DH>
__global__ __launch_bounds__(256) void attn_dq_f32(const T *__restrict__ qkv, const T *__restrict__ o,
                                                   const T *__restrict__ d_o, const float *__restrict__ lse, int Tn,
                                                   int H, int B, T *__restrict__ dqkv, float *__restrict__ dsum) {
  constexpr int R = tile_rows(DH), NB = R / 16;
  typedef Tile<R, DH> TL;
  __shared__ __attribute__((aligned(16))) float sm[2][2][TL::FLOATS];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), kk = lane >> 4;
  const int b = blockIdx.y / H, h = blockIdx.y % H, d = H * DH, sidx = blockIdx.z;
  const size_t ld = 3 * (size_t)d, N = (size_t)B * Tn;
  const T *base = qkv + (size_t)b * Tn * ld + h * DH;
  const int q0 = (gridDim.x - 1 - blockIdx.x) * kOwn, qw = q0 + 16 * wave, q = qw + (lane & 15);
  const int nt = (min(Tn, q0 + kOwn) + R - 1) / R;
  const size_t tok = (size_t)b * Tn + q;
  f4 qf[DH / 16], gf[DH / 16], dq[DH / 16];
  load_own<T, DH>(qf, base + (size_t)q * ld, q < Tn, lane);
  load_own<T, DH>(gf, d_o + (sidx * N + tok) * d + h * DH, q < Tn, lane);
  load_own<T, DH>(dq, o + tok * d + h * DH, q < Tn, lane);
  float D = 0.f;
#pragma unroll
  for (int s = 0; s < DH / 16; ++s)
#pragma unroll
    for (int e = 0; e < 4; ++e) D = fmaf(gf[s][e], dq[s][e], D);
  D = sum_groups(D);
  if (q < Tn && kk == 0) dsum[(sidx * (size_t)B * H + blockIdx.y) * Tn + q] = D;
  zero<DH>(dq);
  const float sc = rsqrtf((float)DH), sc2 = sc * kLog2e;
  const float L2 = q < Tn ? lse[((size_t)b * H + h) * Tn + q] * kLog2e : 0.f;
  TL tk, tv;
  tk.fetch(base + d, ld, 0, Tn, t);
  tv.fetch(base + 2 * d, ld, 0, Tn, t);
  for (int it = 0; it < nt; ++it) {
    float *sk = sm[it & 1][0], *sv = sm[it & 1][1];
    tk.put(sk, t);
    tv.put(sv, t);
    __syncthreads();
    if (it + 1 < nt) {
      tk.fetch(base + d, ld, (it + 1) * R, Tn, t);
      tv.fetch(base + 2 * d, ld, (it + 1) * R, Tn, t);
    }
#pragma unroll
    for (int a = 0; a < NB; ++a) {
      const int kv0 = it * R + 16 * a;
      if (kv0 > qw + 15) break;
      f4 s = {0.f, 0.f, 0.f, 0.f}, dp = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int e4 = 0; e4 < DH / 16; ++e4) {
        const f4 kf = TL::rows(sk, 16 * a, e4, lane), vf = TL::rows(sv, 16 * a, e4, lane);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s = mma(kf[e], qf[e4][e], s);
          dp = mma(vf[e], gf[e4][e], dp);
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int kv = kv0 + 4 * kk + r;
        const float ds = __builtin_amdgcn_exp2f(s[r] * sc2 - L2) * (dp[r] - D);
        s[r] = kv > q || kv >= Tn ? 0.f : ds;
      }
      add_block<TL, DH>(dq, sk, 16 * a, s, lane);
    }
  }
  if (!all_finite<DH>(dq)) {
    zero<DH>(dq);
    for (int u = 0; u < min(Tn, qw + 16); ++u) {
      const T *row = base + u * ld;
      const float p = __builtin_amdgcn_exp2f(dot_row<T, DH>(qf, row + d, lane) * sc2 - L2);
      const float ds = p * (dot_row<T, DH>(gf, row + 2 * d, lane) - D);
      if (u <= q) add_row<T, DH>(dq, ds, row + d, lane);
    }
  }
  if (q < Tn) store_own<T, DH>(dqkv + (sidx * N + tok) * ld + h * DH, dq, sc, lane);
}

// dK, dV; grid (ceil(T/64), B*H, streams); the first key tile is the longest
template <typename T, int DH>
__global__ __launch_bounds__(256) void attn_dkv_f32(const T *__restrict__ qkv, const T *__restrict__ d_o,
                                                    const float *__restrict__ lse, const float *__restrict__ dsum,
                                                    int Tn, int H, int B, T *__restrict__ dqkv) {
  constexpr int R = tile_rows(DH), NB = R / 16;
  typedef Tile<R, DH> TL;
  __shared__ __attribute__((aligned(16))) float sm[2][2][TL::FLOATS];
  __shared__ __attribute__((aligned(16))) float st[2][2][R];  // lse (in powers of two) and dsum of the tile's rows
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), kk = lane >> 4;
  const int b = blockIdx.y / H, h = blockIdx.y % H, d = H * DH, sidx = blockIdx.z;
  const size_t ld = 3 * (size_t)d, N = (size_t)B * Tn;
  const T *base = qkv + (size_t)b * Tn * ld + h * DH, *gbase = d_o + (sidx * N + (size_t)b * Tn) * d + h * DH;
  const float *lrow = lse + ((size_t)b * H + h) * Tn, *drow = dsum + (sidx * (size_t)B * H + blockIdx.y) * Tn;
  const int kv0 = blockIdx.x * kOwn, kw = kv0 + 16 * wave, kv = kw + (lane & 15);
  const int it0 = kv0 / R, nt = (Tn + R - 1) / R;
  f4 kf[DH / 16], vf[DH / 16], dk[DH / 16], dv[DH / 16];
  load_own<T, DH>(kf, base + (size_t)kv * ld + d, kv < Tn, lane);
  load_own<T, DH>(vf, base + (size_t)kv * ld + 2 * d, kv < Tn, lane);
  zero<DH>(dk);
  zero<DH>(dv);
  const float sc = rsqrtf((float)DH), sc2 = sc * kLog2e;
  TL tq, tg;
  float ls = 0.f;
  auto fetch = [&](int it) {
    tq.fetch(base, ld, it * R, Tn, t);
    tg.fetch(gbase, (size_t)d, it * R, Tn, t);
    const int r = it * R + t % R;
    if (t < 2 * R) ls = r < Tn ? (t < R ? lrow[r] * kLog2e : drow[r]) : 0.f;
  };
  fetch(it0);
  for (int it = it0; it < nt; ++it) {
    float *sq = sm[it & 1][0], *sg = sm[it & 1][1];
    tq.put(sq, t);
    tg.put(sg, t);
    if (t < 2 * R) st[it & 1][t / R][t % R] = ls;
    __syncthreads();
    if (it + 1 < nt) fetch(it + 1);
#pragma unroll
    for (int a = 0; a < NB; ++a) {
      const int q0 = it * R + 16 * a;
      if (q0 + 15 < kw || q0 >= Tn) continue;  // every query of the block precedes every key
      f4 s = {0.f, 0.f, 0.f, 0.f}, dp = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int e4 = 0; e4 < DH / 16; ++e4) {
        const f4 qf = TL::rows(sq, 16 * a, e4, lane), gf = TL::rows(sg, 16 * a, e4, lane);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s = mma(qf[e], kf[e4][e], s);
          dp = mma(gf[e], vf[e4][e], dp);
        }
      }
      const f4 l4 = *reinterpret_cast<const f4 *>(&st[it & 1][0][16 * a + 4 * kk]);
      const f4 d4 = *reinterpret_cast<const f4 *>(&st[it & 1][1][16 * a + 4 * kk]);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int q = q0 + 4 * kk + r;
        const bool seen = kv <= q && q < Tn;
        const float p = seen ? __builtin_amdgcn_exp2f(s[r] * sc2 - l4[r]) : 0.f;
        dp[r] = seen ? p * (dp[r] - d4[r]) : 0.f;
        s[r] = p;
      }
      add_block<TL, DH>(dv, sg, 16 * a, s, lane);
      add_block<TL, DH>(dk, sq, 16 * a, dp, lane);
    }
  }
  if (!all_finite<DH>(dv) || !all_finite<DH>(dk)) {
    zero<DH>(dv);
    zero<DH>(dk);
    for (int u = kw; u < Tn; ++u) {
      const T *qr = base + u * ld, *gr = gbase + (size_t)u * d;
      const float p = __builtin_amdgcn_exp2f(dot_row<T, DH>(kf, qr, lane) * sc2 - lrow[u] * kLog2e);
      const float ds = p * (dot_row<T, DH>(vf, gr, lane) - drow[u]);
      if (u < kv) continue;
      add_row<T, DH>(dv, p, gr, lane);
      add_row<T, DH>(dk, ds, qr, lane);
    }
  }
  if (kv < Tn) {
    T *out = dqkv + (sidx * N + (size_t)b * Tn + kv) * ld + d + h * DH;
    store_own<T, DH>(out, dk, sc, lane);
    store_own<T, DH>(out + d, dv, 1.f, lane);
  }
}

// ---- the same with a workgroup's wavefronts on different parts of the streamed axis ------------------------------
// A wavefront's chain over a long row is what a small grid waits for.  Here a workgroup owns 16 queries (keys), its W wavefronts take
// every W-th 16-row block of the streamed axis each, straight from memory - no row is read by two of them - and add up
// what they have through LDS.

// N consecutive elements as fp32, zero where the row does not exist
template <int N, typename T>
__device__ inline void get_row(float (&v)[N], const T *p, bool in) {
  if constexpr (N >= 4) {
#pragma unroll
    for (int i = 0; i < N / 4; ++i) {
      const f4 x = in ? get4(p + 4 * i) : f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int e = 0; e < 4; ++e) v[4 * i + e] = x[e];
    }
  } else if constexpr (N == 2) {
    if constexpr (sizeof(T) == 4) {
      const float2 x = in ? *reinterpret_cast<const float2 *>(p) : make_float2(0.f, 0.f);
      v[0] = x.x;
      v[1] = x.y;
    } else {
      const uint32_t x = in ? *reinterpret_cast<const uint32_t *>(p) : 0;
      v[0] = bf16_to_f32((bf16_t)(x & 0xFFFF));
      v[1] = bf16_to_f32((bf16_t)(x >> 16));
    }
  } else {
    v[0] = in ? ld<T>(p) : 0.f;
  }
}
template <int N, typename T>
__device__ inline void put_row(T *p, const float (&v)[N]) {
  if constexpr (N >= 4) {
#pragma unroll
    for (int i = 0; i < N / 4; ++i) put4(p + 4 * i, f4{v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]});
  } else if constexpr (N == 2) {
    if constexpr (sizeof(T) == 4) *reinterpret_cast<float2 *>(p) = make_float2(v[0], v[1]);
    else *reinterpret_cast<uint32_t *>(p) = pack_bf16x2(v[0], v[1]);
  } else {
    st<T>(p, v[0]);
  }
}

// A 16-row block of the streamed axis as A operand, rows [row0, row0 + 16) of X below `end`: with the rows as matrix rows
// (ByRow: lane's row l & 15, columns 16 s + 4 (l >> 4) + 0..3) and with the columns as matrix rows (ByCol: the lane's rows are
// 4 (l >> 4) + r, and matrix row i of tile dt is column i DH / 16 + dt, so that a lane reads DH / 16 neighbours).
template <typename T, int DH>
struct ByRow {
  f4 v[DH / 16];
  __device__ inline void load(const T *X, size_t ld, int row0, int end, int lane) {
    const int r = row0 + (lane & 15);
    load_own<T, DH>(v, X + (size_t)r * ld, r < end, lane);
  }
};
template <typename T, int DH>
struct ByCol {
  float v[4][DH / 16];
  __device__ inline void load(const T *X, size_t ld, int row0, int end, int lane) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = row0 + 4 * (lane >> 4) + r;
      get_row(v[r], X + (size_t)row * ld + (lane & 15) * (DH / 16), row < end);
    }
  }
};
template <typename T, int DH>
__device__ inline f4 scores(const ByRow<T, DH> &x, const f4 (&own)[DH / 16]) {
  f4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int e4 = 0; e4 < DH / 16; ++e4)
#pragma unroll
    for (int e = 0; e < 4; ++e) s = mma(x.v[e4][e], own[e4][e], s);
  return s;
}
template <typename T, int DH>
__device__ inline void add_cols(f4 (&acc)[DH / 16], const ByCol<T, DH> &x, const f4 &w) {
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int dt = 0; dt < DH / 16; ++dt) acc[dt] = mma(x.v[r][dt], w[r], acc[dt]);
}
// A lane's sums are columns (4 (l >> 4) + e) DH / 16 + dt of its query (key): DH / 4 neighbours from DH / 4 (l >> 4) on.
template <typename T, int DH>
__device__ inline void add_row_cols(f4 (&acc)[DH / 16], float w, const T *X, int lane) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float x[DH / 16];
    get_row(x, X + (4 * (lane >> 4) + e) * (DH / 16), true);
#pragma unroll
    for (int dt = 0; dt < DH / 16; ++dt) acc[dt][e] += x[dt] * w;
  }
}
// The wavefronts' sums meet in LDS: after park() and a barrier, thread t < 256 of the workgroup takes columns
// (t & 15) DH / 16 + 0.. of row t >> 4 from each.
template <int DH, int W>
struct Meet {
  static constexpr int P = DH + 4;
  float sum[W][16][P];
  __device__ inline void park(const f4 (&acc)[DH / 16], int wave, int lane) {
    float *p = sum[wave][lane & 15] + (lane >> 4) * (DH / 4);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int dt = 0; dt < DH / 16; ++dt) p[e * (DH / 16) + dt] = acc[dt][e];
  }
  __device__ inline void take(float (&v)[DH / 16], const float (&weight)[W], int t) const {
#pragma unroll
    for (int i = 0; i < DH / 16; ++i) v[i] = 0.f;
#pragma unroll
    for (int w = 0; w < W; ++w)
#pragma unroll
      for (int i = 0; i < DH / 16; ++i) v[i] = fmaf(sum[w][t >> 4][(t & 15) * (DH / 16) + i], weight[w], v[i]);
  }
};

// grid (ceil(T/16), B*H); the longest rows start first
template <typename T, int DH, int W>
__global__ __launch_bounds__(64 * W) void attn_fwd_split_f32(const T *__restrict__ qkv, int Tn, int H, T *__restrict__ o,
                                                             float *__restrict__ lse) {
  __shared__ __attribute__((aligned(16))) Meet<DH, W> meet;
  __shared__ float ms[W][16], ls[W][16];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), kk = lane >> 4;
  const int b = blockIdx.y / H, h = blockIdx.y % H, d = H * DH;
  const size_t ld = 3 * (size_t)d;
  const T *base = qkv + (size_t)b * Tn * ld + h * DH;
  const int last = gridDim.x - 1 - blockIdx.x, q0 = 16 * last, q = q0 + (lane & 15);  // key blocks 0 .. last
  f4 qf[DH / 16], acc[DH / 16];
  load_own<T, DH>(qf, base + (size_t)q * ld, q < Tn, lane);
  zero<DH>(acc);
  float m = -INFINITY, l = 0.f;
  const float sc = rsqrtf((float)DH) * kLog2e;
  ByRow<T, DH> kf;  // (a block's rows are requested while the block before it is summed up, its columns ahead of its scores)
  if (wave <= last) kf.load(base + d, ld, 16 * wave, Tn, lane);
  for (int a = wave; a <= last; a += W) {
    ByCol<T, DH> vf;
    vf.load(base + 2 * d, ld, 16 * a, Tn, lane);
    f4 s = scores<T, DH>(kf, qf);
    if (a + W <= last) kf.load(base + d, ld, 16 * (a + W), Tn, lane);
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int kv = 16 * a + 4 * kk + r;
      s[r] = kv > q || kv >= Tn ? -INFINITY : s[r] * sc;
      mx = fmaxf(mx, s[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mn = fmaxf(m, mx), at = base_of(mn), alpha = __builtin_amdgcn_exp2f(m - at);
    m = mn;
    l *= alpha;
#pragma unroll
    for (int i = 0; i < DH / 16; ++i) acc[i] *= alpha;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      s[r] = __builtin_amdgcn_exp2f(s[r] - at);
      l += s[r];
    }
    add_cols<T, DH>(acc, vf, s);
  }
  if (!all_finite<DH>(acc)) {
    zero<DH>(acc);
    for (int a = wave; a <= last; a += W)
      for (int u = 16 * a; u < min(Tn, 16 * a + 16); ++u) {
        const T *row = base + u * ld;
        const float p = __builtin_amdgcn_exp2f(dot_row<T, DH>(qf, row + d, lane) * sc - base_of(m));
        if (u <= q) add_row_cols<T, DH>(acc, p, row + 2 * d, lane);
      }
  }
  l = sum_groups(l);
  meet.park(acc, wave, lane);
  if (kk == 0) {
    ms[wave][lane] = m;
    ls[wave][lane] = l;
  }
  __syncthreads();
  if (t < 256) {
    const int qi = t >> 4;
    float mm = -INFINITY, ll = 0.f, w[W], v[DH / 16];
#pragma unroll
    for (int i = 0; i < W; ++i) mm = fmaxf(mm, ms[i][qi]);
#pragma unroll
    for (int i = 0; i < W; ++i) {
      w[i] = __builtin_amdgcn_exp2f(ms[i][qi] - base_of(mm));
      ll = fmaf(ls[i][qi], w[i], ll);
    }
    const float inv = 1.f / ll;
#pragma unroll
    for (int i = 0; i < W; ++i) w[i] *= inv;
    meet.take(v, w, t);
    if (q0 + qi < Tn) {
      put_row(o + ((size_t)b * Tn + q0 + qi) * d + h * DH + (t & 15) * (DH / 16), v);
      if ((t & 15) == 0) lse[((size_t)b * H + h) * Tn + q0 + qi] = (mm + log2f(ll)) * kLn2;
    }
  }
}

// dQ and dsum; grid (ceil(T/16), B*H, streams)
template <typename T, int DH, int W>
__global__ __launch_bounds__(64 * W) void attn_dq_split_f32(const T *__restrict__ qkv, const T *__restrict__ o,
                                                            const T *__restrict__ d_o, const float *__restrict__ lse,
                                                            int Tn, int H, int B, T *__restrict__ dqkv,
                                                            float *__restrict__ dsum) {
  __shared__ __attribute__((aligned(16))) Meet<DH, W> meet;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), kk = lane >> 4;
  const int b = blockIdx.y / H, h = blockIdx.y % H, d = H * DH, sidx = blockIdx.z;
  const size_t ld = 3 * (size_t)d, N = (size_t)B * Tn;
  const T *base = qkv + (size_t)b * Tn * ld + h * DH;
  const int last = gridDim.x - 1 - blockIdx.x, q0 = 16 * last, q = q0 + (lane & 15);
  const size_t tok = (size_t)b * Tn + q;
  f4 qf[DH / 16], gf[DH / 16], dq[DH / 16];
  load_own<T, DH>(qf, base + (size_t)q * ld, q < Tn, lane);
  load_own<T, DH>(gf, d_o + (sidx * N + tok) * d + h * DH, q < Tn, lane);
  load_own<T, DH>(dq, o + tok * d + h * DH, q < Tn, lane);
  float D = 0.f;
#pragma unroll
  for (int s = 0; s < DH / 16; ++s)
#pragma unroll
    for (int e = 0; e < 4; ++e) D = fmaf(gf[s][e], dq[s][e], D);
  D = sum_groups(D);
  if (q < Tn && lane < 16 && wave == 0) dsum[(sidx * (size_t)B * H + blockIdx.y) * Tn + q] = D;
  zero<DH>(dq);
  const float sc = rsqrtf((float)DH), sc2 = sc * kLog2e;
  const float L2 = q < Tn ? lse[((size_t)b * H + h) * Tn + q] * kLog2e : 0.f;
  ByRow<T, DH> kf, vf;
  auto rows = [&](int a) {
    kf.load(base + d, ld, 16 * a, Tn, lane);
    vf.load(base + 2 * d, ld, 16 * a, Tn, lane);
  };
  if (wave <= last) rows(wave);
  for (int a = wave; a <= last; a += W) {
    ByCol<T, DH> kc;
    kc.load(base + d, ld, 16 * a, Tn, lane);
    f4 s = scores<T, DH>(kf, qf);
    const f4 dp = scores<T, DH>(vf, gf);
    if (a + W <= last) rows(a + W);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int kv = 16 * a + 4 * kk + r;
      const float ds = __builtin_amdgcn_exp2f(s[r] * sc2 - L2) * (dp[r] - D);
      s[r] = kv > q || kv >= Tn ? 0.f : ds;
    }
    add_cols<T, DH>(dq, kc, s);
  }
  if (!all_finite<DH>(dq)) {
    zero<DH>(dq);
    for (int a = wave; a <= last; a += W)
      for (int u = 16 * a; u < min(Tn, 16 * a + 16); ++u) {
        const T *row = base + u * ld;
        const float p = __builtin_amdgcn_exp2f(dot_row<T, DH>(qf, row + d, lane) * sc2 - L2);
        const float ds = p * (dot_row<T, DH>(gf, row + 2 * d, lane) - D);
        if (u <= q) add_row_cols<T, DH>(dq, ds, row + d, lane);
      }
  }
  meet.park(dq, wave, lane);
  __syncthreads();
  if (t < 256 && q0 + (t >> 4) < Tn) {
    float w[W], v[DH / 16];
#pragma unroll
    for (int i = 0; i < W; ++i) w[i] = sc;
    meet.take(v, w, t);
    put_row(dqkv + (sidx * N + (size_t)b * Tn + q0 + (t >> 4)) * ld + h * DH + (t & 15) * (DH / 16), v);
  }
}

// dK, dV; grid (ceil(T/16), B*H, streams); the first keys have the most queries
template <typename T, int DH, int W>
__global__ __launch_bounds__(64 * W) void attn_dkv_split_f32(const T *__restrict__ qkv, const T *__restrict__ d_o,
                                                             const float *__restrict__ lse, const float *__restrict__ dsum,
                                                             int Tn, int H, int B, T *__restrict__ dqkv) {
  __shared__ __attribute__((aligned(16))) Meet<DH, W> meet;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), kk = lane >> 4;
  const int b = blockIdx.y / H, h = blockIdx.y % H, d = H * DH, sidx = blockIdx.z;
  const size_t ld = 3 * (size_t)d, N = (size_t)B * Tn;
  const T *base = qkv + (size_t)b * Tn * ld + h * DH, *gbase = d_o + (sidx * N + (size_t)b * Tn) * d + h * DH;
  const float *lrow = lse + ((size_t)b * H + h) * Tn, *drow = dsum + (sidx * (size_t)B * H + blockIdx.y) * Tn;
  const int first = blockIdx.x, kv0 = 16 * first, kv = kv0 + (lane & 15), nb = (Tn + 15) / 16;  // query blocks first .. nb - 1
  f4 kf[DH / 16], vf[DH / 16], dk[DH / 16], dv[DH / 16];
  load_own<T, DH>(kf, base + (size_t)kv * ld + d, kv < Tn, lane);
  load_own<T, DH>(vf, base + (size_t)kv * ld + 2 * d, kv < Tn, lane);
  zero<DH>(dk);
  zero<DH>(dv);
  const float sc = rsqrtf((float)DH), sc2 = sc * kLog2e;
  ByRow<T, DH> qf, gf;
  auto rows = [&](int a) {
    qf.load(base, ld, 16 * a, Tn, lane);
    gf.load(gbase, (size_t)d, 16 * a, Tn, lane);
  };
  if (first + wave < nb) rows(first + wave);
  for (int a = first + wave; a < nb; a += W) {
    ByCol<T, DH> qc, gc;
    float l4[4], d4[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int q = 16 * a + 4 * kk + r;
      l4[r] = q < Tn ? lrow[q] * kLog2e : 0.f;
      d4[r] = q < Tn ? drow[q] : 0.f;
    }
    qc.load(base, ld, 16 * a, Tn, lane);
    gc.load(gbase, (size_t)d, 16 * a, Tn, lane);
    f4 s = scores<T, DH>(qf, kf), dp = scores<T, DH>(gf, vf);
    if (a + W < nb) rows(a + W);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int q = 16 * a + 4 * kk + r;
      const bool seen = kv <= q && q < Tn;
      const float p = seen ? __builtin_amdgcn_exp2f(s[r] * sc2 - l4[r]) : 0.f;
      dp[r] = seen ? p * (dp[r] - d4[r]) : 0.f;
      s[r] = p;
    }
    add_cols<T, DH>(dv, gc, s);
    add_cols<T, DH>(dk, qc, dp);
  }
  if (!all_finite<DH>(dv) || !all_finite<DH>(dk)) {
    zero<DH>(dv);
    zero<DH>(dk);
    for (int a = first + wave; a < nb; a += W)
      for (int u = 16 * a; u < min(Tn, 16 * a + 16); ++u) {
        const T *qr = base + u * ld, *gr = gbase + (size_t)u * d;
        const float p = __builtin_amdgcn_exp2f(dot_row<T, DH>(kf, qr, lane) * sc2 - lrow[u] * kLog2e);
        const float ds = p * (dot_row<T, DH>(vf, gr, lane) - drow[u]);
        if (u < kv) continue;
        add_row_cols<T, DH>(dv, p, gr, lane);
        add_row_cols<T, DH>(dk, ds, qr, lane);
      }
  }
  float w[W], v[DH / 16];
  T *out = dqkv + (sidx * N + (size_t)b * Tn + kv0 + (t >> 4)) * ld + d + h * DH + (t & 15) * (DH / 16);
  const bool mine = t < 256 && kv0 + (t >> 4) < Tn;
  meet.park(dk, wave, lane);
  __syncthreads();
  if (mine) {
#pragma unroll
    for (int i = 0; i < W; ++i) w[i] = sc;
    meet.take(v, w, t);
    put_row(out, v);
  }
  __syncthreads();
  meet.park(dv, wave, lane);
  __syncthreads();
  if (mine) {
#pragma unroll
    for (int i = 0; i < W; ++i) w[i] = 1.f;
    meet.take(v, w, t);
    put_row(out + d, v);
  }
}

// Which form.  The chain of the longest wavefront is what a launch waits for up to about half the CUs' number of workgroups of
// 64 rows; beyond, a tile that four wavefronts share costs less than each reading its own.  Forward / backward, us, of 64 rows
// and split: 1 x 896 tokens, a head of 128, two streams 93 / 270 and 27 / 100; 4 x 1024, two of 128 (128 workgroups) 110 / 310 and
// 60 / 229; 2 x 640, four of 64, two streams (160) 35 / 112 and 18 / 87; but 8 x 256, eight of 64 (256) 18 / 56 and 20 / 78, 8 x 512,
// sixteen of 64 (1024) 94 / 290 and 107 / 446.  A single tile of 64 rows has no chain to cut: 4 x 64, sixteen of 32, two streams
// (128) 12.1 and 12.7.  Up to 256 tokens the chain is short enough that the split form's workgroups also have to go into two
// rounds or so (shared / split, in us, of that many split workgroups): forward, 128 tokens, heads of 128 16.9 / 14.0 (512), 17.2 / 20.8 (576);
// 256 tokens, of 64 16.3 / 15.4 (576), of 128 30.2 / 29.8 (576), 30.1 / 33.1 (640); backward, 128 tokens, of 64 28.6 / 26.4 (512),
// 28.7 / 36.3 (576); 256 tokens, of 64 49.8 / 39.2 (512), 50.3 / 55.5 (576), of 128 88.7 / 74.7 (512), 89.5 / 106.4 (576).  Between 128 and 224
// tokens the shared tiles' last one is short or missing half, and the backward gains a little beyond.  Up to 96 tokens the backward of heads
// of 128 has to go into one round: 96 tokens 38.6 / 25.6 (252), 40.2 / 43.2 (444).
int split_parts(int dh, bool backward, long heads, int Tn) {  // heads: of all batches and streams; 0: tiles of 64 rows
  const long tiles = (Tn + 63) / 64 * heads, split = (Tn + 15) / 16 * heads;
  if (tiles > (Tn <= 64 ? 64 : 160)) return 0;
  const int most = Tn > 256               ? 640
                   : !backward            ? (Tn <= 128 ? 512 : dh == 128 ? 576 : 640)
                   : dh == 128 && Tn < 97 ? 256
                                          : (Tn > 128 && Tn <= 224 ? 560 : 512);
  if (split > most) return 0;
  // Eight wavefronts for long rows of narrow heads, whose blocks take less time than their loads: backward of 2 x 1000 tokens, four heads
  // of 16, 71 -> 62 us with four and 45 with eight; 1 x 576, seven of 32, forward 25 -> 10 -> 7.9.  (At 64 and 128 four are as fast or faster.)
  return dh <= 32 && Tn >= 512 ? 8 : 4;
}
template <int DH, typename F>
void with_waves(int parts, F &&f) {
  if constexpr (DH <= 32) {
    if (parts == 8) return f(std::integral_constant<int, 8>{});
  }
  f(std::integral_constant<int, 4>{});
}

template <typename T, int DH>
hipError_t fwd_t(const void *qkv, int B, int Tn, int H, void *o, float *lse, hipStream_t s) {
  const dim3 grid((Tn + kOwn - 1) / kOwn, B * H), split((Tn + 15) / 16, B * H);
  if (const int parts = split_parts(DH, false, (long)B * H, Tn))
    with_waves<DH>(parts, [&](auto w) {
      constexpr int W = decltype(w)::value;
      hipLaunchKernelGGL((attn_fwd_split_f32<T, DH, W>), split, dim3(64 * W), 0, s, (const T *)qkv, Tn, H, (T *)o, lse);
    });
  else
    hipLaunchKernelGGL((attn_fwd_f32<T, DH>), grid, dim3(256), 0, s, (const T *)qkv, Tn, H, (T *)o, lse);
  return hipGetLastError();
}
template <typename T, int DH>
hipError_t bwd_t(const void *qkv, const void *o, const void *d_o, const float *lse, int ns, int B, int Tn, int H,
                 void *dqkv, float *dsum, hipStream_t s) {
  const dim3 grid((Tn + kOwn - 1) / kOwn, B * H, ns), split((Tn + 15) / 16, B * H, ns);
  if (const int parts = split_parts(DH, true, (long)B * H * ns, Tn)) {
    with_waves<DH>(parts, [&](auto w) {
      constexpr int W = decltype(w)::value;
      hipLaunchKernelGGL((attn_dq_split_f32<T, DH, W>), split, dim3(64 * W), 0, s, (const T *)qkv, (const T *)o, (const T *)d_o,
                         lse, Tn, H, B, (T *)dqkv, dsum);
      hipLaunchKernelGGL((attn_dkv_split_f32<T, DH, W>), split, dim3(64 * W), 0, s, (const T *)qkv, (const T *)d_o, lse, dsum,
                         Tn, H, B, (T *)dqkv);
    });
    return hipGetLastError();
  }
  hipLaunchKernelGGL((attn_dq_f32<T, DH>), grid, dim3(256), 0, s, (const T *)qkv, (const T *)o, (const T *)d_o, lse, Tn,
                     H, B, (T *)dqkv, dsum);
  hipLaunchKernelGGL((attn_dkv_f32<T, DH>), grid, dim3(256), 0, s, (const T *)qkv, (const T *)d_o, lse, dsum, Tn, H, B,
                     (T *)dqkv);
  return hipGetLastError();
}

}  // namespace

hipError_t attention_forward_mfma(const void *qkv, int B, int T, int H, int dh, void *o, float *lse,
                                  hipStream_t s);
hipError_t attention_backward_mfma(const void *qkv, const void *d_o, const float *lse, const float *dsum, int ns,
                                   int B, int T, int H, int dh, void *dqkv, hipStream_t s);

int attention_form_mfma(int dh, int ns, int B, int T, int H);

int attention_form(int dtype, int dh, int ns, int B, int T, int H) {
  if (dtype == 1 && dh >= 64) return attention_form_mfma(dh, ns, B, T, H);
  return split_parts(dh, ns > 0, (long)B * H * (ns > 0 ? ns : 1), T);
}

// Front ends used by the step: bf16 with head widths 64 to 256 runs on the bf16 matrix instructions, fp32
// and bf16 with head widths 16 and 32 on the kernels above.
hipError_t attention_forward(int dtype, const void *qkv, int B, int T, int H, int dh, void *o, float *lse,
                             hipStream_t s) {
  if (dtype == 1) {
    if (dh == 16) return fwd_t<bf16_t, 16>(qkv, B, T, H, o, lse, s);
    if (dh == 32) return fwd_t<bf16_t, 32>(qkv, B, T, H, o, lse, s);
    return attention_forward_mfma(qkv, B, T, H, dh, o, lse, s);
  }
  switch (dh) {
    case 16: return fwd_t<float, 16>(qkv, B, T, H, o, lse, s);
    case 32: return fwd_t<float, 32>(qkv, B, T, H, o, lse, s);
    case 64: return fwd_t<float, 64>(qkv, B, T, H, o, lse, s);
    case 128: return fwd_t<float, 128>(qkv, B, T, H, o, lse, s);
    default: return hipErrorInvalidValue;
  }
}
hipError_t attention_backward(int dtype, const void *qkv, const void *o, const void *d_o, const float *lse,
                              int ns, int B, int T, int H, int dh, void *dqkv, float *dsum, hipStream_t s) {
  if (dtype == 1) {
    if (dh == 16) return bwd_t<bf16_t, 16>(qkv, o, d_o, lse, ns, B, T, H, dqkv, dsum, s);
    if (dh == 32) return bwd_t<bf16_t, 32>(qkv, o, d_o, lse, ns, B, T, H, dqkv, dsum, s);
    return attention_backward_mfma(qkv, d_o, lse, dsum, ns, B, T, H, dh, dqkv, s);
  }
  switch (dh) {
    case 16: return bwd_t<float, 16>(qkv, o, d_o, lse, ns, B, T, H, dqkv, dsum, s);
    case 32: return bwd_t<float, 32>(qkv, o, d_o, lse, ns, B, T, H, dqkv, dsum, s);
    case 64: return bwd_t<float, 64>(qkv, o, d_o, lse, ns, B, T, H, dqkv, dsum, s);
    case 128: return bwd_t<float, 128>(qkv, o, d_o, lse, ns, B, T, H, dqkv, dsum, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace il
