// LayerNorm forward and backward for the pre-LN block.  One 64-lane wavefront owns a
// row; row reductions are wavefront shuffles (no LDS), statistics are fp32.  The
// backward is fused with the residual-gradient add (the gradient stream G is updated in
// place) and with the first stage of the gamma/beta column reductions.
#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "common.h"

namespace il {
namespace {

constexpr int kWaves = 4;         // rows in flight per 256-thread block
constexpr int kLnBwdBlocks = 512;

__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

template <typename T> __device__ inline float round_to(float v);
template <> __device__ inline float round_to<float>(float v) { return v; }
template <> __device__ inline float round_to<bf16_t>(float v) { return bf16_to_f32(f32_to_bf16(v)); }

// Vector access helpers: V consecutive elements per lane (V = 4 when d and every address divide by 4, else 1).
template <typename T, int V> struct Vec;
template <> struct Vec<float, 4> {
  static __device__ inline void load(const float *p, float (&o)[4]) {
    const float4 v = *reinterpret_cast<const float4 *>(p);
    o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
  }
  static __device__ inline void store(float *p, const float (&o)[4]) {
    *reinterpret_cast<float4 *>(p) = make_float4(o[0], o[1], o[2], o[3]);
  }
};
template <> struct Vec<bf16_t, 4> {
  static __device__ inline void load(const bf16_t *p, float (&o)[4]) {
    const uint2 v = *reinterpret_cast<const uint2 *>(p);
    o[0] = bf16_to_f32((bf16_t)(v.x & 0xFFFF)); o[1] = bf16_to_f32((bf16_t)(v.x >> 16));
    o[2] = bf16_to_f32((bf16_t)(v.y & 0xFFFF)); o[3] = bf16_to_f32((bf16_t)(v.y >> 16));
  }
  static __device__ inline void store(bf16_t *p, const float (&o)[4]) {
    uint2 v;
    v.x = pack_bf16x2(o[0], o[1]);
    v.y = pack_bf16x2(o[2], o[3]);
    *reinterpret_cast<uint2 *>(p) = v;
  }
};
template <typename T> struct Vec<T, 1> {
  static __device__ inline void load(const T *p, float (&o)[1]) { o[0] = ld<T>(p); }
  static __device__ inline void store(T *p, const float (&o)[1]) { st<T>(p, o[0]); }
};

// Forward: a lane owns columns (lane + 64 j) * V + (0..V-1), j < J, d <= 64 V J.  Gain and bias are requested with the row
// where the registers they take leave enough wavefronts: after the reductions their latency stands alone.  bf16, us with
// the row / after it: 4096 x 256 3.14 / 3.23, 512 x 1024 3.52 / 3.62, but 8192 x 1280 14.0 / 12.7, 4096 x 2048 12.1 / 10.5;
// fp32, whose gain needs no conversion: 512 x 2048 4.2 / 4.6, 8192 x 2048 21.3 / 22.1, 4096 x 2048 12.9 / 12.4 (alone slower).
template <typename T, int V, int J>
__global__ __launch_bounds__(256) void ln_fwd_kernel(const float *__restrict__ x, const T *__restrict__ gamma,
                                                     const T *__restrict__ beta, float eps, int rows, int d,
                                                     T *__restrict__ y, float *__restrict__ stats,
                                                     float *__restrict__ xcopy) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = blockIdx.x * kWaves + wave;
  if (row >= rows) return;
  const float *xr = x + (size_t)row * d;
  constexpr bool AHEAD = sizeof(T) == 4 || J <= 4;
  float v[J][V], g[J][V], b[J][V];
  auto gain = [&](int j, int c) {
    Vec<T, V>::load(gamma + c, g[j]);
    Vec<T, V>::load(beta + c, b[j]);
  };
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int c = (lane + 64 * j) * V;
    if (c < d) {
      Vec<float, V>::load(xr + c, v[j]);
    } else {
#pragma unroll
      for (int e = 0; e < V; ++e) v[j][e] = 0.f;
    }
  }
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int c = (lane + 64 * j) * V;
    if (AHEAD && c < d) gain(j, c);
  }
#pragma unroll
  for (int j = 0; j < J; ++j)
#pragma unroll
    for (int e = 0; e < V; ++e) s += v[j][e];
  // x - sum / d in one rounding, and the same value for the variance and the result: a mean rounded first costs
  // the result another 2^-24 of the mean wherever 1 / d is not a power of two
  const float invd = 1.f / d, total = wave_sum(s);
  auto centred = [&](float x) { return __builtin_fmaf(-invd, total, x); };
  float q = 0.f, first = 0.f;
#pragma unroll
  for (int j = 0; j < J; ++j)
#pragma unroll
    for (int e = 0; e < V; ++e) {
      const float t = (lane + 64 * j) * V < d ? centred(v[j][e]) : 0.f;
      if (V > 1 && j * V + e == 0) first = t;
      else q = __builtin_fmaf(t, t, q);
      if (V > 1 && j * V + e == 1) q = __builtin_fmaf(first, first, q);
    }
  const float rstd = rsqrtf(__builtin_fmaf(wave_sum(q), invd, eps));
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int c = (lane + 64 * j) * V;
    if (c >= d) continue;
    if (!AHEAD) gain(j, c);
    float o[V];
#pragma unroll
    for (int e = 0; e < V; ++e) o[e] = __builtin_fmaf(centred(v[j][e]) * rstd, g[j][e], b[j][e]);
    Vec<T, V>::store(y + (size_t)row * d + c, o);
    if (xcopy) Vec<float, V>::store(xcopy + (size_t)row * d + c, v[j]);
  }
  if (lane == 0) {
    stats[2 * row] = total * invd;
    stats[2 * row + 1] = rstd;
  }
}

// p[at], with the element's place as one 32-bit byte offset beside a uniform address (a stream is below 4 GiB)
template <typename T>
__device__ inline T *lane_at(T *p, uint32_t at) {
  return reinterpret_cast<T *>(reinterpret_cast<char *>(const_cast<std::remove_const_t<T> *>(p)) + (uint32_t)(at * sizeof(T)));
}

// Backward, d divisible by 4: GW wavefronts share a row (a lane owns columns 4 l + 0..3 for its lane
// number l in the group, d <= 256 GW), a workgroup walks over rows with NG groups.  Bound by its bytes
// (16 per element and stream; 27 us for 8192 x 1024).  One wavefront per row needed 130 registers at
// d = 1024 and 235 at 2048; this form takes 64 to 74.
template <typename T, int GW>
__global__ __launch_bounds__(GW > 4 ? 512 : 256) void ln_bwd_rows_kernel(const T *__restrict__ dy, const float *__restrict__ x,
                                                           const float *__restrict__ stats,
                                                           const T *__restrict__ gamma, int rows, int N, int d, float *G,
                                                           T *Gb, StreamWeights sw, float *__restrict__ partials) {
  constexpr int NG = GW > 4 ? 1 : 4 / GW, GL = 64 * GW;
  __shared__ float red[2][NG][GW][2];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, grp = wave / GW, wg = wave % GW, l = wg * 64 + lane;
  float dg[4], db[4], gm[4];
  const int c = l * 4;
#pragma unroll
  for (int e = 0; e < 4; ++e) { dg[e] = 0.f; db[e] = 0.f; gm[e] = 0.f; }
  if (c < d) Vec<T, 4>::load(gamma + c, gm);
  const float invd = 1.f / d;
  const int step = gridDim.x * NG;
  const int trips = (rows + step - 1) / step;  // the same for every wavefront: the barrier below is theirs together
  for (int it = 0; it < trips; ++it) {
    const int row = it * step + blockIdx.x * NG + grp;
    const bool live = row < rows;
    const int tok = live ? row % N : 0;
    const float w = live ? sw.w[row / N] : 0.f;
    const float mean = stats[2 * tok], rstd = stats[2 * tok + 1];
    const float *xr = x + (size_t)tok * d;
    const T *dyr = dy + (size_t)row * d;
    float *gr = G + (size_t)row * d;
    T *gbr = Gb + (size_t)row * d;
    float xh[4], dv[4], gv[4];
    float s1 = 0.f, s2 = 0.f;
    const bool in = live && c < d;
    if (in) {
      Vec<T, 4>::load(dyr + c, dv);
      Vec<float, 4>::load(xr + c, xh);
      Vec<float, 4>::load(gr + c, gv);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      dv[e] = in ? dv[e] : 0.f;
      xh[e] = in ? (xh[e] - mean) * rstd : 0.f;
      const float t = dv[e] * gm[e];
      s1 += t;
      s2 += t * xh[e];
      dg[e] += w * dv[e] * xh[e];
      db[e] += w * dv[e];
    }
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
    if constexpr (GW > 1) {
      float *r = red[it & 1][grp][wg];
      if (lane == 0) { r[0] = s1; r[1] = s2; }
      __syncthreads();  // (the other half of `red` is written next, so one barrier a row is enough)
      s1 = s2 = 0.f;
#pragma unroll
      for (int k = 0; k < GW; ++k) { s1 += red[it & 1][grp][k][0]; s2 += red[it & 1][grp][k][1]; }
    }
    const float m1 = s1 * invd, m2 = s2 * invd;
    if (in) {
#pragma unroll
      for (int e = 0; e < 4; ++e) gv[e] += rstd * (dv[e] * gm[e] - m1 - xh[e] * m2);
      Vec<float, 4>::store(gr + c, gv);
      Vec<T, 4>::store(gbr + c, gv);
    }
  }
  // column sums of the workgroup: its groups combine through LDS, fixed order
  float *pg = partials + (size_t)blockIdx.x * 2 * d;
  if constexpr (NG == 1) {
    if (c < d) {
      Vec<float, 4>::store(pg + c, dg);
      Vec<float, 4>::store(pg + d + c, db);
    }
  } else {
    __shared__ float4 cols[NG][2][GL];
    cols[grp][0][l] = make_float4(dg[0], dg[1], dg[2], dg[3]);
    cols[grp][1][l] = make_float4(db[0], db[1], db[2], db[3]);
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * GL; i += 256) {
      const int which = i / GL, col = (i % GL) * 4;
      if (col >= d) continue;
      float4 a = cols[0][which][i % GL];
#pragma unroll
      for (int k = 1; k < NG; ++k) {
        const float4 b = cols[k][which][i % GL];
        a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
      }
      *reinterpret_cast<float4 *>(pg + which * d + col) = a;
    }
  }
}

// The same, a workgroup walking over tokens, a token's streams NS at a time: x and the statistics are read once for all of
// them, and their weighted sum - what the weight gradient of the linear map in front of this LayerNorm multiplies
// with - and its column sums are left beside them instead of in a pass of their own, which reads every stream again.
// 72 to 98 registers.  Two streams at a time against one, us: 4096 x 1024, two streams 24.1 / 24.8, 1024 x 768 7.4 / 8.0; at
// GW = 8 it takes 110 registers and 2048 x 2048, three streams 32.2 / 30.1: one at a time there.
template <typename T, int GW, int NS>
__global__ __launch_bounds__(GW > 4 ? 512 : 256) void ln_bwd_sum_kernel(const T *__restrict__ dy, const float *__restrict__ x,
                                                           const float *__restrict__ stats,
                                                           const T *__restrict__ gamma, int ns, int N, int d, float *G,
                                                           T *Gb, StreamWeights sw, float *__restrict__ partials, T *ysum,
                                                           float *__restrict__ ypart) {
  constexpr int NG = GW > 4 ? 1 : 4 / GW, GL = 64 * GW;
  __shared__ float red[2][NG][GW][2 * NS];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, grp = wave / GW, wg = wave % GW, l = wg * 64 + lane;
  float dg[4], db[4], dy1[4], gm[4];
  const int c = l * 4;
#pragma unroll
  for (int e = 0; e < 4; ++e) { dg[e] = 0.f; db[e] = 0.f; dy1[e] = 0.f; gm[e] = 0.f; }
  if (c < d) Vec<T, 4>::load(gamma + c, gm);
  const float invd = 1.f / d;
  const size_t nd = (size_t)N * d;
  const int step = gridDim.x * NG;
  const int trips = (N + step - 1) / step;  // the same for every wavefront: the barrier below is theirs together
  int turn = 0;
  for (int it = 0; it < trips; ++it) {
    const int tok = it * step + blockIdx.x * NG + grp;
    const bool in = tok < N && c < d;
    const int t0 = tok < N ? tok : 0;
    const float mean = stats[2 * t0], rstd = stats[2 * t0 + 1];
    float xh[4] = {0.f, 0.f, 0.f, 0.f}, y[4] = {0.f, 0.f, 0.f, 0.f};
    const uint32_t at = (uint32_t)tok * d + c;
    if (in) Vec<float, 4>::load(lane_at(x, at), xh);
    for (int s0 = 0; s0 < ns; s0 += NS, turn ^= 1) {
      float dv[NS][4], gv[NS][4], sum[2 * NS];
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        const bool live = in && (NS == 1 || s0 + k < ns);
        if (live) {
          Vec<T, 4>::load(lane_at(dy + (s0 + k) * nd, at), dv[k]);
          Vec<float, 4>::load(lane_at(G + (s0 + k) * nd, at), gv[k]);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) dv[k][e] = live ? dv[k][e] : 0.f;
      }
      if (s0 == 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) xh[e] = in ? (xh[e] - mean) * rstd : 0.f;
      }
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        const float w = NS == 1 || s0 + k < ns ? sw.w[s0 + k] : 0.f;
        float s1 = 0.f, s2 = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float t = dv[k][e] * gm[e];
          s1 += t;
          s2 += t * xh[e];
          dg[e] += w * dv[k][e] * xh[e];
          db[e] += w * dv[k][e];
        }
        sum[2 * k] = wave_sum(s1);
        sum[2 * k + 1] = wave_sum(s2);
      }
      if constexpr (GW > 1) {
        float *r = red[turn][grp][wg];
        if (lane == 0) {
#pragma unroll
          for (int k = 0; k < 2 * NS; ++k) r[k] = sum[k];
        }
        __syncthreads();  // (the other half of `red` is written next, so one barrier a turn is enough)
#pragma unroll
        for (int k = 0; k < 2 * NS; ++k) {
          sum[k] = 0.f;
#pragma unroll
          for (int q = 0; q < GW; ++q) sum[k] += red[turn][grp][q][k];
        }
      }
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        if (!in || (NS > 1 && s0 + k >= ns)) continue;
        const float m1 = sum[2 * k] * invd, m2 = sum[2 * k + 1] * invd, w = sw.w[s0 + k];
#pragma unroll
        for (int e = 0; e < 4; ++e) gv[k][e] += rstd * (dv[k][e] * gm[e] - m1 - xh[e] * m2);
        Vec<float, 4>::store(lane_at(G + (s0 + k) * nd, at), gv[k]);
        Vec<T, 4>::store(lane_at(Gb + (s0 + k) * nd, at), gv[k]);
        if (w != 0.f) {  // (uniform) the sum is taken of the stored values
#pragma unroll
          for (int e = 0; e < 4; ++e) y[e] += w * round_to<T>(gv[k][e]);
        }
      }
    }
    if (in) {
      if (ysum) Vec<T, 4>::store(lane_at(ysum, at), y);
#pragma unroll
      for (int e = 0; e < 4; ++e) dy1[e] += y[e];
    }
  }
  // column sums of the workgroup: its groups combine through LDS, fixed order
  float *pg = partials + (size_t)blockIdx.x * 2 * d, *py = ypart + (size_t)blockIdx.x * d;
  if constexpr (NG == 1) {
    if (c < d) {
      Vec<float, 4>::store(pg + c, dg);
      Vec<float, 4>::store(pg + d + c, db);
      Vec<float, 4>::store(py + c, dy1);
    }
  } else {
    __shared__ float4 cols[NG][3][GL];
    cols[grp][0][l] = make_float4(dg[0], dg[1], dg[2], dg[3]);
    cols[grp][1][l] = make_float4(db[0], db[1], db[2], db[3]);
    cols[grp][2][l] = make_float4(dy1[0], dy1[1], dy1[2], dy1[3]);
    __syncthreads();
    for (int i = threadIdx.x; i < 3 * GL; i += 256) {
      const int which = i / GL, col = (i % GL) * 4;
      if (col >= d) continue;
      float4 a = cols[0][which][i % GL];
#pragma unroll
      for (int k = 1; k < NG; ++k) {
        const float4 b = cols[k][which][i % GL];
        a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
      }
      *reinterpret_cast<float4 *>(which == 2 ? py + col : pg + which * d + col) = a;
    }
  }
}

// ... element by element, a wavefront per row: lane owns columns lane + 64 j, j < J.
template <typename T, int V, int J>
__global__ __launch_bounds__(256) void ln_bwd_kernel(const T *__restrict__ dy, const float *__restrict__ x,
                                                     const float *__restrict__ stats,
                                                     const T *__restrict__ gamma, int rows, int N, int d,
                                                     float *G, T *Gb, StreamWeights sw,
                                                     float *__restrict__ partials) {
  __shared__ float red[kWaves][64 * V];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float dg[J][V], db[J][V], gm[J][V];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int c = (lane + 64 * j) * V;
#pragma unroll
    for (int e = 0; e < V; ++e) { dg[j][e] = 0.f; db[j][e] = 0.f; gm[j][e] = 0.f; }
    if (c < d) Vec<T, V>::load(gamma + c, gm[j]);
  }
  const float invd = 1.f / d;
  for (int row = blockIdx.x * kWaves + wave; row < rows; row += gridDim.x * kWaves) {
    const int tok = row % N;
    const float w = sw.w[row / N];
    const float mean = stats[2 * tok], rstd = stats[2 * tok + 1];
    const float *xr = x + (size_t)tok * d;
    const T *dyr = dy + (size_t)row * d;
    float *gr = G + (size_t)row * d;
    T *gbr = Gb + (size_t)row * d;
    float xh[J][V], dxh[J][V], gv[J][V];
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int c = (lane + 64 * j) * V;
      if (c < d) {
        float dyv[V];
        Vec<T, V>::load(dyr + c, dyv);
        Vec<float, V>::load(xr + c, xh[j]);
        Vec<float, V>::load(gr + c, gv[j]);
#pragma unroll
        for (int e = 0; e < V; ++e) {
          xh[j][e] = (xh[j][e] - mean) * rstd;
          dxh[j][e] = dyv[e] * gm[j][e];
          s1 += dxh[j][e];
          s2 += dxh[j][e] * xh[j][e];
          dg[j][e] += w * dyv[e] * xh[j][e];
          db[j][e] += w * dyv[e];
        }
      } else {
#pragma unroll
        for (int e = 0; e < V; ++e) { xh[j][e] = 0.f; dxh[j][e] = 0.f; gv[j][e] = 0.f; }
      }
    }
    const float m1 = wave_sum(s1) * invd, m2 = wave_sum(s2) * invd;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int c = (lane + 64 * j) * V;
      if (c < d) {
#pragma unroll
        for (int e = 0; e < V; ++e) gv[j][e] += rstd * (dxh[j][e] - m1 - xh[j][e] * m2);
        Vec<float, V>::store(gr + c, gv[j]);
        Vec<T, V>::store(gbr + c, gv[j]);
      }
    }
  }
  // block-level column sums: the four wavefronts combine through LDS, fixed order
  float *pg = partials + (size_t)blockIdx.x * 2 * d;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    if (64 * j * V >= d) continue;  // uniform across the block
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      __syncthreads();
#pragma unroll
      for (int e = 0; e < V; ++e) red[wave][lane * V + e] = pass ? db[j][e] : dg[j][e];
      __syncthreads();
      if (wave == 0) {
        const int c = (lane + 64 * j) * V;
#pragma unroll
        for (int e = 0; e < V; ++e) {
          const int i = lane * V + e;
          if (c + e < d) pg[pass * d + c + e] = (red[0][i] + red[1][i]) + (red[2][i] + red[3][i]);
        }
      }
    }
  }
}

// The number of column passes J a width needs: registers per lane, and so wavefronts per SIMD, follow it.
// Widths that divide by 4 take four columns per lane where every vector starts on 16 (bf16: 8) bytes, which an
// odd d_mlp can prevent in fp32, and the caller's x in both types.
template <typename F>
void with_width(int d, bool vec, F &&f) {
#define IL_W(V, J) return f(std::integral_constant<int, V>{}, std::integral_constant<int, J>{})
  if (vec) {
    switch ((d + 255) / 256) {
      case 1: IL_W(4, 1);
      case 2: IL_W(4, 2);
      case 3: IL_W(4, 3);
      case 4: IL_W(4, 4);
      case 5:
      case 6: IL_W(4, 6);
      default: IL_W(4, 8);
    }
  }
  if (d <= 256) IL_W(1, 4);
  IL_W(1, 32);
#undef IL_W
}

// (x of the first block is the caller's, who is asked for no alignment; nullptr is aligned)
template <typename T>
bool vec4(int d, const T *gamma, const T *beta, const float *x, const float *xcopy) {
  return (d & 3) == 0 && (((uintptr_t)gamma | (uintptr_t)beta) & (4 * sizeof(T) - 1)) == 0 &&
         (((uintptr_t)x | (uintptr_t)xcopy) & 15) == 0;
}

template <typename T>
void launch_fwd(hipStream_t s, const float *x, const T *gamma, const T *beta, float eps, int rows, int d, T *y,
                float *stats, float *xcopy) {
  with_width(d, vec4<T>(d, gamma, beta, x, xcopy), [&](auto v, auto j) {
    hipLaunchKernelGGL((ln_fwd_kernel<T, decltype(v)::value, decltype(j)::value>), dim3((rows + kWaves - 1) / kWaves),
                       dim3(256), 0, s, x, gamma, beta, eps, rows, d, y, stats, xcopy);
  });
}
template <typename T>
void launch_bwd(hipStream_t s, const T *dy, const float *x, const float *stats, const T *gamma, int ns, int N, int d,
                float *G, T *Gb, const StreamWeights &sw, float *partials, int *nblk, T *ysum, float *ypart, bool *summed) {
  *summed = false;
  const int rows = ns * N;
  auto by_rows = [&](auto kernel, int threads, int at_once) {
    *nblk = std::min((rows + at_once - 1) / at_once, kLnBwdBlocks);
    hipLaunchKernelGGL(kernel, dim3(*nblk), dim3(threads), 0, s, dy, x, stats, gamma, rows, N, d, G, Gb, sw, partials);
  };
  if (!vec4<T>(d, gamma, gamma, x, G)) {
    if (d <= 256) by_rows(ln_bwd_kernel<T, 1, 4>, 256, kWaves);
    else by_rows(ln_bwd_kernel<T, 1, 32>, 256, kWaves);
    return;
  }
  *summed = ypart != nullptr && d > 256;
  auto launch = [&](auto gw) {
    constexpr int GW = decltype(gw)::value, NG = GW > 4 ? 1 : 4 / GW, threads = GW > 4 ? 512 : 256;
    if (!*summed) return by_rows(ln_bwd_rows_kernel<T, GW>, threads, NG);
    if constexpr (GW > 1) {
      *nblk = std::min((N + NG - 1) / NG, kLnBwdBlocks);
      auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(*nblk), dim3(threads), 0, s, dy, x, stats, gamma, ns, N, d, G, Gb, sw,
                           partials, ysum, ypart);
      };
      if (ns == 1 || GW == 8) go(ln_bwd_sum_kernel<T, GW, 1>);
      else go(ln_bwd_sum_kernel<T, GW, GW == 8 ? 1 : 2>);
    }
  };
  if (d <= 256) launch(std::integral_constant<int, 1>{});
  else if (d <= 512) launch(std::integral_constant<int, 2>{});
  else if (d <= 1024) launch(std::integral_constant<int, 4>{});
  else launch(std::integral_constant<int, 8>{});
}

}  // namespace

int ln_backward_max_blocks() { return kLnBwdBlocks; }

// Forming the sums makes the launch 0.2 to 1.5 us longer, and in a backward it stands in the chain of data gradients that
// the step waits for, where the pass it replaces runs beside them.  It pays where the chain's products fill the
// chip, so that the pass takes time from them.  Steps in us, without / with the sums (bf16, tokens x d, n):
//   4096 x 1024 2 16858 / 16707, 3 (8 components) 23763 / 23383;  2752 x 576 3 11022 / 10903;  3776 x 768 1 16055 / 15986;
//   4096 x 2048 2 73610 / 73170;  2752 x 1984 2 33041 / 32875;  4096 x 512 1 3438 / 3423;  2048 x 1024 2, 2304 x 768 2 equal;
//   2048 x 512 1 1720 / 1732;  4096 x 256 1 2346 / 2364;  1600 x 768 3 4828 / 4844;  960 x 1920 2 25278 / 25385;
//   576 x 256 2 3024 / 3097;  1024 x 2048 2 7486 / 7504;  704 x 448 2 5806 / 5843.
bool ln_backward_sums(int N, int d) {
  return d > 256 && (d & 3) == 0 && N >= 1536 && (long)N * d >= 3l << 19;
}

hipError_t ln_forward(int dtype, const float *x, const void *gamma, const void *beta, float eps, int rows,
                      int d, void *y, float *stats, float *xcopy, hipStream_t s) {
  if (dtype == 0)
    launch_fwd<float>(s, x, (const float *)gamma, (const float *)beta, eps, rows, d, (float *)y, stats, xcopy);
  else
    launch_fwd<bf16_t>(s, x, (const bf16_t *)gamma, (const bf16_t *)beta, eps, rows, d, (bf16_t *)y, stats, xcopy);
  return hipGetLastError();
}

hipError_t ln_backward_residual(int dtype, const void *dy, const float *x, const float *stats, const void *gamma,
                                int ns, int N, int d, float *G, void *Gb, const StreamWeights &sw, float *partials,
                                int *nblk, void *ysum, float *ypart, bool *summed, hipStream_t s) {
  if (dtype == 0)
    launch_bwd<float>(s, (const float *)dy, x, stats, (const float *)gamma, ns, N, d, G, (float *)Gb, sw, partials, nblk,
                      (float *)ysum, ypart, summed);
  else
    launch_bwd<bf16_t>(s, (const bf16_t *)dy, x, stats, (const bf16_t *)gamma, ns, N, d, G, (bf16_t *)Gb, sw, partials,
                       nblk, (bf16_t *)ysum, ypart, summed);
  return hipGetLastError();
}

}  // namespace il
