// bf16 GEMM on the gfx950 matrix cores (v_mfma_f32_32x32x16_bf16), fp32 accumulate,
// with the library's fused epilogues.
//
// Tiling.  A workgroup of WGM x WGN wavefronts owns a BM x BN tile of C and walks K in steps
// of 64.  Each wavefront owns (BM/WGM) x (BN/WGN) = MI x NI MFMA tiles of 32x32, all held in
// accumulator registers.
//
// Operand layouts.  An operand is either "k-contiguous" ([rows, K] row-major: activations
// in forward / dgrad, weights in dgrad) or "k-major" ([K, rows] row-major: weights in
// forward, both operands of a weight gradient).
//
// Staging.  Operand tiles go HBM -> LDS directly (buffer loads with LDS destination): no
// staging registers, no ds_write instructions, and the buffer descriptor's range check
// zero-fills rows or k beyond the operand's edge without a branch.  NSTAGE LDS buffers rotate;
// one barrier per K step.  K-contiguous tiles are read with ds_read_b128, k-major tiles with
// the LDS transposing read (ds_read_b64_tr_b16), which delivers the MFMA operand order
// straight from the [k][row] image.
//
// The grid is one-dimensional; tile ids are regrouped so that the workgroups that land on
// one XCD (id mod 8) work on neighbouring tiles and share their operands in that XCD's L2.
#include <algorithm>
#include <cstring>

#include <hip/hip_ext.h>

#include "common.h"
#include "gemm_tile.h"
#include "lds_dma.h"
#include <type_traits>
#include <utility>

namespace il {
namespace {

constexpr long kPairTiles = 160;  // 256x256 tiles from which that tile is taken
constexpr int EPI_WGRAD_ACC = 9;  // EPI_WGRAD where every problem of the launch accumulates

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u32x4;

__device__ inline void unpack8(const u32x4 v, float (&f)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[2 * i] = bf16_to_f32((bf16_t)(v[i] & 0xFFFFu));
    f[2 * i + 1] = bf16_to_f32((bf16_t)(v[i] >> 16));
  }
}
__device__ inline u32x4 pack8(const float (&f)[8]) {
  u32x4 v;
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = pack_bf16x2(f[2 * i], f[2 * i + 1]);
  return v;
}

// A value from another lane of the same 16-lane row through the data-parallel path of the vector ALU (no
// LDS traffic): CTRL 0xB1 = lane ^ 1, 0x4E = lane ^ 2 (quad permutes), 0x141 = lane 7 - i of each half row.
template <int CTRL>
__device__ inline float dpp_f32(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}

// The largest of three in one instruction.  (fmaxf on values fresh from memory spends another on each to quiet
// signalling NaNs, which no product leaves.)
__device__ inline float max3(float a, float b, float c) {
  float r = a;
#if defined(__HIP_DEVICE_COMPILE__)
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
#endif
  return r;
}

// What the epilogue reads at a row's eight consecutive output columns, besides bias: the pre-activation or
// attention output (bf16), the residual or the accumulated-into output (fp32).
struct Extra { u32x4 q[2]; };
template <int EPI> constexpr bool kExtraBf16 = EPI == EPI_GELU_BWD || EPI == EPI_GELU_BWD_SUM || EPI == EPI_STORE_DOT;
template <int EPI> constexpr bool kBias = EPI == EPI_BIAS || EPI == EPI_BIAS_GELU || EPI == EPI_BIAS_RES;
template <int EPI> constexpr bool kExtraF32 = EPI == EPI_BIAS_RES || EPI == EPI_WGRAD_ACC;
template <int EPI>
__device__ inline Extra load_extra(const GemmArgs &g, int grow, int gcol) {
  Extra x = {};
  if (grow < g.M && gcol < g.N) {
    if constexpr (kExtraBf16<EPI>) {
      x.q[0] = *reinterpret_cast<const u32x4 *>((const bf16_t *)g.aux + (size_t)(grow % g.aux_wrap) * g.ldc + gcol);
    } else if constexpr (kExtraF32<EPI>) {
      const float *p = (EPI == EPI_BIAS_RES ? g.res : (const float *)g.C) + (size_t)grow * g.ldc + gcol;
      x.q[0] = *reinterpret_cast<const u32x4 *>(p);
      x.q[1] = *reinterpret_cast<const u32x4 *>(p + 4);
    }
  }
  return x;
}

// One row's eight consecutive output columns: the epilogue operation and the store.
template <int EPI>
__device__ inline void emit8(const GemmArgs &g, float4 v0, float4 v1, int grow, int gcol, const float (&bv)[8],
                             const Extra &x) {
  if (grow >= g.M || gcol >= g.N) return;
  float v[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
  const size_t o = (size_t)grow * g.ldc + gcol;
  if constexpr (EPI == EPI_STORE) {
    *reinterpret_cast<u32x4 *>((bf16_t *)g.C + o) = pack8(v);
  } else if constexpr (EPI == EPI_STORE_DOT) {
    const u32x4 u = pack8(v);
    *reinterpret_cast<u32x4 *>((bf16_t *)g.C + o) = u;
    float w[8];
    unpack8(u, v);  // (of the stored, rounded values)
    unpack8(x.q[0], w);
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) s = __builtin_fmaf(v[e], w[e], s);
    s += dpp_f32<0xB1>(s);  // lane ^ 1
    s += dpp_f32<0x4E>(s);  // lane ^ 2: the four lanes of a row's 32 columns (N divides by 32: all inside or none)
    if ((gcol & 31) == 0) g.row_stats[(size_t)(gcol >> 5) * g.M + grow] = s;
  } else if constexpr (EPI == EPI_LOGITS) {
    u32x4 h;
#pragma unroll
    for (int i = 0; i < 4; ++i) h[i] = pack_f16x2(v[2 * i], v[2 * i + 1]);
    *reinterpret_cast<u32x4 *>((uint16_t *)g.C + o) = h;
  } else if constexpr (EPI == EPI_BIAS) {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] += bv[e];
    *reinterpret_cast<u32x4 *>((bf16_t *)g.C + o) = pack8(v);
  } else if constexpr (EPI == EPI_BIAS_GELU) {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] += bv[e];
    const u32x4 u = pack8(v);
    *reinterpret_cast<u32x4 *>((bf16_t *)g.C + o) = u;
    unpack8(u, v);  // the activation is taken of the stored (rounded) pre-activation
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = gelu_f(v[e]);
    *reinterpret_cast<u32x4 *>((bf16_t *)g.C2 + o) = pack8(v);
  } else if constexpr (EPI == EPI_BIAS_RES) {
    const float4 r0 = __builtin_bit_cast(float4, x.q[0]), r1 = __builtin_bit_cast(float4, x.q[1]);
    float4 o0 = {v[0] + bv[0] + r0.x, v[1] + bv[1] + r0.y, v[2] + bv[2] + r0.z, v[3] + bv[3] + r0.w};
    float4 o1 = {v[4] + bv[4] + r1.x, v[5] + bv[5] + r1.y, v[6] + bv[6] + r1.z, v[7] + bv[7] + r1.w};
    *reinterpret_cast<float4 *>((float *)g.C + o) = o0;
    *reinterpret_cast<float4 *>((float *)g.C + o + 4) = o1;
  } else if constexpr (EPI == EPI_GELU_BWD) {
    float u[8];
    unpack8(x.q[0], u);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] *= gelu_grad_f(u[e]);
    *reinterpret_cast<u32x4 *>((bf16_t *)g.C + o) = pack8(v);
  } else if constexpr (EPI == EPI_STORE_F32) {
    *reinterpret_cast<float4 *>((float *)g.C + o) = v0;
    *reinterpret_cast<float4 *>((float *)g.C + o + 4) = v1;
  } else {  // EPI_WGRAD, EPI_WGRAD_ACC
    float *c = (float *)g.C + o;
    float4 o0 = {g.scale * v[0], g.scale * v[1], g.scale * v[2], g.scale * v[3]};
    float4 o1 = {g.scale * v[4], g.scale * v[5], g.scale * v[6], g.scale * v[7]};
    if (EPI == EPI_WGRAD_ACC || g.beta) {
      const float4 c0 = EPI == EPI_WGRAD_ACC ? __builtin_bit_cast(float4, x.q[0]) : *reinterpret_cast<const float4 *>(c);
      const float4 c1 = EPI == EPI_WGRAD_ACC ? __builtin_bit_cast(float4, x.q[1]) : *reinterpret_cast<const float4 *>(c + 4);
      o0.x += c0.x; o0.y += c0.y; o0.z += c0.z; o0.w += c0.w;
      o1.x += c1.x; o1.y += c1.y; o1.z += c1.z; o1.w += c1.w;
    }
    *reinterpret_cast<float4 *>(c) = o0;
    *reinterpret_cast<float4 *>(c + 4) = o1;
  }
}

// ---- epilogue shared by the kernels ---------------------------------------------------------
// A lane holds column (lane & 31) and rows 8*(r/4) + 4*(lane>>5) + (r&3) of each 32x32 block.  Each
// wavefront passes strips of 8 (64-wide wave tile) or 16 rows through an LDS region of its own so
// that every lane ends up with 8 consecutive columns of one row: 16-byte bf16 / 32-byte fp32 stores
// and equally wide reads of bias, residual and pre-activation.  No workgroup barrier is involved:
// the region is private to the wavefront, whose LDS operations complete in issue order.
// What the epilogue reads from memory is requested for all rows of a call up front: strip by strip
// each read's latency stood alone, eight times per 64-row wave tile.
template <int WTN>
struct EpiStrip {
  static constexpr int SP = WTN + 4, LPR = WTN / 8, RPP = 64 / LPR, GPS = RPP / 8, NSTRIP = 32 / RPP;
  static constexpr int FLOATS = RPP * SP;  // per wavefront
};
template <int WTN, int EPI, int MI>
struct EpiExtras {
  static constexpr int COUNT = kExtraBf16<EPI> || kExtraF32<EPI> ? MI * EpiStrip<WTN>::NSTRIP : 1;
  Extra x[COUNT];
  int tgt[EPI == EPI_LOGITS ? MI * EpiStrip<WTN>::NSTRIP : 1];
  u32x4 bias;
  __device__ inline void load(const GemmArgs &g, int row0, int col0, int lane) {
    typedef EpiStrip<WTN> E;
    const int gcol = col0 + (lane % E::LPR) * 8, row = row0 + lane / E::LPR;
    if constexpr (kBias<EPI>) {
      bias = u32x4{};
      if (gcol < g.N) bias = *reinterpret_cast<const u32x4 *>((const bf16_t *)g.bias + gcol);
    }
    if constexpr (kExtraBf16<EPI> || kExtraF32<EPI>) {
#pragma unroll
      for (int k = 0; k < COUNT; ++k) x[k] = load_extra<EPI>(g, row + k * E::RPP, gcol);
    }
    if constexpr (EPI == EPI_LOGITS) {
      if (g.row_stats) {
#pragma unroll
        for (int k = 0; k < MI * E::NSTRIP; ++k) tgt[k] = row + k * E::RPP < g.M ? g.row_targets[row + k * E::RPP] : -1;
      }
    }
  }
  // Waits for all of it, that is for what these strips read: of a 256x256 tile's two halves the second waits here behind the
  // first's stores (it was requested ahead of them, fp32 reads apart), and epilogue_gelu_sum() takes its reads as they come.
  // Loads and stores count down one counter in order, and stores behind a condition cannot be
  // counted when compiling: waiting strip by strip, each strip also waited for the strip before to be written (logits
  // of 2048 x 32000 x 256: 85.4 us, now 81.1; GELU' of 16384 x 8192 x 2048: 536 us, now 529).
  __device__ inline void arrived() {
    if constexpr (kBias<EPI>) asm volatile("" : "+v"(bias)::"memory");
    if constexpr (kExtraBf16<EPI> || kExtraF32<EPI>) {
#pragma unroll
      for (int k = 0; k < COUNT; ++k) {
        asm volatile("" : "+v"(x[k].q[0])::"memory");
        if constexpr (kExtraF32<EPI>) asm volatile("" : "+v"(x[k].q[1])::"memory");
      }
    }
    if constexpr (EPI == EPI_LOGITS) {
#pragma unroll
      for (int k = 0; k < MI * EpiStrip<WTN>::NSTRIP; ++k) asm volatile("" : "+v"(tgt[k])::"memory");
    }
  }
};
template <int WTN, int EPI, int MI, int NI>
__device__ inline void epilogue_strips(const GemmArgs &g, floatx16 (&acc)[MI][NI], float *stg, int row0, int col0,
                                       int lane, EpiExtras<WTN, EPI, MI> &ex) {
  typedef EpiStrip<WTN> E;
  constexpr int SP = E::SP;
  const int hh = lane >> 5, lq = lane & 31;
  const int col_l = (lane % E::LPR) * 8, row_in = lane / E::LPR;
  const int gcol = col0 + col_l;
  ex.arrived();
  float bv[8];
  if constexpr (kBias<EPI>) unpack8(ex.bias, bv);
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int p = 0; p < E::NSTRIP; ++p) {
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int gq = 0; gq < E::GPS; ++gq)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            stg[(8 * gq + 4 * hh + e) * SP + j * 32 + lq] = acc[i][j][4 * (p * E::GPS + gq) + e];
      asm volatile("" ::: "memory");
      const float4 v0 = *reinterpret_cast<const float4 *>(stg + row_in * SP + col_l);
      const float4 v1 = *reinterpret_cast<const float4 *>(stg + row_in * SP + col_l + 4);
      asm volatile("" ::: "memory");
      const int grow = row0 + i * 32 + p * E::RPP + row_in;
      if constexpr (EPI == EPI_LOGITS) {
        // Softmax statistics of this row's 64 columns from the fp32 accumulators (before any rounding):
        // the row's eight lanes (consecutive lane ids) each hold eight columns; N is a multiple of 8, so a
        // lane's columns are all inside the matrix or all outside.  These are vector instructions that nothing hides
        // (two wavefronts to a SIMD, both in the epilogue), so they are counted: one selection per lane, not one per
        // column, and the target's logit from the strip in LDS, not by eight comparisons.  2048 x 32000 x 256:
        // 89.8 us with 1943 vector instructions per lane of a 256x256 tile, 85.4 with 1384.
        static_assert((WTN == kStatGroup && E::LPR == 8) || EPI != EPI_LOGITS, "one statistics group per wave-tile row");
        if (g.row_stats) {
          const float v[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
          const bool in = gcol < g.N;
          float m = max3(max3(v[0], v[1], v[2]), max3(v[3], v[4], v[5]), max3(v[6], v[7], v[7]));
          m = in ? m : -INFINITY;
          m = fmaxf(m, dpp_f32<0xB1>(m));   // lane ^ 1
          m = fmaxf(m, dpp_f32<0x4E>(m));   // lane ^ 2
          m = fmaxf(m, dpp_f32<0x141>(m));  // the other quad of the eight lanes
          const float m2 = m * 1.4426950408889634f;
          float se = 0.f;
#pragma unroll
          for (int e = 0; e < 8; ++e) se += __builtin_amdgcn_exp2f(__builtin_fmaf(v[e], 1.4426950408889634f, -m2));
          se = in ? se : 0.f;
          se += dpp_f32<0xB1>(se);
          se += dpp_f32<0x4E>(se);
          se += dpp_f32<0x141>(se);
          if (grow < g.M) {
            if (lane % E::LPR == 0 && col0 < g.N) {
              float *st = g.row_stats + ((size_t)grow * ((g.N + kStatGroup - 1) / kStatGroup) + col0 / kStatGroup) * 2;
              st[0] = m;
              st[1] = se;
            }
            const int tgt = ex.tgt[i * E::NSTRIP + p];
            if (in && (unsigned)(tgt - gcol) < 8) g.row_ztgt[grow] = stg[row_in * SP + tgt - col0];
          }
        }
      }
      emit8<EPI>(g, v0, v1, grow, gcol, bv, ex.x[EpiExtras<WTN, EPI, MI>::COUNT > 1 ? i * E::NSTRIP + p : 0]);
    }
}

// EPI_GELU_BWD_SUM on a wave's two 64 x 64 pieces: of two streams the same tokens (one pre-activation, one
// derivative and one sum for both), of one stream two runs of 64 rows.  Column sums of the pieces' sum, as stored,
// go to row (first row of the piece) / 64 of g.row_stats.  limit: rows beyond it do not exist.
__device__ inline void epilogue_gelu_sum(const GemmArgs &g, floatx16 (&acc)[2][2][2], float *stg, int r0, int r1, int limit0,
                                         int limit1, int col0, int lane, const EpiExtras<64, EPI_GELU_BWD_SUM, 2> (&ex)[2]) {
  typedef EpiStrip<64> E;
  constexpr int SP = E::SP;
  const int hh = lane >> 5, lq = lane & 31, col_l = (lane & 7) * 8, row_in = lane >> 3, gcol = col0 + col_l;
  const bool two = g.streams == 2, in = gcol < g.N;
  float cols[2][8] = {};
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int p = 0; p < 4; ++p) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) stg[h * E::FLOATS + (4 * hh + e) * SP + j * 32 + lq] = acc[h][i][j][4 * p + e];
      asm volatile("" ::: "memory");
      float v[2][8], d[8];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const float4 f = *reinterpret_cast<const float4 *>(stg + h * E::FLOATS + row_in * SP + col_l + 4 * q);
          v[h][4 * q] = f.x; v[h][4 * q + 1] = f.y; v[h][4 * q + 2] = f.z; v[h][4 * q + 3] = f.w;
        }
      asm volatile("" ::: "memory");
      const int row = i * 32 + p * 8 + row_in;
      float sum[8] = {};
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (h == 0 || !two) {
          unpack8(ex[h].x[i * 4 + p].q[0], d);
#pragma unroll
          for (int e = 0; e < 8; ++e) d[e] = gelu_grad_f(d[e]);
        }
        const int grow = (h ? r1 : r0) + row;
        if (!in || grow >= (h ? limit1 : limit0)) continue;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[h][e] *= d[e];
        const u32x4 o = pack8(v[h]);
        *reinterpret_cast<u32x4 *>((bf16_t *)g.C + (size_t)grow * g.ldc + gcol) = o;
        float y[8];
        unpack8(o, y);
        const float w = g.sum_w[two ? h : 0];
        if (w != 0.f) {  // (uniform)
#pragma unroll
          for (int e = 0; e < 8; ++e) sum[e] += w * y[e];
        }
        if (h == 1 || !two) {
          if (g.C2) *reinterpret_cast<u32x4 *>((bf16_t *)g.C2 + (size_t)((two ? r0 : grow - row) + row) * g.ldc + gcol) = pack8(sum);
#pragma unroll
          for (int e = 0; e < 8; ++e) { cols[two ? 0 : h][e] += sum[e]; sum[e] = 0.f; }
        }
      }
    }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (h == 1 && two) break;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float c = cols[h][e];
      c += __shfl_xor(c, 8, 64);
      c += __shfl_xor(c, 16, 64);
      c += __shfl_xor(c, 32, 64);
      cols[h][e] = c;
    }
    const int row = h ? r1 : r0;
    if (lane < 8 && in && row < (h ? limit1 : limit0)) {
      float *o = g.row_stats + (size_t)(row >> 6) * g.N + gcol;
      *reinterpret_cast<float4 *>(o) = make_float4(cols[h][0], cols[h][1], cols[h][2], cols[h][3]);
      *reinterpret_cast<float4 *>(o + 4) = make_float4(cols[h][4], cols[h][5], cols[h][6], cols[h][7]);
    }
  }
}

// ------------------------------------------------------------------------------------------
// Direct loads write 16 bytes per lane at consecutive LDS addresses in lane order, so the
// LDS image of a tile is fixed and the swizzle is applied on the global side: the thread that
// fills LDS chunk position p fetches the logical chunk that belongs there.
//   k-contiguous tile: [row][64 k] (128 bytes per row), chunk c of row r at c ^ g(r)
//   k-major tile:      [k][ROWS]  (ROWS*2 bytes per k),  chunk c of k-row k at c ^ KS(k & 3), KS = 4 for k-rows of
//                      256 bytes or more (all start at bank 0 of the 64 four-byte banks: the four k-rows that one
//                      cycle of a transposing read touches, 64 bytes each, go to the four quarters of the bank
//                      span), 2 for 128-byte k-rows (which alternate between the halves of the span by themselves)
// A k-major fragment is two ds_read_b64_tr_b16: within 16 lanes, lane i points at 4
// consecutive rows-elements of k-row kb + i/4, column group 4(i%4); the instruction hands
// lane j the four k values kb..kb+3 of row j - exactly the MFMA operand order.
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short short4v;

constexpr int kBK = 64;  // K step

template <int ROWS, bool KMAJOR, int NT>
struct DmaTile {
  static constexpr int BYTES = ROWS * kBK * 2;
  static constexpr int NLD = BYTES / (NT * 16);  // loads per thread per K step
  static_assert(BYTES % (NT * 16) == 0 && NLD >= 1, "tile must divide over the threads");
  static constexpr int RB = KMAJOR ? ROWS * 2 : kBK * 2;  // LDS bytes per row
  static constexpr int KS = ROWS >= 128 ? 4 : 2;          // k-major swizzle step, in 16-byte chunks
  uint32_t voff[NLD];
  int kadd[NLD];
  uint32_t kstride;

  __device__ static inline int g(int row) { return (row ^ (row >> 3)) & 7; }

  __device__ inline void init(int row0, int rows, int ld, int t) {
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int p = i * NT + t;
      if constexpr (!KMAJOR) {
        constexpr int CPR = kBK / 8;
        const int row = p / CPR, chunk = (p % CPR) ^ g(row);
        kadd[i] = chunk * 8;
        voff[i] = row0 + row < rows ? ((uint32_t)(row0 + row) * ld + chunk * 8) * 2u : kOob;
        kstride = 2;
      } else {
        constexpr int CPR = ROWS / 8;
        const int krow = p / CPR, chunk = (p % CPR) ^ (KS * (krow & 3));
        kadd[i] = krow;
        voff[i] = row0 + chunk * 8 < rows ? ((uint32_t)krow * ld + row0 + chunk * 8) * 2u : kOob;
        kstride = (uint32_t)ld * 2u;
      }
    }
  }
  // lds: stage base of this operand (wave-uniform); wave: wave id (uniform)
  __device__ inline void issue(BufRsrc rs, char *lds, int wave, int k0, int kend) const {
    const uint32_t adv = (uint32_t)k0 * kstride;
    const uint32_t base = lds_address(lds) + wave * 1024;
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const bool ok = k0 + kadd[i] < kend;
      dma16(rs, base + i * (NT * 16), ok ? voff[i] + adv : kOob);
    }
  }
  // K-contiguous tiles: the swizzled address of fragment (row block i, k
  // slice ks) differs from that of (0, 0) in bits 5-6 only, by an exclusive-or with a constant
  // (32 rows toggle bit 2 of g, a k slice adds 2 to the chunk index).  One lane-dependent base per
  // operand plus a constant per read costs no registers for precomputed addresses, which the
  // multiply loop of the large tile needs for its accumulators.
  static constexpr bool XOR_FORM = !KMAJOR;
  __device__ static inline uint32_t lane_base(uint32_t lds_addr, int rbase0, int lane) {
    const int row = rbase0 + (lane & 31);
    return lds_addr + row * RB + ((((lane >> 5) ^ g(row)) & 7) << 4);
  }
  __device__ static inline bf16x8 frag_x(uint32_t base, int i, int ks) {
    typedef __attribute__((address_space(3))) const bf16x8 *lds_frag;
    const uint32_t a = (base ^ (uint32_t)(((2 * ks) ^ (4 * (i & 1))) << 4)) + i * 32 * RB;
    return *reinterpret_cast<lds_frag>((uintptr_t)a);
  }
  // 32 x 16 MFMA fragment of rows [rbase, rbase+32), k slice ks of the staged K step
  __device__ static inline bf16x8 frag(const char *lds, int rbase, int ks, int lane) {
    if constexpr (!KMAJOR) {
      const int row = rbase + (lane & 31), chunk = 2 * ks + (lane >> 5);
      return *reinterpret_cast<const bf16x8 *>(lds + row * RB + ((chunk ^ g(row)) << 4));
    } else {
      const int g16 = lane >> 4, i = lane & 15;
      const int m = rbase + 16 * (g16 & 1) + 4 * (i & 3);
      const int k = 16 * ks + 8 * (g16 >> 1) + (i >> 2);
      const int col = (((m >> 3) ^ (KS * (i >> 2))) << 4) + ((m >> 2) & 1) * 8;
      union { short4v h[2]; bf16x8 v; } f;
      f.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (__attribute__((address_space(3))) short4v *)(lds + k * RB + col));
      f.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (__attribute__((address_space(3))) short4v *)(lds + (k + 4) * RB + col));
      return f.v;
    }
  }
};

// f(std::integral_constant<int, 0>{}), ..., f(std::integral_constant<int, N - 1>{})
template <class F, int... I>
__device__ inline void static_for_impl(F &&f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ inline void static_for(F &&f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// The prepared problems of one call, as the launchers take them.
struct GemmBatch {
  int count;
  GemmArgs p[kMaxBatch];
};

// Who issues the direct loads.  A wavefront's LDS operations complete in issue order and a direct
// load is one of them, so a wavefront that loads the next tile and then reads fragments of the
// current one waits for its own loads.  With LOADERS four extra wavefronts (one per SIMD) do
// nothing but load, NSTAGE-1 tiles ahead, and the multiplying wavefronts never have a load in
// their LDS queue; without, every wavefront loads its share and then multiplies (the cheaper
// arrangement when many small workgroups share a CU and cover for each other).
// The multiply loop is hand-pipelined where it has the wavefront's LDS queue to itself.
constexpr int kLoaderWaves = 4;
template <int BM, int BN, int WGM, int WGN, int NSTAGE, bool AKM, bool BKM, int EPI, bool LOADERS, int MAX>
__global__ __launch_bounds__(64 * (WGM * WGN + (LOADERS ? kLoaderWaves : 0))) void gemm_dma_kernel(Problems<MAX> batch) {
  constexpr int NC = 64 * WGM * WGN;                // multiplying threads
  constexpr int NL = LOADERS ? 64 * kLoaderWaves : NC;  // threads that share the loading of one tile
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int MI = WTM / 32, NI = WTN / 32;
  constexpr int ABYTES = BM * kBK * 2, STAGE = (BM + BN) * kBK * 2;
  constexpr int EPIB = WGM * WGN * EpiStrip<WTN>::FLOATS * 4;  // epilogue staging reuses the operand buffers
  __shared__ __attribute__((aligned(1024))) char smem[NSTAGE * STAGE > EPIB ? NSTAGE * STAGE : EPIB];

  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = wave / WGN, wn = wave % WGN;

  int tile0;
  GemmArgs g = my_problem(batch, tile0);
  const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
  const MyTile mt = my_tile(g, blockIdx.x - tile0, tiles_m, tiles_n);
  const int m0 = mt.m * BM, n0 = mt.n * BN, kb0 = mt.k0, ke = mt.k1;

  const BufRsrc ra = make_rsrc(g.A, g.a_bytes), rb = make_rsrc(g.B, g.b_bytes);
  typedef DmaTile<BM, AKM, NL> TA;
  typedef DmaTile<BN, BKM, NL> TB;
  TA la;
  TB lb;
  la.init(m0, g.M, g.lda, t % NL);
  lb.init(n0, g.N, g.ldb, t % NL);
  const int lwave = wave % (NL / 64);             // position of this wavefront among the loaders of a tile
  const bool loader = LOADERS && wave >= WGM * WGN;  // this wavefront only loads (uniform)
  constexpr int LPS = TA::NLD + TB::NLD;  // loads per thread per K step
  const int nk = (ke - kb0 + kBK - 1) / kBK;
  auto issue = [&](int kt) {
    char *st = smem + (kt % NSTAGE) * STAGE;
    la.issue(ra, st, lwave, kb0 + kt * kBK, ke);
    lb.issue(rb, st + ABYTES, lwave, kb0 + kt * kBK, ke);
  };

  floatx16 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const uint32_t xa = TA::lane_base(lds_address(smem), wm * WTM, lane);
  const uint32_t xb = TB::lane_base(lds_address(smem) + ABYTES, wn * WTN, lane);
  // K steps kt .. kt+NSTAGE-2 are in flight while step kt is multiplied; one barrier per step:
  // it publishes step kt (every loading thread waited for its own loads of it) and retires the
  // buffer of step kt-1, which the loads issued right after it overwrite.
  if (!LOADERS || loader) {
#pragma unroll
    for (int s = 0; s < NSTAGE - 1; ++s)
      if (s < nk) issue(s);
  }
  if (loader) {
    // the same barriers as the multiplying wavefronts, through the epilogue's, then done
    for (int kt = 0; kt < nk; ++kt) {
      if (nk - 1 - kt >= NSTAGE - 2)
        wait_vmcnt<(NSTAGE - 2) * LPS>();
      else
        wait_vmcnt<0>();
      __syncthreads();
      if (kt + NSTAGE - 1 < nk) issue(kt + NSTAGE - 1);
    }
    __syncthreads();  // (the one barrier between the last multiply and the epilogue's use of the ring)
    return;
  }

  // What the epilogue reads: before the first step, under which its latency passes, where the registers that it then
  // holds through the loop cost no resident workgroup (one 128x128 ring of two steps less on a CU) and do not spill
  // (fp32 reads beside the accumulators of twelve wavefronts).  GELU' of 4096 x 1024 x 256: 8.6 us, now 7.9; FC2 with its
  // residual, 4096 x 256 x 1024: 7.0 us, now 6.6.
  constexpr bool EARLY = LOADERS && (MI * NI == 1 || NSTAGE == 4 || (NSTAGE == 3 && !kExtraF32<EPI>));
  EpiExtras<WTN, EPI, MI> ex;
  if constexpr (EARLY) ex.load(g, m0 + wm * WTM, n0 + wn * WTN, lane);
  for (int kt = 0; kt < nk; ++kt) {
    if constexpr (!LOADERS) {
      if (nk - 1 - kt >= NSTAGE - 2)
        wait_vmcnt<(NSTAGE - 2) * LPS>();
      else
        wait_vmcnt<0>();
    }
    __syncthreads();
    if constexpr (!LOADERS) {
      if (kt + NSTAGE - 1 < nk) issue(kt + NSTAGE - 1);
    }
    const char *sa = smem + (kt % NSTAGE) * STAGE;
    const char *sb = sa + ABYTES;
    const uint32_t soff = (uint32_t)(kt % NSTAGE) * STAGE;  // (added before the exclusive-or: no carry into bits 4-6)
    if constexpr (LOADERS) {
      // Software pipeline over the (k slice, row block) slots of the step: the A fragment of the next
      // slot and, two slots before a new k slice, its B fragments are requested before the MFMAs of
      // the current slot, and the scheduler is held to that order (one group of LDS reads, then the
      // slot's MFMAs), so a read's latency passes under the previous slot's matrix work.
      constexpr int KS = kBK / 16, ARD = AKM ? 2 : 1, BRD = BKM ? 2 : 1;  // LDS instructions per fragment
      auto getA = [&](int ks, int i) {
        return TA::XOR_FORM ? TA::frag_x(xa + soff, i, ks) : TA::frag(sa, wm * WTM + i * 32, ks, lane);
      };
      auto getB = [&](int ks, int j) {
        return TB::XOR_FORM ? TB::frag_x(xb + soff, j, ks) : TB::frag(sb, wn * WTN + j * 32, ks, lane);
      };
      // D slots ahead: two where the accumulators leave room for a third A fragment, else one
      constexpr int D = (MI * NI <= 4 && MI >= 2) ? 2 : 1;
      static_assert(D <= MI || MI == 1, "a k slice's B fragments are requested while the previous slice is in use");
      bf16x8 aq[D + 1], bq[2][NI];
#pragma unroll
      for (int j = 0; j < NI; ++j) bq[0][j] = getB(0, j);
#pragma unroll
      for (int p = 0; p < D; ++p)
        if (p < KS * MI) aq[p] = getA(p / MI, p % MI);
      __builtin_amdgcn_sched_group_barrier(0x100, NI * BRD + D * ARD, 0);
      static_for<KS * MI>([&](auto slot_c) {
        constexpr int slot = decltype(slot_c)::value, ks = slot / MI, i = slot % MI;
        constexpr int ahead = slot + D;
        constexpr bool nextA = ahead < KS * MI;
        constexpr bool nextB = nextA && ahead % MI == 0;
        if constexpr (nextA) aq[ahead % (D + 1)] = getA(ahead / MI, ahead % MI);
        if constexpr (nextB) {
#pragma unroll
          for (int j = 0; j < NI; ++j) bq[(ahead / MI) & 1][j] = getB(ahead / MI, j);
        }
#pragma unroll
        for (int j = 0; j < NI; ++j)
          acc[i][j] =
              __builtin_amdgcn_mfma_f32_32x32x16_bf16(aq[slot % (D + 1)], bq[ks & 1][j], acc[i][j], 0, 0, 0);
        constexpr int reads = (nextA ? ARD : 0) + (nextB ? NI * BRD : 0);
        if constexpr (reads > 0) __builtin_amdgcn_sched_group_barrier(0x100, reads, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, NI, 0);
      });
      continue;
    }
#pragma unroll
    for (int ks = 0; ks < kBK / 16; ++ks) {
      bf16x8 af[MI], bfr[NI];
#pragma unroll
      for (int i = 0; i < MI; ++i)
        af[i] = TA::XOR_FORM ? TA::frag_x(xa + soff, i, ks) : TA::frag(sa, wm * WTM + i * 32, ks, lane);
#pragma unroll
      for (int j = 0; j < NI; ++j)
        bfr[j] = TB::XOR_FORM ? TB::frag_x(xb + soff, j, ks) : TB::frag(sb, wn * WTN + j * 32, ks, lane);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
    }
  }
  if constexpr (!EARLY) ex.load(g, m0 + wm * WTM, n0 + wn * WTN, lane);
  __syncthreads();  // every wavefront is done with the ring
  epilogue_strips<WTN, EPI>(g, acc, reinterpret_cast<float *>(smem) + wave * EpiStrip<WTN>::FLOATS, m0 + wm * WTM,
                            n0 + wn * WTN, lane, ex);
}

// ------------------------------------------------------------------------------------------
// The 256x256 tile.  Eight wavefronts, two per SIMD (w and w + 4), in two groups that take turns: while one
// group's products occupy the matrix units, the other reads its next fragments from LDS and issues direct
// loads; a workgroup barrier hands over.  No wavefront both waits for LDS and feeds the matrix unit, and -
// unlike with separate loader wavefronts, which leave 168 registers to each of twelve - a wavefront has the
// registers for all fragments of 16 products (512 matrix cycles) besides its 128 accumulators.
//
// A wavefront (wm, wn) owns columns 64 wn .. 64 wn + 63 and rows 64 wm .. 64 wm + 63 of both 128-row halves.
// Two K steps are staged, 2 x 64 KB, each operand as two tiles of 128 rows.  A K step is two phases,
//   phase 1: read A half 0 and all of B, products of half 0;  load A half 1 of step s + 1
//   phase 2: read A half 1, products of half 1;               load A half 0 and B of step s + 2
// Every read of a phase has returned before the barrier that ends its reading part (lgkmcnt 0), and the
// next phase's loads come after that barrier, so a load never meets a read of the slot it refills; and a
// load is awaited (vmcnt: eight younger ones may be outstanding, each wavefront for its own, then the
// barrier) two phases after it was issued and read after three - one and a half K steps, where a two-stage
// ring of whole tiles gives one.
//
// Bound: with every CU busy the part holds 1.6-1.7 GHz under its power limit on products of this kind, and
// 8192^3 at 1.44 PFLOP/s is 81-86 % of the matrix units' rate at that clock (with loader wavefronts and a
// persistent grid 1.39; data gradients 8192 x 2048 x 6144: 164 -> 150 us); the counters say busy 86-90 % of the
// CUs' busy cycles in a d = 2048 step's plain-store launches, 59-60 % where the epilogue is heavy.  A K step has
// four barriers; four more (a phase per quadrant) cost 9 %, 16x16x32 products 5 %.
#define IL_FENCE()                         \
  do {                                     \
    asm volatile("" ::: "memory");         \
    __builtin_amdgcn_sched_barrier(0);     \
  } while (0)
template <bool AKM, bool BKM, int EPI, int MAX>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_pair_kernel(Problems<MAX> batch) {
  constexpr int HB = 128 * 64 * 2;  // bytes of half an operand tile
  __shared__ __attribute__((aligned(1024))) char smem[8 * HB];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6), wm = wave >> 2, wn = wave & 3;
  typedef DmaTile<128, AKM, 512> TA;
  typedef DmaTile<128, BKM, 512> TB;
  static_assert(TA::NLD == 2 && TB::NLD == 2, "the load counts below");

  int tile0;
  GemmArgs g = my_problem(batch, tile0);
  // The tile's two halves are 128 rows each: consecutive, or (EPI_GELU_BWD_SUM of two streams stacked over
  // M / 2 tokens) the same tokens of either stream.
  const int half = EPI == EPI_GELU_BWD_SUM && g.streams == 2 ? g.M >> 1 : 0;
  const int tiles_m = half ? (half + 127) / 128 : (g.M + 255) / 256, tiles_n = (g.N + 255) / 256;
  const MyTile mt = my_tile(g, blockIdx.x - tile0, tiles_m, tiles_n);
  const int tm = mt.m, n0 = mt.n * 256, kb0 = mt.k0, ke = mt.k1;
  const int m0 = tm * (half ? 128 : 256), m1 = half ? half + m0 : m0 + 128;
  const int limit0 = half ? half : g.M;
  const int nk = (ke - kb0 + 63) / 64;

  const BufRsrc ra = make_rsrc(g.A, g.a_bytes), rb = make_rsrc(g.B, g.b_bytes);
  TA la[2];
  TB lb[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    la[i].init(i ? m1 : m0, i ? g.M : limit0, g.lda, t);
    lb[i].init(n0 + 128 * i, g.N, g.ldb, t);
  }
  // LDS slot s & 1: A half 0, A half 1, B half 0, B half 1.  A step past the last one loads zeros (every lane
  // is beyond the range), so the load counts hold to the end.
  auto loadA = [&](int s, int i) { la[i].issue(ra, smem + (s & 1) * 4 * HB + i * HB, wave, kb0 + s * 64, ke); };
  auto loadB = [&](int s) {
    lb[0].issue(rb, smem + (s & 1) * 4 * HB + 2 * HB, wave, kb0 + s * 64, ke);
    lb[1].issue(rb, smem + (s & 1) * 4 * HB + 3 * HB, wave, kb0 + s * 64, ke);
  };
  loadA(0, 0);
  loadB(0);
  loadA(0, 1);
  loadA(1, 0);
  loadB(1);

  floatx16 acc[2][2][2];  // [row half][32-row block][32-column block]
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][q][j][r] = 0.f;

  const uint32_t xa = TA::lane_base(lds_address(smem), wm * 64, lane);
  const int bhalf = (2 + (wn >> 1)) * HB;  // this wavefront's columns lie in one half of B
  const uint32_t xb = TB::lane_base(lds_address(smem) + bhalf, (wn & 1) * 64, lane);
  bf16x8 fa[2][4], fb[2][4];  // [block][k slice of 16]
  auto readA = [&](uint32_t slot, int i) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        fa[q][ks] = TA::XOR_FORM ? TA::frag_x(xa + slot + i * HB, q, ks)
                                 : TA::frag(smem + slot + i * HB, wm * 64 + q * 32, ks, lane);
  };
  auto readB = [&](uint32_t slot) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        fb[j][ks] = TB::XOR_FORM ? TB::frag_x(xb + slot, j, ks)
                                 : TB::frag(smem + slot + bhalf, (wn & 1) * 64 + j * 32, ks, lane);
  };
  auto hand_over = [&] {
    IL_FENCE();
    __builtin_amdgcn_s_barrier();
    IL_FENCE();
  };
  auto products = [&](auto half) {
    constexpr int i = decltype(half)::value;
    wait_vmcnt<8>();
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    hand_over();
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int q = 0; q < 2; ++q)
          acc[i][q][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[q][ks], fb[j][ks], acc[i][q][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    hand_over();
  };

  wait_vmcnt<8>();  // A half 0 and B of step 0
  hand_over();
  if (wm == 1) hand_over();  // the second group runs one part behind the first
  for (int s = 0; s < nk; ++s) {
    const uint32_t slot = (uint32_t)(s & 1) * 4 * HB;
    readA(slot, 0);
    readB(slot);
    loadA(s + 1, 1);
    products(std::integral_constant<int, 0>{});
    readA(slot, 1);
    loadA(s + 2, 0);
    loadB(s + 2);
    products(std::integral_constant<int, 1>{});
  }
  wait_vmcnt<0>();           // (the zeros of the steps past the end have landed: the epilogue reuses the slots)
  const int r0 = m0 + wm * 64, r1 = m1 + wm * 64, c0 = n0 + wn * 64;
  EpiExtras<64, EPI, 2> ex[2];  // bf16 reads of both halves fit the registers the fragments leave, fp32 reads of one
  ex[0].load(g, r0, c0, lane);
  if constexpr (!kExtraF32<EPI>) {
    if (!half) ex[1].load(g, r1, c0, lane);
  }
  if (wm == 0) hand_over();
  hand_over();
  if constexpr (EPI == EPI_GELU_BWD_SUM) {
    float *stg = reinterpret_cast<float *>(smem) + 2 * wave * EpiStrip<64>::FLOATS;
    epilogue_gelu_sum(g, acc, stg, r0, r1, limit0, g.M, c0, lane, ex);
  } else {
    float *stg = reinterpret_cast<float *>(smem) + wave * EpiStrip<64>::FLOATS;
    epilogue_strips<64, EPI>(g, acc[0], stg, r0, c0, lane, ex[0]);
    if constexpr (kExtraF32<EPI>) ex[1].load(g, r1, c0, lane);
    epilogue_strips<64, EPI>(g, acc[1], stg, r1, c0, lane, ex[1]);
  }
}

thread_local const KernelTimer *tl_timer = nullptr;  // armed by gemm_time_next()

// The launch, with the armed timer's events on it if there is one.
template <typename P>
hipError_t launch_one(void (*kernel)(P), const P &problems, int workgroups, int threads, hipStream_t s) {
  if (const KernelTimer *t = tl_timer) {
    tl_timer = nullptr;
    hipExtLaunchKernelGGL(kernel, dim3(workgroups), dim3(threads), 0, s, t->start, t->stop, 0, problems);
  } else {
    hipLaunchKernelGGL(kernel, dim3(workgroups), dim3(threads), 0, s, problems);
  }
  return hipGetLastError();
}

template <int BM, int BN, int WGM, int WGN, int NSTAGE, bool AKM, bool BKM, int EPI, bool LOADERS>
hipError_t launch_dma(GemmBatch &b, hipStream_t s) {
  return with_problems<AKM && BKM>(
      b.p, b.count,
      [](const GemmArgs &g) { return TileGrid{(g.M + BM - 1) / BM, (g.N + BN - 1) / BN, BM, BN}; },
      [&](const auto &problems, int tiles) {
        return launch_one(gemm_dma_kernel<BM, BN, WGM, WGN, NSTAGE, AKM, BKM, EPI, LOADERS, std::decay_t<decltype(problems)>::kRoom>, problems,
                          tiles, 64 * (WGM * WGN + (LOADERS ? kLoaderWaves : 0)), s);
      });
}

template <bool AKM, bool BKM, int EPI>
hipError_t launch_pair(GemmBatch &b, hipStream_t s) {
  return with_problems<AKM && BKM>(
      b.p, b.count,
      [](const GemmArgs &g) {
        const int rows = EPI == EPI_GELU_BWD_SUM && g.streams == 2 ? (g.M / 2 + 127) / 128 : (g.M + 255) / 256;
        return TileGrid{rows, (g.N + 255) / 256, 256, 256};
      },
      [&](const auto &problems, int tiles) {
        return launch_one(gemm_pair_kernel<AKM, BKM, EPI, std::decay_t<decltype(problems)>::kRoom>, problems, tiles, 512, s);
      });
}

template <bool AKM, bool BKM, int EPI>
hipError_t pick_tile(GemmBatch &b, hipStream_t s) {
  long t256 = 0, t128 = 0, t64 = 0, t256x128 = 0, t128x256 = 0;
  for (int i = 0; i < b.count; ++i) {
    const long sp = std::max(b.p[i].splits, 1);
    t256x128 += sp * ((b.p[i].M + 255) / 256) * ((b.p[i].N + 127) / 128);
    t128x256 += sp * ((b.p[i].M + 127) / 128) * ((b.p[i].N + 255) / 256);
    t64 += sp * ((b.p[i].M + 63) / 64) * ((b.p[i].N + 63) / 64);
    t256 += sp * ((b.p[i].M + 255) / 256) * ((b.p[i].N + 255) / 256);
    t128 += sp * ((b.p[i].M + 127) / 128) * ((b.p[i].N + 127) / 128);
  }
  if constexpr (EPI == EPI_LOGITS) {
    // a statistics group is the 64 columns of one wave tile: every tile but the 64x64 ones (32-wide wave tiles)
    if (b.p[0].tile == 4 || b.p[0].tile == 5) return hipErrorInvalidValue;
  }
  switch (b.p[0].tile) {
    case 1:
    case 8: return launch_pair<AKM, BKM, EPI>(b, s);
    case 2: return launch_dma<128, 128, 2, 2, 2, AKM, BKM, EPI, true>(b, s);
    case 3: return launch_dma<128, 128, 2, 2, 4, AKM, BKM, EPI, true>(b, s);
    case 4: if constexpr (EPI != EPI_LOGITS) return launch_dma<64, 64, 2, 2, 2, AKM, BKM, EPI, false>(b, s); else break;
    case 5: if constexpr (EPI != EPI_LOGITS) return launch_dma<64, 64, 2, 2, 4, AKM, BKM, EPI, true>(b, s); else break;
    case 6: return launch_dma<256, 128, 4, 2, 3, AKM, BKM, EPI, true>(b, s);
    case 7: return launch_dma<128, 256, 2, 4, 3, AKM, BKM, EPI, true>(b, s);
    default: break;
  }
  // Measured on MI355X, with operands that are not already in cache (inside a training step a
  // weight was last used a step ago).  With enough 256x256 tiles to cover most of the 256 CUs the
  // large tile wins (fewest operand bytes per flop).  Below that the 128x128 tile: two workgroups per
  // CU with two stages when there are more tiles than CUs, one workgroup with four stages in flight
  // when each CU gets at most one.  When even those leave CUs idle, 64x64 tiles shorten each
  // workgroup's K loop, which is what bounds such a launch: loader wavefronts and four stages while at
  // most two workgroups land on a CU (the deeper ring covers the trip to HBM), beyond that up to five
  // plain small workgroups per CU that cover for each other.
  if (t256 >= kPairTiles) return launch_pair<AKM, BKM, EPI>(b, s);
  if (t128 >= 192 && t128 <= 256) return launch_dma<128, 128, 2, 2, 4, AKM, BKM, EPI, true>(b, s);
  // about one 256x128 (or 128x256) tile per CU, three stages: as good as the 128x128 tile on cached
  // operands and 15-20 % better on operands from HBM (fewer bytes per flop, deeper ring)
  if (std::min(t256x128, t128x256) >= 192 && std::min(t256x128, t128x256) <= 256)
    return t128x256 <= t256x128 ? launch_dma<128, 256, 2, 4, 3, AKM, BKM, EPI, true>(b, s)
                                : launch_dma<256, 128, 4, 2, 3, AKM, BKM, EPI, true>(b, s);
  if (t128 > 256) return launch_dma<128, 128, 2, 2, 2, AKM, BKM, EPI, true>(b, s);
  if constexpr (EPI == EPI_LOGITS) {
    return launch_dma<128, 128, 2, 2, 4, AKM, BKM, EPI, true>(b, s);  // (never the 32-wide wave tiles)
  } else {
    if (t64 <= 512) return launch_dma<64, 64, 2, 2, 4, AKM, BKM, EPI, true>(b, s);
    return launch_dma<64, 64, 2, 2, 2, AKM, BKM, EPI, false>(b, s);
  }
}

// argument checks and buffer extents of one problem
hipError_t prepare(GemmArgs &g) {
  if (g.M <= 0 || g.N <= 0 || g.K <= 0) return hipErrorInvalidValue;
  if ((g.N & 7) || (g.ldc & 7) || ((uintptr_t)g.C & 15)) return hipErrorInvalidValue;
  if ((g.lda & 7) || (g.ldb & 7) || ((uintptr_t)g.A & 15) || ((uintptr_t)g.B & 15)) return hipErrorInvalidValue;
  if (g.a_kmajor && (g.M & 7)) return hipErrorInvalidValue;
  if (g.b_kmajor && (g.N & 7)) return hipErrorInvalidValue;
  if (!g.a_kmajor && (g.K & 7)) return hipErrorInvalidValue;
  if (!g.b_kmajor && (g.K & 7)) return hipErrorInvalidValue;
  if (!split_ok(g)) return hipErrorInvalidValue;
  if (g.epi == EPI_STORE_DOT && (!g.row_stats || !g.aux || g.aux_wrap < 1 || (g.N & 31))) return hipErrorInvalidValue;
  if (g.epi == EPI_GELU_BWD_SUM && (!g.row_stats || !g.aux || (g.streams != 1 && (g.streams != 2 || (g.M & 127) || g.aux_wrap != g.M / 2)) ||
                                    ((uintptr_t)g.row_stats & 15) || ((uintptr_t)g.C2 & 15) || g.aux_wrap < 1 || g.splits > 1))
    return hipErrorInvalidValue;
  if (g.epi == EPI_LOGITS && g.row_stats && (!g.row_targets || !g.row_ztgt)) return hipErrorInvalidValue;
  const size_t arows = g.a_kmajor ? (size_t)g.K : (size_t)g.M;
  const size_t brows = g.b_kmajor ? (size_t)g.K : (size_t)g.N;
  const size_t ab = arows * g.lda * 2, bb = brows * g.ldb * 2;  // bytes, below 2 GiB
  if (ab >= 0x7FFFFFFFull || bb >= 0x7FFFFFFFull) return hipErrorInvalidValue;
  g.a_bytes = (uint32_t)ab;
  g.b_bytes = (uint32_t)bb;
  return hipSuccess;
}

// Adds up the parts of a split product, four columns per thread, four parts in flight.
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float *__restrict__ part, int splits, size_t stride,
                                                            int rows, int cols, float *out, int ldc) {
  const int c4 = cols >> 2;
  const size_t total = (size_t)rows * c4;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int p0 = 0; p0 < splits; p0 += 4) {
      float4 b[4];
#pragma unroll
      for (int k = 0; k < 4; ++k)
        b[k] = p0 + k < splits ? *reinterpret_cast<const float4 *>(part + (p0 + k) * stride + 4 * i)
                               : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int k = 0; k < 4; ++k) { a.x += b[k].x; a.y += b[k].y; a.z += b[k].z; a.w += b[k].w; }
    }
    *reinterpret_cast<float4 *>(out + i / c4 * ldc + i % c4 * 4) = a;
  }
}

}  // namespace

const KernelTimer *gemm_time_next(const KernelTimer *t) {
  const KernelTimer *old = tl_timer;
  tl_timer = t;
  return old;
}

// The step uses exactly these (layout, epilogue) combinations; anything else is a
// programming error in the caller and is reported instead of silently taking another path.
hipError_t gemm_bf16_batch(const GemmArgs *list, int count, hipStream_t s) {
  if (count < 1 || count > kMaxBatch) return hipErrorInvalidValue;
  GemmBatch b;
  memset(&b, 0, sizeof(b));
  b.count = count;
  for (int i = 0; i < count; ++i) {
    b.p[i] = list[i];
    if (list[i].a_kmajor != list[0].a_kmajor || list[i].b_kmajor != list[0].b_kmajor || list[i].epi != list[0].epi)
      return hipErrorInvalidValue;
    const hipError_t e = prepare(b.p[i]);
    if (e != hipSuccess) return e;
  }
  const GemmArgs &g = b.p[0];
  const int lay = g.a_kmajor * 2 + g.b_kmajor;
  switch (lay) {
    case 1:  // activations x weights[K,N]: forward linears, head logits
      switch (g.epi) {
        case EPI_STORE: return pick_tile<false, true, EPI_STORE>(b, s);
        case EPI_LOGITS: return pick_tile<false, true, EPI_LOGITS>(b, s);
        case EPI_BIAS: return pick_tile<false, true, EPI_BIAS>(b, s);
        case EPI_BIAS_GELU: return pick_tile<false, true, EPI_BIAS_GELU>(b, s);
        case EPI_BIAS_RES: return pick_tile<false, true, EPI_BIAS_RES>(b, s);
        default: return hipErrorInvalidValue;
      }
    case 0:  // dY x W^T with W stored [N,K]: data gradients
      switch (g.epi) {
        case EPI_STORE: return pick_tile<false, false, EPI_STORE>(b, s);
        case EPI_STORE_DOT: return pick_tile<false, false, EPI_STORE_DOT>(b, s);
        case EPI_GELU_BWD: return pick_tile<false, false, EPI_GELU_BWD>(b, s);
        case EPI_GELU_BWD_SUM: return launch_pair<false, false, EPI_GELU_BWD_SUM>(b, s);
        case EPI_STORE_F32: return pick_tile<false, false, EPI_STORE_F32>(b, s);
        default: return hipErrorInvalidValue;
      }
    case 3:  // X^T dY: weight gradients
      if (g.epi != EPI_WGRAD) return hipErrorInvalidValue;
      for (int i = 0; i < count; ++i)
        if (!list[i].beta) return pick_tile<true, true, EPI_WGRAD>(b, s);
      return pick_tile<true, true, EPI_WGRAD_ACC>(b, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t gemm_bf16(const GemmArgs &g, hipStream_t s) { return gemm_bf16_batch(&g, 1, s); }

// The 256x256 tile has both streams' halves of a token in one lane; it is taken where it is the choice anyway.
bool gemm_gelu_sum(int streams, int tokens, int N) {
  const long rows = streams == 2 ? (tokens + 127) / 128 : (tokens + 255) / 256;
  return (streams == 1 || streams == 2) && rows * ((N + 255) / 256) >= kPairTiles;
}

// Prices every number of parts with every tile (measured microseconds per 64-deep K step of a workgroup:
// the 128x128 tile alone on its CU 0.47 with four stages, two of them with two stages 0.96; 256x256 1.35;
// 64x64 up to two per CU 0.42; fp32 as gemm_f32_us), the rounds its workgroups need, and the traffic of writing and
// adding up the parts at 4 bytes per picosecond.
SplitPlan gemm_split_plan(int dtype, int M, int N, int K, size_t ws_floats) {
  const long steps = (K + 63) / 64, cap = std::min<long>({32, (long)(ws_floats / ((size_t)M * N)), steps / 4});
  auto tiles = [&](int t) { return (long)((M + t - 1) / t) * ((N + t - 1) / t); };
  auto up = [](long a, long b) { return (a + b - 1) / b; };
  SplitPlan best{1, 0};
  double best_us = 1e30;
  for (long sp = 1; sp <= std::max<long>(cap, 1); ++sp) {
    const double add_us = sp < 2 ? 0.0 : 4.0 + 2.0 * sp * M * N * 4.0 / 4e6;
    const long per = up(steps, sp);
    auto take = [&](int tile, double us) {
      if (us + add_us < best_us) { best_us = us + add_us; best = SplitPlan{(int)sp, tile}; }
    };
    auto price = [&](int tile, long wgs, long per_round, double step_us) { take(tile, up(wgs, per_round) * per * step_us); };
    if (dtype == 0) {
      take(2, gemm_f32_us(2, tiles(128) * sp, per));
      take(3, gemm_f32_us(3, up(M, 128) * up(N, 64) * sp, per));
      take(4, gemm_f32_us(4, tiles(64) * sp, per));
    } else {
      price(3, tiles(128) * sp, 256, 0.47);
      price(2, tiles(128) * sp, 512, 0.96);
      price(1, tiles(256) * sp, 256, 1.35);
      price(5, tiles(64) * sp, 512, 0.42);
    }
  }
  return best;
}

hipError_t gemm_splitk(int dtype, const GemmArgs &g, SplitPlan plan, float *ws, hipStream_t s) {
  GemmArgs a = g;
  a.tile = plan.tile;
  if (plan.splits < 2) return dtype == 0 ? gemm_f32(a, s) : gemm_bf16(a, s);
  if (g.epi != EPI_STORE_F32 || !ws || (g.N & 3) || (g.ldc & 3)) return hipErrorInvalidValue;
  a.k_per = ((g.K + 63) / 64 + plan.splits - 1) / plan.splits * 64;
  a.splits = (g.K + a.k_per - 1) / a.k_per;
  a.C = ws;
  a.ldc = g.N;
  const hipError_t e = dtype == 0 ? gemm_f32(a, s) : gemm_bf16(a, s);
  if (e != hipSuccess) return e;
  size_t blocks = ((size_t)g.M * (g.N >> 2) + 255) / 256;
  if (blocks > 2048) blocks = 2048;
  hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)blocks), dim3(256), 0, s, ws, a.splits, (size_t)g.M * g.N, g.M,
                     g.N, (float *)g.C, g.ldc);
  return hipGetLastError();
}

}  // namespace il
