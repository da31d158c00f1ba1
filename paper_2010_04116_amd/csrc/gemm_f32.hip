// fp32 GEMM (il_config.dtype == IL_F32) on the bf16 matrix instructions: every fp32 operand element is the sum of
// three bf16 and a product of two elements the sum of six bf16 products, accumulated in fp32.  Arbitrary M, N, K,
// both operand layouts, the library's fused epilogues.
//
// Precision.  hi + mid + lo holds all 24 bits of every normal operand (taken times 2^24, see split8).  Of the nine partial
// products three are left out, mid lo, lo mid and lo lo: each at most 2^-25 of the whole product, together less than
// 2^-24, and of one sign where the operands are equal.  What remains are the roundings of the accumulation, and
// there are fewer of them than with the fp32 instruction (v_mfma_f32_32x32x2_f32: two k at a time): against 64 bits the
// relative error (2-norm) at 2048 x 512 x 2048 is 3.5e-7 where that instruction gave 8.1e-7, at 256 x 256 x 31992 1.6e-6
// and 3.2e-6, at K = 64 5.5e-8 and 1.4e-7; from K = 64 on no shape, layout or distribution of random operands tried
// (normal, with an offset, over ten decades, probabilities) was worse; below, where accumulation hardly rounds, at most
// 1.4 times as large (K = 1 3.6e-8 and 2.6e-8).  Sums of equal products, whose roundings have one sign, come out either
// way: 512 times 0.998^2 1.5e-8 and 5.2e-6, 512 times 1.732^2 5.1e-7 and 3.6e-8.
// What comes out not finite - an infinity splits into NaN parts, sums from 2^80 on overflow - is computed again with the
// fp32 instruction, 64 x 64 outputs at a time: 2048 x 512 x 2048 33 -> 136 us if every block is,
// whatever the number of values.
//
// Bound: 6 x 32 matrix cycles for 32 x 32 x 16, where the fp32 instruction takes 8 x 64: 2.7 times its rate at equal
// clock.  4096 x 4096 x 2048 558 -> 336 us (205 TFLOP/s, 1.23 PFLOP/s of bf16 products: the clock the power limit
// allows); 2048 x 2048 x 512 with GELU 47 -> 30.5, 4096 x 512 x 2048 74 -> 52, 2048 x 512 x 2048 45 -> 32 us: small
// outputs are bound by what a CU is delivered and converts (64 KB and four products of 64 x 64 x 64 every 0.9 us), not by the
// matrix units.
#include <algorithm>
#include <cstring>
#include <type_traits>

#include "common.h"
#include "gemm_tile.h"
#include "lds_dma.h"

namespace il {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short short4v;
typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u32x4;

// Loading threads of a workgroup, beside the four wavefronts that multiply: eight wavefronts in two per SIMD, so that
// one converts while the other waits (four: 33 -> 36 us at 2048 x 512 x 2048, 328 -> 345 at 4096 x 4096 x 2048).
constexpr int NL = 512;
constexpr int kAhead = 3;  // K steps in flight (four or five change nothing)

// Loads to registers, which the compiler waits for; outside the descriptor's range they return 0.
typedef __amdgpu_buffer_rsrc_t Rsrc;
__device__ inline Rsrc rsrc(const void *base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000);
}
__device__ inline floatx4 load_f32x4(Rsrc r, uint32_t off) {
  return __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
}
__device__ inline float load_f32(Rsrc r, uint32_t off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}

struct GemmBatch {  // the prepared problems of one call
  int count;
  GemmArgs p[kMaxBatch];
};

// One operand tile in LDS: three bf16 planes (hi, mid, lo), each in 16-byte chunks of eight elements that are
// consecutive in memory.  Chunk c of a row sits at
//   k-contiguous [row][BK]:  c ^ g(row): 16 consecutive rows of a vector read go to 16 different places of the banks
//   k-major      [k][ROWS]:  c ^ KS (k & 3): the four k rows of a transposing read go to different quarters
// LB = 4 elements per load needs 16-byte aligned rows and an extent divisible by four along the contiguous
// axis; LB = 1 takes anything.
template <int ROWS, bool KMAJOR, int BK, int LB>
struct Tile {
  static constexpr int RB = KMAJOR ? ROWS * 2 : BK * 2, CPR = RB / 16, PLANE = ROWS * BK * 2;  // bytes, chunks, bytes
  static constexpr int NCH = PLANE / 16 / NL, NLD = 8 / LB;  // chunks per loader thread, loads per chunk
  static constexpr int KS = ROWS >= 128 ? 4 : 2;
  static_assert(PLANE % (16 * NL) == 0, "a plane divides over the loading threads");
  static_assert(BK == 32 || BK == 64, "g below");
  uint32_t voff[NCH][NLD];
  int kadd[NCH];
  uint32_t kstride;
  struct Raw { float v[NCH][8]; };
  __device__ static inline int g(int row) { return BK == 64 ? (row ^ (row >> 3)) & 7 : (row >> 2) & 3; }
  __device__ inline void init(int row0, int rows, int ld, int t) {
    kstride = KMAJOR ? (uint32_t)ld * 4u : 4u;
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int p = i * NL + t, r = p / CPR, c = p % CPR;
      const int row = KMAJOR ? 8 * (c ^ (KS * (r & 3))) : r, k = KMAJOR ? r : 8 * (c ^ g(r));
      kadd[i] = k;
#pragma unroll
      for (int e = 0; e < NLD; ++e) {
        const int re = row0 + row + (KMAJOR ? e * LB : 0);
        voff[i][e] = re < rows ? (KMAJOR ? (uint32_t)k * ld + re : (uint32_t)re * ld + k + e * LB) * 4u : kOob;
      }
    }
  }
  __device__ inline void load(Rsrc rs, int k0, int kend, Raw &raw) const {
    const uint32_t adv = (uint32_t)k0 * kstride;
#pragma unroll
    for (int i = 0; i < NCH; ++i)
#pragma unroll
      for (int e = 0; e < NLD; ++e) {
        const bool in = k0 + kadd[i] + (KMAJOR ? 0 : e * LB) < kend;
        const uint32_t off = in ? voff[i][e] + adv : kOob;
        if constexpr (LB == 4) {
          const floatx4 q = load_f32x4(rs, off);
#pragma unroll
          for (int j = 0; j < 4; ++j) raw.v[i][4 * e + j] = q[j];
        } else {
          raw.v[i][e] = load_f32(rs, off);
        }
      }
  }
  // 32 x 16 operand of rows [rbase, rbase + 32), k slice ks, of one plane
  __device__ static inline bf16x8 frag(const char *lds, int rbase, int ks, int lane) {
    if constexpr (!KMAJOR) {
      const int row = rbase + (lane & 31), c = 2 * ks + (lane >> 5);
      return *reinterpret_cast<const bf16x8 *>(lds + row * RB + ((c ^ g(row)) << 4));
    } else {
      const int g16 = lane >> 4, i = lane & 15;
      const int m = rbase + 16 * (g16 & 1) + 4 * (i & 3), k = 16 * ks + 8 * (g16 >> 1) + (i >> 2);
      const int col = (((m >> 3) ^ (KS * (i >> 2))) << 4) + ((m >> 2) & 1) * 8;
      union { short4v h[2]; bf16x8 v; } f;
      f.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v *)(lds + k * RB + col));
      f.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v *)(lds + (k + 4) * RB + col));
      return f.v;
    }
  }
};

// A float as the sum of three bf16, hi + mid + lo, each the rounded rest of the one before: 8 + 8 + 8 bits and
// two signs hold all 24.  It is taken times 2^24, so that lo of the smallest normal operand is a normal number too, and
// the sums of products times 2^-48 at the end: exact both, at 0 to 3 % of the time (2048 x 512 x 2048 31.2 -> 32.1 us).
// Without it operands below 2^-110 lost lo, 1e-36 times 1e36 ten of its bits.  Eight values become a chunk of each plane.
// (Plain multiplies and subtractions of four bytes: fused ones of eight with a literal made the loop 2 % slower.)
constexpr float kUp = 0x1p24f, kDown = 0x1p-48f;
__device__ inline void split8(const float (&x)[8], u32x4 (&f)[3]) {
#pragma clang fp contract(off)
  float up = kUp;
#if defined(__HIP_DEVICE_COMPILE__)
  asm("" : "+s"(up));
#endif
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float a = x[2 * i] * up, b = x[2 * i + 1] * up;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      uint32_t u = pack_bf16x2(a, b);
      asm("" : "+v"(u));  // (or the low half is converted a second time for its own shift)
      f[k][i] = u;
      if (k < 2) {  // (exact: the rest has the remaining bits only)
        a -= __builtin_bit_cast(float, u << 16);
        b -= __builtin_bit_cast(float, u & 0xFFFF0000u);
      }
    }
  }
}
struct Split {
  bf16x8 p[3];  // hi, mid, lo
};
// Four consecutive columns of one row: the epilogue operation and the store.  x is what it reads there
// (residual, pre-activation, accumulated-into output).
template <int EPI>
constexpr bool kReads = EPI == EPI_BIAS_RES || EPI == EPI_GELU_BWD || EPI == EPI_WGRAD;
__device__ inline float4 load4(const float *p, int n, bool wide) {  // n of the four columns exist
  if (wide) return *reinterpret_cast<const float4 *>(p);
  return make_float4(p[0], n > 1 ? p[1] : 0.f, n > 2 ? p[2] : 0.f, n > 3 ? p[3] : 0.f);
}
__device__ inline void store4(float *p, const float4 v, int n, bool wide) {
  if (wide) {
    *reinterpret_cast<float4 *>(p) = v;
    return;
  }
  p[0] = v.x;
  if (n > 1) p[1] = v.y;
  if (n > 2) p[2] = v.z;
  if (n > 3) p[3] = v.w;
}
template <int EPI>
__device__ inline float4 load_extra(const GemmArgs &g, int row, int col, bool wide) {
  const float *in = EPI == EPI_BIAS_RES ? g.res : (EPI == EPI_GELU_BWD ? (const float *)g.aux : (const float *)g.C);
  if (!kReads<EPI> || (EPI == EPI_WGRAD && !g.beta) || row >= g.M || col >= g.N) return make_float4(0.f, 0.f, 0.f, 0.f);
  return load4(in + (size_t)(EPI == EPI_GELU_BWD ? row % g.aux_wrap : row) * g.ldc + col, g.N - col, wide);
}
template <int EPI>
__device__ inline void emit4(const GemmArgs &g, float4 v, const float4 x, const float4 bias, int row, int col, bool wide) {
  if (row >= g.M || col >= g.N) return;
  if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_GELU || EPI == EPI_BIAS_RES) {
    v.x += bias.x; v.y += bias.y; v.z += bias.z; v.w += bias.w;
  }
  if constexpr (EPI == EPI_BIAS_RES) {
    v.x += x.x; v.y += x.y; v.z += x.z; v.w += x.w;
  }
  if constexpr (EPI == EPI_GELU_BWD) {
    v.x *= gelu_grad_f(x.x); v.y *= gelu_grad_f(x.y); v.z *= gelu_grad_f(x.z); v.w *= gelu_grad_f(x.w);
  }
  if constexpr (EPI == EPI_WGRAD) {
    v.x = g.scale * v.x + x.x; v.y = g.scale * v.y + x.y; v.z = g.scale * v.z + x.z; v.w = g.scale * v.w + x.w;
  }
  const size_t o = (size_t)row * g.ldc + col;
  store4((float *)g.C + o, v, g.N - col, wide);
  if constexpr (EPI == EPI_BIAS_GELU)
    store4((float *)g.C2 + o, make_float4(gelu_f(v.x), gelu_f(v.y), gelu_f(v.z), gelu_f(v.w)), g.N - col, wide);
}

// Four multiplying wavefronts own a BM x BN tile in squares of 64 x 64: four squares of 128 x 128, two of 128 x 64, one
// of 64 x 64.  Wavefronts that share a square share out a K step in slices of 16 (an operand read from LDS then
// serves as many products as in the large tile), and their sums meet in LDS at the end.  Eight loader wavefronts fetch K
// steps ahead into registers, split them - every element once - and write the planes of step kt + 1 while step kt
// is multiplied; one barrier per step publishes them and retires the slot of step kt - 1.  A slice's operands are
// read while the slice before it is multiplied.
template <int BM, int BN>
struct Shape {
  static constexpr int WM = BM / 64, WN = BN / 64, KG = 4 / (WM * WN), BK = KG > 1 ? 64 : 32;
  static constexpr int SL = BK / 16 / KG;  // slices per wavefront and step
  static constexpr int STAGE = (BM + BN) * BK * 6, PITCH = BN + 8;
  static constexpr int RING = 2 * STAGE, SUMS = KG * BM * PITCH * 4, LDS = RING > SUMS ? RING : SUMS;
};
template <int BM, int BN, bool AKM, bool BKM, int LB, int MAX>
__global__ __launch_bounds__(256 + NL) __attribute__((amdgpu_waves_per_eu(3, 3))) void gemm_f32_kernel(Problems<MAX> batch) {
  typedef Shape<BM, BN> S;
  constexpr int WM = S::WM, WN = S::WN, KG = S::KG, SL = S::SL, BK = S::BK;
  typedef Tile<BM, AKM, BK, LB> TA;
  typedef Tile<BN, BKM, BK, LB> TB;
  static_assert(3 * (TA::PLANE + TB::PLANE) == S::STAGE, "stage");
  __shared__ __attribute__((aligned(1024))) char smem[S::LDS];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);

  int tile0;
  GemmArgs g = my_problem(batch, tile0);
  const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
  const MyTile mt = my_tile(g, blockIdx.x - tile0, tiles_m, tiles_n);
  const int m0 = mt.m * BM, n0 = mt.n * BN, kb0 = mt.k0, ke = mt.k1;
  const int nk = (ke - kb0 + BK - 1) / BK;

  float *sums = reinterpret_cast<float *>(smem);
  if (wave >= 4) {  // loader wavefronts
    const Rsrc ra = rsrc(g.A, g.a_bytes), rb = rsrc(g.B, g.b_bytes);
    TA la;
    TB lb;
    la.init(m0, g.M, g.lda, t - 256);
    lb.init(n0, g.N, g.ldb, t - 256);
    constexpr int D = kAhead;  // steps
    typename TA::Raw qa[D];
    typename TB::Raw qb[D];
    auto fetch = [&](int kt, int set) {  // (a step past the last reads as zero)
      la.load(ra, kb0 + kt * BK, ke, qa[set]);
      lb.load(rb, kb0 + kt * BK, ke, qb[set]);
    };
    auto publish = [&](int kt, int set) {
      char *st = smem + (kt & 1) * S::STAGE + (t - 256) * 16;
      u32x4 f[3];
#pragma unroll
      for (int i = 0; i < TA::NCH; ++i) {
        split8(qa[set].v[i], f);
#pragma unroll
        for (int k = 0; k < 3; ++k) *reinterpret_cast<u32x4 *>(st + k * TA::PLANE + i * NL * 16) = f[k];
      }
#pragma unroll
      for (int i = 0; i < TB::NCH; ++i) {
        split8(qb[set].v[i], f);
#pragma unroll
        for (int k = 0; k < 3; ++k) *reinterpret_cast<u32x4 *>(st + 3 * TA::PLANE + k * TB::PLANE + i * NL * 16) = f[k];
      }
    };
#pragma unroll
    for (int u = 0; u < D; ++u) fetch(u, u);
    __builtin_amdgcn_sched_barrier(0);
    publish(0, 0);
    fetch(D, 0);
    [&] {
      for (int kt = 0;;) {
#pragma unroll
        for (int u = 1; u <= D; ++u) {
          __syncthreads();
          if (++kt >= nk) return;
          publish(kt, u % D);
          fetch(kt + D, u % D);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }();
    __syncthreads();  // (every wavefront is done with the ring)
  } else {
    const int kg = wave / (WM * WN), wm = wave / WN % WM, wn = wave % WN;
    floatx16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    struct Operands { Split a[2], b[2]; };
    auto read = [&](int kt, int s) {
      const char *sa = smem + (kt & 1) * S::STAGE, *sb = sa + 3 * TA::PLANE;
      Operands o;
#pragma unroll
      for (int k = 2; k >= 0; --k)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          o.a[i].p[k] = TA::frag(sa + k * TA::PLANE, wm * 64 + 32 * i, kg * SL + s, lane);
          o.b[i].p[k] = TB::frag(sb + k * TB::PLANE, wn * 64 + 32 * i, kg * SL + s, lane);
        }
      return o;
    };
    auto products = [&](const Operands &o) {
      // all but mid lo, lo mid and lo lo, the small ones first
      constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
      for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o.a[i].p[PA[q]], o.b[j].p[PB[q]], acc[i][j], 0, 0, 0);
    };
    __syncthreads();
    Operands cur = read(0, 0);
    for (int kt = 0; kt < nk - 1; ++kt) {
#pragma unroll
      for (int s = 1; s < SL; ++s) {
        const Operands nxt = read(kt, s);
        products(cur);
        cur = nxt;
      }
      __syncthreads();
      const Operands nxt = read(kt + 1, 0);
      products(cur);
      cur = nxt;
    }
#pragma unroll
    for (int s = 1; s < SL; ++s) {
      const Operands nxt = read(nk - 1, s);
      products(cur);
      cur = nxt;
    }
    products(cur);

    // Infinities and values from 2^104 on split into NaN parts, and sums from 2^80 on overflow: what comes out not finite
    // is done again in fp32 products, straight from memory.
    float bad = 0.f, down = kDown;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) bad = __builtin_fmaf(acc[i][j][r], 0.f, bad);
    if (__any(!(bad == 0.f))) {
      down = 1.f;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
      for (int kt = 0; kt < nk; ++kt)
#pragma unroll 1
        for (int e = 0; e < 8 * SL; ++e) {
          const int k = kb0 + kt * BK + kg * SL * 16 + 2 * e + (lane >> 5);
          float a[2], b[2];
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const int m = m0 + wm * 64 + 32 * i + (lane & 31), n = n0 + wn * 64 + 32 * i + (lane & 31);
            a[i] = k < ke && m < g.M ? ((const float *)g.A)[AKM ? (size_t)k * g.lda + m : (size_t)m * g.lda + k] : 0.f;
            b[i] = k < ke && n < g.N ? ((const float *)g.B)[BKM ? (size_t)k * g.ldb + n : (size_t)n * g.ldb + k] : 0.f;
          }
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    }
    __syncthreads();  // every wavefront is done with the ring
    // a lane holds column lane & 31 and rows 8 (r / 4) + 4 (lane >> 5) + (r & 3) of each 32x32 block
    float *mine = sums + (kg * BM + wm * 64 + 4 * (lane >> 5)) * S::PITCH + wn * 64 + (lane & 31);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) mine[(32 * i + 8 * (r >> 2) + (r & 3)) * S::PITCH + 32 * j] = acc[i][j][r] * down;
  }

  // What the epilogue reads is requested for all of a thread's rows before the sums are there.
  constexpr int QPR = BN / 4, RPP = (256 + NL) / QPR, NQ = (BM + RPP - 1) / RPP;  // quads per row, rows per pass, passes
  const bool biased = g.epi == EPI_BIAS || g.epi == EPI_BIAS_GELU || g.epi == EPI_BIAS_RES;
  const bool wide = !((g.ldc | g.N) & 3) && !(((uintptr_t)g.C | (uintptr_t)g.C2 | (uintptr_t)g.bias | (uintptr_t)g.res | (uintptr_t)g.aux) & 15);
  const int row_l = t / QPR, col = n0 + t % QPR * 4;
  const float4 bias = biased && col < g.N ? load4((const float *)g.bias + col, g.N - col, wide) : make_float4(0.f, 0.f, 0.f, 0.f);
  auto finish = [&](auto epi) {
    constexpr int EPI = decltype(epi)::value;
    float4 x[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) x[q] = load_extra<EPI>(g, row_l + q * RPP < BM ? m0 + row_l + q * RPP : g.M, col, wide);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int row = row_l + q * RPP;
      if (row >= BM) break;
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int k = 0; k < KG; ++k) {
        const float4 p = *reinterpret_cast<const float4 *>(sums + (k * BM + row) * S::PITCH + t % QPR * 4);
        v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
      }
      emit4<EPI>(g, v, x[q], bias, m0 + row, col, wide);
    }
  };
  switch (g.epi) {  // (uniform)
    case EPI_BIAS: finish(std::integral_constant<int, EPI_BIAS>{}); break;
    case EPI_BIAS_GELU: finish(std::integral_constant<int, EPI_BIAS_GELU>{}); break;
    case EPI_BIAS_RES: finish(std::integral_constant<int, EPI_BIAS_RES>{}); break;
    case EPI_GELU_BWD: finish(std::integral_constant<int, EPI_GELU_BWD>{}); break;
    case EPI_WGRAD: finish(std::integral_constant<int, EPI_WGRAD>{}); break;
    default: finish(std::integral_constant<int, EPI_STORE>{}); break;
  }
}

template <int BM, int BN>
long tiles_of(const GemmArgs &g) {
  return (long)((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN) * std::max(g.splits, 1);
}
template <int BM, int BN, bool AKM, bool BKM, int LB>
hipError_t launch(GemmBatch &b, hipStream_t s) {
  return with_problems<AKM && BKM>(
      b.p, b.count, [](const GemmArgs &g) { return TileGrid{(g.M + BM - 1) / BM, (g.N + BN - 1) / BN, BM, BN}; },
      [&](const auto &problems, int tiles) {
        hipLaunchKernelGGL((gemm_f32_kernel<BM, BN, AKM, BKM, LB, std::decay_t<decltype(problems)>::kRoom>), dim3(tiles), dim3(256 + NL),
                           0, s, problems);
        return hipGetLastError();
      });
}

template <bool AKM, bool BKM>
hipError_t pick(GemmBatch &b, bool aligned, hipStream_t s) {
  if (!aligned) return launch<64, 64, AKM, BKM, 1>(b, s);
  long t64 = 0, t128x64 = 0, t128 = 0;
  int k = 0;
  for (int i = 0; i < b.count; ++i) {
    t64 += tiles_of<64, 64>(b.p[i]);
    t128x64 += tiles_of<128, 64>(b.p[i]);
    t128 += tiles_of<128, 128>(b.p[i]);
    k = std::max(k, b.p[i].splits > 1 ? b.p[i].k_per : b.p[i].K);
  }
  const long steps = (k + 63) / 64;
  const double us64 = gemm_f32_us(4, t64, steps), us128x64 = gemm_f32_us(3, t128x64, steps), us128 = gemm_f32_us(2, t128, steps);
  int tile = b.p[0].tile;
  if (!tile) tile = us128 <= std::min(us128x64, us64) ? 2 : us128x64 <= us64 ? 3 : 4;
  switch (tile) {
    case 2: return launch<128, 128, AKM, BKM, 4>(b, s);
    case 3: return launch<128, 64, AKM, BKM, 4>(b, s);
    default: return launch<64, 64, AKM, BKM, 4>(b, s);
  }
}

}  // namespace

// Rounds of workgroups, times what one takes: microseconds per 64 of K with the chip full, and about five for start
// and epilogue.  Measured (128x128 / 128x64 / 64x64): 2048x1536x512 24 / 30 / 31 us, 4096x512x2048 64 / 51 / 65,
// 2048x512x2048 - / 43 / 33, 1600x768x3072 87 / 62 / 85, 4096x2048x512 57 / 71 / 91.
double gemm_f32_us(int tile, long workgroups, long steps) {
  const double step_us = tile == 2 ? 2.6 : tile == 3 ? 1.45 : 0.9;
  return (double)((workgroups + 255) / 256) * (5.0 + steps * step_us);
}

hipError_t gemm_f32_batch(const GemmArgs *list, int count, hipStream_t s) {
  if (count < 1 || count > kMaxBatch) return hipErrorInvalidValue;
  GemmBatch b;
  memset(&b, 0, sizeof(b));
  b.count = count;
  bool aligned = true;
  for (int i = 0; i < count; ++i) {
    GemmArgs &g = b.p[i];
    g = list[i];
    if (g.a_kmajor != list[0].a_kmajor || g.b_kmajor != list[0].b_kmajor) return hipErrorInvalidValue;
    if (g.M <= 0 || g.N <= 0 || g.K <= 0 || g.epi < EPI_STORE || g.epi > EPI_WGRAD) return hipErrorInvalidValue;
    if (!split_ok(g)) return hipErrorInvalidValue;
    const size_t ab = (size_t)(g.a_kmajor ? g.K : g.M) * g.lda * 4, bb = (size_t)(g.b_kmajor ? g.K : g.N) * g.ldb * 4;
    if (ab >= 0x7FFFFFFFull || bb >= 0x7FFFFFFFull) return hipErrorInvalidValue;  // 32-bit buffer offsets
    g.a_bytes = (uint32_t)ab;
    g.b_bytes = (uint32_t)bb;
    aligned = aligned && !((g.lda | g.ldb | (g.a_kmajor ? g.M : g.K) | (g.b_kmajor ? g.N : g.K)) & 3) &&
              !(((uintptr_t)g.A | (uintptr_t)g.B) & 15);
  }
  switch (b.p[0].a_kmajor * 2 + b.p[0].b_kmajor) {
    case 0: return pick<false, false>(b, aligned, s);
    case 1: return pick<false, true>(b, aligned, s);
    case 2: return pick<true, false>(b, aligned, s);
    default: return pick<true, true>(b, aligned, s);
  }
}

hipError_t gemm_f32(const GemmArgs &g, hipStream_t s) { return gemm_f32_batch(&g, 1, s); }

}  // namespace il
