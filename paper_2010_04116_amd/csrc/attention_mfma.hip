// Causal attention forward / backward on the gfx950 matrix cores for bf16 and head
// widths 64, 128 and 256.  K/V (forward, dQ) or Q/dO (dK, dV) tiles are LDS-resident, double
// buffered and filled by direct HBM -> LDS loads; scores are never written to memory.
//
// Orientation.  Scores are computed transposed, S^T = K Q^T, with v_mfma_f32_32x32x16_bf16:
// a lane then owns ONE query column (lane & 31) and holds 16 key rows per 32x32 tile in its
// accumulator registers.  Row max / row sum of the softmax are therefore in-register
// reductions plus one exchange with lane ^ 32, and the probabilities go straight from the
// accumulators into the B operand of the second product O^T = V^T P^T without touching LDS:
// the MFMA's k index is only a summation label, so the key order a lane happens to hold
// (rows 4h..4h+3 and 8+4h..8+4h+3 of each 16-key group, h = lane >> 5) is used as is and the
// A operand V^T is fetched in the same order from the [key][dh] tile with the LDS transposing
// read (each source lane may point at any row, so no transposed copy is staged).
//
// The backward recomputes the probabilities from the saved log-sum-exp (kept in powers of two) with
// fixed reduction order (no atomics): some workgroups own a key/value tile and accumulate dK, dV over
// the query tiles at or below the diagonal, the others own a query tile and accumulate dQ.  All of
// them share one launch: the row sums dO.O that both need arrive with dO, from the epilogue of the
// GEMM that produces it (in 32-column pieces, summed here).
#include "common.h"
#include "lds_dma.h"
#include <type_traits>

namespace il {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short short4v;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kNegBig = -1.0e30f;
constexpr int kStages = 2;  // staged tiles (a third was no faster forward and 5 % slower backward)
constexpr floatx16 kZero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

__device__ inline uint4 ldg16(const bf16_t *p) { return *reinterpret_cast<const uint4 *>(p); }
__device__ inline uint32_t pack2(float a, float b) {
  return pack_bf16x2(a, b);
}
union Frag {
  bf16x8 v;
  uint4 q;
  uint2 h[2];
  uint32_t u[4];
  short4v s[2];
};

// A [ROWS tokens] x [DH] tile of a token-major matrix, staged as is ([token][dh]) by direct
// loads (NT threads, 16 bytes each per round).  The 16-byte chunk c of row r sits at chunk
// position c ^ h(r).  LDS has 64 banks of 4 bytes: a ds_read_b128 serves 16 lanes (16 rows x 16
// bytes) per cycle and a transposing ds_read_b64_tr_b16 32 lanes (4 rows x 64 bytes), so h must
// send 16 consecutive rows to 16 different 16-byte positions of the 256-byte bank span and 4
// consecutive rows to 4 different 64-byte quarters of it.  Rows of 256 bytes or more all start at
// bank 0: h(r) = (r & 3) << 2 | (r >> 2) & 3.  Rows of 128 bytes alternate between the two halves
// of the span by themselves (bit 0 of r): h(r) = bit 1 of r << 2 | bit 2 << 1 | bit 3.  (With the
// earlier three-bit h(r) = (r & 3) << 1 | (r >> 2) & 1 the LDS counters showed every second cycle
// of these kernels' LDS activity as a bank conflict.)
template <int ROWS, int DH, int NT = 256>
struct TokTile {
  static constexpr int RB = DH * 2, CPR = DH / 8, BYTES = ROWS * RB, NLD = BYTES / (NT * 16);
  static_assert(BYTES % (NT * 16) == 0 && NLD >= 1, "a tile divides over the threads");
  uint32_t voff[NLD];
  int radd[NLD];
  uint32_t rstride;
  __device__ static inline int h(int r) {
    if constexpr (DH >= 128) return ((r & 3) << 2) | ((r >> 2) & 3);
    return (((r >> 1) & 1) << 2) | (((r >> 2) & 1) << 1) | ((r >> 3) & 1);
  }
  // col0: first element column of this head; ld: elements per token row
  __device__ inline void init(int col0, int ld, int t) {
    rstride = (uint32_t)ld * 2u;
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int p = i * NT + t, row = p / CPR, chunk = (p % CPR) ^ h(row);
      radd[i] = row;
      voff[i] = ((uint32_t)row * ld + col0 + chunk * 8) * 2u;
    }
  }
  // rows [row0, row0 + ROWS) of the matrix; rows >= row_end read as zero
  __device__ inline void issue(BufRsrc rs, char *lds, int wave, int row0, int row_end) const {
    const uint32_t adv = (uint32_t)row0 * rstride;
    const uint32_t base = lds_address(lds) + wave * 1024;
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const bool ok = row0 + radd[i] < row_end;
      dma16(rs, base + i * NT * 16, ok ? voff[i] + adv : kOob);
    }
  }
  // MFMA operand with the tile's rows as matrix rows and dh as k: rows rbase + (lane & 31),
  // dh slice [16 ks, 16 ks + 16)
  __device__ static inline bf16x8 rowfrag(const char *lds, int rbase, int ks, int lane) {
    const int row = rbase + (lane & 31), chunk = 2 * ks + (lane >> 5);
    return *reinterpret_cast<const bf16x8 *>(lds + row * RB + ((chunk ^ h(row)) << 4));
  }
  // MFMA A operand with dh as matrix rows (dt*32 + (lane & 31)) and 16 tokens as k, in the
  // order a lane holds them in a 32x32 accumulator: tokens tok0 + 4h + (0..3), tok0 + 8 + 4h + (0..3).
  __device__ static inline bf16x8 trfrag(const char *lds, int tok0, int dt, int lane) {
    const int g16 = lane >> 4, i = lane & 15;
    const int dcol = dt * 32 + 16 * (g16 & 1) + 4 * (i & 3);
    const int row = tok0 + 4 * (g16 >> 1) + (i >> 2);
    const int sub = ((dcol >> 2) & 1) * 8;
    Frag f;
    f.s[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v *)(
        lds + row * RB + (((dcol >> 3) ^ h(row)) << 4) + sub));
    f.s[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v *)(
        lds + (row + 8) * RB + (((dcol >> 3) ^ h(row + 8)) << 4) + sub));
    return f.v;
  }
  // The same two with one byte offset per lane for all fragments, where registers are short: a dh slice, a dh block
  // and the 8 rows between a fragment's halves are constants exclusive-or'd into the swizzled chunk, and tiles,
  // stages and row blocks constants added (they and RB are multiples of the span the exclusive-or reaches).
  __device__ static inline uint32_t row_offset(int lane) {
    const int row = lane & 31;
    return row * RB + (((lane >> 5) ^ h(row)) << 4);
  }
  __device__ static inline bf16x8 rowfrag_at(const char *lds, uint32_t off, int ks, int add) {
    return *reinterpret_cast<const bf16x8 *>(lds + (off ^ (uint32_t)(ks << 5)) + add);
  }
  __device__ static inline uint32_t tr_offset(int lane) {
    const int g16 = lane >> 4, i = lane & 15, row = 4 * (g16 >> 1) + (i >> 2), dcol = 16 * (g16 & 1) + 4 * (i & 3);
    return row * RB + (((dcol >> 3) ^ h(row)) << 4) + ((dcol >> 2) & 1) * 8;
  }
  __device__ static inline bf16x8 trfrag_at(const char *lds, uint32_t off, int dt, int add) {
    constexpr uint32_t kHalf = (uint32_t)(DH >= 128 ? 2 : 1) << 4;  // h(row) ^ h(row + 8), row < 8
    Frag f;
    f.s[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) short4v *)(lds + (off ^ (uint32_t)(dt << 6)) + add));
    f.s[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) short4v *)(lds + (off ^ (uint32_t)(dt << 6) ^ kHalf) + add + 8 * RB));
    return f.v;
  }
};


// Which causal tile a workgroup takes.  Tiles differ in length (rank 0 = longest, rank nx-1 =
// shortest, lengths in the ratio nx : nx-1 : ... : 1) while the hardware hands workgroups to the
// chip's 8 XCDs round-robin by linear id and, inside an XCD, to its 32 CUs round-robin - the
// natural (x, y) order would give one XCD all the longest tiles and put two of them on each of
// its CUs.  Here every XCD receives the same mix of lengths, the 32 workgroups that start first
// on an XCD are its longest and the 32 that join them on the same CUs its shortest, in opposite
// order, so the two workgroups that share a CU add up to the same work everywhere; later rounds
// likewise.  Only the assignment of work to workgroups changes, never the result.
struct CausalTile {
  int rank, y;
};
__device__ inline CausalTile causal_tile() {
  const int nx = gridDim.x, ny = gridDim.y;
  const int L = blockIdx.x + nx * blockIdx.y;
  if ((ny & 7) != 0) return {(int)blockIdx.x, (int)blockIdx.y};
  const int j = L & 7, s = L >> 3, c = ny >> 3, P = nx * c;  // XCD, slot in the XCD, tiles per length and per XCD
  const int full = P & ~63, rho = s >> 6, w = s & 63;
  int i;  // position in the XCD's list of tiles sorted by decreasing length
  if (s < full)
    i = w < 32 ? 32 * rho + w : P - 1 - (32 * rho + (w - 32));
  else
    i = (full >> 1) + (s - full);
  return {i / c, j + 8 * (i % c)};
}

// ------------------------------------------------------------------ forward -------------
// grid (ceil(T / 32 NW), B*H); NW wavefronts, each owns 32 queries; key tiles of 64.
template <int DH, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(DH > 128 ? 1 : 2, DH > 128 ? 1 : 2))) void
attn_fwd_mfma(const bf16_t *__restrict__ qkv, int T, int H, bf16_t *__restrict__ o, float *__restrict__ lse) {
  constexpr int BQ = 32 * NW, BKV = DH > 128 ? 32 : 64, NA = BKV / 32;
  constexpr bool HOIST = DH <= 64;  // the wider head has no registers to spare for a whole tile of fragments
  constexpr int KT = BKV * DH * 2, STAGE = 2 * KT;
  typedef TokTile<BKV, DH, 64 * NW> Tile;
  __shared__ __attribute__((aligned(16))) char smem[kStages * STAGE];
  const int t = threadIdx.x, lane = t & 63, hh = lane >> 5, lq = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const CausalTile ct = causal_tile();
  const int qt = gridDim.x - 1 - ct.rank;  // the last query tile is the longest
  const int b = ct.y / H, h = ct.y % H;
  const int d = H * DH;
  const size_t ld3 = 3 * (size_t)d;
  const bf16_t *qbase = qkv + (size_t)b * T * ld3 + h * DH;
  const int q0 = qt * BQ, qw0 = q0 + 32 * wave, q = qw0 + lq;
  const int kv_end = min(T, q0 + BQ);
  const int nkv = (kv_end + BKV - 1) / BKV;

  const BufRsrc rs = make_rsrc(qbase, (size_t)T * ld3 * 2 - (size_t)h * DH * 2);
  Tile lk, lv;
  lk.init(d, (int)ld3, t);
  lv.init(2 * d, (int)ld3, t);
  // tile kt goes to slot kt % kStages; a tile past the last one loads zeros, so the load counts hold
  auto issue = [&](int kt) {
    char *st = smem + (kt % kStages) * STAGE;
    const int end = kt < nkv ? T : 0;
    lk.issue(rs, st, wave, kt * BKV, end);
    lv.issue(rs, st + KT, wave, kt * BKV, end);
  };
#pragma unroll
  for (int s = 0; s < kStages - 1; ++s) issue(s);

  Frag qf[DH / 16];
#pragma unroll
  for (int ks = 0; ks < DH / 16; ++ks)
    qf[ks].q = (q < T) ? ldg16(qbase + (size_t)q * ld3 + 16 * ks + 8 * hh) : make_uint4(0, 0, 0, 0);

  floatx16 oacc[DH / 32];
#pragma unroll
  for (int i = 0; i < DH / 32; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[i][r] = 0.f;
  float m = kNegBig, l = 0.f;  // running maximum of the scaled scores, in powers of two
  const float sc = rsqrtf((float)DH) * kLog2e;

  for (int kt = 0; kt < nkv; ++kt) {
    const char *sk = smem + (kt % kStages) * STAGE, *sv = sk + KT;
    const int kv0 = kt * BKV;
    wait_vmcnt<0>();
    __syncthreads();  // tile kt is complete; every wavefront is done with tile kt-1
    const bool live = kv0 <= qw0 + 31;  // some key of the tile is visible to some query of this wavefront
    bf16x8 kf[HOIST ? NA : 1][HOIST ? DH / 16 : 1], vf[HOIST ? NA : 1][2][HOIST ? DH / 32 : 1];
    if constexpr (HOIST) {  // every fragment of the tile is requested ahead of the next loads
      if (live) {
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
          for (int ks = 0; ks < DH / 16; ++ks) kf[a][ks] = Tile::rowfrag(sk, 32 * a, ks, lane);
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
          for (int bq = 0; bq < 2; ++bq)
#pragma unroll
            for (int dt = 0; dt < DH / 32; ++dt) vf[a][bq][dt] = Tile::trfrag(sv, 32 * a + 16 * bq, dt, lane);
      }
    }
    issue(kt + kStages - 1);
    if (!live) continue;
    floatx16 s[NA];
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      s[a] = kZero16;
#pragma unroll
      for (int ks = 0; ks < DH / 16; ++ks)
        s[a] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            HOIST ? kf[HOIST ? a : 0][HOIST ? ks : 0] : Tile::rowfrag(sk, 32 * a, ks, lane), qf[ks].v, s[a], 0, 0, 0);
    }
    float mx = kNegBig;
    // the causal / end-of-sequence mask is compiled into the diagonal tiles' path only
    auto mask_max = [&](auto masked) {
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          if constexpr (decltype(masked)::value) {
            const int kv = kv0 + 32 * a + 8 * (r >> 2) + 4 * hh + (r & 3);
            s[a][r] = ((kv > q) | (kv >= T)) ? kNegBig : s[a][r];
          }
          mx = fmaxf(mx, s[a][r]);
        }
    };
    if (DH > 128 || kv0 + BKV - 1 > qw0 || kv0 + BKV > T)  // (at 256 a second copy of the loop costs more in registers than it saves)
      mask_max(std::true_type{});
    else
      mask_max(std::false_type{});
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mnew = fmaxf(m, mx * sc);
    const float alpha = __builtin_amdgcn_exp2f(m - mnew);
    float rsum = 0.f;
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[a][r], sc, -mnew));
        s[a][r] = p;
        rsum += p;
      }
    l = l * alpha + rsum;
    m = mnew;
#pragma unroll
    for (int i = 0; i < DH / 32; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[i][r] *= alpha;
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int bq = 0; bq < 2; ++bq) {
        Frag pf;
#pragma unroll
        for (int e = 0; e < 4; ++e) pf.u[e] = pack2(s[a][8 * bq + 2 * e], s[a][8 * bq + 2 * e + 1]);
#pragma unroll
        for (int dt = 0; dt < DH / 32; ++dt)
          oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              HOIST ? vf[HOIST ? a : 0][bq][HOIST ? dt : 0] : Tile::trfrag(sv, 32 * a + 16 * bq, dt, lane), pf.v,
              oacc[dt], 0, 0, 0);
      }
  }
  wait_vmcnt<0>();  // (the zeros of the tiles past the end)

  l += __shfl_xor(l, 32, 64);
  if (q < T) {
    const float inv = 1.f / l;
    bf16_t *op = o + ((size_t)b * T + q) * d + h * DH;
#pragma unroll
    for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        uint2 v;
        v.x = pack2(oacc[dt][4 * g] * inv, oacc[dt][4 * g + 1] * inv);
        v.y = pack2(oacc[dt][4 * g + 2] * inv, oacc[dt][4 * g + 3] * inv);
        *reinterpret_cast<uint2 *>(op + dt * 32 + 8 * g + 4 * hh) = v;
      }
    if (hh == 0) lse[((size_t)b * H + h) * T + q] = m + log2f(l);
  }
}

// Row sums dO.O of one head, from the 32-column pieces [d / 32][rows] that came with dO.
template <int DH>
__device__ inline float dsum_of(const float *pieces, size_t rows, size_t row, int h) {
  float s = 0.f;
#pragma unroll
  for (int p = 0; p < DH / 32; ++p) s += pieces[(size_t)(h * (DH / 32) + p) * rows + row];
  return s;
}

// The same value, which the compiler takes for a new one: what is derived from it in a loop is not kept across it.
__device__ inline uint32_t here(uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(v));
#endif
  return v;
}

// The bytes a stage of the dK / dV part holds: Q and each stream's dO as stored, lse and each stream's dsum.
template <int DH>
constexpr int dkv_stage(int streams) { return (1 + streams) * (64 * DH * 2 + 64 * 4); }

// ------------------------------------------------------------------ backward: dQ --------
// Same walk as the forward, for NS streams from sidx on: they share K, V, the scores and the probabilities.
template <int DH, int NS>
__device__ __forceinline__ void attn_bwd_dq_body(const bf16_t *__restrict__ qkv, const bf16_t *__restrict__ d_o,
                                                 const float *__restrict__ lse, const float *__restrict__ dsum, int B,
                                                 int T, int H, int ns, int sidx, bf16_t *__restrict__ dqkv, char *smem) {
  constexpr int BQ = 128, BKV = 64;
  constexpr int KT = BKV * DH * 2, STAGE = 2 * KT;  // K and V tiles as stored
  typedef TokTile<BKV, DH> Tile;
  const int t = threadIdx.x, lane = t & 63, hh = lane >> 5, lq = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const CausalTile ct = causal_tile();
  const int qt = gridDim.x - 1 - ct.rank;
  const int b = ct.y / H, h = ct.y % H;
  const int d = H * DH;
  const size_t ld3 = 3 * (size_t)d, N = (size_t)B * T;
  const bf16_t *qbase = qkv + (size_t)b * T * ld3 + h * DH;
  const int q0 = qt * BQ, qw0 = q0 + 32 * wave, q = qw0 + lq;
  const int kv_end = min(T, q0 + BQ);
  const int nkv = (kv_end + BKV - 1) / BKV;
  const size_t tok = (size_t)b * T + q;

  const BufRsrc rs = make_rsrc(qbase, (size_t)T * ld3 * 2 - (size_t)h * DH * 2);
  Tile lk, lv;
  lk.init(d, (int)ld3, t);
  lv.init(2 * d, (int)ld3, t);
  auto issue = [&](int kt) {  // (past the last tile: zeros)
    char *st = smem + (kt % kStages) * STAGE;
    const int end = kt < nkv ? T : 0;
    lk.issue(rs, st, wave, kt * BKV, end);
    lv.issue(rs, st + KT, wave, kt * BKV, end);
  };
#pragma unroll
  for (int s = 0; s < kStages - 1; ++s) issue(s);

  Frag qf[DH / 16], gf[NS][DH / 16];
#pragma unroll
  for (int ks = 0; ks < DH / 16; ++ks) {
    if (q < T) {
      qf[ks].q = ldg16(qbase + (size_t)q * ld3 + 16 * ks + 8 * hh);
#pragma unroll
      for (int st = 0; st < NS; ++st)
        gf[st][ks].q = ldg16(d_o + ((sidx + st) * N + tok) * d + h * DH + 16 * ks + 8 * hh);
    } else {
      qf[ks].q = make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int st = 0; st < NS; ++st) gf[st][ks].q = make_uint4(0, 0, 0, 0);
    }
  }
  const float sc = rsqrtf((float)DH), sc2 = sc * kLog2e;
  const float l2 = (q < T) ? lse[((size_t)b * H + h) * T + q] : 0.f;
  float dsv[NS];
  floatx16 dq[NS][DH / 32];
#pragma unroll
  for (int st = 0; st < NS; ++st) {
    dsv[st] = (q < T) ? dsum_of<DH>(dsum, ns * N, (sidx + st) * N + tok, h) : 0.f;
#pragma unroll
    for (int i = 0; i < DH / 32; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) dq[st][i][r] = 0.f;
  }

  for (int kt = 0; kt < nkv; ++kt) {
    const char *sk = smem + (kt % kStages) * STAGE, *sv = sk + KT;
    const int kv0 = kt * BKV;
    wait_vmcnt<0>();
    __syncthreads();
    issue(kt + kStages - 1);
    if (kv0 <= qw0 + 31) {
      const bool diag = kv0 + BKV - 1 > qw0 || kv0 + BKV > T;
#pragma unroll(DH > 64 || NS > 1 ? 1 : 2)
      for (int a = 0; a < 2; ++a) {
        floatx16 s = kZero16, dp[NS];  // a constant accumulator input costs no registers to clear
#pragma unroll
        for (int st = 0; st < NS; ++st) dp[st] = kZero16;
#pragma unroll
        for (int ks = 0; ks < DH / 16; ++ks) {
          const bf16x8 kf = Tile::rowfrag(sk, 32 * a, ks, lane);
          const bf16x8 vf = Tile::rowfrag(sv, 32 * a, ks, lane);
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks].v, s, 0, 0, 0);
#pragma unroll
          for (int st = 0; st < NS; ++st)
            dp[st] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, gf[st][ks].v, dp[st], 0, 0, 0);
        }
        auto probs = [&](auto masked) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], sc2, -l2));
            if constexpr (decltype(masked)::value) {
              const int kv = kv0 + 32 * a + 8 * (r >> 2) + 4 * hh + (r & 3);
              p = ((kv > q) | (kv >= T)) ? 0.f : p;
            }
#pragma unroll
            for (int st = 0; st < NS; ++st) dp[st][r] = p * (dp[st][r] - dsv[st]);  // dS^T, without the scale
          }
        };
        if (DH > 128 || diag)
          probs(std::true_type{});
        else
          probs(std::false_type{});
#pragma unroll
        for (int bq = 0; bq < 2; ++bq) {
          Frag pf[NS];
#pragma unroll
          for (int st = 0; st < NS; ++st)
#pragma unroll
            for (int e = 0; e < 4; ++e) pf[st].u[e] = pack2(dp[st][8 * bq + 2 * e], dp[st][8 * bq + 2 * e + 1]);
#pragma unroll
          for (int dt = 0; dt < DH / 32; ++dt) {
            const bf16x8 kf = Tile::trfrag(sk, 32 * a + 16 * bq, dt, lane);
#pragma unroll
            for (int st = 0; st < NS; ++st)
              dq[st][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, pf[st].v, dq[st][dt], 0, 0, 0);
          }
        }
      }
    }
  }
  wait_vmcnt<0>();
  if (q < T) {
#pragma unroll
    for (int st = 0; st < NS; ++st) {
      bf16_t *op = dqkv + ((sidx + st) * N + tok) * ld3 + h * DH;
#pragma unroll
      for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          uint2 v;
          v.x = pack2(dq[st][dt][4 * g] * sc, dq[st][dt][4 * g + 1] * sc);
          v.y = pack2(dq[st][dt][4 * g + 2] * sc, dq[st][dt][4 * g + 3] * sc);
          *reinterpret_cast<uint2 *>(op + dt * 32 + 8 * g + 4 * hh) = v;
        }
    }
  }
}

// ------------------------------------------------------------------ backward: dK, dV ----
// 4 wavefronts, each owns
// 32 keys (a lane owns one key column); query tiles of 64 from the diagonal to the end of the
// sequence.  Scores are computed as S = Q K^T with the query index in the accumulator rows, so P
// and dS feed the products dV^T = dO^T P and dK^T = Q^T dS directly from registers.
// WHAT: 0 = dK and dV in one pass; 1 = dV only; 2 = dK only.  At head width 128 the one-pass form
// holds 64 registers of K / V fragments and 128 of accumulators: it does not fit the 256
// architectural registers, runs one wavefront per SIMD and pays accumulation-register moves.  Split
// into a dV pass (K fragments, 64 accumulator registers) and a dK pass (K and V fragments, 64
// accumulator registers), both fit with two wavefronts per SIMD; the score product is computed in
// both (40 matrix instructions per 32x32 sub-tile instead of 32), which the kernel - bound by
// latency, not by the matrix unit - more than wins back.  NS streams from sidx on share Q, the scores and
// the probabilities.
template <int DH, int WHAT, int NS>
__device__ __forceinline__ void attn_bwd_dkv_body(const bf16_t *__restrict__ qkv, const bf16_t *__restrict__ d_o,
                                                  const float *__restrict__ lse, const float *__restrict__ dsum, int B,
                                                  int T, int H, int ns, int sidx, bf16_t *__restrict__ dqkv,
                                                  char *smem) {
  constexpr bool DO_DV = WHAT != 2, DO_DK = WHAT != 1;
  constexpr int BKV = 128, BQ = 64;
  constexpr int QT = BQ * DH * 2;                 // one staged tile
  constexpr int STAGE = dkv_stage<DH>(NS);
  typedef TokTile<BQ, DH> Tile;
  const int t = threadIdx.x, lane = t & 63, hh = lane >> 5, lk_ = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const CausalTile ct = causal_tile();  // the first key tile is the longest
  const int b = ct.y / H, h = ct.y % H;
  const int d = H * DH;
  const size_t ld3 = 3 * (size_t)d, N = (size_t)B * T;
  const bf16_t *qbase = qkv + (size_t)b * T * ld3 + h * DH;
  const bf16_t *kbase = qbase + d, *vbase = qbase + 2 * d;
  const float *lrow = lse + ((size_t)b * H + h) * T;
  const int kv0 = ct.rank * BKV, kvw0 = kv0 + 32 * wave, kv = kvw0 + lk_;
  const int qt0 = kv0 / BQ, nqt = (T + BQ - 1) / BQ;

  Frag kf[DH / 16], vf[DO_DK ? DH / 16 : 1];
#pragma unroll
  for (int ks = 0; ks < DH / 16; ++ks) {
    if (kv < T) {
      kf[ks].q = ldg16(kbase + (size_t)kv * ld3 + 16 * ks + 8 * hh);
      if constexpr (DO_DK) vf[ks].q = ldg16(vbase + (size_t)kv * ld3 + 16 * ks + 8 * hh);
    } else {
      kf[ks].q = make_uint4(0, 0, 0, 0);
      if constexpr (DO_DK) vf[ks].q = make_uint4(0, 0, 0, 0);
    }
  }
  floatx16 dk[NS][DO_DK ? DH / 32 : 1], dv[NS][DO_DV ? DH / 32 : 1];
#pragma unroll
  for (int st = 0; st < NS; ++st)
#pragma unroll
    for (int i = 0; i < DH / 32; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if constexpr (DO_DK) dk[st][i][r] = 0.f;
        if constexpr (DO_DV) dv[st][i][r] = 0.f;
      }
  const float sc = rsqrtf((float)DH);
  const float sc2 = sc * kLog2e;

  const BufRsrc rq = make_rsrc(qbase, (size_t)T * ld3 * 2 - (size_t)h * DH * 2);
  BufRsrc rg[NS];
#pragma unroll
  for (int st = 0; st < NS; ++st)
    rg[st] = make_rsrc(d_o + ((sidx + st) * N + (size_t)b * T) * d + h * DH, (size_t)T * d * 2 - (size_t)h * DH * 2);
  Tile lq, lg;
  lq.init(0, (int)ld3, t);
  lg.init(0, d, t);
  // Direct loads of the Q and dO tiles, kStages - 1 tiles ahead (past the last tile: zeros); the 64 lse and
  // dsum values of a tile go through registers, one tile ahead: wavefront 0 fetches lse, wavefront 1 + st dsum.
  auto issue = [&](int it) {
    char *base = smem + (it % kStages) * STAGE;
    const int r0 = (qt0 + it) * BQ, end = qt0 + it < nqt ? T : 0;
    lq.issue(rq, base, wave, r0, end);
#pragma unroll
    for (int st = 0; st < NS; ++st) lg.issue(rg[st], base + (1 + st) * QT, wave, r0, end);
  };
  float row_val = 0.f;
  auto fetch_rows = [&](int it) {
    const int r = (qt0 + it) * BQ + lane;
    row_val = 0.f;
    if (r < T && wave == 0) row_val = lrow[r];
    if (DO_DK && r < T && wave >= 1 && wave <= NS)
      row_val = dsum_of<DH>(dsum, ns * N, (sidx + wave - 1) * N + (size_t)b * T + r, h);
  };
  auto put_rows = [&](int it) {
    float *row = reinterpret_cast<float *>(smem + (it % kStages) * STAGE + (1 + NS) * QT);
    if (wave < 1 + NS) row[wave * BQ + lane] = row_val;
  };
  const int nit = nqt - qt0;
  const uint32_t row_off = Tile::row_offset(lane), tr_off = Tile::tr_offset(lane);
  fetch_rows(0);
#pragma unroll
  for (int s = 0; s < kStages - 1; ++s) issue(s);
  put_rows(0);

  for (int it = 0; it < nit; ++it) {
    const int qt = qt0 + it;
    const char *sq = smem + (it % kStages) * STAGE;
    const float *sl = reinterpret_cast<const float *>(sq + (1 + NS) * QT), *sd = sl + BQ;
    const int qb0 = qt * BQ;
    wait_vmcnt<0>();
    __syncthreads();
    fetch_rows(it + 1);
    issue(it + kStages - 1);
#pragma unroll(DH > 64 || NS > 1 ? 1 : 2)
    for (int a = 0; a < BQ / 32; ++a) {
      const int qa0 = qb0 + 32 * a;
      if (qa0 + 31 < kvw0 || qa0 >= T) continue;  // every query of the sub-tile precedes every key
      // (two streams' accumulators leave room for two of the fragments' addresses, and not for the eight that would
      // be kept across the loop: those came back from scratch, each behind a wait for the direct loads in flight)
      uint32_t ro = 0, to = 0;
      if constexpr (NS > 1) {
        ro = here(row_off + (it % kStages) * STAGE + 32 * a * Tile::RB);
        to = here(tr_off + (it % kStages) * STAGE + 32 * a * Tile::RB);
      }
      auto rows = [&](int tile, int ks) {
        if constexpr (NS > 1) return Tile::rowfrag_at(smem, ro, ks, tile * QT);
        return Tile::rowfrag(sq + tile * QT, 32 * a, ks, lane);
      };
      auto trans = [&](int tile, int bq, int dt) {
        if constexpr (NS > 1) return Tile::trfrag_at(smem, to, dt, tile * QT + 16 * bq * Tile::RB);
        return Tile::trfrag(sq + tile * QT, 32 * a + 16 * bq, dt, lane);
      };
      floatx16 s = kZero16, dp = kZero16;
#pragma unroll
      for (int ks = 0; ks < DH / 16; ++ks) {
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rows(0, ks), kf[ks].v, s, 0, 0, 0);
        if constexpr (DO_DK)
          dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rows(1, ks), vf[ks].v, dp, 0, 0, 0);
      }
      const bool diag = qa0 < kvw0 + 31 || qa0 + 32 > T;
      Frag pf[2], sf[2];  // P and dS of the sub-tile, packed to bf16 as they are produced
      auto grads = [&](int st, int g, const float (&p4)[4]) {  // dS of stream st from its dO V^T, four rows
        const float4 d4 = *reinterpret_cast<const float4 *>(sd + st * BQ + 32 * a + 8 * g + 4 * hh);
        const float dv4[4] = {d4.x, d4.y, d4.z, d4.w};
        float s4[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) s4[e] = p4[e] * (dp[4 * g + e] - dv4[e]);  // without the scale
        sf[g >> 1].u[2 * (g & 1)] = pack2(s4[0], s4[1]);
        sf[g >> 1].u[2 * (g & 1) + 1] = pack2(s4[2], s4[3]);
      };
      auto probs = [&](auto masked) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float4 l4 = *reinterpret_cast<const float4 *>(sl + 32 * a + 8 * g + 4 * hh);
          const float lv4[4] = {l4.x, l4.y, l4.z, l4.w};
          float p4[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int r = 4 * g + e;
            float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], sc2, -lv4[e]));
            if constexpr (decltype(masked)::value) {
              const int qq = qa0 + 8 * g + 4 * hh + e;
              p = ((kv > qq) | (qq >= T)) ? 0.f : p;
            }
            p4[e] = p;
            if constexpr (NS > 1) s[r] = p;
          }
          if constexpr (DO_DV) {
            pf[g >> 1].u[2 * (g & 1)] = pack2(p4[0], p4[1]);
            pf[g >> 1].u[2 * (g & 1) + 1] = pack2(p4[2], p4[3]);
          }
          if constexpr (DO_DK) grads(0, g, p4);
        }
      };
      if (DH > 128 || diag)
        probs(std::true_type{});
      else
        probs(std::false_type{});
#pragma unroll
      for (int st = 0; st < NS; ++st) {
        if (DO_DK && st > 0) {
          dp = kZero16;
#pragma unroll
          for (int ks = 0; ks < DH / 16; ++ks)
            dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rows(1 + st, ks),
                                                         vf[DO_DK ? ks : 0].v, dp, 0, 0, 0);
#pragma unroll
          for (int g = 0; g < 4; ++g) grads(st, g, {s[4 * g], s[4 * g + 1], s[4 * g + 2], s[4 * g + 3]});
        }
#pragma unroll
        for (int bq = 0; bq < 2; ++bq) {
#pragma unroll
          for (int dt = 0; dt < DH / 32; ++dt) {
            if constexpr (DO_DV)
              dv[st][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                  trans(1 + st, bq, dt), pf[bq].v, dv[st][dt], 0, 0, 0);
            if constexpr (DO_DK)
              dk[st][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(trans(0, bq, dt),
                                                                   sf[bq].v, dk[st][dt], 0, 0, 0);
          }
        }
      }
    }
    if (it + 1 < nit) put_rows(it + 1);
  }
  wait_vmcnt<0>();
  if (kv < T) {
#pragma unroll
    for (int st = 0; st < NS; ++st) {
      bf16_t *kp = dqkv + ((sidx + st) * N + (size_t)b * T + kv) * ld3 + d + h * DH;
#pragma unroll
      for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          uint2 v;
          if constexpr (DO_DK) {
            v.x = pack2(dk[st][dt][4 * g] * sc, dk[st][dt][4 * g + 1] * sc);
            v.y = pack2(dk[st][dt][4 * g + 2] * sc, dk[st][dt][4 * g + 3] * sc);
            *reinterpret_cast<uint2 *>(kp + dt * 32 + 8 * g + 4 * hh) = v;
          }
          if constexpr (DO_DV) {
            v.x = pack2(dv[st][dt][4 * g], dv[st][dt][4 * g + 1]);
            v.y = pack2(dv[st][dt][4 * g + 2], dv[st][dt][4 * g + 3]);
            *reinterpret_cast<uint2 *>(kp + d + dt * 32 + 8 * g + 4 * hh) = v;
          }
        }
    }
  }
}

// The backward of all streams in one launch, grid (ceil(T/128), B*H, roles * groups of NS streams): blockIdx.z % roles
// selects what a workgroup computes, the longest role first - dK and dV, dQ; or (head width 128) dK, dQ, dV.
// With at least two wavefronts per SIMD demanded, the register budget is the 256 architectural VGPRs and the
// compiler keeps the MFMA accumulators there; without, it places them in the accumulation registers and
// moves every score to a VGPR and back (a third of the vector instructions at head width 64).  Head width
// 256 does not fit that budget (256 + 256 registers and 16 bytes of scratch, dK / dV's need, also for dQ, which
// alone takes 232 + 160); two launches are slower all the same: 32 x 128 tokens, 4 heads 45.2 us against 26.8, two
// streams 49.5 against 45.7, 4 x 512, 8 heads 100.6 against 60.4.
constexpr int bwd_roles(int dh) { return dh == 128 ? 3 : 2; }
template <int DH, int NS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(DH > 128 ? 1 : 2))) void attn_bwd_mfma(
    const bf16_t *__restrict__ qkv, const bf16_t *__restrict__ d_o, const float *__restrict__ lse,
    const float *__restrict__ dsum, int ns, int B, int T, int H, bf16_t *__restrict__ dqkv) {
  __shared__ __attribute__((aligned(256))) char smem[kStages * dkv_stage<DH>(NS)];
  constexpr int R = bwd_roles(DH);
  const int role = blockIdx.z % R, sidx = blockIdx.z / R * NS;
  auto walk = [&](auto streams) {
    constexpr int n = decltype(streams)::value;
    if (role == 1)
      attn_bwd_dq_body<DH, n>(qkv, d_o, lse, dsum, B, T, H, ns, sidx, dqkv, smem);
    else if (role == 0)
      attn_bwd_dkv_body<DH, R == 3 ? 2 : 0, n>(qkv, d_o, lse, dsum, B, T, H, ns, sidx, dqkv, smem);
    else if constexpr (R == 3)
      attn_bwd_dkv_body<DH, 1, n>(qkv, d_o, lse, dsum, B, T, H, ns, sidx, dqkv, smem);
  };
  if (NS > 1 && sidx + NS > ns)
    walk(std::integral_constant<int, 1>{});  // the last of an odd number
  else
    walk(std::integral_constant<int, NS>{});
}

// ------------------------------------------------------------------ small grids ---------
// With few batches and heads a launch waits for the chain of its longest workgroup, tile after tile behind a barrier.
// Here a workgroup owns 32 queries (keys) and its W wavefronts take every W-th 32-row block of the other axis each, staged
// in LDS of their own: no barrier until they add up what they have.  A block's last fragments are requested before
// the next block's loads are issued (a read behind them in a wavefront's queue waits for their data).

// Two 32 x DH tiles of one wavefront, two stages.
template <int DH>
struct Private {
  static constexpr int KT = 32 * DH * 2, STAGE = 2 * KT, BYTES = kStages * STAGE;
  typedef TokTile<32, DH, 64> Tile;
};
// What W wavefronts hold of a 32 x DH result meets in LDS: row = the lane's own query (key).
template <int DH, int W>
struct Meet {
  static constexpr int P = DH + 4, PER = DH / (2 * W);  // columns a thread of the workgroup takes of one row
  float *at;                                            // [W][32][P]
  __device__ inline void park(const floatx16 (&acc)[DH / 32], int wave, int lane) const {
    float *p = at + (wave * 32 + (lane & 31)) * P + 4 * (lane >> 5);
#pragma unroll
    for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<float4 *>(p + 32 * dt + 8 * g) =
            make_float4(acc[dt][4 * g], acc[dt][4 * g + 1], acc[dt][4 * g + 2], acc[dt][4 * g + 3]);
  }
  __device__ static inline int row(int t) { return t / (2 * W); }
  __device__ static inline int col(int t) { return t % (2 * W) * PER; }
  __device__ inline void store(bf16_t *out, const float (&weight)[W], int t) const {  // out: the row's first column
#pragma unroll
    for (int c = 0; c < PER; c += 4) {
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int w = 0; w < W; ++w) {
        const float4 x = *reinterpret_cast<const float4 *>(at + (w * 32 + row(t)) * P + col(t) + c);
        v.x = __builtin_fmaf(x.x, weight[w], v.x);
        v.y = __builtin_fmaf(x.y, weight[w], v.y);
        v.z = __builtin_fmaf(x.z, weight[w], v.z);
        v.w = __builtin_fmaf(x.w, weight[w], v.w);
      }
      *reinterpret_cast<uint2 *>(out + col(t) + c) = make_uint2(pack2(v.x, v.y), pack2(v.z, v.w));
    }
  }
};
template <int DH, int W>
constexpr int split_lds() {
  return W * Private<DH>::BYTES > W * 32 * (DH + 4) * 4 ? W * Private<DH>::BYTES : W * 32 * (DH + 4) * 4;
}

// grid (ceil(T / 32), B*H)
template <int DH, int W>
__global__ __launch_bounds__(64 * W) void attn_fwd_split(const bf16_t *__restrict__ qkv, int T, int H, bf16_t *__restrict__ o,
                                                         float *__restrict__ lse) {
  typedef Private<DH> L;
  typedef typename L::Tile Tile;
  __shared__ __attribute__((aligned(256))) char smem[split_lds<DH, W>()];
  __shared__ float ms[W][32], ls[W][32];
  const int t = threadIdx.x, lane = t & 63, hh = lane >> 5, lq = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const CausalTile ct = causal_tile();
  const int qt = gridDim.x - 1 - ct.rank, b = ct.y / H, h = ct.y % H, d = H * DH;  // key blocks 0 .. qt
  const size_t ld3 = 3 * (size_t)d;
  const bf16_t *qbase = qkv + (size_t)b * T * ld3 + h * DH;
  const int q = 32 * qt + lq;
  char *const mine = smem + wave * L::BYTES;

  const BufRsrc rs = make_rsrc(qbase, (size_t)T * ld3 * 2 - (size_t)h * DH * 2);
  Tile lk, lv;
  lk.init(d, (int)ld3, lane);
  lv.init(2 * d, (int)ld3, lane);
  auto issue = [&](int kt, int stage) {
    lk.issue(rs, mine + stage * L::STAGE, 0, 32 * kt, T);
    lv.issue(rs, mine + stage * L::STAGE + L::KT, 0, 32 * kt, T);
  };
  if (wave <= qt) issue(wave, 0);
  Frag qf[DH / 16];
#pragma unroll
  for (int ks = 0; ks < DH / 16; ++ks)
    qf[ks].q = (q < T) ? ldg16(qbase + (size_t)q * ld3 + 16 * ks + 8 * hh) : make_uint4(0, 0, 0, 0);
  floatx16 oacc[DH / 32];
#pragma unroll
  for (int i = 0; i < DH / 32; ++i) oacc[i] = kZero16;
  float m = kNegBig, l = 0.f;
  const float sc = rsqrtf((float)DH) * kLog2e;

  int stage = 0;
  for (int kt = wave; kt <= qt; kt += W, stage ^= 1) {
    const char *sk = mine + stage * L::STAGE, *sv = sk + L::KT;
    wait_vmcnt<0>();
    floatx16 s = kZero16;
#pragma unroll
    for (int ks = 0; ks < DH / 16; ++ks)
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Tile::rowfrag(sk, 0, ks, lane), qf[ks].v, s, 0, 0, 0);
    bf16x8 vf[2][DH / 32];
#pragma unroll
    for (int bq = 0; bq < 2; ++bq)
#pragma unroll
      for (int dt = 0; dt < DH / 32; ++dt) vf[bq][dt] = Tile::trfrag(sv, 16 * bq, dt, lane);
    if (kt + W <= qt) issue(kt + W, stage ^ 1);
    float mx = kNegBig;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if (kt == qt) {  // (uniform)
        const int kv = 32 * kt + 8 * (r >> 2) + 4 * hh + (r & 3);
        s[r] = ((kv > q) | (kv >= T)) ? kNegBig : s[r];
      }
      mx = fmaxf(mx, s[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mnew = fmaxf(m, mx * sc), alpha = __builtin_amdgcn_exp2f(m - mnew);
    float rsum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], sc, -mnew));
      rsum += s[r];
    }
    l = l * alpha + rsum;
    m = mnew;
#pragma unroll
    for (int i = 0; i < DH / 32; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[i][r] *= alpha;
#pragma unroll
    for (int bq = 0; bq < 2; ++bq) {
      Frag pf;
#pragma unroll
      for (int e = 0; e < 4; ++e) pf.u[e] = pack2(s[8 * bq + 2 * e], s[8 * bq + 2 * e + 1]);
#pragma unroll
      for (int dt = 0; dt < DH / 32; ++dt)
        oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[bq][dt], pf.v, oacc[dt], 0, 0, 0);
    }
  }
  l += __shfl_xor(l, 32, 64);
  if (hh == 0) {
    ms[wave][lq] = m;
    ls[wave][lq] = l;
  }
  __syncthreads();  // every wavefront is done with its tiles
  const Meet<DH, W> meet{reinterpret_cast<float *>(smem)};
  meet.park(oacc, wave, lane);
  __syncthreads();
  const int r = meet.row(t), qr = 32 * qt + r;
  if (qr >= T) return;
  float mm = kNegBig, ll = 0.f, w[W];
#pragma unroll
  for (int i = 0; i < W; ++i) mm = fmaxf(mm, ms[i][r]);
#pragma unroll
  for (int i = 0; i < W; ++i) {
    w[i] = __builtin_amdgcn_exp2f(ms[i][r] - mm);
    ll = __builtin_fmaf(ls[i][r], w[i], ll);
  }
  const float inv = 1.f / ll;
#pragma unroll
  for (int i = 0; i < W; ++i) w[i] *= inv;
  meet.store(o + ((size_t)b * T + qr) * d + h * DH, w, t);
  if (meet.col(t) == 0) lse[((size_t)b * H + h) * T + qr] = mm + log2f(ll);
}

// The backward's roles in one launch, grid (ceil(T / 32), B*H, roles * streams): dK and dV first, then dQ.
template <int DH, int W>
__device__ __forceinline__ void split_dq(const bf16_t *__restrict__ qkv, const bf16_t *__restrict__ d_o,
                                         const float *__restrict__ lse, const float *__restrict__ dsum, int B, int T, int H, int ns,
                                         int sidx, bf16_t *__restrict__ dqkv, char *smem) {
  typedef Private<DH> L;
  typedef typename L::Tile Tile;
  const int t = threadIdx.x, lane = t & 63, hh = lane >> 5, lq = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const CausalTile ct = causal_tile();
  const int qt = gridDim.x - 1 - ct.rank, b = ct.y / H, h = ct.y % H, d = H * DH;
  const size_t ld3 = 3 * (size_t)d, N = (size_t)B * T;
  const bf16_t *qbase = qkv + (size_t)b * T * ld3 + h * DH;
  const int q = 32 * qt + lq;
  const size_t tok = (size_t)b * T + q;
  char *const mine = smem + wave * L::BYTES;
  const BufRsrc rs = make_rsrc(qbase, (size_t)T * ld3 * 2 - (size_t)h * DH * 2);
  Tile lk, lv;
  lk.init(d, (int)ld3, lane);
  lv.init(2 * d, (int)ld3, lane);
  auto issue = [&](int kt, int stage) {
    lk.issue(rs, mine + stage * L::STAGE, 0, 32 * kt, T);
    lv.issue(rs, mine + stage * L::STAGE + L::KT, 0, 32 * kt, T);
  };
  if (wave <= qt) issue(wave, 0);
  Frag qf[DH / 16], gf[DH / 16];
#pragma unroll
  for (int ks = 0; ks < DH / 16; ++ks) {
    qf[ks].q = q < T ? ldg16(qbase + (size_t)q * ld3 + 16 * ks + 8 * hh) : make_uint4(0, 0, 0, 0);
    gf[ks].q = q < T ? ldg16(d_o + (sidx * N + tok) * d + h * DH + 16 * ks + 8 * hh) : make_uint4(0, 0, 0, 0);
  }
  const float sc = rsqrtf((float)DH), sc2 = sc * kLog2e;
  const float l2 = (q < T) ? lse[((size_t)b * H + h) * T + q] : 0.f;
  const float dsv = (q < T) ? dsum_of<DH>(dsum, ns * N, sidx * N + tok, h) : 0.f;
  floatx16 dq[DH / 32];
#pragma unroll
  for (int i = 0; i < DH / 32; ++i) dq[i] = kZero16;
  int stage = 0;
  for (int kt = wave; kt <= qt; kt += W, stage ^= 1) {
    const char *sk = mine + stage * L::STAGE, *sv = sk + L::KT;
    wait_vmcnt<0>();
    floatx16 s = kZero16, dp = kZero16;
#pragma unroll
    for (int ks = 0; ks < DH / 16; ++ks) {
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Tile::rowfrag(sk, 0, ks, lane), qf[ks].v, s, 0, 0, 0);
      dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Tile::rowfrag(sv, 0, ks, lane), gf[ks].v, dp, 0, 0, 0);
    }
    bf16x8 kc[2][DH / 32];
#pragma unroll
    for (int bq = 0; bq < 2; ++bq)
#pragma unroll
      for (int dt = 0; dt < DH / 32; ++dt) kc[bq][dt] = Tile::trfrag(sk, 16 * bq, dt, lane);
    if (kt + W <= qt) issue(kt + W, stage ^ 1);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], sc2, -l2));
      if (kt == qt) {  // (uniform)
        const int kv = 32 * kt + 8 * (r >> 2) + 4 * hh + (r & 3);
        p = ((kv > q) | (kv >= T)) ? 0.f : p;
      }
      dp[r] = p * (dp[r] - dsv);  // dS^T, without the scale
    }
#pragma unroll
    for (int bq = 0; bq < 2; ++bq) {
      Frag pf;
#pragma unroll
      for (int e = 0; e < 4; ++e) pf.u[e] = pack2(dp[8 * bq + 2 * e], dp[8 * bq + 2 * e + 1]);
#pragma unroll
      for (int dt = 0; dt < DH / 32; ++dt)
        dq[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kc[bq][dt], pf.v, dq[dt], 0, 0, 0);
    }
  }
  __syncthreads();
  const Meet<DH, W> meet{reinterpret_cast<float *>(smem)};
  meet.park(dq, wave, lane);
  __syncthreads();
  const int qr = 32 * qt + meet.row(t);
  if (qr >= T) return;
  float w[W];
#pragma unroll
  for (int i = 0; i < W; ++i) w[i] = sc;
  meet.store(dqkv + (sidx * N + (size_t)b * T + qr) * ld3 + h * DH, w, t);
}

// WHAT as for attn_bwd_dkv_body: 0 = dK and dV, 1 = dV only, 2 = dK only.
template <int DH, int W, int WHAT>
__device__ __forceinline__ void split_dkv(const bf16_t *__restrict__ qkv, const bf16_t *__restrict__ d_o,
                                          const float *__restrict__ lse, const float *__restrict__ dsum, int B, int T, int H, int ns,
                                          int sidx, bf16_t *__restrict__ dqkv, char *smem, float (*rows)[2][2][32]) {
  constexpr bool DO_DV = WHAT != 2, DO_DK = WHAT != 1;
  typedef Private<DH> L;
  typedef typename L::Tile Tile;
  const int t = threadIdx.x, lane = t & 63, hh = lane >> 5, lk_ = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const CausalTile ct = causal_tile();  // the first keys have the most queries
  const int own = ct.rank, b = ct.y / H, h = ct.y % H, d = H * DH, nqt = (T + 31) / 32;  // query blocks own .. nqt - 1
  const size_t ld3 = 3 * (size_t)d, N = (size_t)B * T;
  const bf16_t *qbase = qkv + (size_t)b * T * ld3 + h * DH;
  const bf16_t *kbase = qbase + d, *vbase = qbase + 2 * d;
  const float *lrow = lse + ((size_t)b * H + h) * T;
  const int kv = 32 * own + lk_;
  char *const mine = smem + wave * L::BYTES;
  Frag kf[DH / 16], vf[DO_DK ? DH / 16 : 1];
#pragma unroll
  for (int ks = 0; ks < DH / 16; ++ks) {
    kf[ks].q = kv < T ? ldg16(kbase + (size_t)kv * ld3 + 16 * ks + 8 * hh) : make_uint4(0, 0, 0, 0);
    if constexpr (DO_DK) vf[ks].q = kv < T ? ldg16(vbase + (size_t)kv * ld3 + 16 * ks + 8 * hh) : make_uint4(0, 0, 0, 0);
  }
  floatx16 dk[DH / 32], dv[DH / 32];  // (the one that is not asked for is never used)
#pragma unroll
  for (int i = 0; i < DH / 32; ++i) {
    dk[i] = kZero16;
    dv[i] = kZero16;
  }
  const float sc = rsqrtf((float)DH), sc2 = sc * kLog2e;
  const BufRsrc rq = make_rsrc(qbase, (size_t)T * ld3 * 2 - (size_t)h * DH * 2);
  const BufRsrc rg = make_rsrc(d_o + (sidx * N + (size_t)b * T) * d + h * DH, (size_t)T * d * 2 - (size_t)h * DH * 2);
  Tile lq, lg;
  lq.init(0, (int)ld3, lane);
  lg.init(0, d, lane);
  auto issue = [&](int qt, int stage) {
    lq.issue(rq, mine + stage * L::STAGE, 0, 32 * qt, T);
    lg.issue(rg, mine + stage * L::STAGE + L::KT, 0, 32 * qt, T);
  };
  // lse (lanes 0..31) and dsum of a block's rows go through a register, one block ahead
  auto row_value = [&](int qt) {
    const int r = 32 * qt + (lane & 31);
    return r >= T ? 0.f : hh == 0 ? lrow[r] : !DO_DK ? 0.f : dsum_of<DH>(dsum, ns * N, sidx * N + (size_t)b * T + r, h);
  };
  float ahead = 0.f;
  if (own + wave < nqt) {
    ahead = row_value(own + wave);
    issue(own + wave, 0);
  }
  int stage = 0;
  for (int qt = own + wave; qt < nqt; qt += W, stage ^= 1) {
    const char *sq = mine + stage * L::STAGE, *sg = sq + L::KT;
    float(*row)[32] = rows[wave][stage];
    row[hh][lane & 31] = ahead;
    wait_vmcnt<0>();
    floatx16 s = kZero16, dp = kZero16;
#pragma unroll
    for (int ks = 0; ks < DH / 16; ++ks) {
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Tile::rowfrag(sq, 0, ks, lane), kf[ks].v, s, 0, 0, 0);
      if constexpr (DO_DK)
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Tile::rowfrag(sg, 0, ks, lane), vf[ks].v, dp, 0, 0, 0);
    }
    bf16x8 gc[2][DO_DV ? DH / 32 : 1], qc[2][DO_DK ? DH / 32 : 1];
#pragma unroll
    for (int bq = 0; bq < 2; ++bq)
#pragma unroll
      for (int dt = 0; dt < DH / 32; ++dt) {
        if constexpr (DO_DV) gc[bq][dt] = Tile::trfrag(sg, 16 * bq, dt, lane);
        if constexpr (DO_DK) qc[bq][dt] = Tile::trfrag(sq, 16 * bq, dt, lane);
      }
    float4 l4[4], d4[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      l4[g] = *reinterpret_cast<const float4 *>(&row[0][8 * g + 4 * hh]);
      d4[g] = *reinterpret_cast<const float4 *>(&row[1][8 * g + 4 * hh]);
    }
    if (qt + W < nqt) {
      ahead = row_value(qt + W);
      issue(qt + W, stage ^ 1);
    }
    Frag pf[2], sf[2];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float lv4[4] = {l4[g].x, l4[g].y, l4[g].z, l4[g].w}, dv4[4] = {d4[g].x, d4[g].y, d4[g].z, d4[g].w};
      float p4[4], s4[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = 4 * g + e;
        p4[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], sc2, -lv4[e]));
        if (qt == own || qt == nqt - 1) {  // (uniform)
          const int qq = 32 * qt + 8 * g + 4 * hh + e;
          p4[e] = ((kv > qq) | (qq >= T)) ? 0.f : p4[e];
        }
        s4[e] = p4[e] * (dp[r] - dv4[e]);  // without the scale
      }
      pf[g >> 1].u[2 * (g & 1)] = pack2(p4[0], p4[1]);
      pf[g >> 1].u[2 * (g & 1) + 1] = pack2(p4[2], p4[3]);
      sf[g >> 1].u[2 * (g & 1)] = pack2(s4[0], s4[1]);
      sf[g >> 1].u[2 * (g & 1) + 1] = pack2(s4[2], s4[3]);
    }
#pragma unroll
    for (int bq = 0; bq < 2; ++bq)
#pragma unroll
      for (int dt = 0; dt < DH / 32; ++dt) {
        if constexpr (DO_DV) dv[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gc[bq][dt], pf[bq].v, dv[dt], 0, 0, 0);
        if constexpr (DO_DK) dk[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qc[bq][dt], sf[bq].v, dk[dt], 0, 0, 0);
      }
  }
  const Meet<DH, W> meet{reinterpret_cast<float *>(smem)};
  const int kr = 32 * own + meet.row(t);
  bf16_t *out = dqkv + (sidx * N + (size_t)b * T + kr) * ld3 + d + h * DH;
  auto hand_in = [&](const floatx16 (&acc)[DH / 32], float scale, bf16_t *to) {
    float w[W];
#pragma unroll
    for (int i = 0; i < W; ++i) w[i] = scale;
    __syncthreads();  // every wavefront is done with what lies there
    meet.park(acc, wave, lane);
    __syncthreads();
    if (kr < T) meet.store(to, w, t);
  };
  if constexpr (DO_DK) hand_in(dk, sc, out);
  if constexpr (DO_DV) hand_in(dv, 1.f, out + d);
}

// (dK and dV of heads of 256 have registers of their own each: 512 and 310 on the stack together)
constexpr int split_roles(int dh) { return dh > 128 ? 3 : 2; }
template <int DH, int W>
__global__ __launch_bounds__(64 * W) void attn_bwd_split(const bf16_t *__restrict__ qkv, const bf16_t *__restrict__ d_o,
                                                         const float *__restrict__ lse, const float *__restrict__ dsum, int ns, int B,
                                                         int T, int H, bf16_t *__restrict__ dqkv) {
  __shared__ __attribute__((aligned(256))) char smem[split_lds<DH, W>()];
  __shared__ __attribute__((aligned(16))) float rows[W][2][2][32];
  constexpr int R = split_roles(DH);
  const int role = blockIdx.z % R, sidx = blockIdx.z / R;
  if (role == 1)
    split_dq<DH, W>(qkv, d_o, lse, dsum, B, T, H, ns, sidx, dqkv, smem);
  else if (role == 0)
    split_dkv<DH, W, R == 3 ? 2 : 0>(qkv, d_o, lse, dsum, B, T, H, ns, sidx, dqkv, smem, rows);
  else if constexpr (R == 3)
    split_dkv<DH, W, 1>(qkv, d_o, lse, dsum, B, T, H, ns, sidx, dqkv, smem, rows);
}

}  // namespace

// Where the other axis is divided up.  The split forms' workgroups are short, but every wavefront loads its own blocks, and a CU holds few of
// them: one at widths 128 and 256, whose wavefronts have 32 and 64 KB of LDS each; at width 64 (16 KB) two of the forward but one of
// the backward, by its 276 registers.  So they gain while one round holds them all, and a little beyond where rows are
// long; up to 64 tokens there is no chain to cut (at 256 there is: its shared tiles hold 32 keys).  In us, shared / split (workgroups of the split form):
//   forward 64   1 x 576 tokens, 2 heads (36) 11.4 / 7.1;  1 x 1000, 3 (96) 18.2 / 9.7;  2 x 400, 8 (208) 9.7 / 6.5;  8 x 256, 8 (512)
//                7.3 / 6.0;  8 x 200, 12 (672) 7.1 / 9.5;  32 x 64, 6 (384) 4.4 / 5.3
//   forward 128  1 x 672, 6 (126) 19.9 / 11.8;  12 x 208, 3 (252) 10.1 / 6.9;  2 x 1024, 4 (256) 29.2 / 16.0;  4 x 656, 5 (420) 20.1 / 20.6
//   forward 256  1 x 928, 2 (58) 62.0 / 33.6;  16 x 128, 2 (128) 13.5 / 8.9;  4 x 928, 4 (464) 63.7 / 39.9;  32 x 128, 4 (512) 15.0 / 16.3;
//                8 x 32, 2 (16) 6.5 / 6.7
//   backward 64  1 x 576, 2 (72) 18.4 / 9.9;  4 x 96, 8 (192) 6.9 / 5.0;  2 x 400, 8 (416) 15.4 / 10.7;  2 x 256, 14 (448) 11.4 / 11.2;
//                2 x 128, 12, two streams (384) 8.0 / 8.4;  2 x 640, 5, two (800) 20.9 / 25.0;  4 x 64, 9, two (288) 5.1 / 7.5
//   backward 128 1 x 672, 6 (252) 25.3 / 17.9;  2 x 256, 8 (256) 13.8 / 9.5;  2 x 1024, 4 (512) 35.1 / 27.4;  4 x 128, 8, two (512) 10.4 / 13.0;
//                8 x 40, 4, two (256) 6.0 / 7.2;  beyond one round only where the XCDs get the same mix of lengths (causal_tile(): heads of all
//                batches a multiple of eight) or rows are long: 1 x 512, 16 (512) 20.4 / 18.3, but 12 (384) 20.5 / 24.2, 5, three (480)
//                21.1 / 25.3, 5, two (320) 20.3 / 19.0;  1 x 576, 11 (396) 23.3 / 21.7, 14 (504) 23.8 / 25.7;  1 x 1024, 8 (512) 34.0 / 25.6,
//                2, four (512) 34.1 / 39.4;  1 x 2048, 4 (512) 65.8 / 59.9
//   backward 256 1 x 928, 2 (174) 98 / 45;  1 x 64, 1 (6) 12.2 / 7.1;  16 x 128, 2 (384) 24.3 / 15.0;  8 x 128, 3, two (576) 25.1 / 20.4;
//                8 x 104, 4, two (768) 25.0 / 24.2;  4 x 928, 4 (1392) 102 / 118;  16 x 64, 2, two (384) 13.7 / 13.4;
//                8 x 65, 4, three (864) 20.2 / 25.7
constexpr int split_waves(int dh) { return dh > 128 ? 2 : 4; }  // (four at 256: 256 KB of tiles)
bool fwd_splits(int dh, long heads, int T) {
  const long workgroups = (T + 31) / 32 * heads;
  if (dh == 256) return T > 32 && workgroups <= (T >= 512 ? 512 : 256);
  return T > 64 && workgroups <= (dh == 64 ? 512 : 256);
}
bool bwd_splits(int dh, long heads, int ns, int T) {
  const long workgroups = (T + 31) / 32 * heads * ns * split_roles(dh);
  if (dh == 256) return workgroups <= (T > 96 ? 640 : 256);
  const int most = dh == 64 ? (T >= 256 ? 448 : 256) : T < 512 ? 256 : heads % 8 == 0 || T > 1024 ? 512 : T > 512 ? 400 : 288;
  return T > 64 && workgroups <= most;
}

// A workgroup of four wavefronts takes 128 queries; where that leaves CUs without a workgroup, two wavefronts take
// 64, but each of them reads the keys for half as many queries and has more of them to load.  Forward in us, four /
// two wavefronts:
//   width 64   8 x 64 tokens, 8 heads 4.64 / 4.62;  4 x 128, 16: 5.65 / 5.08;  8 x 256, 8: 7.78 / 7.34;
//              2 x 512, 16: 11.45 / 10.99;  longer sequences lose (2 x 900, 8 heads of 32, when that width ran here: 13.6 / 14.2)
//   width 128  4 x 64, 16 heads 5.33 / 6.00;  8 x 256, 4: 10.72 / 11.13;  2 x 512, 16: 16.94 / 18.23  (the two-wavefront
//              form gets 230 + 134 registers from the compiler, one wavefront per SIMD, where four get 256 + 0 and two)
//   width 256  16 x 64, 4 heads 8.62 / 9.01;  8 x 128, 4: 14.39 / 13.33;  4 x 256, 4: 22.14 / 21.93;  2 x 512, 8: 39.0 / 40.0
bool fwd_by_two(int dh, long heads, int T) {
  return dh != 128 && (T + 127) / 128 * heads < 256 && (dh == 64 ? T <= 512 : T > 64 && T <= 256);
}
template <int DH>
hipError_t fwd(const bf16_t *qkv, int B, int T, int H, bf16_t *o, float *lse, hipStream_t s) {
  if (fwd_splits(DH, (long)B * H, T)) {
    constexpr int W = split_waves(DH);
    hipLaunchKernelGGL((attn_fwd_split<DH, W>), dim3((T + 31) / 32, B * H), dim3(64 * W), 0, s, qkv, T, H, o, lse);
    return hipGetLastError();
  }
  if constexpr (DH != 128) {
    if (fwd_by_two(DH, (long)B * H, T)) {
      hipLaunchKernelGGL((attn_fwd_mfma<DH, 2>), dim3((T + 63) / 64, B * H), dim3(128), 0, s, qkv, T, H, o, lse);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((attn_fwd_mfma<DH, 4>), dim3((T + 127) / 128, B * H), dim3(256), 0, s, qkv, T, H, o, lse);
  return hipGetLastError();
}
hipError_t attention_forward_mfma(const void *qkv, int B, int T, int H, int dh, void *o, float *lse,
                                  hipStream_t s) {
  const bf16_t *x = (const bf16_t *)qkv;
  switch (dh) {
    case 64: return fwd<64>(x, B, T, H, (bf16_t *)o, lse, s);
    case 128: return fwd<128>(x, B, T, H, (bf16_t *)o, lse, s);
    case 256: return fwd<256>(x, B, T, H, (bf16_t *)o, lse, s);
    default: return hipErrorInvalidValue;
  }
}

// At head width 64 a workgroup walks two streams together: one read of K, V and Q and one score product and
// exponential serve both, 24 matrix instructions per sub-tile and stream instead of 28, half of the LDS reads for dQ;
// the walk is bound by the latency of its products and reads.  256 registers, the most two wavefronts per SIMD have, none
// spilled.  That leaves half as many workgroups, so it is taken where there are more of them than the 512 that the chip
// holds at a time; at 512 short sequences would gain and long ones lose.  Backward in us, one by one / in pairs (workgroups in pairs):
//   8 x 512 tokens, 16 heads, two streams (1024) 65.0 / 53.0, three streams (2048) 91.6 / 79.3;  4 x 1024, 16 (1024) 91.0 / 76.1;
//   64 x 64, 8 (1024) 22.4 / 20.5;  8 x 200, 12, three (768) 27.6 / 23.8;  3 x 640, 12, three (720) 45.1 / 39.1;
//   8 x 256, 16 (512) 27.1 / 23.4;  4 x 512, 16 (512) 35.2 / 34.8;  2 x 1024, 16 (512) 51.8 / 54.0;  4 x 1024, 8 (512) 49.8 / 52.9;
//   8 x 256, 12 (384) 20.0 / 21.4;  8 x 256, 8 (256) 17.1 / 19.1.
// Wider heads have no registers for a second stream's accumulators.  The streams' weighted sum formed here as well, of
// the rows just stored, cost 15 to 25 us a launch: more than the pass on the other stream that it replaces.
constexpr long kPairedWgs = 640;
bool bwd_pairs(int dh, long heads, int ns, int T) {
  return dh == 64 && ns > 1 && (T + 127) / 128 * heads * bwd_roles(dh) * ((ns + 1) / 2) >= kPairedWgs;
}
template <int DH, int NS>
hipError_t bwd(const bf16_t *qkv, const bf16_t *d_o, const float *lse, const float *dsum, int ns, int B, int T, int H,
               bf16_t *dqkv, hipStream_t s) {
  if (bwd_splits(DH, (long)B * H, ns, T)) {
    constexpr int W = split_waves(DH);
    hipLaunchKernelGGL((attn_bwd_split<DH, W>), dim3((T + 31) / 32, B * H, split_roles(DH) * ns), dim3(64 * W), 0, s, qkv, d_o,
                       lse, dsum, ns, B, T, H, dqkv);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((attn_bwd_mfma<DH, NS>), dim3((T + 127) / 128, B * H, bwd_roles(DH) * ((ns + NS - 1) / NS)), dim3(256), 0,
                     s, qkv, d_o, lse, dsum, ns, B, T, H, dqkv);
  return hipGetLastError();
}
int attention_form_mfma(int dh, int ns, int B, int T, int H) {
  const long heads = (long)B * H;
  if (ns > 0) return bwd_splits(dh, heads, ns, T) ? split_waves(dh) : bwd_pairs(dh, heads, ns, T) ? -2 : 0;
  return fwd_splits(dh, heads, T) ? split_waves(dh) : fwd_by_two(dh, heads, T) ? -1 : 0;
}
hipError_t attention_backward_mfma(const void *qkv, const void *d_o, const float *lse, const float *dsum, int ns,
                                   int B, int T, int H, int dh, void *dqkv, hipStream_t s) {
  const bf16_t *x = (const bf16_t *)qkv, *g = (const bf16_t *)d_o;
  bf16_t *out = (bf16_t *)dqkv;
  const bool pairs = bwd_pairs(dh, (long)B * H, ns, T);
  switch (dh) {
    case 64: return pairs ? bwd<64, 2>(x, g, lse, dsum, ns, B, T, H, out, s) : bwd<64, 1>(x, g, lse, dsum, ns, B, T, H, out, s);
    case 128: return bwd<128, 1>(x, g, lse, dsum, ns, B, T, H, out, s);
    case 256: return bwd<256, 1>(x, g, lse, dsum, ns, B, T, H, out, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace il
