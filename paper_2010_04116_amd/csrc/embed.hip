// Input embedding of the first module (App. B: an embedding matrix in front of the Transformer
// blocks) and its gradient.
//
//   forward :  x0[i, :]   = wte[tokens[i], :] + wpe[i % T, :]                      (fp32 out)
//   backward:  dwpe[t, :] = sum_b dx0[b*T + t, :]
//              dwte[v, :] = sum over the positions i with tokens[i] == v of dx0[i, :]
//
// The token gradient is a scatter-add, done without atomics and with a fixed summation order: a
// workgroup owns a set of vocabulary rows, lists the positions that hit them in ascending order and
// adds those rows of dx0 in that order, in registers.  Every element of dwte and dwpe is the plain
// sequential sum of its rows; a token outside [0, vocab) embeds as zero and receives no gradient.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "../../include/interlock.h"
#include "common.h"

namespace il {
namespace {

__device__ inline void load4(const float *p, float (&o)[4]) {
  const float4 q = *reinterpret_cast<const float4 *>(p);
  o[0] = q.x; o[1] = q.y; o[2] = q.z; o[3] = q.w;
}
__device__ inline void load4(const bf16_t *p, float (&o)[4]) {
  const uint2 q = *reinterpret_cast<const uint2 *>(p);
  o[0] = bf16_to_f32((bf16_t)(q.x & 0xFFFF)); o[1] = bf16_to_f32((bf16_t)(q.x >> 16));
  o[2] = bf16_to_f32((bf16_t)(q.y & 0xFFFF)); o[3] = bf16_to_f32((bf16_t)(q.y >> 16));
}

constexpr int kSegment = 4096;   // positions listed at a time (one LDS list entry each)
// Vocabulary row groups = workgroups of the token-gradient kernel: where dwte exceeds the L2s' 32 MB, kMostGroups (each
// writes fewer rows one after the other); otherwise kMaxGroups, as each group scans all positions.  us with
// kMaxGroups and kMostGroups: 33 MB (vocabulary 32000, d = 256) 24.6 and 30.2, 51 MB (50304, 256) 18.9 and 18.6,
// (20000, 640) 25.1 and 23.1, 134 MB (32768, 1024) 32.4 and 26.3, 412 MB (50304, 2048) 150 and 133.
constexpr int kMaxGroups = 4096, kMostGroups = 8192;
constexpr size_t kManyBytes = 40u * 1000 * 1000;

// Four consecutive columns per lane, two row passes apart in flight by occupancy: bound by the fp32
// rows it writes.  VEC: rows of wte / wpe / x0 take 8- or 16-byte accesses.
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void embed_fwd_kernel(const T *__restrict__ wte, const T *__restrict__ wpe,
                                                        const int32_t *__restrict__ tokens, int N, int Tn, int d,
                                                        int V, float *__restrict__ x0) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int i = blockIdx.x * 4 + wave; i < N; i += gridDim.x * 4) {
    const int tok = tokens[i];
    const bool ok = tok >= 0 && tok < V;
    const T *te = wte + (size_t)(ok ? tok : 0) * d, *pe = wpe + (size_t)(i % Tn) * d;
    float *o = x0 + (size_t)i * d;
    if constexpr (VEC) {
      for (int c = lane * 4; c < d; c += 256) {
        float a[4], b[4];
        load4(te + c, a);
        load4(pe + c, b);
        float4 r;
        r.x = (ok ? a[0] : 0.f) + b[0];
        r.y = (ok ? a[1] : 0.f) + b[1];
        r.z = (ok ? a[2] : 0.f) + b[2];
        r.w = (ok ? a[3] : 0.f) + b[3];
        *reinterpret_cast<float4 *>(o + c) = r;
      }
    } else {
      for (int c = lane; c < d; c += 64) o[c] = (ok ? ld<T>(te + c) : 0.f) + ld<T>(pe + c);
    }
  }
}

template <int VEC> struct Cols { float v[VEC]; };
template <int VEC>
__device__ inline Cols<VEC> load_cols(const float *p) {
  Cols<VEC> r;
  if constexpr (VEC == 4) {
    const float4 q = *reinterpret_cast<const float4 *>(p);
    r.v[0] = q.x; r.v[1] = q.y; r.v[2] = q.z; r.v[3] = q.w;
  } else {
    r.v[0] = *p;
  }
  return r;
}
template <int VEC>
__device__ inline void store_cols(float *p, const Cols<VEC> &r) {
  if constexpr (VEC == 4)
    *reinterpret_cast<float4 *>(p) = make_float4(r.v[0], r.v[1], r.v[2], r.v[3]);
  else
    *p = r.v[0];
}

// Both gradients in one launch.
//
// Workgroups [0, groups): group w owns the vocabulary rows v with v mod groups == w (groups is a power
// of two).  Token frequencies fall off steeply and frequent tokens have neighbouring ids, so rows are
// dealt out round-robin: with blocks of 32 consecutive rows the first workgroup had 45 % of all
// positions of a word-like distribution to add up, one after the other through memory (1.26 ms at
// 4096 positions, d = 1024, vocabulary 32768, where the launch is now bound by writing the 134 MB of
// dwte).  The four wavefronts scan a quarter of a segment of positions each, 16 bytes per lane, and
// append their hits in ascending order to a list each, the next tokens under way; then every row is summed
// from the lists by `nw` wavefronts, one column group of VEC per lane, eight rows of dx0 in flight.  Rows are
// stored once per segment; a later segment (N > kSegment) adds to the rows it hits only.  The hits of a group are
// few (one on average at 4096 positions): held in registers, a row costs one comparison and ballot instead of
// four trips to the LDS (4096 positions, d = 1536, vocabulary 50304: 77 -> 71 us).
//
// The remaining workgroups: dwpe[t, c] = sum_b dx0[b*T + t, c], b ascending.
template <int VEC>
__global__ __launch_bounds__(256) void embed_bwd_kernel(const float *__restrict__ dx0,
                                                        const int32_t *__restrict__ tokens, int N, int B, int Tn, int d,
                                                        int V, int groups, float *__restrict__ dwte,
                                                        float *__restrict__ dwpe) {
  constexpr int QUARTER = kSegment / 4;
  __shared__ uint16_t list_pos[4][QUARTER];  // position within the quarter
  __shared__ uint16_t list_row[4][QUARTER];  // row index within the group (vocab <= 2^24, groups >= 4096 there)
  __shared__ int list_len[4];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  if ((int)blockIdx.x >= groups) {
    const size_t total = (size_t)Tn * d, step = (size_t)(gridDim.x - groups) * 256 * VEC;
    for (size_t i = ((size_t)(blockIdx.x - groups) * 256 + t) * VEC; i < total; i += step) {
      Cols<VEC> s = {};
      for (int b = 0; b < B; ++b) {
        const Cols<VEC> x = load_cols<VEC>(dx0 + (size_t)b * total + i);
#pragma unroll
        for (int e = 0; e < VEC; ++e) s.v[e] += x.v[e];
      }
      store_cols<VEC>(dwpe + i, s);
    }
    return;
  }
  const int w = blockIdx.x, shift = 31 - __builtin_clz(groups);
  const int nrows = w < V ? (V - 1 - w) / groups + 1 : 0;
  const int ncg = (d + VEC - 1) / VEC;                       // column groups of a row
  const int nw = ncg <= 64 ? 1 : (ncg <= 128 ? 2 : 4);       // wavefronts that share one row
  const bool aligned = ((uintptr_t)tokens & 15) == 0;

  for (int seg = 0; seg < N; seg += kSegment) {
    {  // this wavefront's quarter of the segment
      const int base = seg + wave * QUARTER, end = min(N, base + QUARTER);
      int len = 0;
      const auto whole = [&](int i) { return aligned && i + 3 < end; };
      int4 next = {};
      if (whole(base + lane * 4)) next = *reinterpret_cast<const int4 *>(tokens + base + lane * 4);
      for (int i0 = base; i0 < end; i0 += 256) {
        const int i = i0 + lane * 4;
        int tok[4];
        const int4 q = next;
        if (whole(i + 256)) next = *reinterpret_cast<const int4 *>(tokens + i + 256);
        if (whole(i)) {
          tok[0] = q.x; tok[1] = q.y; tok[2] = q.z; tok[3] = q.w;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) tok[e] = i + e < end ? tokens[i + e] : -1;
        }
        bool hit[4], any = false;
        int mine = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          hit[e] = tok[e] >= 0 && tok[e] < V && (tok[e] & (groups - 1)) == w;
          any = any || hit[e];
          mine += hit[e];
        }
        if (__ballot(any) == 0) continue;
        // exclusive prefix of the lanes' hit counts (0..4 each) from the ballots of the count's bits
        const unsigned long long below = (1ull << lane) - 1ull;
        const unsigned long long c1 = __ballot(mine & 1), c2 = __ballot(mine & 2), c4 = __ballot(mine & 4);
        int at = len + __popcll(c1 & below) + 2 * __popcll(c2 & below) + 4 * __popcll(c4 & below);
        len += __popcll(c1) + 2 * __popcll(c2) + 4 * __popcll(c4);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (hit[e]) {
            list_pos[wave][at] = (uint16_t)(i + e - base);
            list_row[wave][at] = (uint16_t)(tok[e] >> shift);
            ++at;
          }
      }
      if (lane == 0) list_len[wave] = len;
    }
    __syncthreads();
    // the four lists, one after the other, are ascending: entry l of all goes to lane l, once for all rows where they fit
    const int o1 = list_len[0], o2 = o1 + list_len[1], o3 = o2 + list_len[2], all = o3 + list_len[3];
    int my_row = -1, my_pos = 0;
    auto fetch = [&](int l) {
      my_row = -1;
      if (l < all) {
        const int q = (l >= o1) + (l >= o2) + (l >= o3), at = l - (q == 0 ? 0 : q == 1 ? o1 : q == 2 ? o2 : o3);
        my_row = list_row[q][at];
        my_pos = q * QUARTER + list_pos[q][at];
      }
    };
    if (all <= 64) fetch(lane);
    for (int r = wave / nw; r < nrows; r += 4 / nw) {
      float *dst = dwte + ((size_t)r * groups + w) * d;
      for (int cg = (wave % nw) * 64 + lane; cg - lane < ncg; cg += nw * 64) {  // (uniform trip count)
        const bool in = cg < ncg;
        const int c = cg * VEC;
        Cols<VEC> acc = {};
        bool touched = seg == 0;
        for (int l0 = 0; l0 < all; l0 += 64) {
          if (all > 64) fetch(l0 + lane);
          unsigned long long m = __ballot(my_row == r);
          if (m == 0) continue;
          if (!touched) {
            if (in) acc = load_cols<VEC>(dst + c);
            touched = true;
          }
          const float *src = dx0 + (size_t)seg * d + c;
          while (m) {  // eight rows requested before the first is added; added in ascending order
            Cols<VEC> x[8];
            int n = 0;
#pragma unroll
            for (int u = 0; u < 8; ++u)
              if (m) {
                const int b = __builtin_ctzll(m);
                m &= m - 1;
                const int p = __builtin_amdgcn_readlane(my_pos, b);
                x[u] = in ? load_cols<VEC>(src + (size_t)p * d) : Cols<VEC>{};
                n = u + 1;
              }
#pragma unroll
            for (int u = 0; u < 8; ++u)
              if (u < n) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc.v[e] += x[u].v[e];
              }
          }
        }
        if (in && touched) store_cols<VEC>(dst + c, acc);
      }
    }
    __syncthreads();  // the lists are rewritten by the next segment
  }
}

}  // namespace
}  // namespace il

extern "C" {

int il_embed_forward(int32_t dtype, const void *wte, const void *wpe, const int32_t *tokens, int32_t batch,
                     int32_t seq, int32_t d_model, int32_t vocab, float *x0, void *stream) {
  using namespace il;
  if (dtype != IL_F32 && dtype != IL_BF16) return IL_E_ARG;
  if (!wte || !wpe || !tokens || !x0 || batch < 1 || seq < 1 || d_model < 1 || vocab < 1) return IL_E_ARG;
  const long long N = (long long)batch * seq;
  if (N > (1 << 24) || vocab > (1 << 24)) return IL_E_SHAPE;
  if ((d_model & 3) == 0 && ((uintptr_t)x0 & 15)) return IL_E_SHAPE;
  const int blocks = (int)((N + 3) / 4 < 4096 ? (N + 3) / 4 : 4096);
  hipStream_t s = (hipStream_t)stream;
  const uintptr_t tab = (uintptr_t)wte | (uintptr_t)wpe;
  const bool vec = (d_model & 3) == 0 && (tab & (dtype == IL_F32 ? 15 : 7)) == 0;
#define IL_EMBED_FWD(TY, VEC)                                                                                     \
  hipLaunchKernelGGL((embed_fwd_kernel<TY, VEC>), dim3(blocks), dim3(256), 0, s, (const TY *)wte, (const TY *)wpe, \
                     tokens, (int)N, seq, d_model, vocab, x0)
  if (dtype == IL_F32) {
    if (vec) IL_EMBED_FWD(float, true); else IL_EMBED_FWD(float, false);
  } else {
    if (vec) IL_EMBED_FWD(bf16_t, true); else IL_EMBED_FWD(bf16_t, false);
  }
#undef IL_EMBED_FWD
  return hipGetLastError() == hipSuccess ? IL_OK : IL_E_HIP;
}

int il_embed_backward(const float *dx0, const int32_t *tokens, int32_t batch, int32_t seq, int32_t d_model,
                      int32_t vocab, float *dwte, float *dwpe, void *stream) {
  using namespace il;
  if (!dx0 || !tokens || !dwte || !dwpe || batch < 1 || seq < 1 || d_model < 1 || vocab < 1) return IL_E_ARG;
  const long long N = (long long)batch * seq;
  if (N > (1 << 24) || vocab > (1 << 24)) return IL_E_SHAPE;
  hipStream_t s = (hipStream_t)stream;
  // the smallest power of two that gives every workgroup one row, up to the most
  const int most = (size_t)vocab * d_model * sizeof(float) > kManyBytes ? kMostGroups : kMaxGroups;
  int groups = 1;
  while (groups < vocab && groups < most) groups *= 2;
  const bool vec = (d_model & 3) == 0 && (((uintptr_t)dx0 | (uintptr_t)dwte | (uintptr_t)dwpe) & 15) == 0;
  const size_t pos = ((size_t)seq * d_model / (vec ? 4 : 1) + 255) / 256;
  const int pblocks = (int)(pos < 1024 ? pos : 1024);
  if (vec)
    hipLaunchKernelGGL(embed_bwd_kernel<4>, dim3(groups + pblocks), dim3(256), 0, s, dx0, tokens, (int)N, batch, seq,
                       d_model, vocab, groups, dwte, dwpe);
  else
    hipLaunchKernelGGL(embed_bwd_kernel<1>, dim3(groups + pblocks), dim3(256), 0, s, dx0, tokens, (int)N, batch, seq,
                       d_model, vocab, groups, dwte, dwpe);
  return hipGetLastError() == hipSuccess ? IL_OK : IL_E_HIP;
}

}  // extern "C"
