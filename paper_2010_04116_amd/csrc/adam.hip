// Optimiser step of the paper's Transformer runs (App. B, training configuration): Adam with bias
// correction, one fused pass over the flat parameter buffer.
//
//   m <- b1 m + (1-b1) g     v <- b2 v + (1-b2) g^2
//   w <- w - lr * (m / (1-b1^t)) / (sqrt(v / (1-b2^t)) + eps)
//
// HBM-bound: per parameter it reads g, m, v, w (16 B) and writes m, v, w (12 B), plus 2 B for the
// bf16 image of w in bf16 mode.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "../../include/interlock.h"
#include "common.h"

namespace il {
namespace {

constexpr size_t kCachedBytes = 350u * 1000 * 1000;

struct AdamScalars { float b1, b2, omb1, omb2, c1, c2, lr, eps; };

__device__ inline float adam_one(float g, float &m, float &v, float w, const AdamScalars &a) {
  m = a.b1 * m + a.omb1 * g;
  v = a.b2 * v + a.omb2 * g * g;
  return w - a.lr * (m * a.c1) / (sqrtf(v * a.c2) + a.eps);
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
template <bool NT>
__device__ inline float4 load4(const float *p, size_t i) {
  const f32x4 *q = reinterpret_cast<const f32x4 *>(p) + i;
  const f32x4 x = NT ? __builtin_nontemporal_load(q) : *q;
  return make_float4(x[0], x[1], x[2], x[3]);
}
template <bool NT>
__device__ inline void store4(float *p, size_t i, const float4 &x) {
  f32x4 *q = reinterpret_cast<f32x4 *>(p) + i;
  const f32x4 y = {x.x, x.y, x.z, x.w};
  if constexpr (NT)
    __builtin_nontemporal_store(y, q);
  else
    *q = y;
}

// BF: also write the bf16 image of the updated fp32 weights.  Buffers are 16-byte aligned
// (8-byte for the bf16 image); the tail (< 4 elements) is handled by the last thread, element-wise.
//
// Bound by HBM.  Four parameters per thread and a workgroup for every 4 T of them, so what the chip has in flight is
// one moving window of each buffer: 8192 workgroups striding over the buffers, two places of each at a time, drew
// 4.0-4.9 TB/s from 42 M parameters on.  NT: the accesses pass the Infinity Cache by, which then keeps no
// lines that the pass would evict before they are used again, and does not write them back in their own order.
// us per pass with the bf16 image (42 M, 128 M, 437 M, 2.43 G parameters): strided 268, 958, 2773, 15068; window 245,
// 731, 2473, 13860; NT in workgroups of 256 226, 657, 2387, 13707, of 1024 203, 614, 2349, 13315 (6.3 TB/s at 128 M).
template <bool BF, bool NT, int T>
__global__ __launch_bounds__(T) void adam_step_kernel(float *__restrict__ w, bf16_t *__restrict__ p,
                                                      const float *__restrict__ g, float *__restrict__ m,
                                                      float *__restrict__ v, size_t count, AdamScalars a) {
  const size_t n4 = count >> 2, stride = (size_t)gridDim.x * T;
  for (size_t i = (size_t)blockIdx.x * T + threadIdx.x; i < n4; i += stride) {
    const float4 gg = load4<NT>(g, i);
    float4 mm = load4<NT>(m, i), vv = load4<NT>(v, i), ww = load4<NT>(w, i);
    ww.x = adam_one(gg.x, mm.x, vv.x, ww.x, a);
    ww.y = adam_one(gg.y, mm.y, vv.y, ww.y, a);
    ww.z = adam_one(gg.z, mm.z, vv.z, ww.z, a);
    ww.w = adam_one(gg.w, mm.w, vv.w, ww.w, a);
    store4<NT>(m, i, mm);
    store4<NT>(v, i, vv);
    store4<NT>(w, i, ww);
    if constexpr (BF) {  // (the forward pass reads it next: through the cache)
      uint2 q;
      q.x = pack_bf16x2(ww.x, ww.y);
      q.y = pack_bf16x2(ww.z, ww.w);
      reinterpret_cast<uint2 *>(p)[i] = q;
    }
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == T - 1)
    for (size_t i = n4 << 2; i < count; ++i) {
      float mm = m[i], vv = v[i];
      const float ww = adam_one(g[i], mm, vv, w[i], a);
      m[i] = mm; v[i] = vv; w[i] = ww;
      if constexpr (BF) p[i] = f32_to_bf16(ww);
    }
}

}  // namespace
}  // namespace il

extern "C" {

double il_lr_schedule(int64_t step, int32_t d_model, int32_t warmup_steps) {
  if (step < 1 || d_model < 1 || warmup_steps < 1) return 0.0;
  const double s = (double)step, w = (double)warmup_steps;
  return std::pow((double)d_model, -0.5) * std::fmin(std::pow(s, -0.5), s * std::pow(w, -1.5));
}

int il_adam_step(int32_t dtype, void *params, float *master, const float *grads, float *m, float *v,
                 size_t count, int64_t step, float lr, float beta1, float beta2, float eps, void *stream) {
  using namespace il;
  if (dtype != IL_F32 && dtype != IL_BF16) return IL_E_ARG;
  if (!params || !grads || !m || !v || step < 1) return IL_E_ARG;
  if ((dtype == IL_BF16) != (master != nullptr)) return IL_E_ARG;
  if (!(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f) || !(eps >= 0.f) || !(lr >= 0.f))
    return IL_E_ARG;
  float *w = dtype == IL_BF16 ? master : (float *)params;
  if (((uintptr_t)w | (uintptr_t)grads | (uintptr_t)m | (uintptr_t)v) & 15) return IL_E_SHAPE;
  if (dtype == IL_BF16 && ((uintptr_t)params & 7)) return IL_E_SHAPE;
  if (count == 0) return IL_OK;
  AdamScalars a;
  a.b1 = beta1; a.b2 = beta2; a.omb1 = 1.f - beta1; a.omb2 = 1.f - beta2;
  a.c1 = (float)(1.0 / (1.0 - std::pow((double)beta1, (double)step)));   // bias corrections in double
  a.c2 = (float)(1.0 / (1.0 - std::pow((double)beta2, (double)step)));
  a.lr = lr; a.eps = eps;
  // Buffers that the 256 MB Infinity Cache holds for the most part stay in it, larger ones go past it.  us, in windows
  // and NT: 16 M parameters 72 and 79 (fp32 mode 63 and 73), 18 M 79 and 87 (72 and 81), 20 M 101 and 96 (85 and 93),
  // 24 M 140 and 116 (121 and 108).
  const bool nt = count > kCachedBytes / (dtype == IL_BF16 ? 18 : 16);
  const size_t T = nt ? 1024 : 256;
  size_t blocks = ((count >> 2) + T - 1) / T;
  if (blocks < 1) blocks = 1;
  if (blocks > (1u << 21)) blocks = 1u << 21;  // (a launch's threads are counted in 32 bits; strided beyond)
  hipStream_t s = (hipStream_t)stream;
#define IL_ADAM(BF, NT, T)                                                                                    \
  hipLaunchKernelGGL((adam_step_kernel<BF, NT, T>), dim3((unsigned)blocks), dim3(T), 0, s, w, (bf16_t *)params, \
                     grads, m, v, count, a)
  if (dtype == IL_BF16) {
    if (nt) IL_ADAM(true, true, 1024); else IL_ADAM(true, false, 256);
  } else {
    if (nt) IL_ADAM(false, true, 1024); else IL_ADAM(false, false, 256);
  }
#undef IL_ADAM
  return hipGetLastError() == hipSuccess ? IL_OK : IL_E_HIP;
}

}  // extern "C"
