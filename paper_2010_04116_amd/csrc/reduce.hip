// Small bandwidth-bound helpers: deterministic two-stage column sums (bias gradients,
// LayerNorm gain/bias gradients), gradient-stream injection / combination, fp32 -> T
// conversion.  No float atomics anywhere: every reduction has a fixed order.
#include <cstdint>

#include "common.h"

namespace il {
namespace {

constexpr int kColBlocksY = 64;   // row splits of the first stage

// V consecutive elements, V * sizeof(T) = 16 bytes (or V = 1)
template <typename T, int V>
__device__ inline void load_vec(const T *p, float (&o)[V]) {
  if constexpr (V == 8) {
    const uint4 q = *reinterpret_cast<const uint4 *>(p);
    const uint32_t u[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      o[2 * e] = bf16_to_f32((bf16_t)(u[e] & 0xFFFF));
      o[2 * e + 1] = bf16_to_f32((bf16_t)(u[e] >> 16));
    }
  } else if constexpr (V == 4) {
    const float4 q = *reinterpret_cast<const float4 *>(p);
    o[0] = q.x; o[1] = q.y; o[2] = q.z; o[3] = q.w;
  } else {
    o[0] = ld<T>(p);
  }
}
template <typename T, int V>
__device__ inline void store_vec(T *p, const float (&v)[V]) {
  if constexpr (V == 8) {
    uint4 q;
    q.x = pack_bf16x2(v[0], v[1]);
    q.y = pack_bf16x2(v[2], v[3]);
    q.z = pack_bf16x2(v[4], v[5]);
    q.w = pack_bf16x2(v[6], v[7]);
    *reinterpret_cast<uint4 *>(p) = q;
  } else if constexpr (V == 4) {
    *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]);
  } else {
    st<T>(p, v[0]);
  }
}

// First stage, fused with the weighted sum over gradient streams: for every token row the kernel
// forms the job's weighted sum of streams in fp32, optionally stores it (rounded to T) for the
// weight-gradient GEMM, and accumulates its column sums (the bias gradient).  ysum may lie on one of the
// streams: a thread has read its elements of all of them before it writes.  Bound by the bytes it
// reads and writes.  Grid (column groups, row splits, jobs); block = 32 column groups of V x 8 row
// lanes with 16-byte accesses (V = 1: 64 columns x 4 row lanes, for columns that do not divide).
template <typename T, int V>
__global__ __launch_bounds__(256) void sum_colsum_kernel(SumColsumJobs jobs) {
  constexpr int CG = V > 1 ? 32 : 64, RL = 256 / CG;
  __shared__ float red[RL][CG * V];
  const SumColsumJob &jb = jobs.job[blockIdx.z];
  const SumTable &tab = jobs.table[jb.table];
  const T *Y = (const T *)jb.Y;
  T *ysum = (T *)jb.ysum;
  float *__restrict__ partials = jb.partials;
  const int N = jobs.N, cols = jb.cols, ns = tab.ns;
  if ((int)blockIdx.x * CG * V >= cols) return;  // uniform: this job is narrower than the widest one
  const int tx = threadIdx.x % CG, ty = threadIdx.x / CG;
  const int c = (blockIdx.x * CG + tx) * V;
  const int per = (N + gridDim.y - 1) / gridDim.y;
  const int r0 = blockIdx.y * per, r1 = min(N, r0 + per);
  float acc[V];
#pragma unroll
  for (int e = 0; e < V; ++e) acc[e] = 0.f;
  if (c < cols)
    for (int r = r0 + ty; r < r1; r += RL) {
      float v[V];
#pragma unroll
      for (int e = 0; e < V; ++e) v[e] = 0.f;
      for (int si = 0; si < ns; ++si) {
        float y[V];
        load_vec<T, V>(Y + ((size_t)tab.row[si] * N + r) * cols + c, y);
#pragma unroll
        for (int e = 0; e < V; ++e) v[e] += tab.w[si] * y[e];
      }
      if (ysum) store_vec<T, V>(ysum + (size_t)r * cols + c, v);
#pragma unroll
      for (int e = 0; e < V; ++e) acc[e] += v[e];
    }
#pragma unroll
  for (int e = 0; e < V; ++e) red[ty][tx * V + e] = acc[e];
  __syncthreads();
  for (int i = threadIdx.x; i < CG * V; i += 256) {
    const int cc = blockIdx.x * CG * V + i;
    if (cc < cols) {
      float v = 0.f;
#pragma unroll
      for (int y = 0; y < RL; ++y) v += red[y][i];
      partials[(size_t)blockIdx.y * cols + cc] = v;
    }
  }
}

// four elements of fp32 (T) at 16 (8) bytes
__device__ inline void store4(float *p, float4 v) { *reinterpret_cast<float4 *>(p) = v; }
__device__ inline void store4(bf16_t *p, float4 v) {
  *reinterpret_cast<uint2 *>(p) = make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
}

// Elementwise passes, bound by their bytes: `quads` groups of four per grid, the last count % 4 elements by
// the grid's last threads (quads = 0: element by element, for addresses off 16 bytes).
template <typename T>
__global__ __launch_bounds__(256) void inject_kernel(const float *__restrict__ src, float *G, T *Gb, size_t quads,
                                                     size_t count, int accumulate) {
  const size_t first = (size_t)blockIdx.x * 256 + threadIdx.x, step = (size_t)gridDim.x * 256;
  for (size_t i = first; i < quads; i += step) {
    float4 v = reinterpret_cast<const float4 *>(src)[i];
    if (accumulate) {
      const float4 g = reinterpret_cast<const float4 *>(G)[i];
      v.x += g.x; v.y += g.y; v.z += g.z; v.w += g.w;
    }
    reinterpret_cast<float4 *>(G)[i] = v;
    store4(Gb + 4 * i, v);
  }
  for (size_t i = 4 * quads + first; i < count; i += step) {
    const float v = src[i] + (accumulate ? G[i] : 0.f);
    G[i] = v;
    st<T>(Gb + i, v);
  }
}

__global__ __launch_bounds__(256) void combine_kernel(const float *__restrict__ G, size_t stride, int nstreams,
                                                      StreamWeights sw, float *__restrict__ out, size_t quads,
                                                      size_t count, int accumulate) {
  const size_t first = (size_t)blockIdx.x * 256 + threadIdx.x, step = (size_t)gridDim.x * 256;
  for (size_t i = first; i < quads; i += step) {
    float4 v = accumulate ? reinterpret_cast<const float4 *>(out)[i] : make_float4(0.f, 0.f, 0.f, 0.f);
    for (int j = 0; j < nstreams; ++j) {
      const float4 g = reinterpret_cast<const float4 *>(G + (size_t)j * stride)[i];
      const float w = sw.w[j];
      v.x += w * g.x; v.y += w * g.y; v.z += w * g.z; v.w += w * g.w;
    }
    reinterpret_cast<float4 *>(out)[i] = v;
  }
  for (size_t i = 4 * quads + first; i < count; i += step) {
    float v = accumulate ? out[i] : 0.f;
    for (int j = 0; j < nstreams; ++j) v += sw.w[j] * G[(size_t)j * stride + i];
    out[i] = v;
  }
}

template <typename T>
__global__ __launch_bounds__(256) void convert_kernel(const float *__restrict__ src, T *__restrict__ dst,
                                                      size_t quads, size_t count) {
  const size_t first = (size_t)blockIdx.x * 256 + threadIdx.x, step = (size_t)gridDim.x * 256;
  for (size_t i = first; i < quads; i += step) store4(dst + 4 * i, reinterpret_cast<const float4 *>(src)[i]);
  for (size_t i = 4 * quads + first; i < count; i += step) st<T>(dst + i, src[i]);
}

__global__ __launch_bounds__(256) void sum_scalar_kernel(const float *__restrict__ v, int n, float scale,
                                                         float *__restrict__ out) {
  constexpr int U = 8;  // loads in flight per thread
  __shared__ float red[256];
  float acc = 0.f;
  for (int i0 = threadIdx.x; i0 < n; i0 += 256 * U) {
    float x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = i0 + 256 * u < n ? v[i0 + 256 * u] : 0.f;
#pragma unroll
    for (int u = 0; u < U; ++u) acc += x[u];
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = red[0] * scale;
}

inline size_t quads_for(size_t count, const void *a, const void *b, const void *c) {
  return (((uintptr_t)a | (uintptr_t)b | (uintptr_t)c) & 15) ? 0 : count / 4;
}
inline int grid_for(size_t quads, size_t count) {
  const size_t b = ((quads ? quads : count) + 255) / 256;
  return (int)(b > 4096 ? 4096 : (b ? b : 1));
}

}  // namespace

int colsum_max_blocks() { return kColBlocksY; }
hipError_t sum_colsum_multi(int dtype, const SumColsumJobs &jobs, int *nblk, hipStream_t s) {
  if (jobs.count < 1 || jobs.count > kMaxSumColsumJobs) return hipErrorInvalidValue;
  int nby = (jobs.N + 31) / 32;
  if (nby > kColBlocksY) nby = kColBlocksY;
  *nblk = nby;
  const int v = dtype == 0 ? 4 : 8;
  int maxc = 0;
  bool vec = true;
  for (int i = 0; i < jobs.count; ++i) {
    const SumColsumJob &j = jobs.job[i];
    if (j.table < 0 || j.table >= kMaxSumTables || jobs.table[j.table].ns > kMaxStreams) return hipErrorInvalidValue;
    maxc = j.cols > maxc ? j.cols : maxc;
    vec = vec && j.cols % v == 0;
  }
  const dim3 grid(vec ? (maxc + 32 * v - 1) / (32 * v) : (maxc + 63) / 64, nby, jobs.count);
  if (dtype == 0) {
    if (vec) hipLaunchKernelGGL((sum_colsum_kernel<float, 4>), grid, dim3(256), 0, s, jobs);
    else hipLaunchKernelGGL((sum_colsum_kernel<float, 1>), grid, dim3(256), 0, s, jobs);
  } else {
    if (vec) hipLaunchKernelGGL((sum_colsum_kernel<bf16_t, 8>), grid, dim3(256), 0, s, jobs);
    else hipLaunchKernelGGL((sum_colsum_kernel<bf16_t, 1>), grid, dim3(256), 0, s, jobs);
  }
  return hipGetLastError();
}

// Several second stages in one launch: grid.y selects the job.  Block = 16 columns x 16 partial lanes;
// fixed summation order.  A thread has up to 32 partials to add and nothing else to do: bound by the latency of
// its loads, so eight are in flight.
__global__ __launch_bounds__(256) void colsum_final_multi_kernel(ColsumJobs jobs) {
  constexpr int U = 8;
  __shared__ float red[16][17];
  const ColsumJob &jb = jobs.job[blockIdx.y];
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const int c = blockIdx.x * 16 + tx;
  if (blockIdx.x * 16 >= jb.cols) return;  // uniform across the block
  float acc = 0.f;
  if (c < jb.cols) {
    const float *__restrict__ col = jb.partials + c;
    for (int p0 = ty; p0 < jb.nblk; p0 += 16 * U) {
      float v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = p0 + 16 * u < jb.nblk ? col[(size_t)(p0 + 16 * u) * jb.cols] : 0.f;
#pragma unroll
      for (int u = 0; u < U; ++u) acc += v[u];
    }
  }
  red[ty][tx] = acc;
  __syncthreads();
  if (ty == 0 && c < jb.cols) {
    float v = jb.accumulate ? jb.out[c] : 0.f;
#pragma unroll
    for (int y = 0; y < 16; ++y) v += red[y][tx];
    jb.out[c] = v;
  }
}

hipError_t colsum_final_multi(const ColsumJobs &jobs, hipStream_t s) {
  if (jobs.count < 1) return hipSuccess;
  if (jobs.count > kMaxColsumJobs) return hipErrorInvalidValue;
  int maxc = 0;
  for (int i = 0; i < jobs.count; ++i) maxc = jobs.job[i].cols > maxc ? jobs.job[i].cols : maxc;
  hipLaunchKernelGGL(colsum_final_multi_kernel, dim3((maxc + 15) / 16, jobs.count), dim3(256), 0, s, jobs);
  return hipGetLastError();
}

hipError_t stream_inject(int dtype, const float *src, float *G, void *Gb, size_t count, int accumulate,
                         hipStream_t s) {
  const size_t quads = quads_for(count, src, G, Gb);
  if (dtype == 0)
    hipLaunchKernelGGL(inject_kernel<float>, dim3(grid_for(quads, count)), dim3(256), 0, s, src, G, (float *)Gb, quads,
                       count, accumulate);
  else
    hipLaunchKernelGGL(inject_kernel<bf16_t>, dim3(grid_for(quads, count)), dim3(256), 0, s, src, G, (bf16_t *)Gb,
                       quads, count, accumulate);
  return hipGetLastError();
}

hipError_t stream_combine(const float *G, size_t stride, int nstreams, StreamWeights sw, float *out,
                          size_t count, int accumulate, hipStream_t s) {
  const size_t quads = (stride & 3) ? 0 : quads_for(count, G, out, out);
  hipLaunchKernelGGL(combine_kernel, dim3(grid_for(quads, count)), dim3(256), 0, s, G, stride, nstreams, sw, out,
                     quads, count, accumulate);
  return hipGetLastError();
}

hipError_t convert_f32(int dtype, const float *src, void *dst, size_t count, hipStream_t s) {
  const size_t quads = quads_for(count, src, dst, dst);
  if (dtype == 0)
    hipLaunchKernelGGL(convert_kernel<float>, dim3(grid_for(quads, count)), dim3(256), 0, s, src, (float *)dst, quads,
                       count);
  else
    hipLaunchKernelGGL(convert_kernel<bf16_t>, dim3(grid_for(quads, count)), dim3(256), 0, s, src, (bf16_t *)dst,
                       quads, count);
  return hipGetLastError();
}

hipError_t sum_scalar(const float *rowloss, int rows, float scale, float *loss_out, hipStream_t s) {
  hipLaunchKernelGGL(sum_scalar_kernel, dim3(1), dim3(256), 0, s, rowloss, rows, scale, loss_out);
  return hipGetLastError();
}

}  // namespace il
