/*
 * interlock_test.h - test and profiling hooks of libinterlock.  Not part of the training-step
 * boundary (interlock.h): these two calls exist so that tests and micro-benchmarks can reach single
 * kernels and per-kernel-class timings.  Same conventions: device pointers owned by the caller,
 * every function returns a status code or a count, nothing is printed.
 */
#ifndef INTERLOCK_TEST_H
#define INTERLOCK_TEST_H

#include "interlock.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Profiling (cfg.profile != 0): synchronises the stream and returns, per kernel class,
 * launches and total milliseconds since the last call, measured with HIP events recorded
 * on the library's stream before and after each launch group (`ms`; this includes the few
 * microseconds an event costs between launches), the algorithmic flops and bytes of those
 * launches, and for the bf16 GEMM classes `kernel_ms`: the execution time of the MFMA GEMM
 * kernels alone, from events attached to each dispatch (0 for the other classes).  With
 * cfg.profile == 1 everything runs on the caller's stream (no internal side stream); with
 * cfg.profile == 2 the step runs on both streams as it does unprofiled and only `kernel_ms`,
 * the launches, flops and bytes of the GEMM classes are filled (`ms` stays 0): the GEMM kernels'
 * durations inside the real step, other kernels running beside them.
 * `names` receives pointers to static strings; any output array may be NULL.  Returns the
 * number of classes written (<= cap), or a negative status code.
 */
int il_profile_read(il_ctx *ctx, int32_t cap, const char **names, int64_t *launches, double *ms,
                    double *flops, double *bytes, double *kernel_ms);

/*
 * Kernel-level test hook: one GEMM launch of the library's own kernels, outside any step, so
 * that tests and micro-benchmarks can reach each tile configuration and epilogue directly.
 *   C[M,N] = epilogue( sum_k A(m,k) B(k,n) )
 * dtype: il_dtype of A, B (and of C for the bf16/fp32-typed epilogues, see `epi`);
 * a_kmajor / b_kmajor: 0 = operand stored [rows, K] row-major, 1 = stored [K, rows] row-major;
 * epi: 0 store (T) | 1 +bias (T) | 2 +bias, C = pre-activation, C2 = GELU (T, T) |
 *      3 +bias +res (fp32 out) | 4 * GELU'(aux[row % aux_wrap]) (T) | 5 store fp32 |
 *      6 C = scale*acc (+ C if beta) (fp32) | 7 the head's logits tile (bf16 operands, forward layout only, not
 *      the 64x64 tiles): C = acc as IEEE half, clamped to the finite range; if C2 is given also the softmax
 *      statistics of the fp32 accumulators: C2 = fp32 [M][G][2], G = ceil(N / 64), (max, sum of exp(z - max)) of
 *      every group of 64 columns, followed by fp32 [M] target logits z[row, aux[row]] with aux = int32 [M]
 *      targets (rows whose target is outside [0, N) are left unwritten) |
 *      8 store (T) and, in C2 = fp32 [N / 32][M], the sums over 32 columns each of C as stored times
 *      aux[row % aux_wrap] (bf16 operands, N a multiple of 32, data-gradient layout only) |
 *      9 as 4 for `beta` (1 or 2) streams stacked over M / beta rows, a multiple of 64, aux with as many rows, ldc = N
 *      (bf16, data-gradient layout only): C2 = bf16 [M / beta][N], scale * stream 0 + stream 1 of C as stored, followed
 *      by fp32 [M / beta / 64][N], its column sums over runs of 64 rows before it was rounded;
 * tile: 0 = library's choice, else for fp32 2 = 128x128, 3 = 128x64, any other 64x64 (operands whose rows do not
 *       divide by four always take the last), and for bf16 ("+4" = four wavefronts that only load)
 *       1 = 256x256 / 8 wavefronts in two groups that take turns, 2 = 128x128 / 4+4, two K steps staged, 3 = 128x128 / 4+4, four staged,
 *       4 = 64x64 / 4 wavefronts, 5 = 64x64 / 4+4, four staged, 6 = 256x128 / 8+4, three staged,
 *       7 = 128x256 / 8+4, three staged, 8 = the same as 1.
 * All pointers are device pointers; unused ones may be NULL.  Returns an il_status.
 */
int il_test_gemm(int32_t dtype, const void *A, const void *B, int32_t M, int32_t N, int32_t K, int32_t lda,
                 int32_t ldb, int32_t a_kmajor, int32_t b_kmajor, int32_t epi, void *C, void *C2, int32_t ldc,
                 const void *bias, const float *res, const void *aux, int32_t aux_wrap, float scale,
                 int32_t beta, int32_t tile, void *stream);

/*
 * Kernel-level test hook: C[M,N] (fp32, row pitch ldc) = A[M,K] B[N,K]^T with K in `splits` parts (fewer if a part
 * would be empty), each a whole number of 64-deep steps, whose products go to ws (fp32 [splits][M][N]) and are added
 * up in order; with the plan of a head's dx: il_gemm_split_plan returns the number of parts the library would choose
 * within ws_floats, and the tile through *tile.  N and ldc multiples of 4; otherwise as il_test_gemm.
 */
int il_test_gemm_splitk(int32_t dtype, const void *A, const void *B, int32_t M, int32_t N, int32_t K, int32_t splits,
                        int32_t tile, float *ws, float *C, int32_t ldc, void *stream);
int il_gemm_split_plan(int32_t dtype, int32_t M, int32_t N, int32_t K, size_t ws_floats, int32_t *tile);

/*
 * Host function: the output tile (*tile_m, *tile_n) that a GEMM launch of tiles_m x tiles_n tiles of edge_m x edge_n
 * over K (in one part) gives its workgroup number `workgroup`.
 */
int il_gemm_tile_of(int32_t tiles_m, int32_t tiles_n, int32_t edge_m, int32_t edge_n, int32_t K, int32_t workgroup,
                    int32_t *tile_m, int32_t *tile_n);

/*
 * Kernel-level test hook: the library's causal attention by itself.
 * qkv: dtype [batch*seq, 3*heads*width] (Q | K | V, heads contiguous); o: dtype [batch*seq, heads*width]; lse: fp32
 * [batch, heads, seq] (in the unit the backward of the same dtype and width wants).  The forward always runs;
 * the backward follows if d_o (dtype [streams*batch*seq, heads*width]) is given, into dqkv (dtype
 * [streams*batch*seq, 3*heads*width]).  dsum: fp32 [streams*batch*seq * max(heads, heads*width/32)], scratch -
 * except where il_attention_wants_dsum() is 1: there the caller provides the row sums of d_o * o over 32 columns
 * each, [heads*width/32][streams*batch*seq], as the GEMM that makes d_o leaves them (with o of an earlier call).
 * IL_E_SHAPE: the widths and extents il_init refuses, or streams outside [1, 16].
 */
int il_test_attention(int32_t dtype, const void *qkv, int32_t batch, int32_t seq, int32_t heads, int32_t width,
                      void *o, float *lse, const void *d_o, int32_t streams, void *dqkv, float *dsum, void *stream);
int il_attention_wants_dsum(int32_t dtype, int32_t width);
/*
 * Host function: the kernels that such a call takes, the forward (streams = 0) or the backward.  *form receives 0: a
 * workgroup's four wavefronts share tiles of the other axis; 2, 4 or 8: that many wavefronts divide it up; -1: two wavefronts
 * share tiles (forward); -2: as 0, two streams to a workgroup (backward).  Same errors as il_test_attention.
 */
int il_attention_form(int32_t dtype, int32_t width, int32_t batch, int32_t seq, int32_t heads, int32_t streams, int32_t *form);

/*
 * Kernel-level test hook: one LayerNorm forward.  x: fp32 [rows, d]; gamma, beta: dtype [d]; y: dtype [rows, d]; stats:
 * fp32 [rows, 2], mean and 1 / sqrt(variance + eps); xcopy: fp32 [rows, d], a copy of x, or NULL.  d <= 2048.
 */
int il_test_layernorm(int32_t dtype, const float *x, const void *gamma, const void *beta, float eps, int32_t rows, int32_t d,
                      void *y, float *stats, float *xcopy, void *stream);

/*
 * Kernel-level test hook: one LayerNorm backward of `streams` (1 to 16) gradient streams stacked over `tokens` rows.
 * dy: dtype [streams * tokens, d]; x, stats, gamma: the forward's; G: fp32 [streams * tokens, d], to which the gradient at x
 * is added; Gb: G as dtype; weights: streams floats (host); partials: fp32 [512][2 d], of which *blocks rows are written:
 * partial column sums of weight * dy * xhat and of weight * dy.  If ypart (fp32 [512][d]) is given, *summed says
 * whether the weighted sum of the streams' Gb was formed (d > 256, divisible by four, vectors aligned): its partial column sums, *blocks rows of ypart, and the sum
 * itself, dtype [tokens, d], in ysum unless that is NULL.
 */
int il_test_layernorm_backward(int32_t dtype, const void *dy, const float *x, const float *stats, const void *gamma, int32_t streams,
                               int32_t tokens, int32_t d, float *G, void *Gb, const float *weights, float *partials, void *ysum,
                               float *ypart, int32_t *blocks, int32_t *summed, void *stream);

/* ---- measured peaks of the board (reported beside the nominal 2.5 PFLOP/s and 8 TB/s) ------------- */

/*
 * Matrix-unit-only loop: 512 workgroups of four wavefronts, each issuing `iters` x 4 independent
 * v_mfma_f32_32x32x16_bf16 on register operands (no memory traffic), timed with HIP events on `stream`
 * (the call synchronises).  scratch: device, at least 1 KiB (never written in practice).
 * *tflops_out receives the achieved dense bf16 TFLOP/s.  IL_E_ARG for NULL pointers or iters outside
 * [1, 2^22].
 */
int il_measure_mfma_peak(float *scratch, int32_t iters, void *stream, double *tflops_out);

/*
 * Streaming copy dst[0..bytes) = src[0..bytes) in two forms, each run for `reps` launches after one
 * warm-up launch and timed with HIP events on `stream` (the call synchronises): `stream_copy_kernel`
 * (16 bytes per lane, plain loads and stores) and `stream_copy4_kernel` (four 16-byte vectors in flight
 * per lane, non-temporal loads and stores).  *gbs_out receives the better (bytes read + bytes written) /
 * time in GB/s.  Each launch reads and writes exactly `bytes`, so `stream_copy_kernel` is also the kernel
 * of known traffic against which a profiler's HBM byte counters are scaled.  dst and src are device
 * pointers, 16-byte aligned, bytes a multiple of 16 (IL_E_SHAPE otherwise); they may not overlap.
 */
int il_measure_copy_peak(void *dst, const void *src, size_t bytes, int32_t reps, void *stream, double *gbs_out);

#ifdef __cplusplus
}
#endif
#endif /* INTERLOCK_TEST_H */
