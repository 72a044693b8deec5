/*
 * dfa_bench.h - measurement aids of the dilated flash attention library.  They are exported by the
 * same shared library but are no part of the operator's interface (dfa.h): a benchmark harness times
 * launches with them and measures what the matrix cores sustain on their own.
 */
#ifndef DFA_BENCH_H
#define DFA_BENCH_H

#include "dfa.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Times `iters` back-to-back dfa_forward launches with HIP events recorded on `stream`
 * (the stream the kernel runs on) and returns the mean milliseconds per launch in *ms.
 * Arguments as dfa_forward.  Synchronises `stream`.  For benchmarks.
 */
int dfa_forward_timed(const void *q, const void *k, const void *v,
                      dfa_strides_t sq, dfa_strides_t sk, dfa_strides_t sv,
                      int32_t B, int32_t H, int32_t N, int32_t D, dfa_dtype_t dt, float scale,
                      const dfa_branch_t *branches, int32_t nb, const int32_t *head_offsets,
                      void *out, float *lse, void *workspace, size_t workspace_bytes, void *stream,
                      int32_t iters, float *ms);

/*
 * Comparison path of the input-size sweep: dense softmax attention over all N tokens (Eq. 2 with one segment,
 * w = N, r = 1) computed the plain way, with the score matrix held in memory - the "FlashAttention off" side of
 * the paper's ablation (section 4.3, Fig. 4).  Four launches on `stream`: S = Q K^T (batched matrix-core
 * product), row softmax in place, a transpose of V, O = P V.
 *   q, k, v, strides, B, H, N, D, scale   as in dfa_forward, bf16 only; N % 256 == 0 and N <= 4096
 *   out         device bf16 [B, N, H, D];  lse device fp32 [B, H, N] or NULL
 *   workspace   device, 16-byte aligned, dfa_dense_unfused_workspace_bytes() = room for the bf16 scores
 *               [B, H, N, N] and V^T [B, H, D, N]; DFA_ERR_WORKSPACE when smaller
 * Scores and probabilities are rounded to bf16 on their way through memory.
 */
size_t dfa_dense_unfused_workspace_bytes(int32_t B, int32_t H, int32_t N, int32_t D);
int dfa_dense_unfused(const void *q, const void *k, const void *v,
                      dfa_strides_t sq, dfa_strides_t sk, dfa_strides_t sv,
                      int32_t B, int32_t H, int32_t N, int32_t D, float scale,
                      void *out, float *lse, void *workspace, size_t workspace_bytes, void *stream);

/*
 * Which kernels a call launches for a shape, and with which plan (no GPU needed).  The library picks the form by its
 * own estimate of the times, so this is what tests and benchmarks ask when they mean one form in particular.
 *   backward   0: dfa_forward (dfa_forward_static, dfa_encoder_stack), 1: dfa_backward
 *   launch     out, host
 *   tiles, rows, segs, block_mult, items   out, host, NULL to skip: as dfa_plan_describe_forward, of the plan that is
 *              launched.  Where launch->cut is set every entry of segs is a block of at most 32 keys (one of a single key
 *              has stride 0).
 */
#define DFA_FORM_TILES 0    /* bf16: tiles of 256 rows; fp32: tiles of 256 or of 32 rows */
#define DFA_FORM_SHORT 1    /* bf16: tiles of 64 rows, whose walk is shared out inside the workgroup */
#define DFA_FORM_SPLIT 2    /* bf16 forward: tiles of 256 rows, walks shared out over workgroups (DFA_FORM_TILES without a workspace) */
typedef struct {
    int32_t form;           /* DFA_FORM_* */
    int32_t packed;         /* some tile packs several row groups */
    int32_t cut;            /* the key lists are cut into blocks */
    int32_t n_tiles, n_rows, n_segs, n_items;
    int64_t threads;        /* of the call's largest kernel launch (a grid holds fewer than 2^32) */
} dfa_launch_t;
int dfa_launch_describe(int32_t backward, dfa_dtype_t dt, int32_t B, int32_t H, int32_t N,
                        const dfa_branch_t *branches, int32_t nb, const int32_t *head_offsets, dfa_launch_t *launch,
                        int32_t *tiles, int32_t *rows, int32_t *segs, int32_t *block_mult, int32_t *items);

/*
 * The same plan as its kernels read it in device memory, for tests of that layout (no GPU needed).  Arguments as dfa_launch_describe.
 *   image   out, host: the plan's size and where its parts are (bytes from its start).  start_bytes > 0: a short forward, whose plan is
 *           one record of that many bytes per workgroup; otherwise rows at 0, segs, items, and of a split forward the shares of its
 *           n_shares workgroups, each one's item, and the blocks of partial results of each item
 *   bytes   out, host, NULL to skip: image->bytes bytes
 */
typedef struct {
    int64_t bytes, start_bytes, segs, items, shares, share_items, item_parts, block_mult, n_shares;
} dfa_launch_image_t;
int dfa_launch_image(int32_t backward, dfa_dtype_t dt, int32_t B, int32_t H, int32_t N,
                     const dfa_branch_t *branches, int32_t nb, const int32_t *head_offsets, dfa_launch_image_t *image, void *bytes);

/*
 * Measurement aid (no part of the operator): what the matrix cores sustain on their own, the
 * ceiling that the kernels' MFMA rooflines are also quoted against.  Runs a loop of
 * independent v_mfma_f32_32x32x16_bf16 on the whole chip (two waves per SIMD, no memory
 * traffic) on the default stream and synchronises.
 *   random_operands  0: small constant operands; 1: pseudo-random bf16 operands (more bits
 *                    toggle, the sustained clock is lower)
 *   tflops           out, host: achieved TFLOP/s
 *   shader_mhz       out, host: shader clock during the loop (cycle counter / 100 MHz wall counter)
 * Allocates and frees a few bytes of device memory.
 */
int dfa_mfma_peak(int32_t random_operands, float *tflops, float *shader_mhz);

#ifdef __cplusplus
}
#endif
#endif /* DFA_BENCH_H */
