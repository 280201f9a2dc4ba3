/*
 * alr_debug.h -- kernel-level test hooks of the rollout library.
 *
 * These entry points expose single kernels of the library so that tests can
 * check them in isolation and benchmarks can time them.  They are not needed
 * to run the rollout.
 */
#ifndef ALR_DEBUG_H
#define ALR_DEBUG_H

#include <stdint.h>

#include "alr.h"

#ifdef __cplusplus
extern "C" {
#endif

/* C[M,N] (fp32, row-major) = A[M,K] * W[N,K]^T, on the library's GEMM kernel
 * for `dtype` (ALR_BF16: bf16 MFMA with fp32 accumulation; ALR_F32: fp32 FMA).
 * A, W, C are device pointers, row-major and contiguous; N and K must be
 * multiples of 64 (ALR_E_UNSUPPORTED otherwise).  `tile` picks the bf16
 * kernel: 0 = the library's choice for this shape; W staged through LDS:
 * 1 = 256x128, 2 = 128x128, 3 = 64x128, 4 = 256x256 (8 waves), 5 = 256x256
 * (4 waves); 17 = 256x256 with the operands copied straight into LDS and a
 * hand-scheduled K loop, one tile per workgroup; 18 = split-K over that kernel
 * (K slices of at least 192 summed in slice order by a second kernel; 2 or 4
 * slices, the unsplit kernel when K allows none); 19 = the kernel of 17 run
 * persistently (one workgroup per CU looping over the tiles, the next tile's
 * first K steps copied during the current tile's epilogue); 20 = split-K over the
 * 64x128 kernel of 3 (2 or 4 slices, each a multiple of 64; the unsplit kernel of
 * 3 when K allows no split); 21 = 19 with the tiles past the last full round of
 * one tile per CU cut over K, into as many slices (of at least 192) as idle CUs
 * and the scratch (256 KB a slice of a tile) allow.  17 to 19 and 21 run as 3
 * when K < 192.  Other values: ALR_E_INVALID_ARG.  Tiles 18 and 20 need a device
 * scratch buffer of at least 2*M*N*4 bytes for the partial sums (up to 4*M*N*4
 * are used when given), tile 21 one of any size; ALR_E_WORKSPACE otherwise.
 * Enqueued on `stream`. */
alr_status alr_debug_gemm(int32_t dtype, const void* A, const void* W, float* C, int32_t M,
                          int32_t N, int32_t K, int32_t tile, void* scratch,
                          size_t scratch_bytes, alr_stream stream);

/* Work plan of the decode attention for a rollout request (host only, no GPU
 * needed; the same planner alr_rollout runs).  n_seq sequences of lengths
 * seq_len[] laid out as alr_prefill lays them out (keys of sequence i from the
 * sum of the earlier lengths; its transposed values from the sum of the
 * earlier lengths each rounded up to 64), n_anchor anchors as for
 * alr_check_rollout, a device of n_cu compute units.  Writes the key-chunk
 * length in 64-key tiles to *ct_out, the simulated makespan (tiles, an item
 * costing its tiles + 3) to *makespan_out and the number of work items,
 * padding included, to *n_items_out; if items_out is not NULL, item b (run on
 * XCD b % 8) as 6 int32 at items_out[6 b]: first anchor in sorted order (by
 * sequence, then position, then the caller's index), anchor count (0 for
 * padding), kv head, first key, end key (exclusive), partial-output index.
 * ALR_E_UNSUPPORTED when the config's attention has no plan (fp32, or a head
 * size other than 64 and 128), ALR_E_WORKSPACE when the items exceed
 * max_items, the statuses of alr_check_config / alr_check_rollout otherwise. */
alr_status alr_debug_decode_plan(const alr_config* cfg, int32_t n_cu, int32_t n_seq,
                                 const int32_t* seq_len, int32_t n_anchor,
                                 const int32_t* anchor_seq, const int32_t* anchor_pos,
                                 int32_t* ct_out, int32_t* makespan_out, int32_t* n_items_out,
                                 int32_t* items_out, int32_t max_items);

/* Kernel launch sites whose device time can be measured with alr_profile_*. */
typedef enum {
  ALR_PROF_PREFILL_QKV = 1,   /* prefill QKV GEMM (+RoPE, shared K/V store)        */
  ALR_PROF_PREFILL_ATTN = 2,  /* prefill causal attention                           */
  ALR_PROF_PREFILL_O = 3,     /* prefill attention-output GEMM (+residual)          */
  ALR_PROF_PREFILL_GU = 4,    /* prefill gate|up GEMM (+SwiGLU)                     */
  ALR_PROF_PREFILL_DOWN = 5,  /* prefill down GEMM (+residual, features)            */
  ALR_PROF_DECODE_QKV = 6,    /* rollout-step QKV GEMM (+RoPE, private K/V append)  */
  ALR_PROF_DECODE_ATTN = 7,   /* rollout-step anchor-branched attention             */
  ALR_PROF_DECODE_O = 8,
  ALR_PROF_DECODE_GU = 9,
  ALR_PROF_DECODE_DOWN = 10,
  ALR_PROF_LM_GEMM = 11,      /* output-head GEMM (logits into the caller's rows)   */
  ALR_PROF_LM_FINALIZE = 12,  /* log-sum-exp, greedy argmax, in-place log-softmax   */
  ALR_PROF_DECODE_COMBINE = 13, /* merge of decode-attention chunk partials (bf16)  */
  ALR_PROF_COUNT = 14
} alr_prof_site;

/* Kernel that a bf16 product of the model takes at a launch site (host only, no GPU
 * needed; the choice the compute calls make): `rows` rows at a GEMM site above, on a
 * device of n_cu compute units, in a context of this config and these limits.  `cols`
 * is the width of an output-head product that covers a panel of the vocabulary (corpus
 * labels), a multiple of 64; 0, and at every other site, the site's own.  Writes the kernel to
 * *kernel_out (0 = 32x64, 1 = 64x64, 2 = 128x64, 3 = 128x128 tiles of the few-row kernel, 4 =
 * 128x128 LDS-staged, 5 = 256x256, 6 = 64x128 LDS-staged), its K slices, summed by a reduce, to *splits_out, and the K
 * slices of the tiles past the last full round to *tail_out (1: not sliced).
 * ALR_E_UNSUPPORTED for fp32, ALR_E_INVALID_ARG for a site without a GEMM or bad counts, the
 * statuses of alr_check_config otherwise. */
alr_status alr_debug_gemm_plan(const alr_config* cfg, const alr_limits* lim, int32_t n_cu,
                               int32_t site, int32_t rows, int32_t cols, int32_t* kernel_out,
                               int32_t* splits_out, int32_t* tail_out);

/* Start timing every launch at `site` with HIP events recorded on the launch
 * stream, for up to `capacity` launches (later launches are not timed).
 * Creates 2*capacity events (host-side HIP objects, no device buffers). */
alr_status alr_profile_start(alr_ctx* ctx, int32_t site, int32_t capacity);

/* Stop timing; waits for the last recorded event and returns the summed
 * device time (ms) and the number of timed launches.  Destroys the events. */
alr_status alr_profile_stop(alr_ctx* ctx, double* total_ms, int32_t* launches);

#ifdef __cplusplus
}
#endif

#endif /* ALR_DEBUG_H */
