/*
 * specformer_aux.h -- measurement and tuning aids of libspecformer (gfx950).  Not part of the decoding
 * path: bench and sweep programs use these to time kernel classes, to calibrate hardware byte counters and
 * to override the automatic kernel choices of ONE context.
 */
#ifndef SPECFORMER_AUX_H
#define SPECFORMER_AUX_H
#include "specformer.h"
#ifdef __cplusplus
extern "C" {
#endif

/* Force the linear kernels' tile configuration (1..sf_linear_num_tiles()) and split-K factor for every
 * later launch of this context; 0 = automatic choice.  A forced pair whose partial tiles do not fit the
 * workspace makes the launch fail with SF_EHIP.  Tiles 15-17 and 26-28 leave a fused norm's row sums of squares in the workspace,
 * public operations included. host. */
sf_status sf_tune_linear(sf_ctx *ctx, int32_t tile, int32_t split_k);
int32_t sf_linear_num_tiles(void);
/* The K split of a bf16 linear layer of M rows whose weight [N][K] is also used with up to plan_M >= M rows, and the ring
 * kernel's tile (1-14) for it: *split_k is the same for every M <= plan_M (so a row's result does not depend on the rows
 * batched with it), *tile follows M; *tile_rows = rows per workgroup of that tile.  A launch with nothing forced keeps this
 * split and may run on another kernel, with the same bits: sf_linear_choice.  Pure host arithmetic, no GPU needed.  host
 * pointers. */
sf_status sf_linear_config(int32_t M, int32_t plan_M, int32_t N, int32_t K, size_t workspace_bytes,
                           int32_t *tile, int32_t *split_k, int32_t *tile_rows);
/* What a launch of that layer runs on.  flags: SF_LINEAR_*.  In: *tile and *split_k as given to sf_tune_linear (0: automatic).
 * Out: *kernel SF_KERNEL_*, *tile its tile (streaming kernel: 16-column tiles per wave), *split_k the split.  A block tile
 * forced on a layer that the block kernel does not take comes back as ring tile 10, which is what runs.  Pure host
 * arithmetic.  host pointers. */
enum { SF_KERNEL_RING = 0, SF_KERNEL_BLOCK = 1, SF_KERNEL_STREAM = 2 };
enum {
  SF_LINEAR_GLU = 1,       /* the SwiGLU gate (N = 2F)                      */
  SF_LINEAR_NORM = 2,      /* the fused RMSNorm                             */
  SF_LINEAR_ARGMAX = 4,    /* arg-max partials (LM head)                    */
  SF_LINEAR_UNALIGNED = 8, /* x does not start on a 16-byte boundary        */
  SF_LINEAR_OP = 16        /* a public operation, whose workspace may be shared between streams; without it a step's layer */
};
sf_status sf_linear_choice(int32_t M, int32_t plan_M, int32_t N, int32_t K, size_t workspace_bytes, int32_t flags,
                           int32_t *kernel, int32_t *tile, int32_t *split_k);
/* Force the attention's split-KV chunk size in 32-key tiles (>= 16) for this context; 0 = automatic. host. */
sf_status sf_tune_attention(sf_ctx *ctx, int32_t chunk_tiles);

/* Between sf_profile_begin and sf_profile_end every kernel launch of this context is bracketed by a pair
 * of HIP events on its stream.  sf_profile_end waits for the last one and returns, per kernel class, the
 * summed duration in ms and the number of launches (host arrays of n_class >= SF_N_KERNEL_CLASSES
 * entries).  Classes: 0 linear (GEMM), 1 attention, 2 attention split-KV combine, 3 RMSNorm, 4 rotary +
 * K/V append, 5 SwiGLU gate, 6 embedding / hook copies, 7 arg-max pass over stored logits, 8 arg-max
 * finish / accept-commit. */
#define SF_N_KERNEL_CLASSES 9
sf_status sf_profile_begin(sf_ctx *ctx);
sf_status sf_profile_end(sf_ctx *ctx, double *ms, int32_t *launches, int32_t n_class);
/* A plain device-to-device copy kernel (`calib_copy_kernel`) of `bytes` (multiple of 16, 16-byte aligned
 * pointers) that reads and writes every byte exactly once: the dispatch of known size against which
 * hardware byte counters (FETCH_SIZE, WRITE_SIZE) are scaled. */
sf_status sf_calib_copy(void *dst, const void *src, size_t bytes, void *stream);

#ifdef __cplusplus
}
#endif
#endif
