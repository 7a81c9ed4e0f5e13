/*
 * mst_mlp.h -- C ABI of the mini-sequence MLP library (hand-written HIP for
 *              gfx950 / MI355X).
 *
 * The operation is the MLP block of the Mini-Sequence Transformer paper:
 * Algorithm 1 (forward) and Algorithm 3 (backward with recomputation of the
 * intermediates).  The block is the Llama MLP of the paper's model listing
 * (Appendix C): three bias-free linear layers and SiLU,
 *
 *     O = ( silu(X Wg^T) * (X Wu^T) ) Wd^T            (Theorem 1)
 *
 * The token dimension S (the paper's N; batch folded in) is split into M
 * mini-sequences of C = ceil(S / M) rows (Algorithm 1, line 1).  For chunk i
 * the forward pass forms the C x I intermediate A_i = silu(X_i Wg^T) * (X_i Wu^T)
 * in the workspace, writes O_i = A_i Wd^T into rows i*C.. of O (Algorithm 1,
 * lines 3 and 5) and reuses the workspace for the next chunk, so that the
 * workspace holds one C x I intermediate instead of S x I.  Rows are
 * independent, so a call takes them in groups that need not be the chunks: as
 * many as there is memory for, in the workspace and in rows of the output that
 * are not written yet.  The backward pass recomputes
 * the chunk's gate and up projections and forms (Algorithm 3, lines 4-5)
 *
 *     dA_i  = dO_i Wd
 *     dG_i  = dA_i * U_i * silu'(G_i)        dU_i = dA_i * silu(G_i)
 *     dX_i  = dG_i Wg + dU_i Wu              (rows i*C.. of dX)
 *     dWg  += dG_i^T X_i     dWu += dU_i^T X_i     dWd += dO_i^T A_i
 *
 * By the paper's exactness claim (Section 3.1) the result does not depend on M.
 *
 * Readings of the paper fixed by this interface:
 *   - the activation acts on the gate branch only (the model listing's
 *     gate_proj / up_proj / down_proj / act_fn), although Theorem 1 prints it
 *     around the product;
 *   - weights are stored as the listing's Linear layers store them,
 *     [out_features, in_features] row-major: Wg, Wu [I, d], Wd [d, I];
 *   - "grad MLP" of Algorithm 3 is the exact derivative of the block above.
 *
 * Conventions
 *   - Every pointer is a DEVICE pointer owned by the caller, except where
 *     "host" is written.  The library allocates no device memory and keeps no
 *     state between calls (profiling events aside).
 *   - All work is enqueued on `stream` (a hipStream_t passed as void*); the
 *     calls return without waiting for the GPU.
 *   - Return value: MST_OK (0) or a negative error code of mst_lmhead.h
 *     (MST_ERR_BAD_SHAPE also covers I).  Argument errors are found on the
 *     host before anything is launched.
 *   - Requirements: d % 8 == 0, I % 8 == 0; X, Wg, Wu, Wd, dO, O, dX, dWg,
 *     dWu, dWd 16-byte aligned; workspace 256-byte aligned;
 *     1 <= M <= S; d, I < 2^22; I * d < 2^31; ceil(S/M) * I < 2^30.
 *   - Arithmetic: bf16 operands, fp32 MFMA accumulation; silu, its derivative
 *     and the products in fp32 on the accumulators; A, dA, dG, dU rounded to
 *     bf16 (nearest even) before the GEMMs that consume them; O and dX
 *     rounded to bf16; the three weight gradients fp32, accumulated in a fixed
 *     order without atomics, which depends on S, d, I and M alone and on
 *     whether dX overlaps an input (bit-identical across calls, whatever
 *     workspace they are handed).
 */
#ifndef MST_MLP_H
#define MST_MLP_H

#include "mst_lmhead.h"

#ifdef __cplusplus
extern "C" {
#endif

/* host: "mst-mlp <version> (gfx950)" */
const char* mst_mlp_version(void);

/*
 * Bytes of workspace the two calls need (host, pure).
 *   fwd: one chunk of A, C * I bf16.  A larger one is used, for the A of more rows at a time; so are the rows of O that are
 *        not written yet, unless O overlaps an input.
 *   bwd: three chunk-sized bf16 buffers (dA reused for dG, dU, A) = 3 * C * I * 2 bytes.
 * Either output pointer may be NULL.
 */
mst_status mst_mlp_workspace_bytes(int64_t S, int64_t d, int64_t I, int32_t M,
                                   size_t* fwd_bytes, size_t* bwd_bytes);

/*
 * Chunk policy of the paper's chunk-based variant (Section 3.3): a constant
 * chunk size equal to the hidden size, C = d, i.e. M = S / d to the nearest
 * integer and at least 1 (no split when S <= d).  Host, pure; 0 on bad shapes.
 */
int32_t mst_mlp_suggest_m(int64_t S, int64_t d, int64_t I);

/*
 * Forward (Algorithm 1).
 *   X  [S, d] bf16 row-major      block input
 *   Wg [I, d] bf16 row-major      gate projection
 *   Wu [I, d] bf16 row-major      up projection
 *   Wd [d, I] bf16 row-major      down projection
 *   O  [S, d] bf16 row-major      out, fully overwritten
 */
mst_status mst_mlp_fwd(const void* X, const void* Wg, const void* Wu, const void* Wd,
                       int64_t S, int64_t d, int64_t I, int32_t M,
                       void* workspace, size_t workspace_bytes,
                       void* O, void* stream);

/*
 * Backward (Algorithm 3).  Nothing is kept from the forward call: the gate and
 * up projections of every chunk are recomputed.  The rows are taken in groups,
 * not necessarily of whole chunks: one to three of dG, dU and A of a group may
 * be kept in rows of dX that are not final yet.  A dX that overlaps X or dO has
 * to begin at least C rows before it (the groups are then the chunks, one after
 * the other); it must not overlap a weight.
 *   dO  [S, d] bf16      upstream gradient of O
 *   dX  [S, d] bf16      out, fully overwritten
 *   dWg [I, d] fp32      out, fully overwritten (first group stores, later ones accumulate)
 *   dWu [I, d] fp32      out
 *   dWd [d, I] fp32      out
 */
mst_status mst_mlp_bwd(const void* X, const void* Wg, const void* Wu, const void* Wd, const void* dO,
                       int64_t S, int64_t d, int64_t I, int32_t M,
                       void* workspace, size_t workspace_bytes,
                       void* dX, float* dWg, float* dWu, float* dWd, void* stream);

/*
 * Which block tiles the launches of a group of `rows` rows take (host, pure; a test aid).  All give the same O and dX
 * bit for bit.  info[0..2] = gate/up (forward and backward), info[3..5] = down, info[6..8] = dA and info[9..11] = dX
 * where they have launches of their own (mst_mlp_da_in_gateup, mst_mlp_dx_tile), each as
 * {MST_MLP_TILE_* of the launch, or of its end; leading columns (of I, d, I, d) that a launch of 256 x 256 tiles of its
 * own takes before it, 0 for none; 1 where 256 x 256 tiles are laid out in super-tiles}; info[12..13] = the weight
 * gradients of a call whose largest group has `rows` rows: {MST_MLP_TILE_256, _64 or _64_LONE; 1 where the tiles are dealt out
 * evenly over the XCDs}.
 */
enum {
  MST_MLP_TILE_256 = 0,   /* 256 x 256, one workgroup per compute unit                  */
  MST_MLP_TILE_128,       /* 128 x 128, two                                             */
  MST_MLP_TILE_128_LONE,  /* 128 x 128, one, software-pipelined                         */
  MST_MLP_TILE_64,        /* 64 x 64, four                                              */
  MST_MLP_TILE_64_LONE,   /* 64 x 64, one, software-pipelined                           */
  MST_MLP_TILE_64_LONG,   /* the same with K steps of 128                               */
  MST_MLP_TILE_32,        /* 32 x 32, K steps of 128 (not gate/up)                      */
  MST_MLP_TILE_128X256    /* 128 (weights) x 256 (rows), one (gate/up and down)         */
};
mst_status mst_mlp_tile_info(int64_t rows, int64_t d, int64_t I, int64_t* info);

/*
 * How dX of a group of `rows` rows is computed, in a call whose largest group has that many; first: it is the call's first.  One of MST_MLP_DX_*, -1 on bad shapes (host, pure; a test aid).  dX has the same bits either way.
 */
enum {
  MST_MLP_DX_OWN = 0,     /* in a launch of its own, with the tiles that mst_mlp_tile_info names   */
  MST_MLP_DX_SHARED_256,  /* by the launch of the weight gradients, 256 x 256 tiles                */
  MST_MLP_DX_SHARED_128,  /* the same, 128 (hidden index) x 256 or 128 (rows, see below)           */
  MST_MLP_DX_SHARED_64,   /* the same, 64 x 64 tiles, as those of the weight gradients             */
  MST_MLP_DX_SHARED_32    /* the same, 32 x 32                                                     */
};
int32_t mst_mlp_dx_tile(int64_t rows, int64_t d, int64_t I, int32_t first);
/* Rows of that tile: 256 or 128 of MST_MLP_DX_SHARED_128, 256, 64 or 32 of the others, 0 of _OWN; -1 on bad shapes. */
int32_t mst_mlp_dx_tile_rows(int64_t rows, int64_t d, int64_t I, int32_t first);

/*
 * The groups of rows that a call takes, each with the launches that the queries around this one name for its rows (host, pure;
 * test aids): their number, -1 for bad arguments; info of the first `room` of them.
 * mst_mlp_fwd_groups: per group {rows, 1 where its A is kept in the rows of O behind it, 0 in the workspace}; output_overlaps:
 * whether O overlaps an input.
 * mst_mlp_bwd_groups: per group {rows; how many of dG, dU and A are in the rows of dX behind it; MST_MLP_DX_* and the rows of
 * that tile; 1 where dA is computed by the launch of gate/up's backward; MST_MLP_TILE_* of the weight gradients, which have
 * those of the largest group}; dx_overlaps: whether dX overlaps an input.
 */
int64_t mst_mlp_fwd_groups(int64_t S, int64_t d, int64_t I, int32_t M, size_t workspace_bytes, int32_t output_overlaps,
                           int64_t room, int64_t* info);
int64_t mst_mlp_bwd_groups(int64_t S, int64_t d, int64_t I, int32_t M, int32_t dx_overlaps, int64_t room, int64_t* info);

/*
 * Which products of `rows` rows, the first of their call, load rows that are not whole cache lines line by line, their operands
 * beginning on one (host, pure; a test aid): a sum of MST_MLP_LINES_*, -1 on bad shapes.  The same bits either way.
 */
enum {
  MST_MLP_LINES_DOWN = 1,
  MST_MLP_LINES_DA = 2,
  MST_MLP_LINES_DX = 4    /* in a launch of its own or beside the weight gradients (mst_mlp_dx_tile) */
};
int32_t mst_mlp_line_panels(int64_t rows, int64_t d, int64_t I);

/*
 * 1 where dA of a group of `rows` rows is computed by the launch of gate/up's backward, 0 where it has a launch of its own
 * (with the tiles that mst_mlp_tile_info names), -1 on bad shapes (host, pure; a test aid).
 */
int32_t mst_mlp_da_in_gateup(int64_t rows, int64_t d, int64_t I);

/*
 * Workgroup -> tile map of the 256 x 256 launches (host-only test aid; the kernels call the same functions), as
 * mst_tile_of_workgroup in mst_lmhead.h: whole super-tiles of 8 x 4 tiles per XCD where they divide as well over the
 * XCDs as single tiles do, an equal share of the tiles for every XCD elsewhere and for all smaller tiles.
 */
int32_t mst_mlp_tile_grid(int32_t n_slow, int32_t n_fast);
int32_t mst_mlp_tile_of_workgroup(int32_t n_slow, int32_t n_fast, int32_t workgroup, int32_t* slow, int32_t* fast);

/*
 * Per-kernel timing (host), as in mst_lmhead.h: mst_mlp_profile_enable(every)
 * brackets every `every`-th launch of each kernel kind of the two calls above
 * with HIP events on the caller's stream (0 = off); collect adds, per kind, the
 * elapsed milliseconds, the number of launches they cover and (if the pointer
 * is not NULL) the number of all launches while timing was on (arrays of
 * length MST_MLP_PROFILE_KINDS) and clears the record.  A product that ends in
 * a second launch of smaller tiles is timed, and counted, as one.
 */
enum {
  MST_MLP_K_GATEUP = 0,   /* A_i = silu(X_i Wg^T) * (X_i Wu^T)                       */
  MST_MLP_K_DOWN,         /* O_i = A_i Wd^T                                          */
  MST_MLP_K_DA,           /* dA_i = dO_i Wd                                          */
  MST_MLP_K_GATEUP_BWD,   /* recomputed gate/up GEMM + dG_i, dU_i, A_i epilogue; with
                             dA_i in it where one launch serves both                 */
  MST_MLP_K_DX,           /* dX_i = dG_i Wg + dU_i Wu                                */
  MST_MLP_K_DW,           /* dWg += dG_i^T X_i, dWu += dU_i^T X_i, dWd += dO_i^T A_i; with
                             dX_i in it where one launch serves both                 */
  MST_MLP_PROFILE_KINDS
};
mst_status mst_mlp_profile_enable(int every);
mst_status mst_mlp_profile_collect(double* ms_per_kind, int64_t* launches_per_kind, int64_t* issued_per_kind);
const char* mst_mlp_profile_kind_name(int kind);

#ifdef __cplusplus
}
#endif
#endif /* MST_MLP_H */
