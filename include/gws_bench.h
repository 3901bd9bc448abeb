/*
 * libgws -- measurement aids.  Not part of the method: these calls move the bytes of the
 * GaussWS forward and backward passes (paper Eq. 3, Eq. 4) with the launch shape, loads and
 * stores of gws_sample_fwd / gws_sample_bwd and none of their arithmetic, so that a benchmark
 * can put the rate of the sampling kernels next to the rate the memory system allows for the
 * same access pattern.  Same conventions as gws.h: device pointers owned by the caller, host
 * descriptor array read before the call returns, asynchronous on the given stream, gws_status
 * returned, nothing launched on error.
 */
#ifndef GWS_BENCH_H
#define GWS_BENCH_H

#include "gws.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Copies w to w_hat for n tensors with the launch shape, loads and stores of gws_sample_fwd.
 * Its rate is the ceiling the memory system sets for that access pattern, against which the
 * forward pass is read.  Uses fields w, w_hat, rows, cols, ld.                              */
int gws_copy_tiles(const gws_tensor* t, int n, void* stream);

/* Step one of Eq. 3 alone: writes max_{b_l}|w| (exact, as fp32) of every 32x32 block into
 * `scale`, for n tensors, with the launch shape and loads of gws_sample_bwd.  It reads
 * each element once and writes 4 bytes per block, so its rate is the ceiling the memory
 * system sets for the backward pass.  Uses fields w, scale, rows, cols, ld.                 */
int gws_block_absmax(const gws_tensor* t, int n, void* stream);

/* gws_sample_bwd with the launch shape chosen by the caller, to measure the choices the library makes:
 *   variant  -1 = the library's choice; 0, 2 = the kernel for any shape with four, with up to eight wavefronts a
 *            SIMD; 1 = the whole-tile kernel (used only where every tensor of a launch has rows % 32 == 0,
 *            cols % 256 == 0 and an aliased dL/dw)
 *   per_x    column tiles (256 columns) one workgroup walks; 0 = the library's choice
 * Same results as gws_sample_bwd whatever the choice.                                                  */
int gws_sample_bwd_tuned(const gws_tensor* t, int n, uint64_t step, int variant, int per_x, void* stream);

/* The same for gws_sample_fwd; its whole-tile kernel takes one column tile a workgroup: with per_x above 1
 * variant 1 is the library's choice of 0 and 2.                                                        */
int gws_sample_fwd_tuned(const gws_tensor* t, int n, int fmt, uint64_t step, int variant, int per_x, void* stream);

/* gws_gemm_bf16_sample_next with the riding forced: the GEMM (none at all if M == 0) is followed in the same
 * grid by `extra_workgroups` (1 .. 4096) workgroups that sample `next` (rows a multiple of 32, columns of 64),
 * whatever the library's own estimate of whether the sampling fits beside the GEMM's last round says.
 * rider: 0 = the riding loop for any such weight, 1 = the loop for weights of whole 32 x 256 tiles (falls back
 * to 0 for other weights).  Same w_hat and scale bytes as gws_gemm_bf16_sample_next; Y is the 256-tile GEMM's,
 * whichever GEMM that call would choose.                                                                    */
int gws_gemm_bf16_ride_probe(const void* x, int64_t M, int64_t K, int64_t ldx, const void* w, int64_t N, int64_t ldw,
                             int w_is_nk, void* y, int64_t ldy, const gws_tensor* next, int fmt, uint64_t step,
                             int extra_workgroups, int rider, void* stream);

/* How many of the weights next[0 .. n_next) gws_gemm_bf16_sample_next_n would let ride in the launch of an
 * M x K x N GEMM with a [K x N] weight on the current device (a prefix of the list); host function, launches nothing.
 * _layout: the same for either layout of the weight.                                                          */
int gws_ride_plan(int64_t M, int64_t K, int64_t N, const gws_tensor* next, int n_next);
int gws_ride_plan_layout(int64_t M, int64_t K, int64_t N, int w_is_nk, const gws_tensor* next, int n_next);

/* Which kernel a call takes on the current device (without one: on 256 compute units), so that a test can aim at one.
 * Host functions, launch nothing; 0 for sizes that the call refuses.  The choice goes by sizes and leading dimensions,
 * and may change from one version of the library to the next.
 * gws_gemm_form: of gws_gemm_bf16 (sampled 0), of gws_linear_fwd_mode with GWS_LINEAR_IN_OPERAND (1), and of
 * gws_linear_fwd with w_hat (2: a GEMM that is not a _SAMPLE one is preceded by the sampling kernel), Y lying apart from
 * the operands.                                                                                                */
#define GWS_GEMM_STREAM 1           /* 16 .. 128 x 16 .. 64 tiles, K split over wavefronts */
#define GWS_GEMM_MIDDLE 2           /* 128 x 128 or 128 x 96 tiles, any edge */
#define GWS_GEMM_LARGE 3            /* 256 x 256 tiles, whole ones */
#define GWS_GEMM_LARGE_EDGE 4       /* 256 x 256 tiles, any edge */
#define GWS_GEMM_NARROW 5           /* 256 x 192 tiles, any edge */
#define GWS_GEMM_ANY_SHAPE 6        /* 128 x 128 tiles, K-steps of 32 */
#define GWS_GEMM_STREAM_SAMPLE 7    /* K split as in 1, the weight sampled in the operand load */
#define GWS_GEMM_ROWS_SAMPLE 8      /* 256 x 256 or 128 x 128 tiles, the weight sampled in the operand load */
#define GWS_GEMM_ANY_SHAPE_SAMPLE 9 /* the same on the tiles of 6 */
int gws_gemm_form(int64_t M, int64_t K, int64_t ldx, int64_t N, int64_t ldw, int w_is_nk, int sampled);
/* gws_gemm_tile: of the same call, the part of Y that a workgroup of that kernel makes, rows << 16 | columns (of the stream kernel in
 * whole MFMA tiles of 16 x 16, also where it keeps eight rows or eight columns of one: gws_gemm_stream_tile).                     */
int gws_gemm_tile(int64_t M, int64_t K, int64_t ldx, int64_t N, int64_t ldw, int w_is_nk, int sampled);
/* gws_gemm_stream_tile: of the same call where its kernel is GWS_GEMM_STREAM (0 otherwise), how that kernel is launched:
 * rows << 24 | columns << 16 | fetching << 8 | parts, with the rows and columns of Y that a workgroup stores (eight of a tile among
 * them), the workgroups a tile that only fetch the weight into the L2s, and whether each XCD takes a contiguous part of the tiles. */
uint32_t gws_gemm_stream_tile(int64_t M, int64_t K, int64_t ldx, int64_t N, int64_t ldw, int w_is_nk, int sampled);

/* gws_linear_bwd_w_form: of gws_linear_bwd_w_ws for this weight (rows, cols) over M tokens with that much workspace, X, dY and
 * dW being rows that start on 128-byte lines (contiguous ones do); _rows: the same for either, on_lines = 0 where some do not. */
#define GWS_BWD_W_WIDE 1            /* a workgroup per 256 x 256 tile */
#define GWS_BWD_W_NARROW 2          /* a workgroup per 256 x 192 tile */
#define GWS_BWD_W_PIECES_64 3       /* a workgroup per 64 x 64 piece, the tokens split over its wavefronts */
#define GWS_BWD_W_PIECES_128 4      /* the same with pieces of 128 x 64 */
#define GWS_BWD_W_PIECES_96 5       /* of 96 x 96 */
#define GWS_BWD_W_PIECES_128_128 6  /* of 128 x 128 */
#define GWS_BWD_W_PIECES_32 7       /* of 64 x 32 */
#define GWS_BWD_W_SPLIT 16          /* + parts: the tokens of a 256 x 256 tile split over so many workgroups */
int gws_linear_bwd_w_form(const gws_tensor* w, int64_t M, size_t workspace_bytes);
int gws_linear_bwd_w_form_rows(const gws_tensor* w, int64_t M, size_t workspace_bytes, int on_lines);

/* The Box-Muller basis draws R of a word of noise by thresholds on z^2 (hardware logarithm and cosine) unless z^2 comes
 * near one, and by its defined sequence of fp32 operations there.  Both ways over the words first .. first + n - 1 (at most
 * 2^32 of them), added to out (device, three uint64 that the caller clears):
 *   out[0]  words for which the thresholds alone decide and give another R than the sequence
 *   out[1]  words that are left to the sequence
 *   out[2]  (maximum) of those that the thresholds would decide wrongly, the distance from the threshold, in units of
 *           2^-24 of the window's width: how much of the half window, 2^23, the hardware's errors need              */
int gws_box_muller_check(uint64_t first, uint64_t n, void* out, void* stream);

#ifdef __cplusplus
}
#endif
#endif /* GWS_BENCH_H */
