/*
 * zqfp_probe.h -- measurement probes exported by libzqfp next to its C ABI
 * (zqfp.h).  They are tooling for the benchmark, no part of the W4A8 path: two
 * kernels that show what the device itself sustains, so that roofline
 * fractions can be quoted against measured ceilings as well as published peaks.
 */
#ifndef ZQFP_PROBE_H
#define ZQFP_PROBE_H

#include <stddef.h>
#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Both only enqueue work on `stream` (a hipStream_t as void*); the caller times it.
 * Error codes are those of zqfp.h.
 *
 * zqfp_probe_stream_read -- a plain streaming read of `bytes` bytes at `src`
 *   (device, 16-byte aligned; the last bytes % (workgroups * 32 KB) are not
 *   read).  sink: device, >= 4 * workgroups bytes, written at most once per
 *   workgroup with a value that means nothing.
 * zqfp_probe_mfma -- `iters` rounds of 32 independent
 *   v_mfma_scale_f32_16x16x128_f8f6f4 instructions (FP8 x FP4) per wave, 8 waves
 *   per workgroup, operands held in registers: 2 * 16*16*128 * 32 * 8 * iters *
 *   workgroups floating-point operations in total.  operands: device, 4096
 *   bytes of anything; sink: device, >= 2048 * workgroups bytes.
 *
 * Return ZQFP_OK, ZQFP_E_NULL, ZQFP_E_SHAPE (non-positive sizes), ZQFP_E_ALIGN
 * or ZQFP_E_HIP.
 */
int zqfp_probe_stream_read(const void *src, int64_t bytes, void *sink,
                           int workgroups, void *stream);
int zqfp_probe_mfma(const void *operands, void *sink, int iters,
                    int workgroups, void *stream);

/*
 * zqfp_probe_force_tile_plan -- tuning hook for sweeps and tests: every following
 * zqfp_w4a8_gemm* call with more than 16 tokens (and zqfp_gemm_workspace_bytes,
 * which must agree with it) uses bm x bn output tiles, `kg` wave groups per
 * workgroup and `ksplit` slices of K (1 = none) instead of planning them from
 * the problem size.  Tile shapes: 64x128, 64x192, 64x256 with kg 1 or 2,
 * 64x64, 64x96, 64x128 with kg 4, 128x128, 128x192, 128x256, 256x256 with kg
 * 1; ksplit 1..64 (capped at the number of k-tiles).  E4M3 weights have 64x128
 * (kg 1 or 2) and 128x128.  (0, 0, 0, 0) returns to automatic planning.
 * Process-wide, not meant for concurrent use with GEMM calls of other threads.
 * Returns ZQFP_OK or ZQFP_E_SHAPE.
 *
 * zqfp_probe_force_tile_kind -- the same where a shape has several kernels:
 * 64x128 with kg 1 for E4M3 weights, three LDS stages and at most two workgroups
 * per compute unit (occ 2) or two stages and three workgroups (occ 3, also what
 * occ 0 and the call above take).  Any other shape takes occ 0 only.
 */
int zqfp_probe_force_tile_plan(int bm, int bn, int ksplit, int kg);
int zqfp_probe_force_tile_kind(int bm, int bn, int ksplit, int kg, int occ);

/*
 * zqfp_probe_tile_plan -- what the tiled kernel would take for a problem of this
 * size if it served it (zqfp_probe_gemm_form says whether it does): plan[0..5]
 * (host) = tile rows, tile columns, wave groups, workgroups per compute unit
 * (where a shape has several kernels), K slices, k-tiles per slice.  Host only.
 * Returns ZQFP_OK, ZQFP_E_SHAPE, ZQFP_E_MODE or ZQFP_E_NULL.
 */
int zqfp_probe_tile_plan(int64_t M, int64_t K, int64_t N, int wbits, int accum,
                         int have_workspace, int *plan);

/*
 * zqfp_probe_force_decode_waves -- tuning hook: 8 (default) or 16 waves per
 * workgroup of the decode GEMM (at most 16 tokens) where K <= 4096.
 * Process-wide.  Returns ZQFP_OK or ZQFP_E_SHAPE.
 */
int zqfp_probe_force_decode_waves(int nw);

/*
 * zqfp_probe_gemm_form -- which kernel serves zqfp_w4a8_gemm* (wbits 4) or
 * zqfp_w8a8_gemm (wbits 8) for a problem of this size, rank (0: no low-rank
 * correction) and accumulation mode, with a workspace or without one.  Host
 * only: nothing is enqueued.  Returns ZQFP_FORM_*, ZQFP_E_SHAPE or
 * ZQFP_E_MODE.
 */
#define ZQFP_FORM_DECODE 1 /* persistent, at most 16 tokens (long K in chunks through the workspace) */
#define ZQFP_FORM_MID 2    /* a few dozen tokens, long K, few channels: operands straight into registers */
#define ZQFP_FORM_TILE 3   /* tiles through LDS (K slices through the workspace) */
#define ZQFP_FORM_STREAM 4 /* weight-streaming, E4M3 weights only */
int zqfp_probe_gemm_form(int64_t M, int64_t K, int64_t N, int G, int wbits,
                         int r, int accum, int have_workspace);

/*
 * zqfp_probe_left_form -- how a quantizer call forms the left factor T of a
 * rank-r correction.  kind: 0 zqfp_quantize_act_fp8, 1 RMS normalisation, 2
 * layer normalisation (with or without a residual), 3 ReLU, 4 gated unit;
 * in_place: H lies over X or over the second operand.  Host only: nothing is
 * enqueued.  Returns ZQFP_LEFT_* or ZQFP_E_SHAPE.
 */
#define ZQFP_LEFT_BLOCKS 1 /* a workgroup per token and 4 or 8 ranks (or, rank 8, a wave per token) */
#define ZQFP_LEFT_ONE 2    /* a workgroup per token with all sums */
#define ZQFP_LEFT_APART 3  /* a launch of its own behind the quantizer */
int zqfp_probe_left_form(int64_t M, int64_t K, int r, int kind, int in_place);

#ifdef __cplusplus
}
#endif
#endif /* ZQFP_PROBE_H */
