/*
 * sqp_test_hooks.h -- test and benchmark hooks of libsqp.so.  NOT part of the product ABI
 * (that is sqp.h): process-wide switches that override the launch plan the library would
 * pick, plan queries that need no GPU, and two calibration kernels for the benchmark.  None
 * is thread-safe; a test sets a switch, makes its calls and resets it (0 / -1 = automatic).
 */
#ifndef SQP_TEST_HOOKS_H
#define SQP_TEST_HOOKS_H

#include <stddef.h>

#ifdef __cplusplus
extern "C" {
#endif
#pragma GCC visibility push(default) /* the library is built with hidden visibility: these are its exports */

/* Weight-streaming path (M <= 64 rows) of sqp_w4a16_gemm. */
void sqp_debug_set_decode_max_m(int m);            /* rows up to which that path is used (default 64) */
void sqp_debug_set_decode_split(int split);        /* force the number of K parts; 0 = automatic */
void sqp_debug_set_decode_plan(int nw, int split); /* force strips per workgroup and K parts; (0, 0) = automatic */
void sqp_debug_set_decode_kw(int kw);              /* waves per strip: 0 = automatic, 1 = never two, 2 = two wherever built */
void sqp_debug_set_decode_kp(int kp);              /* two chunks per iteration (twice the waves): 0 = automatic, 1 = never,
                                                      2 = where the rules would with enough chunks, 3 = wherever built */
void sqp_debug_set_decode_slice(int mode);         /* column-slice kernel (M <= 32): 0 = automatic, -1 = never, 1 = always with
                                                      32-column slices, 2 = always with 64-column slices (eight waves) */
void sqp_debug_set_slice_plan(int tb, int wv, int grouped); /* tb > 0: column slices of 16 tb columns, wv waves (eight where that many are
                                                      not built for the rows), for every call they cover */
/* Whether a layer fills the chip with slices of 32 (0) or 64 (1) columns and takes the column-slice kernel for
 * that alone (-1: the launch plan decides by N, K and the group).  Host arithmetic only. */
int sqp_debug_decode_slice_choice(int M, int N, int K, int group);
/* The slices a call takes with a workspace set: columns / 16 and waves per workgroup (0, 0: the strip kernel below or the
 * generic one). */
void sqp_debug_decode_slice_plan(int M, int N, int K, int group, int *tb, int *wv);
/* The plan by strips for a shape: strips per workgroup, K parts, k-steps of one group up to 128 k
 * (0 = the generic one-thread-per-element kernel).  Calls with up to 16 rows and groups that are
 * multiples of 128 run it.  Host arithmetic only. */
void sqp_debug_decode_plan(int M, int N, int K, int group, int *nw, int *split, int *kspg);

/* What a call of the strip kernel launches: strips per workgroup, K parts, waves per strip and chunks
 * per iteration (0: by rules on the number of workgroups).  Host arithmetic only. */
void sqp_debug_decode_launch(int M, int N, int K, int group, int *nw, int *split, int *kw, int *kp);

/* Tiled matrix-core path (M > 64). */
void sqp_debug_set_prefill_tiles(int mode);        /* 0 = automatic, 1 = full tiles only, 2 = half-width tiles only */
void sqp_debug_set_prefill_shape(int shape);       /* 0 = automatic, 1 = 128 x 512 full tiles, 2 = 256 x 256 */
void sqp_debug_set_prefill_ksplit(int k);          /* -1 = automatic, 0 or 1 = never, k >= 2 = k parts */
void sqp_debug_set_prefill_variant(int rt, int nt, int parts);  /* one launch of tiles of 32 rt rows x 128 nt columns, K parts
                                                      (rt 3 to 6 with nt 2, 4 or 5 with nt 3, or 4 with nt 4; parts > 1 with nt 2; nt 2 + 16:
                                                      half the columns, the waves halve K, K % 128 == 0); 0 = automatic */
/* The plan in 128-row tiles for a shape on a chip of `cus` compute units: full tiles of the first
 * launch, half-width tiles of the second, K parts.  Host arithmetic only. */
void sqp_debug_prefill_plan(int M, int N, int K, int cus, long *full, long *half, int *ksplit);

void sqp_debug_set_row_blocks(int mt, int split, int kp);  /* more than 64 rows (K % 128 == 0, groups of 32, 64
                                                      and multiples of 128): the strip kernel in row blocks of
                                                      16 mt rows (3, 4), K parts, chunks per iteration; 0 = automatic, -1 = never */
/* What a call takes of these: rows / 16 (0: the tiled kernel), K parts, chunks per iteration; without a
 * workspace (0), with one of the reported size (1) or as large as it likes (2).  Host arithmetic only. */
void sqp_debug_row_blocks(int M, int N, int K, int group, int cus, int workspace, int *out3);

/* How an alpha search runs: sets of prepared operands that fit a region of `bytes` (-1: not even its factors and sums
 * fit: single calls in turn), alphas per launch, whether the next ones are prepared beside them; bytes 0: the
 * buffers of sqp_alpha_search.  Host arithmetic only. */
void sqp_debug_search_plan(int T, int N, int K, int group, int n_alpha, size_t bytes, int *out3);

/* The launches that a call's workspace and scratch sizes are reported for: returns their number (1 or 2) and their
 * (rt, nt, tiles, K parts) in out8.  The plan above, or one round of tiles of another height where that is faster, and with K
 * parts for few left-over tiles; workspace and scratch as large as it likes.  Host arithmetic only. */
int sqp_debug_prefill_launches(int M, int N, int K, int group, int cus, int *out8);

/* What a call launches in their place with `room` bytes for its K parts (workspace or its own scratch, whichever the
 * shape uses): as above, with (rt, nt, tiles, K parts, 2 where the waves halve K) in out10; 0: refused. */
int sqp_debug_prefill_choice(int M, int N, int K, int group, int cus, size_t room, int *out10);

/* Calibration kernels for the benchmark: a plain device copy of `bytes` (a multiple of 16)
 * whose traffic is known, and a loop of nothing but independent 32x32x16 fp16 matrix
 * instructions (data: 64 KiB of fp16 on the device, out: blocks * 256 floats; flops of the
 * launch = blocks * 4 * iters * 16 * 32768). */
int sqp_debug_plain_copy(const void *src, void *dst, size_t bytes, void *stream);
/* A plain streaming read of `bytes` (a multiple of 16; whole passes of 8 x blocks x 256 x 16 bytes
 * are read, the rest is skipped) by `blocks` workgroups of 256 threads, with (nt != 0) or without
 * the non-temporal hint; sink: 4 bytes.  The rate depends on the grid: three workgroups per
 * compute unit (768) read faster than thousands. */
int sqp_debug_read_probe(const void *src, size_t bytes, int nt, int blocks, void *sink, void *stream);
int sqp_debug_mfma_ceiling(const void *data, float *out, int blocks, int iters, void *stream);

#pragma GCC visibility pop
#ifdef __cplusplus
}
#endif
#endif /* SQP_TEST_HOOKS_H */
