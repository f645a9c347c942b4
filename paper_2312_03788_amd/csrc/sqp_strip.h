// Interface between the launch plans of the weight-streaming GEMM (sqp_gemm_decode.hip) and the
// translation units that instantiate its strip kernel (sqp_strip_kernel.h).
#pragma once
#include "sqp_common.h"

// Strips per workgroup, K parts; waves per strip and chunk and chunks per iteration (0: by the
// rules at the launch); 16-row tiles of a row block (calls of more than 64 rows).
struct SqpStripPlan {
    int nw, split;
    int kw, kp;
    int mt = 0;
};

// 16-row tiles of the kernel variant a call takes.
static inline int sqp_strip_row_tiles(int M) { return M <= 16 ? 1 : (M <= 32 ? 2 : (M <= 48 ? 3 : 4)); }

// The split a launch really runs with, and the bytes of fp32 partial tiles it leaves in the workspace (blocks: of
// 16 mt rows).
int sqp_strip_split(int mt, int nw, int kspg, int blocks, int N, int K, int split, size_t *partial_bytes);
// Whether workgroups that walk chunks / split chunks take two per iteration.
bool sqp_strip_two_chunks(int chunks, int split);
extern int sqp_strip_kw_hook, sqp_strip_kp_hook;  // test hooks (0 = automatic)

// The launches, by what a chunk holds: cpg chunks of 128 k per group (groups of 128 cpg); two or four
// groups per chunk of 128 k; one group of 64 or 32 per chunk (K not a multiple of 128).
#define SQP_STRIP_ARGS                                                                                                        \
    const SqpStripPlan &p, int M, int N, int K, int cpg, const h16 *x, const uint32_t *packed, const h16 *scales,            \
        const uint8_t *zeros, h16 *y, int epi, const SqpWorkspace &ws, hipStream_t st
int sqp_strip_g128_rows32(SQP_STRIP_ARGS);  // up to 32 rows
int sqp_strip_g128_rows64(SQP_STRIP_ARGS);  // 33 to 64 rows
int sqp_strip_g64(SQP_STRIP_ARGS);
int sqp_strip_g32(SQP_STRIP_ARGS);
int sqp_strip_one_group(int group, SQP_STRIP_ARGS);
int sqp_strip_row_blocks(int group, SQP_STRIP_ARGS);  // more than 64 rows (K % 128 == 0)
