// Interface between the launch plans of the weight-streaming GEMM (sqp_gemm_decode.hip) and the
// translation units that instantiate its column-slice kernel (sqp_slice_kernel.h).
#pragma once
#include "sqp_common.h"

// Columns per lane (a slice is 16 of them), waves per workgroup, whether four adjacent slices share an XCD.
// tb == 0: the call does not take the column-slice kernel.
struct SqpSlicePlan {
    int tb, wv;
    bool grouped;
};

// Up to 32 rows, groups of 32, 64 (K a multiple of the group) or of cpg chunks of 128 k.
#define SQP_SLICE_ARGS                                                                                                  \
    const SqpSlicePlan &p, int M, int N, int K, int cpg, const h16 *x, const uint32_t *packed, const h16 *scales,      \
        const uint8_t *zeros, h16 *y, int epi, hipStream_t st
int sqp_slice_g128(SQP_SLICE_ARGS);
int sqp_slice_g256(SQP_SLICE_ARGS);
int sqp_slice_g64(SQP_SLICE_ARGS);
int sqp_slice_g32(SQP_SLICE_ARGS);
