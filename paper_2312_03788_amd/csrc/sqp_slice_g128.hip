// Column-slice kernel: groups of 128.
#include "sqp_slice_kernel.h"

int sqp_slice_g128(SQP_SLICE_ARGS)
{
    return dispatch_slices<4, false>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, st);
}
