// Column-slice kernel: groups of several chunks of 128 k.
#include "sqp_slice_kernel.h"

int sqp_slice_g256(SQP_SLICE_ARGS)
{
    return dispatch_slices<4, true>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, st);
}
