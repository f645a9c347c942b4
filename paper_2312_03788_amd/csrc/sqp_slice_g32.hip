// Column-slice kernel: groups of 32.
#include "sqp_slice_kernel.h"

int sqp_slice_g32(SQP_SLICE_ARGS)
{
    return dispatch_slices<1, false>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, st);
}
