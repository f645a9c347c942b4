// Column-slice kernel: groups of 64.
#include "sqp_slice_kernel.h"

int sqp_slice_g64(SQP_SLICE_ARGS)
{
    return dispatch_slices<2, false>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, st);
}
