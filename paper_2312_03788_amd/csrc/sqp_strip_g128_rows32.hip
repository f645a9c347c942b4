// Strip kernel: groups of 128 and multiples, up to 32 rows.
#include "sqp_strip_kernel.h"

int sqp_strip_g128_rows32(SQP_STRIP_ARGS)
{
    if (sqp_strip_row_tiles(M) == 1) return dispatch_mt<1, 4, 4>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, ws, st);
    return dispatch_mt<2, 4, 4>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, ws, st);
}
