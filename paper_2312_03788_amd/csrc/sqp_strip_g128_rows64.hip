// Strip kernel: groups of 128 and multiples, 33 to 64 rows.
#include "sqp_strip_kernel.h"

int sqp_strip_g128_rows64(SQP_STRIP_ARGS)
{
    if (sqp_strip_row_tiles(M) == 3) return dispatch_mt<3, 4, 4>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, ws, st);
    return dispatch_mt<4, 4, 4>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, ws, st);
}
