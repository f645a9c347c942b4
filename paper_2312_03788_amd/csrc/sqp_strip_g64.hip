// Strip kernel: groups of 64, two per chunk of 128 k.
#include "sqp_strip_kernel.h"

int sqp_strip_g64(SQP_STRIP_ARGS)
{
    switch (sqp_strip_row_tiles(M)) {
        case 1: return dispatch_mt<1, 4, 2>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, ws, st);
        case 2: return dispatch_mt<2, 4, 2>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, ws, st);
        case 3: return dispatch_mt<3, 4, 2>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, ws, st);
        default: return dispatch_mt<4, 4, 2>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, ws, st);
    }
}
