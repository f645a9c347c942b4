// Strip kernel: chunks of one group of 64 or 32 (K not a multiple of 128).
#include "sqp_strip_kernel.h"

namespace {
template <int KSPG>
int by_rows(SQP_STRIP_ARGS)
{
    switch (sqp_strip_row_tiles(M)) {
        case 1: return dispatch_mt<1, KSPG, KSPG>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, ws, st);
        case 2: return dispatch_mt<2, KSPG, KSPG>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, ws, st);
        case 3: return dispatch_mt<3, KSPG, KSPG>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, ws, st);
        default: return dispatch_mt<4, KSPG, KSPG>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, ws, st);
    }
}
}  // namespace

int sqp_strip_one_group(int group, SQP_STRIP_ARGS)
{
    if (group == 32) return by_rows<1>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, ws, st);
    return by_rows<2>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, ws, st);
}
