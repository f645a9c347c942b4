// Strip kernel in row blocks of 48 or 64 rows: calls of more than 64 rows, one launch.
#include "sqp_strip_kernel.h"

namespace {

template <int MT, int KP, int GS>
int launch_blocks(int M, int N, int K, int cpg, int split, const h16 *x, const uint32_t *packed, const h16 *scales, const uint8_t *zeros,
                  h16 *y, int epi, const SqpWorkspace &cws, hipStream_t st)
{
    const int tiles = (N + 127) / 128, blocks = (M + 16 * MT - 1) / (16 * MT);
    size_t need = 0;
    split = sqp_strip_split(MT, 2, 4, blocks, N, K, split, &need);
    Workspace ws = {nullptr, nullptr};
    if (split > 1) {
        if (!cws.partial || !cws.tickets || need > cws.partial_bytes) return SQP_ERR_WORKSPACE;
        ws.partial = cws.partial;
        ws.tickets = cws.tickets;
    }
    if (parts_together(tiles, split, blocks)) {
        w4a16_decode_kernel<MT, 2, 4, 2, KP, GS, true, true><<<dim3(tiles, split, blocks), 2 * 2 * KP * 64, 0, st>>>(
            M, N, K, cpg, x, packed, scales, zeros, y, ws, epi);
        return sqp_launch_status();
    }
    w4a16_decode_kernel<MT, 2, 4, 2, KP, GS, true><<<dim3(tiles, split, blocks), 2 * 2 * KP * 64, 0, st>>>(
        M, N, K, cpg, x, packed, scales, zeros, y, ws, epi);
    return sqp_launch_status();
}

template <int MT, int GS>
int by_chunks(const SqpStripPlan &p, int M, int N, int K, int cpg, const h16 *x, const uint32_t *packed, const h16 *scales,
              const uint8_t *zeros, h16 *y, int epi, const SqpWorkspace &ws, hipStream_t st)
{
    if (p.kp == 2 && cpg == 1) return launch_blocks<MT, 2, GS>(M, N, K, cpg, p.split, x, packed, scales, zeros, y, epi, ws, st);
    return launch_blocks<MT, 1, GS>(M, N, K, cpg, p.split, x, packed, scales, zeros, y, epi, ws, st);
}

template <int GS>
int by_rows(const SqpStripPlan &p, int M, int N, int K, int cpg, const h16 *x, const uint32_t *packed, const h16 *scales,
            const uint8_t *zeros, h16 *y, int epi, const SqpWorkspace &ws, hipStream_t st)
{
    if (p.mt == 3) return by_chunks<3, GS>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, ws, st);
    return by_chunks<4, GS>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, ws, st);
}

}  // namespace

int sqp_strip_row_blocks(int group, SQP_STRIP_ARGS)
{
    if (K % 128 != 0 || (group != 32 && group != 64 && group % 128 != 0)) return SQP_ERR_SHAPE;  // (a plan's mistake)
    if (group == 32) return by_rows<1>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, ws, st);
    if (group == 64) return by_rows<2>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, ws, st);
    return by_rows<4>(p, M, N, K, cpg, x, packed, scales, zeros, y, epi, ws, st);
}
