// Quantisation loss of one linear layer, Eq. 4 of arXiv 2312.03788:
//   E = || X W - X_hat W_hat ||_F^2,   W_hat = dequantised 4-bit weights (Eq. 1),
// with X_hat = X diag(s)^-1 and the quantised W_hat of diag(s) W (Eq. 5), as the search over the
// smoothing strength alpha needs it (Sec 2.2: alpha is chosen to minimise the loss).
//
// The two products are never rounded to fp16: that would swamp their difference.  Two kernels:
//
//   loss_split_kernel (K a multiple of 128, groups of 32 or a multiple of 64: every layer of the
//     paper's models): acc = X W over all of K, then acc -= X_hat W_hat over all of K, one fp32
//     accumulator per output element throughout.  X W does not depend on alpha, so the search
//     runs the first half once, keeps the accumulators (fp32) in device memory, and starts the
//     second half of every alpha from them: half the matrix work per alpha, and the same bits as
//     a single call, which runs both halves in one launch.
//   quant_loss_kernel (any other K or group): both products interleaved k-step by k-step.
//
// A workgroup owns a 128 x 128 tile, squares and sums its accumulators in fp64 and writes one
// partial; a second kernel adds the partials in a fixed order, so the result does not depend on
// scheduling.
#include "sqp_common.h"
#include "sqp_quantize_tile.h"
#include "sqp_w4_unpack.h"

namespace {

constexpr int LBM = 128, LBN = 128, LBK = 64, LPAD = 8;  // row stride 144 bytes: 16-byte reads of 32 rows spread over the banks

// ---------------------------------------------------------------- both halves, one after the other
//
// Eight waves: wave (kh, wm, wn) owns rows 64 wm .. +64 and columns 64 wn .. +64 of the tile (2 x 2
// tiles of v_mfma_f32_32x32x16_f16) for the k's of half kh of every 128-k stage; the two halves'
// sums meet in LDS.  A wave tile of 64 x 64 and not smaller, because the reads of X_hat from LDS
// bound the kernel otherwise: 64 x 32 per wave asks for 128 bytes per clock and compute unit, all
// that LDS gives, 64 x 64 for half of it.  The K halves give two waves per SIMD (one unpacks while
// the other multiplies) without smaller tiles.
//   X W: tiles through registers into LDS, W transposed on the way (8 rows x 2 columns per
//     thread, v_perm_b32), the next stage's loads in flight while one is multiplied.
//   X_hat W_hat: X_hat by direct global->LDS loads into a ring of three 32 KB slots (rows of
//     256 bytes, 16-byte pieces XOR-swizzled by row so that a read of 32 rows spreads over the
//     banks), packed words straight into registers (a word is one lane's B operand), two stages in
//     flight, one barrier per stage; loads and waits in assembly as in the GEMM kernels.  The search
//     stores X_hat with every 8 k in the order of the unpacked codes (MODE 2): no permute here.
// Column mapping: accumulator tile t, lane l: column 64 wn + 2 (l % 32) + t (two adjacent columns
// per lane: 8-byte loads of packed words).
// MODE: 0 = both halves, partials[block];  1 = X W only, accumulators to yacc;  2 = X_hat W_hat
// starting from yacc, partials[block].  yacc: [block][wm, wn][register / 4][lane][4] floats.
// What bounds it: the memory pipeline (48 KB per stage and compute unit out of L2), the unpack and the
// matrix cores take 0.4 to 0.5 us of a stage each and overlap in part: 1.0 us per stage (1.2 with all
// loads of a stage issued at once).  Reads from LDS and a fourth ring slot change nothing.
// Measured on 512 x 5120 x 5120 (160 tiles): second half 46 us, first half 75 us, both in one call
// 114 us, where the interleaved kernel takes 147 (8192 x 8192: 188 against 230).  The loss is off its
// 64-bit value by up to 7e-8 relative, as with the interleaved kernel.
constexpr int SBK = 128;                      // k per stage
constexpr int SSLOT = LBM * SBK * 2;          // bytes of X_hat per stage
constexpr int SROW = SBK + LPAD;              // halves per LDS row of the X W tiles

// PREP (MODE 2; 0 or the group size): the workgroups past row loss_rows of the grid, as many as the loss
// leaves compute units idle, prepare the next alpha meanwhile: weight tiles smoothed and quantised in
// turn, activations divided.
struct NextAlpha {
    const float *s;            // [K] its smoothing factors
    const uint4 *x, *w;        // activations, unsmoothed weight
    uint4 *x_hat;              // what it fills
    uint32_t *packed;
    uint16_t *scales;
    uint8_t *zeros;
    int loss_rows, workgroups;
};
template <int MODE, bool G32, int PREP>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
loss_split_kernel(int M, int N, int K, int group, const h16 *__restrict__ x, const h16 *__restrict__ w,
                  const h16 *__restrict__ xh, const uint32_t *__restrict__ packed, const h16 *__restrict__ scales,
                  const uint8_t *__restrict__ zeros, float *__restrict__ yacc, double *__restrict__ partials, NextAlpha next)
{
    constexpr int D = 3;                      // ring slots / register stages of the second half
    __shared__ __attribute__((aligned(1024))) unsigned char lds[D * SSLOT];
    __shared__ double red[8];
    if constexpr (PREP != 0) {
        if ((int)blockIdx.y >= next.loss_rows) {
            typedef QuantizeTile<PREP, 512> Tile;
            static_assert(sizeof(Tile) <= sizeof(lds), "the quantiser's LDS fits the ring");
            const int wg = ((int)blockIdx.y - next.loss_rows) * gridDim.x + blockIdx.x;
            if (wg >= next.workgroups) return;
            const int tx = (N + 255) / 256, tiles = tx * ((K + 255) / 256);
            for (int t = wg; t < tiles; t += next.workgroups)
                quantize_tile<PREP, 512, true>(t % tx, t / tx, N, K, next.w, next.s, next.packed, next.scales, next.zeros,
                                               *reinterpret_cast<Tile *>(lds));
            const int KO = K >> 3;
            const float4 *s4 = reinterpret_cast<const float4 *>(next.s);
            for (long i = (long)wg * 512 + threadIdx.x; i < (long)M * KO; i += (long)next.workgroups * 512) {
                const int ko = (int)(i % KO);
                next.x_hat[i] = code_order(smooth_x8(next.x[i], s4[2 * ko], s4[2 * ko + 1]));
            }
            return;
        }
    }
    static_assert(2 * 128 * SROW * 2 <= D * SSLOT && 4 * 64 * 64 * 4 <= D * SSLOT, "the tiles of X W and the exchange reuse the ring");

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kh = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;
    const int l32 = lane & 31, kb = lane >> 5;
    const int m0 = blockIdx.y * LBM, n0 = blockIdx.x * LBN;
    const long block = (long)blockIdx.y * gridDim.x + blockIdx.x;
    const int stages = K / SBK;
    const int ncol = n0 + wn * 64 + 2 * l32;                   // this lane's two columns (N is even: both in or out)
    const bool ncol_ok = ncol < N;

    f32x16 acc[2][2];
#pragma unroll
    for (int mt = 0; mt < 2; mt++)
#pragma unroll
        for (int t = 0; t < 2; t++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc[mt][t][r] = 0.f;

    // the second half's waves (kh == 1) hand their sums to the first's: acc(kh = 0) += acc(kh = 1)
    auto join = [&]() {
        f32x4 *ex = reinterpret_cast<f32x4 *>(lds) + (size_t)(wave & 3) * 16 * 64 + lane;
        __syncthreads();
        if (kh == 1) {
#pragma unroll
            for (int q = 0; q < 16; q++) {
                const f32x16 &a = acc[q >> 3][(q >> 2) & 1];
                ex[q * 64] = f32x4{a[(q & 3) * 4], a[(q & 3) * 4 + 1], a[(q & 3) * 4 + 2], a[(q & 3) * 4 + 3]};
            }
        }
        __syncthreads();
        if (kh == 0) {
#pragma unroll
            for (int q = 0; q < 16; q++) {
                const f32x4 v = ex[q * 64];
#pragma unroll
                for (int r = 0; r < 4; r++) acc[q >> 3][(q >> 2) & 1][(q & 3) * 4 + r] += v[r];
            }
        } else {
#pragma unroll
            for (int mt = 0; mt < 2; mt++)
#pragma unroll
                for (int t = 0; t < 2; t++)
#pragma unroll
                    for (int r = 0; r < 16; r++) acc[mt][t][r] = 0.f;
        }
        __syncthreads();
    };

    if constexpr (MODE != 2) {
        // ---- X W
        h16 (*sx)[SROW] = reinterpret_cast<h16 (*)[SROW]>(lds);
        h16 (*sw)[SROW] = reinterpret_cast<h16 (*)[SROW]>(lds + 128 * SROW * 2);
        const int arow = tid >> 2, apart = tid & 3;            // X: row, 32-half part of the 128 k
        const int agrow = m0 + arow < M ? m0 + arow : M - 1;   // rows past M: duplicates, masked at the end
        const int wkb = tid >> 6, wcp = tid & 63;              // W: k-blocks wkb and wkb + 8 of 8 rows, column pair
        const int wcol = n0 + 2 * wcp < N ? n0 + 2 * wcp : 0;  // columns past N likewise
        const h16 *px = x + (size_t)agrow * K + apart * 32;
        const h16 *pw = w + (size_t)(wkb * 8) * N + wcol;
        const int wrow = (wcp >> 5) * 64 + (wcp & 31);         // LDS row of the pair's first column; the second's is 32 further
        u32x4 rx[4];
        uint32_t rw[2][8];
        auto fetch = [&]() {
#pragma unroll
            for (int j = 0; j < 4; j++) rx[j] = *reinterpret_cast<const u32x4 *>(px + j * 8);
#pragma unroll
            for (int h = 0; h < 2; h++)
#pragma unroll
                for (int i = 0; i < 8; i++) rw[h][i] = *reinterpret_cast<const uint32_t *>(pw + (size_t)(h * 64 + i) * N);
            px += SBK;
            pw += (size_t)SBK * N;
        };
        fetch();
        for (int s = 0; s < stages; s++) {
#pragma unroll
            for (int j = 0; j < 4; j++) *reinterpret_cast<u32x4 *>(&sx[arow][apart * 32 + j * 8]) = rx[j];
#pragma unroll
            for (int h = 0; h < 2; h++) {
                uint4 c0, c1;  // the low halves of the 8 rows; the high halves
                c0.x = __builtin_amdgcn_perm(rw[h][1], rw[h][0], 0x05040100u); c1.x = __builtin_amdgcn_perm(rw[h][1], rw[h][0], 0x07060302u);
                c0.y = __builtin_amdgcn_perm(rw[h][3], rw[h][2], 0x05040100u); c1.y = __builtin_amdgcn_perm(rw[h][3], rw[h][2], 0x07060302u);
                c0.z = __builtin_amdgcn_perm(rw[h][5], rw[h][4], 0x05040100u); c1.z = __builtin_amdgcn_perm(rw[h][5], rw[h][4], 0x07060302u);
                c0.w = __builtin_amdgcn_perm(rw[h][7], rw[h][6], 0x05040100u); c1.w = __builtin_amdgcn_perm(rw[h][7], rw[h][6], 0x07060302u);
                *reinterpret_cast<uint4 *>(&sw[wrow][h * 64 + wkb * 8]) = c0;
                *reinterpret_cast<uint4 *>(&sw[wrow + 32][h * 64 + wkb * 8]) = c1;
            }
            __syncthreads();
            if (s + 1 < stages) fetch();
#pragma unroll
            for (int ks = 0; ks < 4; ks++) {
                const int kk = kh * 64 + ks * 16 + kb * 8;
                h16x8 a[2], b[2];
#pragma unroll
                for (int i = 0; i < 2; i++) {
                    a[i] = *reinterpret_cast<const h16x8 *>(&sx[wm * 64 + i * 32 + l32][kk]);
                    b[i] = *reinterpret_cast<const h16x8 *>(&sw[wn * 64 + i * 32 + l32][kk]);
                }
#pragma unroll
                for (int mt = 0; mt < 2; mt++)
#pragma unroll
                    for (int t = 0; t < 2; t++)
                        acc[mt][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[mt], b[t], acc[mt][t], 0, 0, 0);
            }
            __syncthreads();
        }
        join();
        if constexpr (MODE == 1) {
            if (kh == 0) {
                f32x4 *yo = reinterpret_cast<f32x4 *>(yacc) + ((size_t)block * 4 + wave) * 16 * 64 + lane;
#pragma unroll
                for (int q = 0; q < 16; q++) {
                    const f32x16 &a = acc[q >> 3][(q >> 2) & 1];
                    yo[q * 64] = f32x4{a[(q & 3) * 4], a[(q & 3) * 4 + 1], a[(q & 3) * 4 + 2], a[(q & 3) * 4 + 3]};
                }
            }
            return;
        }
    } else {
        if (kh == 0) {
            const f32x4 *yi = reinterpret_cast<const f32x4 *>(yacc) + ((size_t)block * 4 + wave) * 16 * 64 + lane;
#pragma unroll
            for (int q = 0; q < 16; q++) {
                const f32x4 v = yi[q * 64];
#pragma unroll
                for (int r = 0; r < 4; r++) acc[q >> 3][(q >> 2) & 1][(q & 3) * 4 + r] = v[r];
            }
        }
    }

    if constexpr (MODE != 1) {
        // ---- - X_hat W_hat
        constexpr int NQ = G32 ? 2 : 1;       // quantisation groups per half stage (64 k)
        constexpr int OX = 4, OW = 4 + 2 * NQ;  // loads per wave and stage: X_hat, words and group parameters
        const UnpackConsts uc = SQP_UNPACK_CONSTS;
        struct Stage {
            u32x2 w[4];       // per k-step of 16: the packed words of the lane's two columns
            uint32_t sc[NQ];  // two fp16 steps
            uint32_t zr[NQ];  // two zero points, one byte each
        };
        const int col = ncol_ok ? ncol : 0;
        const uint32_t voff_w = (uint32_t)(kb * N + col) * 4u, voff_s = (uint32_t)col * 2u, voff_z = (uint32_t)col;
        const long wrow2 = (long)N * 8;       // two packed rows (one k-step) in bytes
        // wave-uniform byte pointers, stepped per stage; past the last stage they stop and the
        // look-ahead re-reads it
        const unsigned char *wq = reinterpret_cast<const unsigned char *>(packed) + (long)kh * 4 * wrow2;
        const unsigned char *xq = reinterpret_cast<const unsigned char *>(xh);
        const int hpg = G32 ? 1 : __builtin_amdgcn_readfirstlane(group / 64);  // half stages per group (G32: two groups per half stage)
        int kin = hpg == 1 ? 0 : kh;           // position of this wave's half stage in its group
        int prow = G32 ? kh * 2 : (hpg == 1 ? kh : 0);  // parameter row of the half stage being issued
        int ist = 0;                           // stage being issued
        // X_hat: wave w copies blocks w, w + 8, ... of the stage (a block = 4 rows x 256 bytes); lane i
        // of a block handles row i / 16 and fetches piece (i % 16) ^ (row % 16) of it
        uint32_t xoff[OX];
#pragma unroll
        for (int j = 0; j < OX; j++) {
            const int row = (wave + 8 * j) * 4 + (lane >> 4);
            const int grow = m0 + row < M ? m0 + row : M - 1;
            xoff[j] = (uint32_t)grow * (uint32_t)K * 2u + (uint32_t)(((lane & 15) ^ (row & 15)) * 16);
        }
        // One quarter of a stage's loads (spread over the k-steps of the stage in progress: all at once they
        // fill the memory pipeline and hold the waves up in front of their arithmetic).
        auto issue_part = [&](Stage &st, int slot, int part) {
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(xq + xoff[part]),
                                             (__attribute__((address_space(3))) void *)(lds + slot * SSLOT + (wave + 8 * part) * 1024), 16, 0, 0);
            const unsigned char *base = wq + part * wrow2;  // wave-uniform
            asm volatile("global_load_dwordx2 %0, %1, %2" : "=v"(st.w[part]) : "v"(voff_w), "s"(base) : "memory");
            if (part < NQ) {
                const long row = (long)__builtin_amdgcn_readfirstlane(prow + part) * N;  // wave-uniform
                const unsigned char *sg = reinterpret_cast<const unsigned char *>(scales) + row * 2, *zg = zeros + row;
                asm volatile("global_load_dword %0, %1, %2" : "=v"(st.sc[part]) : "v"(voff_s), "s"(sg) : "memory");
                asm volatile("global_load_ushort %0, %1, %2" : "=v"(st.zr[part]) : "v"(voff_z), "s"(zg) : "memory");
            }
            if (part < 3) return;
            // step to the next stage, unless this was the last
            const bool more = ist + 1 < stages;
            ist += more ? 1 : 0;
            wq += more ? 8 * wrow2 : 0;
            xq += more ? SBK * 2 : 0;
            if constexpr (G32) {
                prow += more ? 4 : 0;
            } else {                           // groups of 64: two rows per stage
                kin += more ? 2 : 0;
                if (kin >= hpg) { kin -= hpg; prow++; }
                if (kin >= hpg) { kin -= hpg; prow++; }
            }
        };
        auto issue = [&](Stage &st, int slot) {
#pragma unroll
            for (int i = 0; i < 4; i++) issue_part(st, slot, i);
        };
        auto landed = [&](Stage &st) {         // all but the youngest stage's loads have arrived
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(OX + OW) : "memory");
#pragma unroll
            for (int ks = 0; ks < 4; ks++) asm volatile("" : "+v"(st.w[ks]));
#pragma unroll
            for (int g = 0; g < NQ; g++) {
                asm volatile("" : "+v"(st.sc[g]));
                asm volatile("" : "+v"(st.zr[g]));
            }
        };
        // LDS address of this lane's A fragment (row 64 wm + l32, + 32 for the second row tile) in slot 0
        const uint32_t xrd = (uint32_t)(size_t)lds + (uint32_t)((wm * 64 + l32) * 256);
        const int xkey = l32 & 15;
        // stage st in `slot`, with the loads into stage nst and slot nslot in between
        auto compute = [&](const Stage &st, int slot, Stage &nst, int nslot) {
            u32x4 xa[2][2];
            auto read_a = [&](int ks) {
                const uint32_t a = xrd + (uint32_t)(slot * SSLOT) + (uint32_t)(((kh * 8 + ks * 2 + kb) ^ xkey) * 16);
                asm volatile("ds_read_b128 %0, %1" : "=&v"(xa[ks & 1][0]) : "v"(a) : "memory");
                asm volatile("ds_read_b128 %0, %1 offset:8192" : "=&v"(xa[ks & 1][1]) : "v"(a) : "memory");
            };
            read_a(0);
            h16x2 neg_hi[NQ][2], neg_lo[NQ][2], delta[NQ][2];
#pragma unroll
            for (int g = 0; g < NQ; g++)
#pragma unroll
                for (int t = 0; t < 2; t++) {
                    const uint32_t z = (st.zr[g] >> (8 * t)) & 0xffu;
                    neg_hi[g][t] = neg_hi_of(z);
                    neg_lo[g][t] = neg_lo_of(z);
                    const uint32_t sw = st.sc[g] ^ 0x80008000u;  // the negated steps
                    delta[g][t] = __builtin_bit_cast(h16x2, __builtin_amdgcn_perm(sw, sw, t ? 0x03020302u : 0x01000100u));
                }
            // The fragments of the next k-step are on their way from LDS, and its words are unpacked
            // between the MFMAs of this one (the scheduler is told so: left alone it puts the read and
            // its wait next to each other and the unpack in front of the MFMAs).
            h16x8 b[2][2];
            auto unpack = [&](int ks) {
                const int g = G32 ? ks >> 1 : 0;
#pragma unroll
                for (int t = 0; t < 2; t++) b[ks & 1][t] = dequant_word_scaled(st.w[ks][t], neg_hi[g][t], neg_lo[g][t], delta[g][t], uc);
            };
            unpack(0);
#pragma unroll
            for (int ks = 0; ks < 4; ks++) {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
                for (int mt = 0; mt < 2; mt++) asm volatile("" : "+v"(xa[ks & 1][mt]));
                if (ks < 3) read_a(ks + 1);
                issue_part(nst, nslot, ks);
                __builtin_amdgcn_sched_barrier(0);
                if (ks < 3) unpack(ks + 1);
#pragma unroll
                for (int mt = 0; mt < 2; mt++) {
                    // (MODE 2: the search stores X_hat in the order of the unpacked codes)
                    const h16x8 a = MODE == 2 ? __builtin_bit_cast(h16x8, xa[ks & 1][mt]) : permute_x(xa[ks & 1][mt]);
#pragma unroll
                    for (int t = 0; t < 2; t++)
                        acc[mt][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b[ks & 1][t], acc[mt][t], 0, 0, 0);
                }
                if constexpr (MODE != 2) __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);  // first operand: 4 VALU
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // 1 MFMA
                __builtin_amdgcn_sched_group_barrier(0x002, 7, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 7, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 7, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 7, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        Stage st[D];
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // nothing of the compiler's own is counted below
        issue(st[0], 0);
        issue(st[1], 1);
        const int nblk = (stages + D - 1) / D;
        for (int b = 0; b < nblk; b++) {
#pragma unroll
            for (int d = 0; d < D; d++) {
                // Stage s = b D + d has landed for this wave; after the barrier for all of them,
                // and no wave reads the slot of stage s - 1 any more, which is filled next.
                // Stages past the end only keep the load counts in step.
                landed(st[d]);
                asm volatile("s_barrier" ::: "memory");
                if (b * D + d < stages) compute(st[d], d, st[(d + 2) % D], (d + 2) % D);
                else issue(st[(d + 2) % D], (d + 2) % D);
            }
        }
        // the look-ahead loads still in flight land in registers and slots that nothing else may use before
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
        for (int j = 0; j < D; j++) {
#pragma unroll
            for (int ks = 0; ks < 4; ks++) asm volatile("" ::"v"(st[j].w[ks]));
#pragma unroll
            for (int g = 0; g < NQ; g++) {
                asm volatile("" ::"v"(st[j].sc[g]));
                asm volatile("" ::"v"(st[j].zr[g]));
            }
        }
        join();

        // ---- sum of squares of the tile.  Register r of row tile mt: row 8*(r/4) + 4*(lane/32) + r%4
        double ss = 0.0;
        if (kh == 0) {
#pragma unroll
            for (int mt = 0; mt < 2; mt++)
#pragma unroll
                for (int t = 0; t < 2; t++)
#pragma unroll
                    for (int r = 0; r < 16; r++) {
                        const int row = m0 + wm * 64 + mt * 32 + 8 * (r >> 2) + 4 * kb + (r & 3);
                        if (row < M && ncol_ok) ss += (double)acc[mt][t][r] * (double)acc[mt][t][r];
                    }
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) ss += __shfl_xor(ss, off, 64);
        if (lane == 0) red[wave] = ss;
        __syncthreads();
        if (tid == 0) partials[block] = (red[0] + red[1]) + (red[2] + red[3]);
    }
}

// Whether loss_split_kernel covers a shape.
bool loss_split_covers(int K, int group) { return K % SBK == 0 && (group == 32 || group % 64 == 0); }

template <int MODE>
void launch_loss_split(int M, int N, int K, int group, const void *x, const void *w, const void *x_hat, const uint32_t *packed,
                       const void *scales, const uint8_t *zeros, float *yacc, double *partials, hipStream_t st)
{
    const dim3 grid((N + LBN - 1) / LBN, (M + LBM - 1) / LBM);
    if (group == 32)
        loss_split_kernel<MODE, true, 0><<<grid, 512, 0, st>>>(M, N, K, group, (const h16 *)x, (const h16 *)w, (const h16 *)x_hat, packed,
                                                               (const h16 *)scales, zeros, yacc, partials, NextAlpha());
    else
        loss_split_kernel<MODE, false, 0><<<grid, 512, 0, st>>>(M, N, K, group, (const h16 *)x, (const h16 *)w, (const h16 *)x_hat, packed,
                                                                (const h16 *)scales, zeros, yacc, partials, NextAlpha());
}

// The second half of one alpha beside the preparation of the next (groups of 32, 64, 128, 256).
void launch_loss_and_next(int M, int N, int K, int group, const void *x_hat, const uint32_t *packed, const void *scales,
                          const uint8_t *zeros, float *yacc, double *partials, NextAlpha next, hipStream_t st)
{
    const int gx = (N + LBN - 1) / LBN, gy = (M + LBM - 1) / LBM;
    next.loss_rows = gy;
    const dim3 grid(gx, gy + (next.workgroups + gx - 1) / gx);
#define SQP_LOSS_NEXT(G32, G) \
    loss_split_kernel<2, G32, G><<<grid, 512, 0, st>>>(M, N, K, group, nullptr, nullptr, (const h16 *)x_hat, packed, (const h16 *)scales, zeros, yacc, partials, next)
    if (group == 32) SQP_LOSS_NEXT(true, 32);
    else if (group == 64) SQP_LOSS_NEXT(false, 64);
    else if (group == 128) SQP_LOSS_NEXT(false, 128);
    else SQP_LOSS_NEXT(false, 256);
#undef SQP_LOSS_NEXT
}

// ---------------------------------------------------------------- both products interleaved
//
// One contraction over the concatenated inner dimension [X, X_hat] * [W; -W_hat]: per k-step one
// MFMA with the fp16 weights and one with the negated dequantised codes; eight waves with tiles of
// 64 x 32, all tiles through registers into LDS, packed words unpacked in registers.  The global
// loads of the next k-step are issued before the current one is multiplied.

// FULL: M and N are multiples of the tile and K of the k-step, so no access needs a bounds check.
template <bool FULL>
__global__ void __launch_bounds__(512)
quant_loss_kernel(int M, int N, int K, int group, const h16 *__restrict__ x, const h16 *__restrict__ w,
                  const h16 *__restrict__ xh, const uint32_t *__restrict__ packed, const h16 *__restrict__ scales,
                  const uint8_t *__restrict__ zeros, double *__restrict__ partials)
{
    __shared__ __attribute__((aligned(16))) h16 sx[LBM][LBK + LPAD];
    __shared__ __attribute__((aligned(16))) h16 sxh[LBM][LBK + LPAD];
    __shared__ __attribute__((aligned(16))) h16 sw[LBN][LBK + LPAD];  // transposed: [column][k]
    __shared__ double red[8];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 2, wn = wave & 3;                   // wave tile: rows wm*64 .. +64, columns wn*32 .. +32
    const int l32 = lane & 31, kb = lane >> 5;
    const int m0 = blockIdx.y * LBM, n0 = blockIdx.x * LBN;
    const UnpackConsts uc = SQP_UNPACK_CONSTS;

    f32x16 acc[2];
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int r = 0; r < 16; r++) acc[i][r] = 0.f;

    // loader roles
    const int arow = tid >> 2, apart = tid & 3;               // X, X_hat: row, 16-half part of the 64 k
    int agrow = m0 + arow;
    if (!FULL && agrow >= M) agrow = M - 1;                    // rows past M: duplicates, masked at the end
    const int wkb = tid >> 6, wcp = tid & 63;                  // W: k-block of 8 rows, column pair
    const int wcol = n0 + 2 * wcp;
    const int qcol = n0 + wn * 32 + l32;                       // packed words: this lane's column
    const bool wcol_ok = FULL || wcol < N, qcol_ok = FULL || qcol < N;
    // per-thread pointers at this thread's piece of k-step 0, advanced by one step per iteration
    const h16 *px = x + (size_t)agrow * K + apart * 16;
    const h16 *ph = xh + (size_t)agrow * K + apart * 16;
    const h16 *pw = w + (size_t)(wkb * 8) * N + (wcol_ok ? wcol : 0);
    const uint32_t *pq = packed + (size_t)kb * N + (qcol_ok ? qcol : 0);
    const bool one_group = group % LBK == 0;                   // a k-step lies within one quantisation group

    // Software pipeline over the k-steps: the global loads of step k0 + LBK are in flight (into
    // registers) while step k0 is multiplied out of LDS; two waves per SIMD cover each other's waits.
    uint4 rx[2], rh[2];     // X and X_hat: this thread's 2 x 8 halves of its row
    uint32_t rw[8];         // W: 8 rows x one column pair
    uint32_t rword[4], rz[4], rd[4];  // packed word, zero point, negated step per k sub-step
    auto fetch = [&](int k0) {
#pragma unroll
        for (int j = 0; j < 2; j++) {
            const bool ok = FULL || k0 + apart * 16 + j * 8 < K;
            rx[j] = ok ? *reinterpret_cast<const uint4 *>(px + j * 8) : make_uint4(0, 0, 0, 0);
            rh[j] = ok ? *reinterpret_cast<const uint4 *>(ph + j * 8) : make_uint4(0, 0, 0, 0);
        }
        const bool wok = FULL || (wcol_ok && k0 + wkb * 8 < K);          // K is a multiple of 8: a block of 8 rows is in or out as a whole
#pragma unroll
        for (int i = 0; i < 8; i++) rw[i] = wok ? *reinterpret_cast<const uint32_t *>(pw + (size_t)i * N) : 0u;
        const int gstep = k0 / group;
#pragma unroll
        for (int ks = 0; ks < 4; ks++) {
            const int kk = k0 + ks * 16 + kb * 8;
            rword[ks] = 0; rz[ks] = 0; rd[ks] = 0;
            if (FULL || (qcol_ok && kk < K)) {
                const size_t gi = (size_t)(one_group ? gstep : kk / group) * N + qcol;
                rword[ks] = pq[(size_t)(ks * 2) * N];
                rz[ks] = zeros[gi];
                rd[ks] = __builtin_bit_cast(uint16_t, scales[gi]) ^ 0x8000u;  // -Delta
            }
        }
        px += LBK; ph += LBK; pw += (size_t)LBK * N; pq += (size_t)(LBK / 8) * N;
    };
    fetch(0);
    for (int k0 = 0; k0 < K; k0 += LBK) {
        // ---- registers -> LDS
#pragma unroll
        for (int j = 0; j < 2; j++) {
            *reinterpret_cast<uint4 *>(&sx[arow][apart * 16 + j * 8]) = rx[j];
            *reinterpret_cast<uint4 *>(&sxh[arow][apart * 16 + j * 8]) = rh[j];
        }
        {
            uint4 c0, c1;  // column wcol: the low halves of the 8 rows; column wcol + 1: the high halves
            c0.x = __builtin_amdgcn_perm(rw[1], rw[0], 0x05040100u); c1.x = __builtin_amdgcn_perm(rw[1], rw[0], 0x07060302u);
            c0.y = __builtin_amdgcn_perm(rw[3], rw[2], 0x05040100u); c1.y = __builtin_amdgcn_perm(rw[3], rw[2], 0x07060302u);
            c0.z = __builtin_amdgcn_perm(rw[5], rw[4], 0x05040100u); c1.z = __builtin_amdgcn_perm(rw[5], rw[4], 0x07060302u);
            c0.w = __builtin_amdgcn_perm(rw[7], rw[6], 0x05040100u); c1.w = __builtin_amdgcn_perm(rw[7], rw[6], 0x07060302u);
            *reinterpret_cast<uint4 *>(&sw[2 * wcp][wkb * 8]) = c0;
            *reinterpret_cast<uint4 *>(&sw[2 * wcp + 1][wkb * 8]) = c1;
        }
        // ---- packed words of this wave's 32 columns: registers only
        h16x8 bq[4];
#pragma unroll
        for (int ks = 0; ks < 4; ks++)
            bq[ks] = dequant_word_scaled(rword[ks], neg_hi_of(rz[ks]), neg_lo_of(rz[ks]),
                                         __builtin_bit_cast(h16x2, rd[ks] * 0x00010001u), uc);
        __syncthreads();
        if (k0 + LBK < K) fetch(k0 + LBK);
#pragma unroll
        for (int ks = 0; ks < 4; ks++) {
            h16x8 ax[2], ah[2];
#pragma unroll
            for (int mt = 0; mt < 2; mt++) {
                const int row = wm * 64 + mt * 32 + l32;
                ax[mt] = *reinterpret_cast<const h16x8 *>(&sx[row][ks * 16 + kb * 8]);
                ah[mt] = permute_x(*reinterpret_cast<const u32x4 *>(&sxh[row][ks * 16 + kb * 8]));
            }
            const h16x8 bw = *reinterpret_cast<const h16x8 *>(&sw[wn * 32 + l32][ks * 16 + kb * 8]);
#pragma unroll
            for (int mt = 0; mt < 2; mt++) {
                acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ax[mt], bw, acc[mt], 0, 0, 0);
                acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah[mt], bq[ks], acc[mt], 0, 0, 0);
            }
        }
        __syncthreads();
    }

    // ---- sum of squares of the tile.  Accumulator register r of tile mt: row
    // 8*(r/4) + 4*(lane/32) + r%4 of the 32-row tile, column lane%32.
    double ss = 0.0;
#pragma unroll
    for (int mt = 0; mt < 2; mt++)
#pragma unroll
        for (int r = 0; r < 16; r++) {
            const int row = m0 + wm * 64 + mt * 32 + 8 * (r >> 2) + 4 * kb + (r & 3);
            if (FULL || (row < M && qcol_ok)) ss += (double)acc[mt][r] * (double)acc[mt][r];
        }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) ss += __shfl_xor(ss, off, 64);
    if (lane == 0) red[wave] = ss;
    __syncthreads();
    if (tid == 0)
        partials[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = ((red[0] + red[1]) + (red[2] + red[3])) + ((red[4] + red[5]) + (red[6] + red[7]));
}

// Adds n partials in a fixed order: thread t takes t, t + 256, ..., then a tree over the block.
// One workgroup per loss (block b: partials b n .. b n + n - 1 to out[b]).
__global__ void __launch_bounds__(256) sum_partials_kernel(const double *__restrict__ partials, long n, double *__restrict__ out)
{
    __shared__ double s[256];
    partials += (size_t)blockIdx.x * n;
    double a = 0.0;
    for (long i = threadIdx.x; i < n; i += 256) a += partials[i];
    s[threadIdx.x] = a;
    __syncthreads();
    for (int half = 128; half >= 1; half >>= 1) {
        if ((int)threadIdx.x < half) s[threadIdx.x] += s[threadIdx.x + half];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[blockIdx.x] = s[0];
}

// Index of the smallest of n values, the lowest index on ties (n is a grid of alphas: tiny).
__global__ void argmin_kernel(const double *__restrict__ v, int n, int *__restrict__ best)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    int b = 0;
    for (int i = 1; i < n; i++)
        if (v[i] < v[b]) b = i;
    *best = b;
}

}  // namespace

extern "C" long sqp_quant_loss_scratch_doubles(int M, int N)
{
    if (M <= 0 || N <= 0) return 0;
    return (long)((M + LBM - 1) / LBM) * (long)((N + LBN - 1) / LBN);
}

extern "C" int sqp_quant_loss(int M, int N, int K, int group, const void *x, const void *w, const void *x_hat,
                              const uint32_t *packed, const void *scales, const uint8_t *zeros, double *scratch,
                              double *loss, void *stream)
{
    if (!x || !w || !x_hat || !packed || !scales || !zeros || !scratch || !loss) return SQP_ERR_NULL;
    if (M <= 0) return SQP_ERR_SHAPE;
    int rc = sqp_check_quant_shape(N, K, group);
    if (rc) return rc;
    if (sqp_too_big(M, K) || sqp_too_big(M, N)) return SQP_ERR_SHAPE;
    if (sqp_misaligned(x) || sqp_misaligned(w) || sqp_misaligned(x_hat) || sqp_misaligned(packed) ||
        sqp_misaligned(scales) || sqp_misaligned(zeros))
        return SQP_ERR_ALIGN;
    if ((reinterpret_cast<uintptr_t>(scratch) & 7u) || (reinterpret_cast<uintptr_t>(loss) & 7u)) return SQP_ERR_ALIGN;
    const int gy = (M + LBM - 1) / LBM, gx = (N + LBN - 1) / LBN;
    if (gy > 65535) return SQP_ERR_SHAPE;
    hipStream_t st = (hipStream_t)stream;
    if (loss_split_covers(K, group))
        launch_loss_split<0>(M, N, K, group, x, w, x_hat, packed, scales, zeros, nullptr, scratch, st);
    else if (M % LBM == 0 && N % LBN == 0 && K % LBK == 0)
        quant_loss_kernel<true><<<dim3(gx, gy), 512, 0, st>>>(M, N, K, group, (const h16 *)x, (const h16 *)w, (const h16 *)x_hat,
                                                             packed, (const h16 *)scales, zeros, scratch);
    else
        quant_loss_kernel<false><<<dim3(gx, gy), 512, 0, st>>>(M, N, K, group, (const h16 *)x, (const h16 *)w, (const h16 *)x_hat,
                                                              packed, (const h16 *)scales, zeros, scratch);
    sum_partials_kernel<<<1, 256, 0, st>>>(scratch, (long)gx * gy, loss);
    return sqp_launch_status();
}

extern "C" int sqp_alpha_search(int T, int N, int K, int group, int n_alpha, const float *alphas, const void *x_cal,
                                const void *w, float *amax, float *s, void *x_hat, void *w_s, uint32_t *packed,
                                void *scales, uint8_t *zeros, double *scratch, double *loss, int *best, void *stream)
{
    if (!alphas || !x_cal || !w || !amax || !s || !x_hat || !w_s || !packed || !scales || !zeros || !scratch || !loss || !best)
        return SQP_ERR_NULL;
    if (T <= 0 || n_alpha <= 0 || n_alpha > 4096) return SQP_ERR_SHAPE;
    int rc = sqp_check_quant_shape(N, K, group);
    if (rc) return rc;
    if (sqp_too_big(T, K) || sqp_too_big(T, N)) return SQP_ERR_SHAPE;
    if ((T + LBM - 1) / LBM > 65535 || K / group > 65535) return SQP_ERR_SHAPE;
    for (int i = 0; i < n_alpha; i++)
        if (!(alphas[i] >= 0.0f && alphas[i] <= 1.0f)) return SQP_ERR_ARG;
    if (sqp_misaligned(x_cal) || sqp_misaligned(w) || sqp_misaligned(amax) || sqp_misaligned(s) || sqp_misaligned(x_hat) ||
        sqp_misaligned(w_s) || sqp_misaligned(packed) || sqp_misaligned(scales) || sqp_misaligned(zeros))
        return SQP_ERR_ALIGN;
    if ((reinterpret_cast<uintptr_t>(scratch) & 7u) || (reinterpret_cast<uintptr_t>(loss) & 7u) ||
        (reinterpret_cast<uintptr_t>(best) & 3u))
        return SQP_ERR_ALIGN;
    // every check any step below would make has passed: from here on only launch errors can occur
    hipStream_t st = (hipStream_t)stream;
    rc = sqp_channel_absmax(T, K, N, x_cal, w, amax, st);
    // X W once for all alphas.  Its accumulators, the factors of all alphas and the tile sums live in
    // w_s, which the search otherwise fills with the smoothed weight: here the quantisation
    // smooths the weight as it reads it, and w_s gets the last alpha's smoothed weight at the end.
    // Taken wherever they fit there, i.e. from about K = 2 T on (4 bytes per element of the padded
    // [T][N] against 2 per element of [K][N]); shorter K runs the single calls in turn.
    // Measured, 21 alphas on 512 x 5120 x 5120: 4.71 -> 1.26 ms.
    const size_t blocks = (size_t)((T + LBM - 1) / LBM) * ((N + LBN - 1) / LBN);
    const size_t ybytes = blocks * LBM * LBN * sizeof(float), fbytes = (size_t)n_alpha * K * sizeof(float);
    if (loss_split_covers(K, group) && ybytes + fbytes + n_alpha * blocks * sizeof(double) <= (size_t)K * N * sizeof(h16)) {
        float *yacc = (float *)w_s, *factors = (float *)((unsigned char *)w_s + ybytes);
        double *tile_sums = (double *)((unsigned char *)w_s + ybytes + fbytes);
        if (rc == SQP_OK) rc = sqp_smooth_factors(K, n_alpha, alphas, amax, factors, st);
        if (rc == SQP_OK) rc = sqp_smooth_factor(K, alphas[n_alpha - 1], amax, s, st);
        if (rc != SQP_OK) return rc;
        launch_loss_split<1>(T, N, K, group, x_cal, w, nullptr, nullptr, nullptr, nullptr, yacc, nullptr, st);
        // Where the loss tiles leave at least a quarter of the chip idle (160 of 256 on 512 x 5120), the next
        // alpha is prepared there meanwhile, into a second set of buffers behind the tile sums; the last
        // alpha uses the caller's set.  Per alpha on 512 x 5120 x 5120: 69 us one after the other, 56 beside.
        const int idle = sqp_compute_units() - (int)(blocks < 65536 ? blocks : 65536);
        auto up256 = [](size_t v) { return (v + 255) & ~(size_t)255; };
        const size_t rows = (size_t)(K / group);
        const size_t at_packed = up256(ybytes + fbytes + n_alpha * blocks * sizeof(double));
        const size_t at_scales = up256(at_packed + (size_t)K / 8 * N * 4), at_zeros = up256(at_scales + rows * N * 2);
        const size_t at_x = up256(at_zeros + rows * N), end = at_x + (size_t)T * K * sizeof(h16);
        const bool beside = 4 * idle >= sqp_compute_units() && (group == 32 || group == 64 || group == 128 || group == 256) &&
                            end <= (size_t)K * N * sizeof(h16);
        unsigned char *const base = (unsigned char *)w_s;
        struct {
            void *x_hat;
            uint32_t *packed;
            void *scales;
            uint8_t *zeros;
        } set[2] = {{x_hat, packed, scales, zeros}, {base + at_x, (uint32_t *)(base + at_packed), base + at_scales, base + at_zeros}};
        for (int i = 0; i < n_alpha && rc == SQP_OK; i++) {
            const auto &cur = set[beside ? (n_alpha - 1 - i) & 1 : 0], &nxt = set[beside ? (n_alpha - i) & 1 : 0];
            if (!beside || i == 0)
                rc = sqp_smooth_quantize(T, N, K, group, x_cal, w, factors + (size_t)i * K, cur.x_hat, cur.packed, cur.scales, cur.zeros, st);
            if (beside && i + 1 < n_alpha) {
                const NextAlpha next = {factors + (size_t)(i + 1) * K, (const uint4 *)x_cal, (const uint4 *)w, (uint4 *)nxt.x_hat,
                                        nxt.packed, (uint16_t *)nxt.scales, nxt.zeros, 0, idle};
                launch_loss_and_next(T, N, K, group, cur.x_hat, cur.packed, cur.scales, cur.zeros, yacc, tile_sums + i * blocks, next, st);
            } else {
                launch_loss_split<2>(T, N, K, group, nullptr, nullptr, cur.x_hat, cur.packed, cur.scales, cur.zeros, yacc, tile_sums + i * blocks, st);
            }
        }
        sum_partials_kernel<<<n_alpha, 256, 0, st>>>(tile_sums, (long)blocks, loss);
        argmin_kernel<<<1, 64, 0, st>>>(loss, n_alpha, best);
        // x_hat and w_s as the single calls leave them
        if (rc == SQP_OK) rc = sqp_smooth_apply_x(T, K, x_cal, s, x_hat, stream);
        if (rc == SQP_OK) rc = sqp_smooth_apply_w(K, N, w, s, w_s, stream);
        return rc != SQP_OK ? rc : sqp_launch_status();
    }
    for (int i = 0; i < n_alpha && rc == SQP_OK; i++) {
        rc = sqp_smooth_factor(K, alphas[i], amax, s, st);
        if (rc == SQP_OK) rc = sqp_smooth_apply_x(T, K, x_cal, s, x_hat, stream);
        if (rc == SQP_OK) rc = sqp_smooth_apply_w(K, N, w, s, w_s, stream);
        if (rc == SQP_OK) rc = sqp_quantize_pack(N, K, group, w_s, packed, scales, zeros, stream);
        if (rc == SQP_OK) rc = sqp_quant_loss(T, N, K, group, x_cal, w, x_hat, packed, scales, zeros, scratch, loss + i, stream);
    }
    if (rc != SQP_OK) return rc;
    argmin_kernel<<<1, 64, 0, st>>>(loss, n_alpha, best);
    return sqp_launch_status();
}
