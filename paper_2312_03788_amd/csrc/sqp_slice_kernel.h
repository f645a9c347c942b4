// Column-slice variant of the weight-streaming W4A16 GEMM (decode, up to 32 rows): y = x * w_hat, Eq. 3 of
// arXiv 2312.03788 with w_hat = (code - Z) * Delta of Eq. 1, group-wise along K (Sec 2.2).
//
// The strip kernel splits K across workgroups to fill the chip, and the hand-over of partial
// sums between workgroups (through memory, with a ticket) costs a fixed few microseconds per
// launch - as much as streaming the whole layer on the narrowest ones.  Here a workgroup owns a
// slice of 16 TB output columns (16, 32 or 64) over ALL of K and K is split between its waves
// instead: wave w takes the chunks (128 k each) w, w + WV, w + 2 WV, ...; the waves never meet
// in the main loop (each fetches the activations of its own chunks into LDS slots of
// its own, so there is no barrier) and add their fp32 sums through LDS at the end, in wave
// order: no workspace, no tickets, and the result does not depend on scheduling.
// The price: every workgroup fetches all of x (from L2), workgroups x rows x K x 2 bytes per
// launch.  Only the blocks of four rows that hold real rows are fetched.
//
// Column mapping: lane (lc = lane % 16, lk = lane / 16) holds the TB adjacent columns
// n0 + TB lc ... (one load per k-step: their packed words, k-block lk), which are
// the B operands of TB v_mfma_f32_16x16x32_f16 (column block b = every TB-th column of the
// slice, starting at b); their steps Delta are one load, their zero points another.  With the
// fused SiLU(gate)*up output a lane's columns are whole (gate, up) pairs (TB >= 2).
//
// Unpack: the exact fp16 differences code - Z (dequant_word) are multiplied, a group is summed in fp32, and its
// sum is added with one FMA by its step.  Rows are repeated in the 16-row operand so that up to 4 (8) rows need
// only 1 (2) of the 4 registers of a lane scaled.  (The nibbles masked out of a word are fp16 denormals that the
// matrix cores take as they are: four operations of nine less per word, with Z sum x taken off a group's sum
// afterwards.  That subtracts two sums of the size Z sum |x| - a column whose codes are all Z did not give
// 0, errors grew by up to 3 % behind the fp16 rounding - and it was no faster: 0.5 % slower in the mean of
// 6814 calls, 1 % faster at one to four rows.)
//
// What bounds it: up to 8 rows on wide layers the vector instructions beside the loads, on narrow layers the
// latency of a wave's chunks, with many rows the activations.
// us per launch, weights from HBM, strip kernel or 32- and 64-column slices of eight waves alone -> now, 1 / 8 / 16
// rows: 1024->1024 6.3 / 6.5 / 6.6 -> 2.4 / 2.5 / 2.7, 4096->1024 7.2 / 7.3 / 7.4 -> 4.4 / 5.0 / 5.9,
// 4096->4096 5.7 / 6.2 / 7.1 -> 4.8 / 5.3 / 6.1, 4096->12288 8.2 / 8.8 / 9.7 -> 7.5 / 8.1 / 9.1,
// 4096->22016 13.4 / 14.1 / 15.8 -> 11.6 / 13.0 / 15.0, 12288->4096 at one row 10.6 -> 9.7; with each word unpacked in
// front of the MFMAs of the one before (up to 16 rows, groups of 64 and more) 4096->12288 at one row 7.31 -> 7.17 (weights
// in the last-level cache: 6.28 -> 6.02), 4096->22016 10.63 -> 10.44 there, 8192->44032 at four rows 34.6 -> 33.8, 4096->4096
// as before.
// Three and four stages per wave are slower everywhere (again, also with loads masked instead of skipped
// at the end).
#pragma once
#include <type_traits>

#include "sqp_common.h"
#include "sqp_slice.h"
#include "sqp_w4_unpack.h"

namespace {

// MT: 16-row tiles.  TB: columns per lane.  WV: waves per workgroup, each with two stages (registers for
// the weight side, LDS slots for the activations): one chunk is in flight while one is consumed.
// XB: blocks of four activation rows that are fetched (M <= 4 XB).
// GS: k-steps of a chunk that belong to one group: four, two (groups of 64) or one (groups of 32).
// CPG: groups of several chunks (GS == 4).
template <int MT, int TB, int WV, int XB, int GS, bool CPG>
__global__ void __launch_bounds__(WV * 64) __attribute__((amdgpu_waves_per_eu(MT == 1 && TB == 4 && WV == 8 && GS >= 2 ? 4 : 1)))
w4a16_decode_slice_kernel(int M, int N, int K, int cpg, int grouped, const h16 *__restrict__ x, const uint32_t *__restrict__ packed,
                          const h16 *__restrict__ scales, const uint8_t *__restrict__ zeros, h16 *__restrict__ y, int epi)
{
    constexpr int NQ = 4 / GS;            // groups per chunk
    constexpr int XSTAGE = XB * 1024;     // one chunk of x: 4 XB rows of 256 bytes, as 1 KB blocks of four rows
    // Row i of the matrix operand is row i / RS of x: a lane's accumulator registers 4 lk + r then repeat, and
    // RR of the four are distinct.
    constexpr int RR = XB == 1 ? 1 : (XB == 2 ? 2 : 4), RS = 4 / RR;
    static_assert(TB == 1 || TB == 2 || TB == 4, "columns per lane");
    static_assert(MT == 1 ? XB <= 4 : XB > 4 && XB <= 8, "row tiles");
    static_assert(!CPG || GS == 4, "several chunks per group");
    constexpr int RING = WV * 2 * XSTAGE, EXCH = WV * MT * RR * TB * 256;  // the exchange of sums at the end reuses the rings
    __shared__ __attribute__((aligned(1024))) unsigned char xring[RING > EXCH ? RING : EXCH];
    static_assert(sizeof(xring) <= 160 * 1024, "LDS of a workgroup");

    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lc = lane & 15, lk = lane >> 4;
    // Workgroups go to the eight XCDs in turn.  grouped: four adjacent slices run on one XCD, so that the
    // 128-byte lines of weights, steps and zero points they share come through one L2 once.
    int slice = blockIdx.x;
    if (grouped && slice < ((int)gridDim.x & ~31)) slice = (slice & ~31) + (slice & 7) * 4 + ((slice >> 3) & 3);
    const int n0 = slice * (16 * TB);
    const int chunks = (K + 127) / 128;
    const int tail_ks = GS < 4 ? (K - (chunks - 1) * 128) / 32 : 4;  // k-steps of the last chunk
    // lanes past the last column read column 0 instead; their results are never stored
    const int nout = n0 + TB * lc;
    const int ncol = nout < N ? nout : 0;
    // this wave's chunks: wv, wv + WV, ...  (none when the layer has fewer chunks than waves)
    const int nmine = wv < chunks ? (chunks - wv + WV - 1) / WV : 0;
    const int c0 = wv < chunks ? wv : 0;
    const bool my_tail = GS < 4 && tail_ks < 4 && c0 + (nmine - 1) * WV == chunks - 1;  // this wave's last chunk is a short one

    float acc[MT][TB][RR];
#pragma unroll
    for (int mt = 0; mt < MT; mt++)
#pragma unroll
        for (int b = 0; b < TB; b++)
#pragma unroll
            for (int r = 0; r < RR; r++) acc[mt][b][r] = 0.f;

    typedef typename std::conditional<TB == 1, uint32_t, uint32_t __attribute__((ext_vector_type(TB == 1 ? 2 : TB)))>::type wvec;  // the packed words of the lane's columns
    typedef typename std::conditional<TB == 4, u32x2, uint32_t>::type svec;                                                       // their fp16 steps
    struct Stage {
        wvec w[4];       // per k-step
        svec sc[NQ];     // per group
        uint32_t zr[NQ];  // zero points, one byte each
    };

    // Addresses: a wave-uniform byte pointer per stream (stepped on the scalar unit) plus a
    // per-lane 32-bit offset that never changes.
    const uint32_t voff_w = (uint32_t)(lk * N + ncol) * 4u;
    const uint32_t voff_s = (uint32_t)ncol * 2u, voff_z = (uint32_t)ncol;
    const long wstep1 = (long)N * 16;  // one k-step: four packed rows, in bytes
    const long dw = (long)WV * 4 * wstep1;
    const int drem = CPG ? WV % cpg : 0;
    const long drow = CPG ? WV / cpg : WV * NQ;
    const long row0 = CPG ? c0 / cpg : (long)c0 * NQ;
    int rem = CPG ? c0 % cpg : 0, cis = c0;  // position of the chunk being issued in its group; that chunk
    const unsigned char *wq = reinterpret_cast<const unsigned char *>(packed) + (long)c0 * 4 * wstep1;
    const unsigned char *sq = reinterpret_cast<const unsigned char *>(scales) + row0 * N * 2, *zq = zeros + row0 * N;
    const unsigned char *xq = reinterpret_cast<const unsigned char *>(x) + (long)c0 * 256;

    // Activations of a chunk: XB direct global->LDS loads of 1 KB (four rows of 256 bytes
    // each).  Lane i of a block handles row i / 16 of the block and fetches piece
    // (i % 16) ^ (row % 16) of that row, so that a row's pieces (whole 128-byte lines) come from
    // adjacent lanes, while in LDS (where the hardware puts lane i at byte 16 i of the block)
    // the pieces the 16 rows need for one k-step fall into 16 different bank groups.  Rows past
    // M re-read row M - 1.
    unsigned char *const ring = xring + wv * (2 * XSTAGE);
    uint32_t xoff[XB];
#pragma unroll
    for (int j = 0; j < XB; j++) {
        const int row = j * 4 + (lane >> 4);
        const int rowc = row < M ? row : M - 1;
        xoff[j] = (uint32_t)rowc * (uint32_t)K * 2u + (uint32_t)(((lane ^ row) & 15) * 16);
    }

    // Loads of one chunk, the weight side in assembly so that this kernel decides when to wait for them (a stage
    // must not be read before `landed`) and with the non-temporal hint (every weight byte
    // is read once per launch).  A short last chunk (K not a multiple of 128) reads its last k-step and
    // group again in the place of those past K, and the first piece of each row of x; compute clears
    // those fragments of x.
    auto issue = [&](Stage &s, int slot) {
        const bool tail = GS < 4 && tail_ks < 4 && cis == chunks - 1;  // wave-uniform
#pragma unroll
        for (int j = 0; j < XB; j++) {
            uint32_t xo = xoff[j];
            if constexpr (GS < 4)
                if (tail) {
                    const int piece = (lane ^ (j * 4 + (lane >> 4))) & 15;
                    if (piece >= tail_ks * 4) xo -= (uint32_t)(piece * 16);
                }
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(xq + xo),
                                             (__attribute__((address_space(3))) void *)(ring + slot * XSTAGE + j * 1024), 16, 0, 0);
        }
        const unsigned char *b0 = wq, *b1 = b0 + wstep1, *b2 = b1 + wstep1, *b3 = b2 + wstep1;
        if (GS < 4 && tail) {
            b1 = tail_ks > 1 ? b1 : b0;
            b2 = tail_ks > 2 ? b2 : b1;
            b3 = b2;
        }
#define SQP_SLICE_WORDS(OP)                                                                                                  \
    asm volatile(OP " %0, %4, %5 nt\n\t" OP " %1, %4, %6 nt\n\t" OP " %2, %4, %7 nt\n\t" OP " %3, %4, %8 nt"                 \
                 : "=&v"(s.w[0]), "=&v"(s.w[1]), "=&v"(s.w[2]), "=&v"(s.w[3])                                               \
                 : "v"(voff_w), "s"(b0), "s"(b1), "s"(b2), "s"(b3)                                                          \
                 : "memory")
        if constexpr (TB == 1) SQP_SLICE_WORDS("global_load_dword");
        else if constexpr (TB == 2) SQP_SLICE_WORDS("global_load_dwordx2");
        else SQP_SLICE_WORDS("global_load_dwordx4");
#undef SQP_SLICE_WORDS
        const unsigned char *sb = sq, *zb = zq;
#pragma unroll
        for (int q = 0; q < NQ; q++) {
#define SQP_SLICE_PARAMS(OS, OZ)                                                           \
    asm volatile(OS " %0, %2, %4 nt\n\t" OZ " %1, %3, %5 nt"                               \
                 : "=&v"(s.sc[q]), "=&v"(s.zr[q])                                          \
                 : "v"(voff_s), "v"(voff_z), "s"(sb), "s"(zb)                              \
                 : "memory")
            if constexpr (TB == 1) SQP_SLICE_PARAMS("global_load_ushort", "global_load_ubyte");
            else if constexpr (TB == 2) SQP_SLICE_PARAMS("global_load_dword", "global_load_ushort");
            else SQP_SLICE_PARAMS("global_load_dwordx2", "global_load_dword");
#undef SQP_SLICE_PARAMS
            const bool more = !tail || (q + 1) * GS < tail_ks;
            sb += more ? (long)N * 2 : 0;
            zb += more ? (long)N : 0;
        }
        wq += dw;
        xq += WV * 256;
        sq += drow * N * 2;
        zq += drow * N;
        if constexpr (GS < 4) cis += WV;
        if constexpr (CPG) {
            rem += drem;
            const bool wrap = rem >= cpg;
            rem -= wrap ? cpg : 0;
            sq += wrap ? (long)N * 2 : 0;
            zq += wrap ? (long)N : 0;
        }
    };
    auto landed = [&](Stage &s) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // one chunk is in flight at a time
#pragma unroll
        for (int ks = 0; ks < 4; ks++) asm volatile("" : "+v"(s.w[ks]));
#pragma unroll
        for (int q = 0; q < NQ; q++) {
            asm volatile("" : "+v"(s.sc[q]));
            asm volatile("" : "+v"(s.zr[q]));
        }
    };

    // LDS byte addresses of this lane's A fragments (row lc of the operand) in slot 0, per k-step and row tile
    // (operand rows past the fetched ones repeat fetched rows: defined data, unused results)
    uint32_t xrd[4][MT];
#pragma unroll
    for (int mt = 0; mt < MT; mt++) {
        int row = mt * 16 + lc / RS;
        if (row >= 4 * XB) row -= 4 * XB - 16 * mt;
        const uint32_t at = (uint32_t)(size_t)ring + (uint32_t)((row >> 2) * 1024 + (row & 3) * 256);
#pragma unroll
        for (int ks = 0; ks < 4; ks++) xrd[ks][mt] = at + (uint32_t)((((ks * 4 + lk) ^ row) & 15) * 16);
    }
    auto word_of = [](const Stage &s, int ks, int b) -> uint32_t {
        if constexpr (TB == 1) return s.w[ks];
        else return s.w[ks][b];
    };
    auto zero_of = [](const Stage &s, int q, int b) -> uint32_t { return (s.zr[q] >> (8 * b)) & 0xffu; };
    auto step_of = [](const Stage &s, int q, int b) -> float {
        uint32_t pair;
        if constexpr (TB == 4) pair = s.sc[q][b >> 1];
        else pair = s.sc[q];
        const h16x2 v = __builtin_bit_cast(h16x2, pair);
        return (float)((b & 1) ? v.y : v.x);
    };

    auto compute = [&](Stage &s, auto SLOT, bool tail) {
        constexpr int slot = decltype(SLOT)::value;
        // The A fragments are read with instructions written in assembly: the compiler cannot
        // tell which ring slot a direct load filled and would wait for every outstanding load.
        u32x4 xa[4][MT];
#pragma unroll
        for (int ks = 0; ks < 4; ks++)
#pragma unroll
            for (int mt = 0; mt < MT; mt++)
                asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(xa[ks][mt]) : "v"(xrd[ks][mt]), "n"(slot * XSTAGE) : "memory");
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int ks = 0; ks < 4; ks++)
#pragma unroll
            for (int mt = 0; mt < MT; mt++) asm volatile("" : "+v"(xa[ks][mt]));  // no use ahead of the wait
        // A short last chunk: no activations past K, and no step of a group past it (the last group's, read again, may be
        // infinite, and infinity times a sum of 0 is NaN).  Branches: the asm statements keep the compiler
        // from selects, which every chunk would pay for (32 of 220 vector instructions in groups of 64).
        if constexpr (GS < 4)
            if (tail) {
#pragma unroll
                for (int ks = 1; ks < 4; ks++)
                    if (ks >= tail_ks) {
#pragma unroll
                        for (int mt = 0; mt < MT; mt++) {
                            xa[ks][mt] = u32x4{0, 0, 0, 0};
                            asm volatile("" : "+v"(xa[ks][mt]));
                        }
                        if (ks % GS == 0) {
                            s.sc[ks / GS] = svec{};
                            asm volatile("" : "+v"(s.sc[ks / GS]));
                        }
                    }
            }
        // The accumulators are kept whole until a sum of theirs has been read (the asm statements behind the
        // FMAs): a register that nothing reads would otherwise be free for an instruction in assembly while
        // the MFMA still writes it, and the compiler adds no wait states for those.
        // AHEAD: a word is unpacked in front of the matrix instructions of the word before it (the scheduler is kept to
        // that): right behind its own unpack, an MFMA waits, and where a sum moved to other registers
        // with each MFMA, what followed waited for the old ones (5 wait states per word, a third of the loop's time).
        // Not in groups of 32, whose sums are scaled after every k-step, nor with two row tiles, where every word feeds two
        // MFMAs anyway.  us, compiler's order / ahead: groups of 32 at one to four rows on 16385 to 32768 columns, where
        // some compute units hold two workgroups, 1216->24576 6.1 / 7.5, 3008->17464 12.2 / 12.5; 17 to 32 rows 4096->8192 in
        // groups of 64 7.51 / 7.67, 1536->38152 in groups of 256 18.5 / 19.1, 700 calls 0.6 % in the mean.
        constexpr bool AHEAD = MT == 1 && GS > 1;
        const UnpackConsts uc = unpack_consts();  // (here: held across the loop they cost the last of these shapes 3 %)
        const f32x4 none = {0.f, 0.f, 0.f, 0.f};
        auto unpacked = [&](int i) {
            const int ks = i / TB, b = i % TB;
            const uint32_t z = zero_of(s, ks / GS, b);
            return dequant_word(word_of(s, ks, b), neg_hi_of(z), neg_lo_of(z), uc);
        };
        h16x8 next;
        if constexpr (AHEAD) next = unpacked(0);
#pragma unroll
        for (int q = 0; q < NQ; q++) {
            f32x4 g[MT][TB];
#pragma unroll
            for (int ks = q * GS; ks < q * GS + GS; ks++) {
                h16x8 a[MT];
#pragma unroll
                for (int mt = 0; mt < MT; mt++) a[mt] = permute_x(xa[ks][mt]);
#pragma unroll
                for (int b = 0; b < TB; b++) {
                    const int i = ks * TB + b;
                    const h16x8 w = AHEAD ? next : unpacked(i);
                    if constexpr (AHEAD) {
                        if (i + 1 < 4 * TB) next = unpacked(i + 1);
                        __builtin_amdgcn_sched_barrier(0);
                    }
#pragma unroll
                    for (int mt = 0; mt < MT; mt++) g[mt][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[mt], w, ks == q * GS ? none : g[mt][b], 0, 0, 0);
                    if constexpr (AHEAD) __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int b = 0; b < TB; b++) {
                const float d = step_of(s, q, b);
#pragma unroll
                for (int mt = 0; mt < MT; mt++) {
#pragma unroll
                    for (int r = 0; r < RR; r++) acc[mt][b][r] = fmaf(d, g[mt][b][r * RS], acc[mt][b][r]);
                    asm volatile("" : "+v"(acc[mt][b][0]) : "v"(g[mt][b]));
                }
            }
        }
    };

    // Software pipeline over the wave's own chunks: the next one is in flight while one is consumed.
    // Slot and stage of chunk i + 1 were consumed in iteration i - 1 by this same wave (its LDS
    // reads have been waited for), so no barrier is needed.  Nothing is issued past the last chunk
    // (wave-uniform branches): look-ahead loads that fetched its activations again cost the wait for
    // them at the end (1 to 4 % per launch).
    constexpr std::integral_constant<int, 0> S0 = {};
    constexpr std::integral_constant<int, 1> S1 = {};
    Stage st[2];
    if (nmine > 0) issue(st[0], 0);
    for (int i = 0; i < nmine; i += 2) {
        landed(st[0]);
        if (i + 1 < nmine) issue(st[1], 1);
        compute(st[0], S0, my_tail && i == nmine - 1);
        if (i + 1 < nmine) {
            landed(st[1]);
            if (i + 2 < nmine) issue(st[0], 0);
            compute(st[1], S1, my_tail && i + 1 == nmine - 1);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (nothing is in flight here: for the reader of the assembly)

    // ---- the waves add their sums through LDS (the rings are idle once every wave is here), in
    // wave order: wave v < MT RR adds and stores register v % RR of row tile v / RR, i.e. the rows
    // 16 mt + RR lk + r.  [wave][mt][r][lane] of TB floats.
    __syncthreads();
    typedef float fvec __attribute__((ext_vector_type(TB == 1 ? 2 : TB)));
    typedef typename std::conditional<TB == 1, float, fvec>::type sums;
    sums *ex = reinterpret_cast<sums *>(xring);
#pragma unroll
    for (int mt = 0; mt < MT; mt++)
#pragma unroll
        for (int r = 0; r < RR; r++) {
            sums v;
            if constexpr (TB == 1) v = acc[mt][0][r];
            else {
#pragma unroll
                for (int b = 0; b < TB; b++) v[b] = acc[mt][b][r];
            }
            ex[((wv * MT + mt) * RR + r) * 64 + lane] = v;
        }
    __syncthreads();
    if (nout >= N) return;
    for (int part = wv; part < MT * RR; part += WV) {
        const int m = (part / RR) * 16 + RR * lk + part % RR;
        if (m >= M) continue;
        sums sum = ex[part * 64 + lane];
#pragma unroll
        for (int w = 1; w < WV; w++) sum += ex[(w * MT * RR + part) * 64 + lane];
        // epi == 0: the fp16 values themselves, y [M][N].  epi == 1: the lane's columns are
        // (gate, up) pairs of a merged, interleaved gate/up projection and the output is
        // SiLU(gate) * up, y [M][N/2] (the LlamaMLP activation of Fig. 5, from the fp32 sums).
        if constexpr (TB == 1) {
            y[(size_t)m * N + nout] = (h16)sum;
        } else if (epi == 0) {
            typedef h16 hvec __attribute__((ext_vector_type(TB)));
            hvec o;
#pragma unroll
            for (int b = 0; b < TB; b++) o[b] = (h16)sum[b];
            *reinterpret_cast<hvec *>(y + (size_t)m * N + nout) = o;
        } else {
            h16 *out = y + (size_t)m * (N >> 1) + (nout >> 1);
            if constexpr (TB == 2) {
                out[0] = (h16)(sqp_silu(sum[0]) * sum[1]);
            } else {
                h16x2 o;
                o.x = (h16)(sqp_silu(sum[0]) * sum[1]);
                o.y = (h16)(sqp_silu(sum[2]) * sum[3]);
                *reinterpret_cast<h16x2 *>(out) = o;
            }
        }
    }
}

template <int MT, int TB, int WV, int XB, int GS, bool CPG>
int launch_slices(bool grouped, int M, int N, int K, int cpg, const h16 *x, const uint32_t *packed, const h16 *scales, const uint8_t *zeros, h16 *y,
                  int epi, hipStream_t st)
{
    w4a16_decode_slice_kernel<MT, TB, WV, XB, GS, CPG>
        <<<(N + 16 * TB - 1) / (16 * TB), WV * 64, 0, st>>>(M, N, K, cpg, grouped, x, packed, scales, zeros, y, epi);
    return sqp_launch_status();
}

// Up to 16 rows, by the blocks of four rows that hold real rows.
template <int TB, int WV, int GS, bool CPG>
int slices_rows16(bool grouped, int M, int N, int K, int cpg, const h16 *x, const uint32_t *packed, const h16 *scales, const uint8_t *zeros, h16 *y,
                  int epi, hipStream_t st)
{
    if (M <= 4) return launch_slices<1, TB, WV, 1, GS, CPG>(grouped, M, N, K, cpg, x, packed, scales, zeros, y, epi, st);
    if (M <= 8) return launch_slices<1, TB, WV, 2, GS, CPG>(grouped, M, N, K, cpg, x, packed, scales, zeros, y, epi, st);
    if (M <= 12) return launch_slices<1, TB, WV, 3, GS, CPG>(grouped, M, N, K, cpg, x, packed, scales, zeros, y, epi, st);
    return launch_slices<1, TB, WV, 4, GS, CPG>(grouped, M, N, K, cpg, x, packed, scales, zeros, y, epi, st);
}

template <int GS, bool CPG>
int dispatch_slices(const SqpSlicePlan &p, int M, int N, int K, int cpg, const h16 *x, const uint32_t *packed, const h16 *scales,
                    const uint8_t *zeros, h16 *y, int epi, hipStream_t st)
{
    const bool g = p.grouped;
    if (M > 16) {
        if (p.tb == 1) return launch_slices<2, 1, 8, 8, GS, CPG>(g, M, N, K, cpg, x, packed, scales, zeros, y, epi, st);
        if (p.tb == 2) return launch_slices<2, 2, 8, 8, GS, CPG>(g, M, N, K, cpg, x, packed, scales, zeros, y, epi, st);
        return launch_slices<2, 4, 8, 8, GS, CPG>(g, M, N, K, cpg, x, packed, scales, zeros, y, epi, st);
    }
    // 16 waves exist for up to four rows, four for up to eight in groups of 64 and more: eight otherwise
    if constexpr (GS > 1)
        if (p.tb == 4 && p.wv == 4 && M <= 8) {
            if (M <= 4) return launch_slices<1, 4, 4, 1, GS, CPG>(g, M, N, K, cpg, x, packed, scales, zeros, y, epi, st);
            return launch_slices<1, 4, 4, 2, GS, CPG>(g, M, N, K, cpg, x, packed, scales, zeros, y, epi, st);
        }
    if (p.wv == 16 && M <= 4 && p.tb == 1) return launch_slices<1, 1, 16, 1, GS, CPG>(g, M, N, K, cpg, x, packed, scales, zeros, y, epi, st);
    if (p.wv == 16 && M <= 4 && p.tb == 2) return launch_slices<1, 2, 16, 1, GS, CPG>(g, M, N, K, cpg, x, packed, scales, zeros, y, epi, st);
    if (p.tb == 1) return slices_rows16<1, 8, GS, CPG>(g, M, N, K, cpg, x, packed, scales, zeros, y, epi, st);
    if (p.tb == 2) return slices_rows16<2, 8, GS, CPG>(g, M, N, K, cpg, x, packed, scales, zeros, y, epi, st);
    return slices_rows16<4, 8, GS, CPG>(g, M, N, K, cpg, x, packed, scales, zeros, y, epi, st);
}

}  // namespace
