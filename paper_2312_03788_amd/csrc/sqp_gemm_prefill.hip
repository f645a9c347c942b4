// Tiled matrix-core W4A16 GEMM for large M (prefill): y = x * w_hat, Eq. 3 of
// arXiv 2312.03788 with w_hat = fp16((code - Z) * Delta) of Eq. 1, group-wise along K.
//
// A workgroup of 4 waves (one per SIMD, the whole register file each) computes a 128 x 512
// tile of y, the waves side by side on the same 128 rows (or a 256 x 256 tile, waves 2 x 2);
// a wave owns 128 rows x 128 columns as 4 x 4 accumulator tiles of v_mfma_f32_32x32x16_f16
// (256 fp32 registers per lane).
//   - Weights never pass through LDS: one dwordx4 load per lane fetches, for k-block
//     (lane / 32), the packed words of 4 adjacent columns; a word is 8 consecutive k of one
//     column, i.e. one lane's B operand of the 32x32x16 MFMA (column = lane % 32).  The word
//     is unpacked in registers to the fp16 dequantised weights (16 VALU ops, in the order of k) and each B
//     operand feeds 4 MFMAs (the 4 row tiles); each activation fragment feeds 4 as well, as it comes from
//     LDS (4 VALU ops per MFMA).
//   - Activations are the shared operand: a 128 x 64 (256 x 64) slice of x per stage is copied
//     once per workgroup straight into a four-slot LDS ring (direct global->LDS loads of whole
//     128-byte lines, pieces XOR-swizzled so that the 16-byte reads of one k-step spread over
//     all banks) and every wave reads its A operands from there.
//   - With a single wave per SIMD the order of issue is the schedule, so the MFMAs and the
//     vector instructions of a k-step are written out in issue order (see the stream below):
//     while the 16 MFMAs of one k-step run, the activation fragments of the next arrive from
//     LDS and the next weight words are unpacked; the hand-over to the next stage (wait for
//     its loads, barrier) sits inside the last k-step, so the pipeline never drains.
//   - Loads, waits and the per-stage barrier are explicit (assembly), as in the decode
//     kernel: two stages stay in flight while one is consumed, issued between its MFMAs.
// What bounds it: the matrix cores; below a full chip with the unpack's issue slots on top (1024 x 8192 x 8192, 128 tiles: 115
// us, 100 without the unpack, which is about what the MFMAs alone take), on a full one under the power limit.  us per call (M x K x N): tiles numbered
// along a row of the output over all XCDs -> one compact run of tiles per XCD -> with the unpack in the order of k, no
// padded stages (the loop of three used to round a K part of 16 up to 18) and an epilogue that reads one row tile at a
// time (it used to spill, and every reload waited for the stores under way) -> with half the scalar instructions
// per stage and every LDS read and load between two MFMAs instead of in clusters in front of a k-step:
// 512 x 4096 x 22016 111 -> 109 -> 95 -> 88, 1000 x 4096 x 12288 108 -> 107 -> 95 -> 91, 4096 x 4096 x 4096 128 -> 126 ->
// 113 -> 109, 2048 x 8192 x 10240 318 -> 318 -> 296 -> 279, 2048 x 8192 x 44032 1330 -> 1300 -> 1210 -> 1145 (1.29 PFLOP/s).
// Eight waves of 128 x 64 (two per SIMD) needed fewer cycles per MFMA, but the chip then
// clocked lower under its power limit and the result was a little slower, so one wave per SIMD
// it is.
#include <type_traits>

#include "sqp_common.h"
#include "sqp_strip.h"
#include "sqp_w4_unpack.h"

namespace {

constexpr int BK = 64;

// Which tile a workgroup takes.  The tiles are numbered in groups of up to gm rows of tiles, row index fastest
// within a column, so that consecutive numbers are compact blocks; workgroups are dealt to the eight XCDs in turn, so
// each XCD gets one run of consecutive numbers.  The workgroups that an XCD has resident then share its L2: of a stage's 16 KB of activations and 16 KB of weights per 128 x 512 tile
// it fetches 12 blocks for 32 tiles (8 rows x 4 columns) instead of about 35 with column-major numbers over all XCDs.
// Launches in K parts keep the tiles dealt over all XCDs, a part behind the other: with runs they are up to 3 us slower
// (328x6208x1168 19.2 -> 21.9 with the tiles of a part together, 18.4 with the parts of a tile; 196x3136x3320 21.3 ->
// 22.7, 22.4) and nothing faster (160x8192x8192 33.0 -> 32.9, 33.1).
struct TileMap {
    int tile0;   // number of the launch's first tile
    int tn, tm;  // columns and rows of tiles
    int gm;      // rows per group
    int halves;  // 1: the launch's tiles are the left and right halves of the numbered ones (tile0 counts halves)
};
constexpr int XCDS = 8;

// Workgroup w of `total`: its place when every XCD has one run.
__device__ __forceinline__ uint32_t xcd_run(uint32_t w, uint32_t total)
{
    const uint32_t xcd = w % XCDS, len = total / XCDS, more = total % XCDS;
    return xcd * len + (xcd < more ? xcd : more) + w / XCDS;
}

__device__ __forceinline__ void tile_at(const TileMap &m, uint32_t i, int &row, int &col)
{
    const uint32_t n = (m.tile0 + i) >> m.halves;
    const uint32_t g = n / (uint32_t)(m.gm * m.tn), in = n - g * (uint32_t)(m.gm * m.tn);
    const uint32_t left = m.tm - g * m.gm, rows = left < (uint32_t)m.gm ? left : m.gm;
    const uint32_t c = in / rows;
    row = (int)(g * m.gm + in - c * rows);
    col = (int)(m.halves ? 2 * c + ((m.tile0 + i) & 1) : c);
}

// Final store of 8 adjacent columns of row m: the fp16 values themselves, y [M][N], or with epi the (gate, up) pairs'
// SiLU(gate) * up, y [M][N/2].
__device__ __forceinline__ void store_octet(h16 *y, int m, int N, int n, int epi, const f32x4 &a, const f32x4 &b)
{
    if (epi != 0) {
        h16x4 o;
        o.x = (h16)(sqp_silu(a.x) * a.y); o.y = (h16)(sqp_silu(a.z) * a.w);
        o.z = (h16)(sqp_silu(b.x) * b.y); o.w = (h16)(sqp_silu(b.z) * b.w);
        *reinterpret_cast<h16x4 *>(y + (size_t)m * (N >> 1) + (n >> 1)) = o;
        return;
    }
    h16x8 o;
    o.s0 = (h16)a.x; o.s1 = (h16)a.y; o.s2 = (h16)a.z; o.s3 = (h16)a.w;
    o.s4 = (h16)b.x; o.s5 = (h16)b.y; o.s6 = (h16)b.z; o.s7 = (h16)b.w;
    *reinterpret_cast<h16x8 *>(y + (size_t)m * N + n) = o;
}

// RT, NT: 32-row and 32-column MFMA tiles per wave; WM: waves along the rows, the other 4 / WM along
// the columns.  A workgroup owns 32 RT WM rows x 32 NT (4 / WM) columns:
//   <4, 4, 1>: 128 x 512, the four waves side by side on the same 128 rows.  Every packed word
//           is then loaded and unpacked by exactly one wave, and a workgroup stages half as
//           many activation bytes per matrix instruction as with the square tile.
//   <4, 4, 2>: 256 x 256, waves 2 x 2 (the two waves of a column pair unpack the same words).
//   <4, 2, *>: the same with half the columns (128 x 256 / 256 x 128), used for the tiles left over
//           after the last full round so that the tail of a launch costs half a round, and for
//           the K-split launches.
//   <4, 3, 1>, <5, 3, 1>: 128 or 160 x 384 (quicker_launch).
//   <3, 2, 1>, <5, 2, 1>, <6, 2, 1>: 96, 160 or 192 rows x 256 columns, K-split launches of row
//           counts that would leave much of a 128-row tile empty.
// KH = 2: the waves of a column pair halve K between them, stage by stage (a stage is 128 k then), and add their sums
// through LDS at the end: tiles of half the columns in half as many K parts (see plan_launches).
// G32: quantisation groups of 32 rows, i.e. two groups per 64-row stage (the steps and zero
// points of both are loaded per stage and the unpack switches sets after the second k-step);
// otherwise the group is a multiple of 64 rows.
template <int RT, int NT, int WM, int KH, bool G32>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(KH == 1 && NT == 2 && RT <= 4 && WM == 1 ? 2 : 1)))
w4a16_prefill_kernel(int M, int N, int K, int group, TileMap map, const h16 *__restrict__ x,
                     const uint32_t *__restrict__ packed, const h16 *__restrict__ scales,
                     const uint8_t *__restrict__ zeros, h16 *__restrict__ y, float *__restrict__ part, int epi)
{
    constexpr int W = 4;                   // waves: one per SIMD
    constexpr int WNW = W / WM / KH;       // waves along the columns
    constexpr int BM = 32 * RT * WM;       // rows per workgroup
    constexpr int WN = 32 * NT;            // columns per wave
    static_assert(NT >= 2 && NT <= 4, "a lane's columns are one load");
    static_assert(NT != 3 || (WM == 1 && KH == 1 && !G32), "three columns per lane");
    static_assert(KH == 1 || (WM == 1 && !G32), "waves that halve K");
    typedef uint32_t wvec __attribute__((ext_vector_type(NT)));
    typedef std::conditional_t<NT == 4, u32x2, uint32_t> scvec;
    constexpr int PL = NT == 3 ? 3 : 1;    // loads that a lane's steps take, and its zero points
    constexpr int D = 3;                   // register stages of packed weights (two in flight)
    constexpr int XD = KH == 1 ? 4 : 3;    // LDS slots of activations
    constexpr int XHALF = BM * BK * 2;     // 64 k of activations: blocks of 8 rows x 128 bytes
    constexpr int XSTAGE = KH * XHALF;
    constexpr int OX = KH * (BM / 8) / W;  // direct loads per wave per stage (one per 1 KB block), spread over its four k-steps
    constexpr int WGN = WNW * WN;          // columns per workgroup
    constexpr int NQ = G32 ? 2 : 1;        // quantisation groups per stage
    constexpr int OW = 4 + 2 * NQ * PL;
    static_assert(2 * (OX + OW) < 64, "vmcnt field");
    __shared__ __attribute__((aligned(1024))) unsigned char xring[XD * XSTAGE];
    static_assert(sizeof(xring) <= 160 * 1024, "LDS of a workgroup");

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = KH == 1 ? wave / WNW : 0, wn = wave % WNW, kh = KH == 1 ? 0 : wave / WNW;
    const int l32 = lane & 31, kb = lane >> 5;
    // K split across gridDim.y workgroups (part != nullptr): this one takes stages
    // [stage0, stage0 + stages) and leaves its fp32 sums in part[blockIdx.y][blockIdx.x][BM][WGN].
    int trow, tcol;
    tile_at(map, gridDim.y == 1 ? xcd_run(blockIdx.x, gridDim.x) : blockIdx.x, trow, tcol);
    const int nbase = tcol * WGN;
    const int m0 = trow * BM;
    const int n0 = nbase + wn * WN;
    const int stages_all = K / (BK * KH);
    const int stage0 = (int)((uint32_t)stages_all * blockIdx.y / gridDim.y);
    const int stages = (int)((uint32_t)stages_all * (blockIdx.y + 1) / gridDim.y) - stage0;
    const int spg = G32 ? 1 : group / BK;  // stages per quantisation group (G32: two groups per stage)

    int ncol = n0 + NT * l32;
    if (NT == 3 && ncol + 2 >= N && ncol < N) ncol = N - 3;  // (the columns of the lane before again: none past the row is read)
    if (ncol >= N) ncol = 0;

    f32x16 acc[RT][NT];
#pragma unroll
    for (int mt = 0; mt < RT; mt++)
#pragma unroll
        for (int t = 0; t < NT; t++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc[mt][t][r] = 0.f;

    struct Stage {
        wvec w[4];    // per k-step: packed words of the lane's NT columns
        scvec sc[NQ * PL];     // NT fp16 steps (per group of the stage; three columns: one each, no load is aligned to them)
        uint32_t zr[NQ * PL];  // NT zero points, one byte each
    };

    // The loading side walks the stages with one 32-bit scalar offset per stream (buffer loads; a row's place is in the
    // lanes' offsets); past the last stage the offsets stop, so that the look-ahead of the branch-free stages re-reads
    // the last one (cache hits).  Every scalar instruction costs the wave as much as a vector one: 30 per stage, where
    // 64-bit pointers with a clamp each took 56.
    const rsrc_t w_buf = buffer_of(packed, (uint32_t)(K / 8) * (uint32_t)N * 4u);
    const rsrc_t s_buf = buffer_of(scales, (uint32_t)(K / group) * (uint32_t)N * 2u), z_buf = buffer_of(zeros, (uint32_t)(K / group) * (uint32_t)N);
    const uint32_t wstage = (uint32_t)N * 32u;    // eight packed rows (64 k) in bytes
    const int first = stage0 * KH + kh;           // this wave's first 64 k
    uint32_t w_at = (uint32_t)first * wstage;
    const uint32_t w_most = w_at + (uint32_t)(stages - 1) * (KH * wstage);
    const int prow_step = KH / spg, kin_step = KH % spg;  // groups and part of one that a stage advances by
    int kin = first % spg;                        // position of the stage being issued inside its group
    uint32_t z_at = (uint32_t)(first / spg) * (uint32_t)(N * NQ);  // zero points of its group; the steps are at twice that
    const uint32_t z_most = (uint32_t)((first + (stages - 1) * KH) / spg) * (uint32_t)(N * NQ);
    const uint32_t z_inc = (uint32_t)prow_step * (uint32_t)(N * NQ), z_wrap = z_inc + (uint32_t)(N * NQ);
    uint32_t x_at = (uint32_t)stage0 * (KH * BK * 2);
    const uint32_t x_most = x_at + (uint32_t)(stages - 1) * (KH * BK * 2), x_bytes = (uint32_t)M * (uint32_t)K * 2u;
    uint32_t voff_w[4], voff_s[NQ * PL], voff_z[NQ * PL];
#pragma unroll
    for (int ks = 0; ks < 4; ks++) voff_w[ks] = (uint32_t)((kb + 2 * ks) * N + ncol) * 4u;
#pragma unroll
    for (int g = 0; g < NQ * PL; g++) {
        voff_z[g] = NT == 3 ? (uint32_t)(ncol + g) : (uint32_t)(g * N + ncol);
        voff_s[g] = voff_z[g] * 2u;
    }
    // load j of the OW on the weight side of a stage
    auto issue_w = [&](Stage &s, int j) {
        if (j < 4) {
            if constexpr (NT == 4)
                asm volatile("buffer_load_dwordx4 %0, %1, %2, %3 offen" : "=v"(s.w[j]) : "v"(voff_w[j]), "s"(w_buf), "s"(w_at) : "memory");
            else if constexpr (NT == 3)
                asm volatile("buffer_load_dwordx3 %0, %1, %2, %3 offen" : "=v"(s.w[j]) : "v"(voff_w[j]), "s"(w_buf), "s"(w_at) : "memory");
            else
                asm volatile("buffer_load_dwordx2 %0, %1, %2, %3 offen" : "=v"(s.w[j]) : "v"(voff_w[j]), "s"(w_buf), "s"(w_at) : "memory");
        } else if ((j & 1) == 0) {
            const int g = (j - 4) >> 1;
            if constexpr (NT == 3)
                asm volatile("buffer_load_ushort %0, %1, %2, %3 offen" : "=v"(s.sc[g]) : "v"(voff_s[g]), "s"(s_buf), "s"(z_at * 2u) : "memory");
            else if constexpr (NT == 4)
                asm volatile("buffer_load_dwordx2 %0, %1, %2, %3 offen" : "=v"(s.sc[g]) : "v"(voff_s[g]), "s"(s_buf), "s"(z_at * 2u) : "memory");
            else
                asm volatile("buffer_load_dword %0, %1, %2, %3 offen" : "=v"(s.sc[g]) : "v"(voff_s[g]), "s"(s_buf), "s"(z_at * 2u) : "memory");
        } else {
            const int g = (j - 4) >> 1;
            if constexpr (NT == 3)
                asm volatile("buffer_load_ubyte %0, %1, %2, %3 offen" : "=v"(s.zr[g]) : "v"(voff_z[g]), "s"(z_buf), "s"(z_at) : "memory");
            else if constexpr (NT == 4)
                asm volatile("buffer_load_dword %0, %1, %2, %3 offen" : "=v"(s.zr[g]) : "v"(voff_z[g]), "s"(z_buf), "s"(z_at) : "memory");
            else
                asm volatile("buffer_load_ushort %0, %1, %2, %3 offen" : "=v"(s.zr[g]) : "v"(voff_z[g]), "s"(z_buf), "s"(z_at) : "memory");
        }
    };
    auto landed = [&](Stage &s, auto after) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(decltype(after)::value) : "memory");
#pragma unroll
        for (int ks = 0; ks < 4; ks++) asm volatile("" : "+v"(s.w[ks]));
#pragma unroll
        for (int g = 0; g < NQ * PL; g++) {
            asm volatile("" : "+v"(s.sc[g]));
            asm volatile("" : "+v"(s.zr[g]));
        }
    };

    // Activations: wave w copies blocks w, w+4, ... of the stage (a block = 8 rows x 128 bytes).  Lane i of a block handles row i / 8 of the block and fetches piece
    // (i % 8) ^ key(row) of that row's 128 bytes, key(row) = (row / 2) % 8; the hardware puts
    // lane i at byte 16*i of the block.
    uint32_t xoff[OX];
#pragma unroll
    for (int j = 0; j < OX; j++) {
        const int b = (wave + W * j) % (BM / 8);  // (KH == 2: the blocks of the second 64 k follow those of the first)
        const int row = b * 8 + (lane >> 3);
        int grow = m0 + row;
        if (grow >= M) grow = M - 1;
        const int piece = (lane & 7) ^ ((row >> 1) & 7);
        xoff[j] = (uint32_t)grow * (uint32_t)K * 2u + (uint32_t)((wave + W * j) / (BM / 8) * (BK * 2) + piece * 16);
    }
    auto issue_x = [&](int slot, int j) {
        copy16_to_lds(x, x_bytes, xoff[j], x_at, xring + slot * XSTAGE + (wave + W * j) * 1024);
    };
    // all loads of the stage have been issued: step the offsets up to the last stage's
    auto advance = [&]() {
        w_at = min(w_at + KH * wstage, w_most);
        x_at = min(x_at + KH * BK * 2, x_most);
        kin += kin_step;
        const bool wrap = kin >= spg;
        kin -= wrap ? spg : 0;
        z_at = min(z_at + (wrap ? z_wrap : z_inc), z_most);
    };
    const uint32_t xrd0 = (uint32_t)(size_t)xring +
                          (uint32_t)(kh * XHALF + ((wm * 32 * RT + l32) >> 3) * 1024 + ((wm * 32 * RT + l32) & 7) * 128);
    const int xkey = (l32 >> 1) & 7;

    // fragment of row tile mt of a k-step
    auto read_a = [&](u32x4 (&xa)[RT], int slot, int ks, int mt) {
        const uint32_t poff = xrd0 + (uint32_t)(slot * XSTAGE) + (uint32_t)((((ks * 2 + kb) ^ xkey)) * 16);
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(xa[mt]) : "v"(poff), "n"(mt * 4096) : "memory");
    };
    auto wait_a = [&](u32x4 (&xa)[RT]) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int mt = 0; mt < RT; mt++) asm volatile("" : "+v"(xa[mt]));
    };

    // Per-stage constants of the unpack: (-(1024 + Z), -(64 + Z)) and the step in both halves of a register
    // (one set per quantisation group of the stage).  A stage past the end (calls of fewer stages than the loop's three)
    // gets a step of 0 and adds nothing.
    h16x2 neg[NQ][NT], delta[NQ][NT];
    auto stage_consts = [&](const Stage &s, bool live) {
        const uint32_t sel_even = live ? 0x01000100u : 0x0c0c0c0cu;  // byte selectors of v_perm_b32
        const uint32_t sel_odd = live ? 0x03020302u : 0x0c0c0c0cu;   // (0x0c selects a zero byte)
#pragma unroll
        for (int g = 0; g < NQ; g++)
#pragma unroll
            for (int t = 0; t < NT; t++) {
                const uint32_t z = NT == 3 ? s.zr[t] : (s.zr[g] >> (8 * t)) & 0xffu;
                neg[g][t] = neg_pair_of(z);
                uint32_t sw;
                if constexpr (NT == 4) sw = s.sc[g][t >> 1];
                else if constexpr (NT == 3) sw = s.sc[t];
                else sw = s.sc[g];
                delta[g][t] = __builtin_bit_cast(h16x2, __builtin_amdgcn_perm(sw, sw, NT != 3 && (t & 1) ? sel_odd : sel_even));
            }
    };

    // One continuous software pipeline over all k-steps.  While the 16 MFMAs of a k-step
    // issue, the A fragments of the next k-step come from LDS and the next weight word is
    // unpacked.  The hand-over to the next stage happens inside the last k-step of a stage
    // (wait for the next stage's loads, barrier, new constants), so the first LDS reads and
    // the first unpack of a stage are hidden like any other.  Ring discipline: at the barrier in
    // the last k-step of stage s-1 every wave has that stage's last fragments in registers, so its LDS
    // slot (three are enough; four where they fit anyway) and weight registers (three stages) may be refilled during
    // stage s with the loads of stage s+2.
    Stage stg[D];
    u32x4 xa[2][RT];         // A operands as they lie in memory: [k-step parity][row tile]
    uint32_t bq[2][NT][4];   // B operands (dequantised weights): [k-step parity][column tile]

    // ---- The instruction stream of one k-step, in issue order, written out by hand.
    // With one wave per SIMD the order of issue is the schedule: measured on this chip, an
    // independent vector instruction costs 4 cycles and up to 4 of them hide behind a
    // 32x32x16 MFMA, but one that depends on the instruction just before it costs about 8, and
    // the compiler's own order left many such pairs.  So every MFMA and every vector
    // instruction of the k-step is a volatile asm statement (these keep their order), grouped
    // so that a result is used no sooner than 4 instructions later: MFMA i (row tile i / NT, column tile
    // i % NT), then its share of the unpack of the next k-step's B operands.
    // The unpack takes each byte of a word to both halves of a register, under the high bytes of 1024.0 and 64.0, and
    // masks the other nibble of each half out: pairs in the order of k, as the activations have theirs, so that
    // those go to the matrix core as they come from LDS.  (One shift, four and-ors per word give pairs four apart: 3
    // instructions less per word, but 4 more per 32 x 16 activations in every wave, 17 to 19 per word and column tile
    // instead of 16 with 4 x 4 tiles and up to 25 with 6 x 2.)
    // The compiler does not look inside asm statements, so the wait states it would insert
    // are guaranteed by the order itself: vector write -> MFMA read needs 2 (every operand is
    // written >= 4 instructions ahead), vector write -> packed-math read needs 1.
    auto mfma = [&](f32x16 &c, const u32x4 &a4, const uint32_t (&bv)[4]) {
        const u32x4 b4 = {bv[0], bv[1], bv[2], bv[3]};
        asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+a"(c) : "v"(a4), "v"(b4));
    };
    constexpr int NMF = RT * NT;                        // MFMAs per k-step
    constexpr int NV = 16 * NT;                         // vector instructions per k-step
    uint32_t high_bytes = PAIR_HIGH_BYTES;
    asm volatile("" : "+v"(high_bytes));

    // Vector instruction e of a k-step in issue order: the four steps of the unpack one after the other, each over the NT words of
    // the next k-step, four instructions a word; wn = those words, kn = that k-step's position in its stage (it
    // selects the quantisation group's constants)
    auto valu = [&](int e, int cur, const wvec &wn, int kn) {
        const int step = e / (4 * NT), t = e / 4 % NT, j = e % 4;
        uint32_t &b = bq[cur ^ 1][t][j];
        const int qs = G32 ? (kn >> 1) : 0;
        if (step == 0) asm volatile("v_perm_b32 %0, %1, %2, %3" : "=v"(b) : "v"(high_bytes), "v"(wn[t]), "s"(PAIR_SELECT + 0x00010001u * j));
        else if (step == 1) asm volatile("v_and_b32 %0, %1, %0" : "+v"(b) : "s"(PAIR_MASK));
        else if (step == 2) asm volatile("v_pk_add_f16 %0, %0, %1" : "+v"(b) : "v"(neg[qs][t]));
        else asm volatile("v_pk_mul_f16 %0, %0, %1" : "+v"(b) : "v"(delta[qs][t]));
    };

#pragma unroll
    for (int p = 0; p < 2; p++) {
#pragma unroll
        for (int j = 0; j < OX; j++) issue_x(p, j);
#pragma unroll
        for (int j = 0; j < OW; j++) issue_w(stg[p], j);
        advance();
    }
    landed(stg[0], std::integral_constant<int, OX + OW>());
    asm volatile("s_barrier" ::: "memory");
    stage_consts(stg[0], true);
#pragma unroll
    for (int mt = 0; mt < RT; mt++) read_a(xa[0], 0, 0, mt);
    // first operands of the pipeline, by the ordinary helper
#pragma unroll
    for (int t = 0; t < NT; t++) {
        const u32x4 bw = __builtin_bit_cast(u32x4, dequant_word_pairs(stg[0].w[0][t], neg[0][t], delta[0][t]));
        bq[0][t][0] = bw.x; bq[0][t][1] = bw.y; bq[0][t][2] = bw.z; bq[0][t][3] = bw.w;
    }
    wait_a(xa[0]);
    asm volatile("s_nop 3" ::: "memory");  // compiler-issued vector writes above -> asm MFMA reads below

    int slot = 0;  // ring slot of the stage being consumed
    // One stage, with the registers of its place in the ring of D.
    auto stage = [&](auto place) {
        constexpr int d = decltype(place)::value;
        Stage &cur_s = stg[d];
        Stage &next_s = stg[(d + 1) % D];
        Stage &fill_s = stg[(d + 2) % D];
        const int slot_next = slot + 1 < XD ? slot + 1 : 0, slot_fill = slot + 2 < XD ? slot + 2 : slot + 2 - XD;
#pragma unroll
        for (int ks = 0; ks < 4; ks++) {
            const int cur = ks & 1, nxt = cur ^ 1;
            if (ks == 3) {
                landed(next_s, std::integral_constant<int, OX + OW>());
                asm volatile("s_barrier" ::: "memory");
                stage_consts(next_s, d == D - 1 || stages > d + 1);
            }
            const wvec wn = ks < 3 ? cur_s.w[ks + 1] : next_s.w[0];
            // Behind the MFMAs, one each: the fragments of the next k-step, then this one's share of the loads of stage
            // s + 2 (all of them are issued by the end of k-step 2).
            const int x0 = OX * ks / 3, x1 = ks < 3 ? OX * (ks + 1) / 3 : x0, w0 = OW * ks / 3, w1 = ks < 3 ? OW * (ks + 1) / 3 : w0;
#pragma unroll
            for (int i = 0; i < NMF; i++) {
                mfma(acc[i / NT][i % NT], xa[cur][i / NT], bq[cur][i % NT]);
                if (i < RT) {
                    if (ks < 3) read_a(xa[nxt], slot, ks + 1, i);
                    else read_a(xa[nxt], slot_next, 0, i);
                }
#pragma unroll
                for (int e = i * NV / NMF; e < (i + 1) * NV / NMF; e++) valu(e, cur, wn, (ks + 1) & 3);
                if (i >= RT) {
#pragma unroll
                    for (int l = (i - RT) * (x1 - x0 + w1 - w0) / (NMF - RT); l < (i - RT + 1) * (x1 - x0 + w1 - w0) / (NMF - RT); l++) {
                        if (l < x1 - x0) issue_x(slot_fill, x0 + l);
                        else issue_w(fill_s, w0 + l - (x1 - x0));
                    }
                }
            }
            if (ks == 2) advance();
            wait_a(xa[nxt]);
        }
        slot = slot_next;
    };
    // The compiler does not know that the asm statements above wrote the accumulators with MFMAs, so it will not insert the
    // wait states a matrix result needs before another instruction may read it (up to 18): they are spent wherever
    // control flow ends a run of stages (there the compiler may copy accumulators; the build checks that it does not do
    // so earlier).
    auto settle = [&]() {
        asm volatile("s_nop 15\n\ts_nop 15" : "+a"(acc[0][0]), "+a"(acc[0][1]), "+a"(acc[1][0]), "+a"(acc[1][1]), "+a"(acc[2][0]), "+a"(acc[2][1]));
#pragma unroll
        for (int i = 0; i < NMF; i++)
            if (i / NT > 2 || i % NT > 1) asm volatile("" : "+a"(acc[i / NT][i % NT]));
    };
    typedef std::integral_constant<int, 0> First;
    typedef std::integral_constant<int, 1> Second;
    typedef std::integral_constant<int, 2> Third;
    int blocks = stages < D ? 1 : stages / D;
    do {
        stage(First());
        stage(Second());
        stage(Third());
    } while (--blocks > 0);
    settle();
    if (stages > D && stages % D > 0) {
        stage(First());
        settle();
        if (stages % D > 1) {
            stage(Second());
            settle();
        }
    }
    // Drain the clamped look-ahead loads: their destination registers are dead as far as the compiler can
    // tell, but the hardware still writes them when the data arrives, so the empty uses keep every stage
    // allocated until the wait has completed.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int j = 0; j < D; j++) {
#pragma unroll
        for (int ks = 0; ks < 4; ks++) asm volatile("" ::"v"(stg[j].w[ks]));
#pragma unroll
        for (int g = 0; g < NQ * PL; g++) {
            asm volatile("" ::"v"(stg[j].sc[g]));
            asm volatile("" ::"v"(stg[j].zr[g]));
        }
    }

    // epilogue: accumulator register r of tile (mt, t): row 8*(r/4) + 4*(lane/32) + r%4 of the
    // 32-row tile, column NT*(lane%32) + t of the wave's 32*NT
    // (`ready` in front of each row tile's stores: the compiler would otherwise read all accumulators first, spill, and
    // wait for the stores under way wherever it reloads: 7 us of a 130 us launch.)
    auto ready = [&](int mt) {
#pragma unroll
        for (int t = 0; t < NT; t++) asm volatile("" : "+v"(acc[mt][t])::"memory");
    };
    if constexpr (KH == 2) {
        // The two waves of a column pair finish every other row tile each: sums of the first half + of the second.
        f32x4 *ex = reinterpret_cast<f32x4 *>(xring) + (size_t)wn * (RT * NT * 4 * 64) + lane;
        static_assert(WNW * RT * NT * 4096 <= sizeof(xring), "the exchange reuses the ring");
        asm volatile("s_barrier" ::: "memory");  // (all loads into LDS have landed, all reads of it too)
#pragma unroll
        for (int mt = 0; mt < RT; mt++) {
            ready(mt);
            if ((mt & 1) != kh) {
#pragma unroll
                for (int t = 0; t < NT; t++)
#pragma unroll
                    for (int q = 0; q < 4; q++)
                        ex[((mt * NT + t) * 4 + q) * 64] = f32x4{acc[mt][t][4 * q], acc[mt][t][4 * q + 1], acc[mt][t][4 * q + 2], acc[mt][t][4 * q + 3]};
            }
        }
        __syncthreads();
#pragma unroll
        for (int mt = 0; mt < RT; mt++)
            if ((mt & 1) == kh) {
#pragma unroll
                for (int t = 0; t < NT; t++)
#pragma unroll
                    for (int q = 0; q < 4; q++) {
                        const f32x4 v = ex[((mt * NT + t) * 4 + q) * 64];
#pragma unroll
                        for (int r = 0; r < 4; r++) acc[mt][t][4 * q + r] += v[r];
                    }
            }
    }
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int e_l32 = tid & 31, e_kb = (tid >> 5) & 1, e_wave = tid >> 6;
    auto mine = [&](int mt) { return KH == 1 || (mt & 1) == kh; };  // wave-uniform
    const int nloc = (e_wave % WNW) * WN + NT * e_l32;   // first column within the tile
    const int nout = nbase + nloc;
    const int mloc0 = (KH == 1 ? e_wave / WNW : 0) * 32 * RT + 4 * e_kb, mrow0 = m0 + mloc0;
    if (NT == 2 && part != nullptr) {  // (launches in K parts are of half-width tiles)
        float *ptile = part + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * (BM * WGN) + nloc;
#pragma unroll
        for (int mt = 0; mt < RT; mt++) {
            if (!mine(mt)) continue;
            ready(mt);
#pragma unroll
            for (int r = 0; r < 16; r++) {
                const int mo = mt * 32 + 8 * (r >> 2) + (r & 3);
                if (mrow0 + mo < M && nout < N) {
                    float *p = ptile + (size_t)(mloc0 + mo) * WGN;
                    *reinterpret_cast<float2 *>(p) = make_float2(acc[mt][0][r], acc[mt][1][r]);
                }
            }
        }
        return;
    }
    if constexpr (NT == 3) {
        // Three columns per lane are no aligned store, nor whole (gate, up) pairs: a row tile at a time goes through this
        // wave's part of the ring and out in octets of a row.
        constexpr int STRIDE = WN + 4;  // floats per row of the exchange
        static_assert(W * 32 * STRIDE * 4 <= sizeof(xring) || RT < 4, "the exchange reuses the ring");
        if constexpr (W * 32 * STRIDE * 4 <= sizeof(xring)) {
            float *ex = reinterpret_cast<float *>(xring) + e_wave * (32 * STRIDE);
            const int n0 = nbase + e_wave * WN, own = NT * e_l32, ecol = own + 2 >= N - n0 && own < N - n0 ? N - 3 - n0 : own;
            // What a lane reads other lanes of its wave have written: the hardware keeps a wave's LDS accesses in order, and the
            // fences tell the compiler to (they cost no instruction).
            auto across_lanes = [&]() {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            };
            asm volatile("s_barrier" ::: "memory");  // (all loads into LDS have landed, all reads of it too)
#pragma unroll
            for (int mt = 0; mt < RT; mt++) {
                if (mt > 0) across_lanes();
                ready(mt);
#pragma unroll
                for (int r = 0; r < 16; r++)
#pragma unroll
                    for (int t = 0; t < NT; t++) ex[(8 * (r >> 2) + 4 * e_kb + (r & 3)) * STRIDE + ecol + t] = acc[mt][t][r];
                across_lanes();
#pragma unroll
                for (int i = 0; i < 32 * WN / 8 / 64; i++) {
                    const int o = i * 64 + (tid & 63), row = o / (WN / 8), col = o % (WN / 8) * 8;
                    const f32x4 a = *reinterpret_cast<const f32x4 *>(ex + row * STRIDE + col), b = *reinterpret_cast<const f32x4 *>(ex + row * STRIDE + col + 4);
                    const int m = m0 + mt * 32 + row, n = n0 + col;
                    if (m < M && n < N) store_octet(y, m, N, n, epi, a, b);
                }
            }
        }
        return;
    }
    if (nout < N) {
        h16 *ycol = y + nout;
#pragma unroll
        for (int mt = 0; mt < RT; mt++) {
            if (!mine(mt)) continue;
            ready(mt);
#pragma unroll
            for (int r = 0; r < 16; r++) {
                const int m = mrow0 + mt * 32 + 8 * (r >> 2) + (r & 3);
                if (m < M) {
                    if (epi != 0) {
                        // adjacent columns are (gate j, up j): y [M][N/2] = SiLU(gate) * up
                        h16 *yh = y + (size_t)m * (N >> 1) + (nout >> 1);
                        if constexpr (NT == 4) {
                            h16x2 o;
                            o.x = (h16)(sqp_silu(acc[mt][0][r]) * acc[mt][1][r]);
                            o.y = (h16)(sqp_silu(acc[mt][2][r]) * acc[mt][3][r]);
                            *reinterpret_cast<h16x2 *>(yh) = o;
                        } else {
                            *yh = (h16)(sqp_silu(acc[mt][0][r]) * acc[mt][1][r]);
                        }
                    } else if constexpr (NT == 4) {
                        h16x4 o;
                        o.x = (h16)acc[mt][0][r]; o.y = (h16)acc[mt][1][r];
                        o.z = (h16)acc[mt][2][r]; o.w = (h16)acc[mt][3][r];
                        *reinterpret_cast<h16x4 *>(ycol + (size_t)m * N) = o;
                    } else {
                        h16x2 o;
                        o.x = (h16)acc[mt][0][r]; o.y = (h16)acc[mt][1][r];
                        *reinterpret_cast<h16x2 *>(ycol + (size_t)m * N) = o;
                    }
                }
            }
        }
    }
}

// y = fp16(sum over the K parts, in part order) of the fp32 partial tiles part[parts][tiles][bm][wgn]
// that a launch left: 8 adjacent columns per thread.  grid: (bm wgn / 2048, tiles); wgn 128 or 256.
__global__ void __launch_bounds__(256) splitk_reduce_kernel(const float *__restrict__ part, int M, int N, int bm, int wgn, TileMap map,
                                                            int parts, h16 *__restrict__ y, int epi)
{
    const int e = (blockIdx.x * 256 + threadIdx.x) * 8;      // element of the tile
    const int row = wgn == 256 ? e >> 8 : e >> 7, col = e & (wgn - 1);
    int trow, tcol;
    tile_at(map, blockIdx.y, trow, tcol);
    const int m = trow * bm + row, n = tcol * wgn + col;
    if (m >= M || n >= N) return;
    const f32x4 *p = reinterpret_cast<const f32x4 *>(part + (size_t)blockIdx.y * bm * wgn + e);
    const size_t stride = (size_t)gridDim.y * bm * wgn / 4;  // one part, in 16-byte pieces
    f32x4 a = p[0], b = p[1];
    for (int s = 1; s < parts; s++) {
        const f32x4 *q = p + s * stride;
        a += q[0];
        b += q[1];
    }
    store_octet(y, m, N, n, epi, a, b);
}

}  // namespace

int sqp_compute_units()
{
    static int cus = 0;  // same on every device of a node
    if (cus == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            n = 256;
        cus = n;
    }
    return cus;
}

// Test/benchmark hooks.  Tiles: 0 = automatic tile choice, 1 = full tiles only, 2 = half tiles
// only.  K split: -1 = automatic, 0 or 1 = never, k >= 2 = k parts.  Shape: 0 = automatic,
// 1 = 128 x 512 full tiles (waves 1 x 4), 2 = 256 x 256 (waves 2 x 2).
static int g_tile_mode = 0, g_ksplit = -1, g_tile_shape = 0;
extern "C" void sqp_debug_set_prefill_tiles(int mode) { g_tile_mode = mode; }
extern "C" void sqp_debug_set_prefill_ksplit(int k) { g_ksplit = k; }
extern "C" void sqp_debug_set_prefill_shape(int shape) { g_tile_shape = shape; }

// The weight-streaming kernel, 64 rows at a time.
static int decode_in_row_blocks(int M, int N, int K, int group, const h16 *x, const uint32_t *packed,
                                const h16 *scales, const uint8_t *zeros, h16 *y, int epi, const SqpWorkspace &ws, hipStream_t stream)
{
    const size_t ystride = epi != 0 ? (size_t)(N >> 1) : (size_t)N;
    for (int mb = 0; mb < M; mb += 64) {
        int rows = M - mb < 64 ? M - mb : 64;
        int rc = sqp_gemm_decode(rows, N, K, group, x + (size_t)mb * K, packed, scales, zeros, y + (size_t)mb * ystride, epi, ws, stream);
        if (rc) return rc;
    }
    return SQP_OK;
}

// Group sizes the tiled kernel covers (others run in row blocks).
static bool tiled_covers(int K, int group) { return group % BK == 0 || (group == 32 && K % BK == 0); }

// What the row blocks of a call need: blocks of 64 rows and a last one of fewer, whose plan may split where
// theirs does not.
static size_t most_of_row_blocks(size_t (*bytes)(int, int, int, int), int M, int N, int K, int group)
{
    const size_t whole = M >= 64 ? bytes(64, N, K, group) : 0, last = M % 64 ? bytes(M % 64, N, K, group) : 0;
    return whole > last ? whole : last;
}

// Launch plan of the tiled path: `full` full tiles (128 x 512 with wm == 1, 256 x 256 with
// wm == 2) in a first launch, then `half` half-width tiles (starting at full tile `full`), the
// latter times `ksplit` K parts.
struct TilePlan {
    long full, half;
    int ksplit, wm;
};

static TilePlan plan_tiles(int M, int N, int K, int group, int cus, bool have_workspace)
{
    const int wm = (g_tile_shape == 2 && group != 32) ? 2 : 1;  // groups of 32: the 128 x 512 shape only
    const int bm = 128 * wm, fulln = (4 / wm) * 128;
    const int tn = (N + fulln - 1) / fulln, tm = (M + bm - 1) / bm;
    const long tiles = (long)tn * tm;
    const int stages = K / BK;
    TilePlan p = {tiles, 0, 1, wm};
    // (1) Too few tiles to occupy the chip even as half-width tiles: split K as well.  Half
    // tiles times K parts fill the compute units; every part leaves an fp32 [M][N] matrix in
    // the workspace and a second kernel adds the parts in order (deterministic).
    int ksplit = 1;
    if (g_tile_mode == 0 && 4 * tiles <= cus) {
        ksplit = (int)(cus / (2 * tiles));
        if (ksplit > stages / 8) ksplit = stages / 8;   // at least 8 stages per part
        if (ksplit > 16) ksplit = 16;
    }
    if (g_ksplit >= 0) ksplit = g_ksplit;
    if (ksplit > stages) ksplit = stages;
    if (!have_workspace) ksplit = 1;
    if (ksplit >= 2) {
        p.full = 0;
        p.half = 2 * tiles;
        p.ksplit = ksplit;
        return p;
    }
    // (2) One workgroup per compute unit is resident, so a launch proceeds in rounds of `cus`
    // tiles.  When the last round would be at most half full, its tiles are done as twice
    // as many half-width tiles by a second launch, which then costs about half a round.
    const long rounds = tiles / cus, left = tiles - rounds * cus;
    long full = (left > 0 && 2 * left <= cus) ? rounds * cus : tiles;
    if (g_tile_mode == 1) full = tiles;
    if (g_tile_mode == 2) full = 0;
    p.full = full;
    p.half = 2 * (tiles - full);
    return p;
}

// Test hook: the plan for a shape on a chip of `cus` compute units (no launch, no GPU needed).
extern "C" void sqp_debug_prefill_plan(int M, int N, int K, int cus, long *full, long *half, int *ksplit)
{
    const TilePlan p = plan_tiles(M, N, K, 128, cus, true);
    *full = p.full;
    *half = p.half;
    *ksplit = p.ksplit;
}

// Estimated time of a 64-row stage of K for tiles of 32 rt rows x 256 columns.
static const double stage_us[7] = {0, 0, 0, 0.72, 0.77, 0.97, 1.11};

// What a call launches: up to two launches of tiles of 32 rt rows x 32 nt columns per wave, each over
// `tiles` tiles from tile0 of a grid with tn columns of tiles, in `parts` K parts (1: straight to y).  With nt == 2
// behind a launch of full tiles, tile0 counts half tiles and tn full ones (halves).
struct TileLaunch {
    int rt, nt;
    long tile0, tiles;
    int tn, parts;
    bool halves;
    int kh;  // 2: waves that halve K, tiles of half the columns
};
static int tile_columns(const TileLaunch &l, int wm) { return l.nt * 128 / wm / l.kh; }
struct LaunchPlan {
    int wm, count;
    bool own;  // K parts go to the call's own scratch, not to the workspace
    TileLaunch l[2];
};

// Test hook: one launch of this variant over the whole output (0: automatic).
static int g_force_rt = 0, g_force_nt = 0, g_force_parts = 0, g_force_kh = 1;
extern "C" void sqp_debug_set_prefill_variant(int rt, int nt, int parts)
{
    g_force_rt = rt;
    g_force_nt = nt & 15;
    g_force_kh = nt >= 16 ? 2 : 1;
    g_force_parts = parts;
}

static size_t launch_partial_bytes(const TileLaunch &l, int wm)
{
    return l.parts >= 2 ? (size_t)l.parts * l.tiles * (32 * l.rt * wm) * tile_columns(l, wm) * sizeof(float) : 0;
}

// room_ws, room_own: bytes there are for partial sums in the workspace and in the call's own scratch (0:
// none).  The workspace serves the shapes whose 128-row tiles are too few for the chip even at half
// width; all others split only where the call brings its own scratch, because the workspace is shared
// and callers may run those shapes beside calls that use it.
// A plan in 128-row tiles that needs more is returned as it is and refused by the caller; the
// estimates below only take what fits.
static LaunchPlan plan_launches(int M, int N, int K, int group, int cus, size_t room_ws, size_t room_own)
{
    const bool own = g_force_rt == 0 && plan_tiles(M, N, K, group, cus, true).ksplit < 2;
    const size_t room = own ? room_own : room_ws;
    const bool have_workspace = room > 0;
    const TilePlan p = plan_tiles(M, N, K, group, cus, have_workspace);
    LaunchPlan q = {p.wm, 0, own, {}};
    const int stages = K / BK, tnf = (N + (4 / p.wm) * 128 - 1) / ((4 / p.wm) * 128);
    if (g_force_rt > 0 && group != 32) {
        const int kh = g_force_kh == 2 && g_force_nt == 2 && K % (2 * BK) == 0 ? 2 : 1;
        const int wg = 128 * g_force_nt / kh;
        const int tn = (N + wg - 1) / wg, tm = (M + 32 * g_force_rt - 1) / (32 * g_force_rt);
        q.wm = 1;
        q.count = 1;
        int parts = g_force_nt == 2 && have_workspace ? g_force_parts : 1;
        if (parts > stages / kh) parts = stages / kh;
        q.l[0] = TileLaunch{g_force_rt, g_force_nt, 0, (long)tn * tm, tn, parts < 1 ? 1 : parts, false, kh};
        return q;
    }
    const bool hooked = g_tile_mode != 0 || g_tile_shape != 0 || g_ksplit >= 0;
    // Everything in one round of the chip: the variant and the number of K parts with the least estimated time.
    // The estimate (us) ranks plans: per 64-row stage of K 0.72 / 0.77 / 0.97 / 1.11 for tiles of 96 / 128 / 160 /
    // 192 rows x 256 columns and 1.43 for 128 x 512, plus the fp32 parts' way out and back at 5.6 TB/s;
    // more than 12 parts never won.  It leaves out what all plans share, so it is low throughout: 609
    // measured launches of 51 shapes take 6.7 us more, those with K parts another 1.8 for the reduction's
    // launch (with both, rms 6 %).  The plan it picks is 0.5 % slower than the best one measured in the
    // mean of the shapes and 5.5 % at worst, with the reduction's cost in it 0.4 % and 5.5 %.
    // Groups of 32 keep the plan in 128-row tiles: only its two tiles are built for two groups per stage.
    // What it buys (us, 128-row tiles only -> chosen): 8192->8192 at 72 / 150 / 190 / 320 / 640 rows
    // 33.6 -> 27.7, 47.0 -> 37.9, 47.6 -> 39.8, 71.1 -> 56.7, 116 -> 96; 4096->22016 at 80 / 160 / 320 rows
    // 43.7 -> 35.4, 65.5 -> 47.9, 99 -> 76; 8192->10240 at 160 rows 56 -> 43: a 128-row tile computes
    // rows that are not there.
    if (!hooked && group != 32) {
        const double part_us = (double)M * N * 8 / 5.6e6;
        double best = 0;
        const long tiles44 = (long)((N + 511) / 512) * ((M + 127) / 128);
        if (tiles44 <= cus) {
            best = stages * 1.43;
            q.wm = 1;
            q.count = 1;
            q.l[0] = TileLaunch{4, 4, 0, tiles44, (N + 511) / 512, 1, false, 1};
        }
        const int tn = (N + 255) / 256;
        for (int rt = 3; rt <= 6; rt++) {
            const long tiles = (long)tn * ((M + 32 * rt - 1) / (32 * rt));
            int most = have_workspace ? (int)(cus / tiles) : 1;
            if (most > stages / 8) most = stages / 8;  // at least 8 stages per part
            if (most > 12) most = 12;
            if (tiles > cus) continue;
            for (int parts = 1; parts <= (most > 1 ? most : 1); parts++) {
                const double t = (stages + parts - 1) / parts * stage_us[rt] + (parts > 1 ? parts * part_us : 0.0);
                const TileLaunch l = {rt, 2, 0, tiles, tn, parts, false, 1};
                if (launch_partial_bytes(l, 1) <= room && (q.count == 0 || t < best)) {
                    best = t;
                    q.count = 1;
                    q.l[0] = l;
                }
            }
        }
        if (q.count) return q;
    }
    if (p.full > 0) q.l[q.count++] = TileLaunch{4, 4, 0, p.full, tnf, 1, false, 1};
    if (p.half > 0) {
        int parts = p.ksplit;
        while (!hooked && parts > 1 && launch_partial_bytes(TileLaunch{4, 2, 0, p.half, 0, parts, true, 1}, p.wm) > room) parts--;
        // Few tiles left over after the whole rounds: split in K as well, as far as they then fill the
        // chip once.
        if (!hooked && p.full > 0 && have_workspace) {
            int most = (int)(cus / p.half);
            if (most > stages / 8) most = stages / 8;
            if (most > 16) most = 16;
            const double part_us = (double)p.half * 128 * 256 * 8 / 4.5e6;
            double best = stages * 0.77;
            for (int n = 2; n <= most; n++) {
                const double t = (stages + n - 1) / n * 0.77 + n * part_us + 3;  // (3: the reduction's launch)
                if (t < best && launch_partial_bytes(TileLaunch{4, 2, 0, p.half, 0, n, true, 1}, 1) <= room) {
                    best = t;
                    parts = n;
                }
            }
        }
        q.l[q.count++] = TileLaunch{4, 2, 2 * p.full, p.half, tnf, parts, true, 1};
    }
    return q;
}

// Test hook: the launches that a call's sizes are reported for (no GPU needed): up to two of (rt, nt, tiles, parts).
extern "C" int sqp_debug_prefill_launches(int M, int N, int K, int group, int cus, int *out8)
{
    const LaunchPlan q = plan_launches(M, N, K, group, cus, SIZE_MAX, SIZE_MAX);
    for (int i = 0; i < q.count; i++) {
        out8[4 * i] = q.l[i].rt;
        out8[4 * i + 1] = q.l[i].nt;
        out8[4 * i + 2] = (int)q.l[i].tiles;
        out8[4 * i + 3] = q.l[i].parts;
    }
    return q.count;
}

static size_t plan_partial_bytes(const LaunchPlan &q)
{
    size_t need = 0;
    for (int i = 0; i < q.count; i++) {
        const size_t b = launch_partial_bytes(q.l[i], q.wm);
        need = b > need ? b : need;
    }
    return need;
}

// Estimated time (us) of one launch of tiles with all that belongs to it, on a chip that it fills once:
// a + stages * (b + l * workgroups / compute units) + (h + p * MB), the last two with K parts (MB: their fp32 sums
// written and read); a stage is 64 k, 128 with waves that halve K.  Up to one workgroup per compute unit, or two of the
// variants that leave half the registers.  Fitted to 9085 launches of 294 shapes (65 to 1536 rows, N 1024 to 24576,
// K 1024 to 16384, groups of 128): rms 2.7 to 5.0 % by variant.  Beyond four parts each costs 0.2 us at least, however few
// its bytes: the reduction waits for one after the other (5004 launches of 527 other shapes, most of them of few tiles:
// without it 4.7 to 8.7 %, waves that halve K and 9 to 12 parts of less than 0.2 MB 13 % too low).  It keeps calls of few columns
// and a long K with the row blocks: 308x9088x136 in groups of 64 12.5 us, 14.8 in tiles of 12 parts; 219 of 6771 drawn calls,
// 1.10 times faster in the mean.  0: not covered.
static double launch_us(const TileLaunch &l, int M, int N, int K, int cus)
{
    struct Cost { double a, b, l, h, p; };
    static const Cost one[4] = {{7.36, 0.465, 0.112, 1.75, 0.164}, {8.72, 0.479, 0.206, 1.35, 0.140}, {9.94, 0.558, 0.278, 1.39, 0.119}, {10.87, 0.648, 0.318, 1.23, 0.113}};
    static const Cost halves[4] = {{6.76, 0.460, 0.174, 1.81, 0.214}, {7.20, 0.494, 0.266, 2.28, 0.188}, {8.69, 0.576, 0.346, 1.58, 0.187}, {9.20, 0.660, 0.387, 1.53, 0.185}};
    static const Cost two[2] = {{8.92, 0.545, 0.350, 3.09, 0.080}, {10.60, 0.734, 0.409, 1.19, 0.094}}, wide = {8.65, 0.951, 0.372, 0, 0};
    static const Cost three[2] = {{7.72, 0.729, 0.411, 0, 0}, {8.51, 0.876, 0.453, 0, 0}};
    const long groups = l.tiles * l.parts;
    if (groups > 2L * cus || (groups > cus && (l.nt != 2 || l.kh == 2 || l.rt > 4))) return 0;
    const Cost &c = l.nt == 4 ? wide : l.nt == 3 ? three[l.rt - 4] : l.kh == 2 ? halves[l.rt - 3] : groups > cus ? two[l.rt - 3] : one[l.rt - 3];
    const int stages = (K / (BK * l.kh) + l.parts - 1) / l.parts;
    const double part_us = c.p * ((double)M * N * 8e-6), more_us = part_us < 0.2 ? 0.2 : part_us;
    const double parts_us = l.parts > 4 ? 4 * part_us + (l.parts - 4) * more_us : l.parts * part_us;
    const double t = c.a + stages * (c.b + c.l * (double)groups / cus) + (l.parts > 1 ? c.h + parts_us : 0.0);
    // (activations that two L2s would not hold, read by twice as many columns of tiles: measured 10 to 18 % longer, 5 % with
    // whole-K waves)
    return l.kh == 2 && l.parts > 1 && 2.0 * M * K > 8e6 ? 1.12 * t : t;
}

// Of a plan that is one launch of at most one workgroup per compute unit, or one full round of the chip and few tiles left
// over: a quicker one, if there is one by 3 % by the
// estimate, whose parts fit the room that the plan's have.  Tiles of half the columns whose waves halve K need half
// the K parts (or none) for as many workgroups, at the price of twice the activations per compute unit; tiles of 96 and
// 128 rows x 256 columns leave half of the registers, so that two workgroups per compute unit hide each other's
// waits; 128 or 160 rows x 384 columns fill one round where 128 x 512 leave a third of the chip idle or spill over.  The sizes reported to callers are those of the plan itself: what they have stored goes on to hold.
// us per call, weights from HBM, the same kernels with the plan -> with the quicker one: 160x8192x8192 36.9 -> 34.4,
// 160x4096x22016 42.6 -> 39.1, 300x5120x15360 57.9 -> 52.2, 490x2816x5840 29.2 -> 23.2, 999x2176x3832 26.6 -> 22.2,
// 403x3072x22792 73.7 -> 65.7, 512x4096x22016 91.0 -> 83.3, 772x3456x18968 113.0 -> 90.5; over the fitted shapes the pick is
// 0.5 % behind the best in the mean.
static double quicker_launch(LaunchPlan &q, int M, int N, int K, int group, int cus, size_t room)
{
    const bool hooked = g_tile_mode != 0 || g_tile_shape != 0 || g_ksplit >= 0 || g_force_rt > 0;
    if (hooked || group == 32 || q.wm != 1) return 0;
    double best = launch_us(q.l[0], M, N, K, cus);
    if (best == 0) return 0;
    if (q.count == 2) {
        TileLaunch rest = q.l[1];
        rest.halves = false;
        best += launch_us(rest, 128, (int)(rest.tiles * 256), K, cus);
    }
    double least = best * 0.97;
    const int stages = K / BK;
    for (int rt = 3; rt <= 6; rt++)
        for (int kh = 1; kh <= (K % (2 * BK) == 0 ? 2 : 1); kh++) {
            const int wg = 256 / kh, tn = (N + wg - 1) / wg;
            const long tiles = (long)tn * ((M + 32 * rt - 1) / (32 * rt)), slots = rt <= 4 && kh == 1 ? 2 * cus : cus;
            for (int parts = 1; parts <= 12 && tiles * parts <= slots; parts++) {
                const TileLaunch l = {rt, 2, 0, tiles, tn, parts, false, kh};
                if (parts > 1 && (stages < 8 * parts || launch_partial_bytes(l, 1) > room)) break;
                const double t = launch_us(l, M, N, K, cus);
                if (t < least) {
                    least = best = t;
                    q.count = 1;
                    q.l[0] = l;
                }
            }
        }
    const int tn = (N + 383) / 384;
    for (int rt = 4; rt <= 5; rt++) {
        const TileLaunch l = {rt, 3, 0, (long)tn * ((M + 32 * rt - 1) / (32 * rt)), tn, 1, false, 1};
        const double t = l.tiles <= cus ? launch_us(l, M, N, K, cus) : 0;
        if (t > 0 && t < least) {
            least = best = t;
            q.count = 1;
            q.l[0] = l;
        }
    }
    return best;
}

// Estimated time (us) of the launches of a plan, without what all launches share: see plan_launches.
static double launches_us(const LaunchPlan &q, int K, int group, int cus)
{
    double t = 0;
    for (int i = 0; i < q.count; i++) {
        const TileLaunch &l = q.l[i];
        const long rounds = (l.tiles * l.parts + cus - 1) / cus;
        t += rounds * ((K / BK + l.parts - 1) / l.parts) * (l.nt == 4 ? 1.43 : stage_us[l.rt]);
        if (l.parts > 1) t += 2.0 * launch_partial_bytes(l, q.wm) / 5.6e6 + 1.8;
    }
    return t + (group == 32 ? 2.0 : 0.0);
}

// Test hook: row blocks of 16 mt rows with this K split and kp chunks per iteration (0: automatic, -1: never).
static SqpStripPlan g_row_blocks = {0, 0, 0, 0, 0};
extern "C" void sqp_debug_set_row_blocks(int mt, int split, int kp) { g_row_blocks = SqpStripPlan{2, split, 2, kp, mt}; }

// Groups the row blocks cover: their chunks of 128 k hold whole groups or are parts of one (the tiled kernel also takes
// 192, 320 and other odd multiples of 64, whose ends lie inside a chunk).
static bool row_blocks_cover(int K, int group) { return K % 128 == 0 && (group == 32 || group == 64 || group % 128 == 0); }

// Calls of more than 64 rows on layers too small for the tiled kernel: the strip kernel in row blocks of 48 or
// 64 rows, all in one launch (mt 0: none).  A tile of the tiled kernel takes 9 us at K = 1024 and 50 at K = 8192
// with a compute unit to itself, however few tiles there are, and splitting its K costs a second launch
// and the fp32 parts through memory; the strip kernel's workgroups are small, walk K with two waves per SIMD
// and hand partial tiles over in the same launch.  It reads the weights once per row block (the second and
// later ones from L2 or the last-level cache) and unpacks them again, so it loses once the chip is full:
// taken where its estimated time is below that of the tiles (launch_us; 8 % below plan_launches' coarser estimate and
// the 6.7 us that it leaves out).
// The estimate: A + iterations * (B + L * workgroups / compute units) + (H + S * parts), the last two terms with
// more than one K part (B and L 6 % below the fit since the kernel's iterations are that much shorter: 91 other calls); at
// most one eight-wave workgroup (kp = 2) or two four-wave ones per compute unit.
// Fitted to 13700 launches of 1547 shapes (65 to 1024 rows, N 768 to 24576, K 512 to 8192, groups of 32, 64, 128
// and 256, weights from HBM): rms 3 to 6 %, the choice 1 % behind the best variant in the mean.  On 945 other calls
// that take row blocks, drawn over these ranges: 1.46 times faster than the tiles in the geometric mean, 1.5 % of
// them more than 3 % slower, at worst 12 % (the sweep is among the profiles).  us, tiles -> row blocks, groups of 128:
// 1024->1024 at 65 rows 12.1 -> 8.2, 1024->4096 at 160 rows 15.4 -> 9.2, 4096->4096 at 128 rows 21.7 -> 13.8, 2048->8192 at
// 256 rows 26.0 -> 15.3, 8192->8192 at 65 / 128 rows 26.6 -> 25.0 / 32.8 -> 28.8 (at 160 rows 38.4 against 39.6).
// limit: bytes of partial tiles the call may leave in its workspace.
static SqpStripPlan row_blocks_plan(int M, int N, int K, int group, int cus, double tiles_us, size_t limit)
{
    struct Cost { double a, b, l, h, s; };
    static const Cost cost[2][3] = {  // 48 and 64 rows; kp = 1 with up to one and two workgroups per unit, kp = 2
        {{3.92, 0.612, 0.058, 2.14, 0.28}, {5.25, 0.710, 0.143, 1.77, 0.40}, {4.83, 0.964, 0.090, 1.60, 0.22}},
        {{4.19, 0.692, 0.074, 2.03, 0.31}, {5.75, 0.771, 0.198, 1.68, 0.47}, {5.11, 1.085, 0.141, 1.58, 0.29}},
    };
    SqpStripPlan best = {2, 1, 2, 1, 0};
    if (M <= 64 || !row_blocks_cover(K, group)) return best;
    if ((long)((N + 127) / 128) * ((M + 63) / 64) > 2 * cus) return best;  // (no launch below fits: long prompts end here)
    const int chunks = K / 128;
    double least = tiles_us;
    for (int mt = 3; mt <= 4; mt++) {
        const long blocks = (M + 16 * mt - 1) / (16 * mt), tiles = (N + 127) / 128 * blocks;
        size_t part = 0;  // bytes of one K part's tiles (two for all: none where the tickets do not reach)
        if (2 <= chunks && sqp_strip_split(mt, 2, 4, (int)blocks, N, K, 2, &part) == 2) part /= 2;
        for (int kp = 1; kp <= (group > 128 ? 1 : 2); kp++) {
            for (int split = 1; split == 1 || 2 * split <= chunks; split++) {  // at least two chunks per part
                const long groups = tiles * split;
                if (groups > (kp == 2 ? cus : 2 * cus)) break;
                if (split > 1 && (part == 0 || part * split > limit)) break;
                const Cost &c = cost[mt - 3][kp == 2 ? 2 : (groups > cus ? 1 : 0)];
                const int iterations = ((chunks + split - 1) / split + kp - 1) / kp;
                double t = c.a + iterations * (c.b + c.l * groups / cus) + (split > 1 ? c.h + c.s * split : 0.0);
                if (group < 128) t *= 1.05;  // steps and zero points of more groups
                if (t < least) {
                    least = t;
                    best = SqpStripPlan{2, split, 2, kp, mt};
                }
            }
        }
    }
    return best;
}

// What a call takes beside the tiled launches q: none where those are forced by a test hook.  us: their estimated
// time, 0 where launch_us has none.
static SqpStripPlan row_blocks_for(const LaunchPlan &q, int M, int N, int K, int group, int cus, size_t limit, double us)
{
    const bool hooked = g_tile_mode != 0 || g_tile_shape != 0 || g_ksplit >= 0 || g_force_rt > 0;
    if (g_row_blocks.mt > 0 && row_blocks_cover(K, group)) return g_row_blocks;
    if (hooked || g_row_blocks.mt < 0) return SqpStripPlan{2, 1, 2, 1, 0};
    return row_blocks_plan(M, N, K, group, cus, us > 0 ? us : (launches_us(q, K, group, cus) + 6.7) / 1.08, limit);
}

static size_t row_blocks_bytes(const SqpStripPlan &p, int M, int N, int K)
{
    size_t bytes = 0;
    if (p.mt) sqp_strip_split(p.mt, p.nw, 4, (M + 16 * p.mt - 1) / (16 * p.mt), N, K, p.split, &bytes);
    return bytes;
}

// The launches with as large a workspace as they like.  The bytes they leave there are 0 for shapes that report
// none and never touch it.
static LaunchPlan preferred_launches(int M, int N, int K, int group, int cus)
{
    return plan_launches(M, N, K, group, cus, SIZE_MAX, 0);
}

static size_t partial_bytes(int M, int N, int K, int group, int cus)
{
    const LaunchPlan q = preferred_launches(M, N, K, group, cus);
    const size_t tiles = plan_partial_bytes(q);
    if (tiles == 0 && g_row_blocks.mt <= 0) return 0;  // (a forced plan says what it needs)
    // (row blocks as the launches above would leave them, not as a quicker launch would)
    const size_t rows = row_blocks_bytes(row_blocks_for(q, M, N, K, group, cus, SIZE_MAX, 0), M, N, K);
    return rows > tiles ? rows : tiles;
}

size_t sqp_gemm_prefill_partial_bytes(int M, int N, int K, int group)
{
    if (!tiled_covers(K, group)) return most_of_row_blocks(sqp_gemm_decode_partial_bytes, M, N, K, group);
    return partial_bytes(M, N, K, group, sqp_compute_units());
}

// Scratch that a call may ask for its own K parts (the static array's size).
static constexpr size_t OWN_MOST = 48u << 20;

size_t sqp_gemm_prefill_scratch_bytes(int M, int N, int K, int group)
{
    if (!tiled_covers(K, group)) return 0;
    LaunchPlan q = plan_launches(M, N, K, group, sqp_compute_units(), SIZE_MAX, SIZE_MAX);
    const size_t bytes = plan_partial_bytes(q);
    if (q.own) quicker_launch(q, M, N, K, group, sqp_compute_units(), OWN_MOST);
    return q.own ? (plan_partial_bytes(q) > bytes ? plan_partial_bytes(q) : bytes) : 0;  // (also where row blocks run and leave it untouched: 1 shape in 200)
}

// What a workspace has to hold at least for a call not to be refused: the K parts of the plan in 128-row
// tiles as [parts][M][N].  With less than the preferred plan's bytes, one that fits runs, of row blocks too.
// tiles: bytes of the preferred launches.
static size_t least_bytes(size_t tiles, int M, int N, int K, int group, int cus)
{
    if (g_force_rt > 0 || tiles == 0) return tiles;
    const TilePlan p = plan_tiles(M, N, K, group, cus, true);
    const size_t base = p.ksplit >= 2 ? (size_t)p.ksplit * M * N * sizeof(float) : 0;
    return base < tiles ? base : tiles;
}

size_t sqp_gemm_prefill_least_bytes(int M, int N, int K, int group)
{
    if (!tiled_covers(K, group)) return most_of_row_blocks(sqp_gemm_decode_least_bytes, M, N, K, group);
    const int cus = sqp_compute_units();
    return least_bytes(plan_partial_bytes(preferred_launches(M, N, K, group, cus)), M, N, K, group, cus);
}

// What a call runs with these bytes for K parts in its workspace and in its own scratch: row blocks (rows.mt > 0) or
// tiled launches.
struct CallPlan {
    LaunchPlan q;
    SqpStripPlan rows;
    bool refused;  // a workspace below the least size
};

static CallPlan plan_call(int M, int N, int K, int group, int cus, size_t room_ws, size_t room_own)
{
    // The preferred launches are looked for once: they are what runs wherever their parts fit the workspace, unless
    // the call brings scratch for a shape that has no parts there.
    CallPlan c = {preferred_launches(M, N, K, group, cus), {2, 1, 2, 1, 0}, true};
    const size_t tiles = plan_partial_bytes(c.q);
    if (room_ws > 0 && room_ws < least_bytes(tiles, M, N, K, group, cus)) return c;
    if (c.q.own ? room_own > 0 : room_ws < tiles) c.q = plan_launches(M, N, K, group, cus, room_ws, room_own);
    if (plan_partial_bytes(c.q) > (c.q.own ? room_own : room_ws)) return c;
    c.refused = false;
    // What is chosen in their place has the room that the shape reports and no more, however large the buffer is: every
    // sufficient one gives the same launches and so the same bits (a caller's exact one, the static array, one
    // that has grown for other shapes), and a shape that reports no workspace leaves nothing there, beside whichever
    // call is using it.
    const size_t room = c.q.own ? OWN_MOST : tiles, here = c.q.own ? room_own : room_ws;
    const double us = quicker_launch(c.q, M, N, K, group, cus, here < room ? here : room);
    // Parts of row blocks go to the workspace where the shape reports one: the others may run beside calls that
    // use it.  (They may be larger than the tiles': the size reported is looked for only then.)
    const size_t limit = tiles > 0 ? room_ws : 0;
    c.rows = row_blocks_for(c.q, M, N, K, group, cus, limit, us);
    if (row_blocks_bytes(c.rows, M, N, K) > tiles) {
        const size_t most = partial_bytes(M, N, K, group, cus);
        if (limit > most) c.rows = row_blocks_for(c.q, M, N, K, group, cus, most, us);
    }
    return c;
}

// Test hook: the tiled launches of a call with `room` bytes for K parts (no GPU needed): up to two of (rt, nt, tiles, parts,
// kh); 0: refused.
extern "C" int sqp_debug_prefill_choice(int M, int N, int K, int group, int cus, size_t room, int *out10)
{
    const CallPlan c = plan_call(M, N, K, group, cus, room, room);
    if (c.refused) return 0;
    for (int i = 0; i < c.q.count; i++) {
        const TileLaunch &l = c.q.l[i];
        const int v[5] = {l.rt, l.nt, (int)l.tiles, l.parts, l.kh};
        for (int j = 0; j < 5; j++) out10[5 * i + j] = v[j];
    }
    return c.q.count;
}

// Test hook: the row blocks of a call (rows / 16, K parts, chunks per iteration; rows 0: none), without a workspace (0),
// with one of the reported size (1) or as large as it likes (2).  Host arithmetic only.
extern "C" void sqp_debug_row_blocks(int M, int N, int K, int group, int cus, int workspace, int *out3)
{
    SqpStripPlan p = {2, 0, 2, 0, 0};
    if (tiled_covers(K, group))
        p = plan_call(M, N, K, group, cus, workspace == 0 ? 0 : workspace == 1 ? partial_bytes(M, N, K, group, cus) : SIZE_MAX, 0).rows;
    out3[0] = p.mt;
    out3[1] = p.split;
    out3[2] = p.kp;
}

// Rows per group of the numbering: 8 for full tiles, whose stage takes as many bytes of x per row of tiles as of
// weights per column (8 x 4 of the 32 that an XCD holds: 12 blocks of 16 KB, 5.7 x 5.7 would be the least), 4 for tiles
// of half the columns; groups of equal size where the rows do not divide.  One row per group in launches of K parts alone
// (291x5952x1072 18.9 us, 20.4 with groups of four).
static TileMap tile_map(const TileLaunch &l, int wm, int M)
{
    const int bm = 32 * l.rt * wm, most = l.halves || l.nt >= 3 ? 8 / wm : l.parts > 1 ? 1 : 4;
    const int tm = (M + bm - 1) / bm, groups = (tm + most - 1) / most;
    return TileMap{(int)l.tile0, l.tn, tm, (tm + groups - 1) / groups, l.halves};
}

template <int RT, int NT, int WM, bool G32, int KH = 1>
static void launch_variant(const TileLaunch &l, int M, int N, int K, int group, const h16 *x, const uint32_t *packed, const h16 *scales,
                           const uint8_t *zeros, h16 *y, int epi, float *part, hipStream_t stream)
{
    w4a16_prefill_kernel<RT, NT, WM, KH, G32><<<dim3((unsigned)l.tiles, l.parts), 256, 0, stream>>>(
        M, N, K, group, tile_map(l, WM, M), x, packed, scales, zeros, y, l.parts >= 2 ? part : nullptr, epi);
}

int sqp_gemm_prefill(int M, int N, int K, int group, const h16 *x, const uint32_t *packed,
                     const h16 *scales, const uint8_t *zeros, h16 *y, int epi, const SqpWorkspace &ws, hipStream_t stream)
{
    if (!tiled_covers(K, group))
        return decode_in_row_blocks(M, N, K, group, x, packed, scales, zeros, y, epi, ws, stream);
    const CallPlan c = plan_call(M, N, K, group, sqp_compute_units(), ws.partial ? ws.partial_bytes : 0, ws.own ? ws.own_bytes : 0);
    if (c.refused) return SQP_ERR_WORKSPACE;
    const SqpStripPlan &rows = c.rows;
    const LaunchPlan &q = c.q;
    float *const part = q.own ? ws.own : ws.partial;
    if (rows.mt) return sqp_strip_row_blocks(group, rows, M, N, K, group <= 128 ? 1 : group / 128, x, packed, scales, zeros, y, epi, ws, stream);
    for (int i = 0; i < q.count; i++) {
        const TileLaunch &l = q.l[i];
#define SQP_TILES(RT, NT, WM, G32) launch_variant<RT, NT, WM, G32>(l, M, N, K, group, x, packed, scales, zeros, y, epi, part, stream)
#define SQP_TILES_KH(RT) launch_variant<RT, 2, 1, false, 2>(l, M, N, K, group, x, packed, scales, zeros, y, epi, part, stream)
        if (group == 32) {
            if (l.nt == 4) SQP_TILES(4, 4, 1, true);
            else SQP_TILES(4, 2, 1, true);
        } else if (q.wm == 2) {
            if (l.nt == 4) SQP_TILES(4, 4, 2, false);
            else SQP_TILES(4, 2, 2, false);
        } else if (l.nt == 4) {
            SQP_TILES(4, 4, 1, false);
        } else if (l.nt == 3) {
            if (l.rt == 5) SQP_TILES(5, 3, 1, false);
            else SQP_TILES(4, 3, 1, false);
        } else if (l.kh == 2) {
            switch (l.rt) {
                case 3: SQP_TILES_KH(3); break;
                case 5: SQP_TILES_KH(5); break;
                case 6: SQP_TILES_KH(6); break;
                default: SQP_TILES_KH(4); break;
            }
        } else {
            switch (l.rt) {
                case 3: SQP_TILES(3, 2, 1, false); break;
                case 5: SQP_TILES(5, 2, 1, false); break;
                case 6: SQP_TILES(6, 2, 1, false); break;
                default: SQP_TILES(4, 2, 1, false); break;
            }
        }
#undef SQP_TILES
#undef SQP_TILES_KH
        if (l.parts >= 2) {
            const int bm = 32 * l.rt * q.wm, wgn = tile_columns(l, q.wm);
            splitk_reduce_kernel<<<dim3(bm * wgn / 2048, (unsigned)l.tiles), 256, 0, stream>>>(part, M, N, bm, wgn, tile_map(l, q.wm, M), l.parts, y, epi);
        }
    }
    return sqp_launch_status();
}
