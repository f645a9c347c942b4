// Weight-streaming W4A16 GEMM for small M (decode): y = x * w_hat, Eq. 3 of
// arXiv 2312.03788 with w_hat = (code - Z) * Delta of Eq. 1, group-wise along K (Sec 2.2).
//
// The kernel is bound by the HBM stream of packed weights, and on this chip that stream is
// limited by how many cache-line requests a compute unit's vector L1 keeps in flight: the
// L1 handles requests in order, so every request that is not a weight line (activations,
// steps, zero points) takes a place a weight line could have had.  The design follows:
//   - A workgroup of NW waves covers 64*NW output columns; each wave owns a 64-column strip
//     and every wave walks the same range of K.  One dwordx4 load per lane fetches, for
//     k-block (lane / 16), the packed words of 4 adjacent columns: a word is 8 consecutive k
//     of one column, which is exactly one lane's B operand of v_mfma_f32_16x16x32_f16
//     (column = lane % 16, k-block = lane / 16).
//   - The activations of a K chunk are fetched ONCE per workgroup, as whole 128-byte lines,
//     by direct global->LDS loads into a ring of D slots, and every wave takes its A operands
//     from there (row = lane % 16, permuted to the nibble order of the unpack).
//   - The codes become exact fp16 integers (code - Z) with 9 VALU ops per word: the nibbles
//     are OR-ed into the mantissa of 1024.0 (bits 3:0) or 64.0 (bits 7:4) and the offset
//     (1024 + Z or 64 + Z) is subtracted with a packed fp16 add, which is exact.
//   - The MFMA accumulates one chunk in fp32, then the step Delta (a per-lane scalar in the
//     16x16 accumulator layout: column = lane % 16) scales it into the running sum:
//     sum_k x (q - Z) Delta = Delta * sum_k x (q - Z).  (The 48- and 64-row variants multiply the
//     unpacked weights by Delta instead, which is less vector work there.)
//   - Weight loads and all waits are written in assembly: D - 1 chunks of weights stay in
//     flight per wave while one is consumed, and the compiler's conservative waits (it cannot
//     tell ring slots apart) would serialise that.
// What bounds it beside the stream: the instructions a wave issues, one every four to five cycles (a wave alone and two of
// a SIMD alike).  us per launch, weights from HBM, before -> with the scalar work of an iteration cut from 70
// instructions to 25 -> with the words unpacked between the matrix instructions of the one before (and no wait
// states behind the unpack): 16 rows 8192->10240 13.9 -> 13.2 -> 12.8, 22016->8192 22.8 -> 22.2 -> 21.5, 8192->44032 39.3 ->
// 38.9 -> 38.7; 48 rows 5120->27648 27.7 -> 26.5 -> 25.8, 5120->15360 20.0 -> 19.1 -> 18.5; 20 rows in groups of 64
// 4096->22016 19.5 -> 17.9 -> 17.5; 28 rows in groups of 32 23.3 -> 20.7 -> 20.1.
// With SPLIT > 1 workgroups along K, fp32 partial tiles go to a workspace and the workgroup
// that arrives last (atomic ticket) adds them in split order, so the result does not depend
// on scheduling.
#pragma once
#include <type_traits>

#include "sqp_common.h"
#include "sqp_strip.h"
#include "sqp_w4_unpack.h"

// Pipeline depth (stages of weights per wave, slots of activations): three, i.e. two chunks in
// flight per wave while one is consumed; the 32-row variant runs best with four (three with two
// chunks per iteration, whose activation slots are twice as large).  (With the
// streaming hint, masked look-ahead loads and up to eight waves per workgroup three beats four by
// 1-10 % on most shapes; deeper pipelines were slower.)  SQP_DECODE_DEPTH overrides it for experiments.
#ifdef SQP_DECODE_DEPTH
#define SQP_DEPTH_OF(MT, KP) SQP_DECODE_DEPTH
#else
#define SQP_DEPTH_OF(MT, KP) ((MT) == 2 && (KP) == 1 ? 4 : 3)
#endif

namespace {

struct Workspace {
    float *partial;      // [tiles][SPLIT][NW][REGS][64]
    unsigned *tickets;   // [tiles], zero between launches
};

// Final store of 4 adjacent columns n .. n+3 of row m.  epi == 0: the fp16 values themselves,
// y [M][N].  epi == 1: the columns are (gate j, up j, gate j+1, up j+1) of a merged,
// interleaved gate/up projection and the output is SiLU(gate) * up, y [M][N/2] (the LlamaMLP
// activation of Fig. 5, formed from the fp32 sums before any rounding).
__device__ __forceinline__ void store_row4(h16 *y, int m, int N, int n, int epi, float a0, float a1, float a2, float a3)
{
    if (epi == 0) {
        h16x4 o;
        o.x = (h16)a0; o.y = (h16)a1; o.z = (h16)a2; o.w = (h16)a3;
        *reinterpret_cast<h16x4 *>(y + (size_t)m * N + n) = o;
    } else {
        h16x2 o;
        o.x = (h16)(sqp_silu(a0) * a1);
        o.y = (h16)(sqp_silu(a2) * a3);
        *reinterpret_cast<h16x2 *>(y + (size_t)m * (N >> 1) + (n >> 1)) = o;
    }
}

// a / b of wave-uniform values, a < 2^20: the error of the reciprocal and the product is far below the distance
// of (a + 1/2) / b from a whole number.
__device__ __forceinline__ unsigned small_divide(unsigned a, unsigned b)
{
    return __builtin_amdgcn_readfirstlane((unsigned)(((float)a + 0.5f) * __builtin_amdgcn_rcpf((float)b)));
}

// Split-K tickets: one per 128-byte line (atomics on one line are served one after the other).
constexpr int TICKET_STRIDE = 32;

// MT: 16-row tiles of x (M <= 16*MT).  NW: 64-column strips per workgroup.
// KSPG: k-steps (of 32) per chunk; a quantisation group is cpg chunks (cpg = 1 unless the
// group is a multiple of 128 above 128).
// KW: waves per strip and chunk.  With KW = 2 a strip's two waves share every chunk, each taking
// half of its k-steps, and add their sums through LDS at the end: two waves per SIMD, whose
// instructions the hardware interleaves, where a launch has only one workgroup per compute
// unit and a single wave's dependent vector instructions would leave issue slots empty.
// KP: chunks per iteration.  With KP = 2 the workgroup has twice the waves and takes two
// consecutive chunks per iteration, one per half of its waves (same purpose as KW = 2, without
// making a wave's share of a chunk smaller); the halves add up through LDS like KW's.
// GS: k-steps of a chunk that belong to one quantisation group: KSPG, or two and one where a chunk of
// four k-steps holds two groups of 64 or four of 32 (cpg is 1 then).
// RB: a grid of row blocks (z) of 16 MT rows, as many calls next to each other (calls of more than 64 rows).
// SAME: workgroups are renumbered such that the K parts of a tile run on the same XCD (except at the ends of an
// XCD's run), as they do by themselves where the tiles are a multiple of 8.  The hand-over is faster there: 4096->6912
// at 64 rows (54 tiles, 4 parts) 17.9 -> 14.4 us, 4096->1792 at 24 rows 10.4 -> 9.2; 4, 6 and 9 % in the mean of odd tile
// counts at 17 to 32, 33 to 48 and 49 to 64 rows, nothing up to 16.  A variant, not a branch: the
// arithmetic before the first load costs 0.1 us.
template <int MT, int NW, int KSPG, int KW, int KP, int GS, bool RB = false, bool SAME = false>
__global__ void __launch_bounds__(NW * KW * KP * 64) __attribute__((amdgpu_waves_per_eu(KW * KP >= 2 ? 2 : (MT == 1 && NW >= 4 && KSPG < 4 * GS ? 3 : 1))))
w4a16_decode_kernel(int M, int N, int K, int cpg, const h16 *__restrict__ x, const uint32_t *__restrict__ packed,
                    const h16 *__restrict__ scales, const uint8_t *__restrict__ zeros, h16 *__restrict__ y,
                    Workspace ws, int epi)
{
    constexpr int D = SQP_DEPTH_OF(MT, KP);  // register stages of packed weights
    constexpr int XD = D;                  // LDS slots of activations
    constexpr int P = D - 1;               // chunks in flight ahead of the one being consumed
    constexpr int REGS = MT * 4 * 4;       // fp32 accumulator registers per lane
    constexpr int BN = 64 * NW;
    // One chunk of x in LDS: MT*16 rows of KSPG*64 bytes, stored as 1 KB blocks, one per
    // direct load instruction: a block holds 16/KSPG rows, PP = 4*KSPG 16-byte pieces each.
    constexpr int PP = 4 * KSPG;
    constexpr int RPB = 16 / KSPG;         // rows per block
    constexpr int CBLOCKS = MT * KSPG;     // blocks per chunk
    constexpr int XBLOCKS = CBLOCKS * KP;  // blocks per iteration (KP consecutive chunks)
    constexpr int XSTAGE = XBLOCKS * 1024;
    constexpr int WAVES = NW * KW * KP;
    constexpr int KS = KSPG / KW;                // k-steps of a chunk this wave takes
    static_assert(KS * KW == KSPG, "k-steps divide among a strip's waves");
    constexpr int OX = (XBLOCKS + WAVES - 1) / WAVES;  // direct loads per wave per chunk (at most)
    // When the blocks do not divide evenly among the waves, waves XREM and above copy one block
    // fewer (none, where a chunk has fewer blocks than the workgroup has waves): every block is
    // fetched exactly once per workgroup, and such a wave waits on a count of its own.
    constexpr int XREM = XBLOCKS % WAVES;
    constexpr int GPC = KSPG / GS;               // groups per chunk
    constexpr int NQ = KS > GS ? KS / GS : 1;    // groups in this wave's share of a chunk
    constexpr int SQ = KS / NQ;                  // k-steps of one group there
    constexpr int OW = KS + 2 * NQ;              // weight-side loads per wave per chunk
    // With three and four row tiles the per-chunk scaling of 48 or 64 accumulator registers costs more
    // vector work than multiplying the unpacked weights by the step (4 packed multiplies per word, as
    // in the tiled kernel), so those variants accumulate fp16(w_hat) products directly: 33 to 64 rows
    // give the products of the rounded weight whichever variant runs.
    constexpr bool SCALED_B = MT >= 3;
    static_assert((P - 1) * (OX + OW) < 64, "vmcnt field");
    constexpr int EXCHANGE = (KW * KP - 1) * NW * REGS * 256;  // bytes of the sums a strip's waves exchange at the end
    __shared__ __attribute__((aligned(1024))) unsigned char xring[XD * XSTAGE > EXCHANGE ? XD * XSTAGE : EXCHANGE];
    static_assert(sizeof(xring) + 16 <= 160 * 1024, "LDS of a workgroup");
    __shared__ unsigned ticket_s;

    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);    // wave-uniform, kept scalar
    const int wave = wv % NW, kh = (wv / NW) % KW, ph = wv / (NW * KW);   // strip, which k-steps of a chunk, which chunk of an iteration
    const int lc = lane & 15, lk = lane >> 4;
    const int split = gridDim.y;
    int col = blockIdx.x, sidx = blockIdx.y, block = RB ? blockIdx.z : 0;
    if constexpr (SAME) {
        // Workgroups are dealt to the 8 XCDs in turn: each takes one run of (column tile, row block, part).
        const unsigned blocks = RB ? gridDim.z : 1u, all = gridDim.x * split * blocks;
        const unsigned id = blockIdx.x + gridDim.x * (blockIdx.y + split * (RB ? blockIdx.z : 0u)), xcd = id & 7u, more = all & 7u;
        const unsigned p = xcd * (all >> 3) + (xcd < more ? xcd : more) + (id >> 3), u = small_divide(p, split);
        sidx = p - u * split;
        col = RB ? small_divide(u, blocks) : u;
        block = u - col * blocks;
    }
    const int n0 = col * BN + wave * 64;
    const int tile = block * gridDim.x + col;  // of the partial tiles and tickets
    if constexpr (RB) {
        x += (size_t)block * (16 * MT) * K;
        y += (size_t)block * (16 * MT) * (epi == 0 ? N : N >> 1);
        M -= block * (16 * MT);
        M = M < 16 * MT ? M : 16 * MT;
    }
    const int chunks = K / (32 * KSPG);
    // this workgroup's chunk range (all waves walk it together)
    const int g0 = (int)((long)chunks * sidx / split), g1 = (int)((long)chunks * (sidx + 1) / split);

    // lanes past the last column read column 0 instead; their results are never stored
    int ncol = n0 + 4 * lc;
    if (ncol >= N) ncol = 0;

    f32x4 acc[MT][4];
#pragma unroll
    for (int mt = 0; mt < MT; mt++)
#pragma unroll
        for (int t = 0; t < 4; t++) acc[mt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    const UnpackConsts uc = unpack_consts();

    struct Stage {
        u32x4 w[KS];
        u32x2 sc[NQ];     // per group: 4 fp16 steps
        uint32_t zr[NQ];  // 4 zero points, one byte each
    };

    // Weight-side addresses are a scalar base (advanced on the scalar unit) plus a per-lane
    // 32-bit offset that never changes, so the loads cost no vector arithmetic.  The loads are
    // written in assembly so that this kernel, not the compiler, decides when to wait for
    // them: a stage must not be read before `landed` below.  They carry the non-temporal hint:
    // every weight byte is read once per launch, and a plain streaming probe reads 12-15 % faster
    // with it on this chip (the kernel gains about 2 %).  Row blocks read it once each and go without
    // (5 % in the mean of 45 shapes, up to 15).
    // A wave issues one instruction every four to five cycles at best, scalar ones among them, so the loop keeps its
    // scalar work short (25 instructions per iteration where pointers clamped at the end of the range, 64-bit adds
    // per row and a mask formed in a vector register took 70): one base per stream, stepped by a constant, with the rows of
    // an iteration in the lanes' offsets; past the range the bases run on and only the execution mask tells.
    const long wstep1 = (long)N * 16;                            // one k-step: 4 packed rows, in bytes
    // An iteration covers KP consecutive chunks; this wave's are g0 + ph, g0 + ph + KP, ...  (with
    // KP = 2 and an odd range the second half of the waves has one chunk fewer; a wave without
    // any chunk points at g0 and never computes).  The activations are fetched per iteration
    // for all KP chunks by all waves together.
    const int nsup = (g1 - g0 + KP - 1) / KP;                    // iterations of this workgroup
    const int nown = g0 + ph < g1 ? (g1 - g0 - ph + KP - 1) / KP : 0;  // and of this wave
    const int cs = nown > 0 ? g0 + ph : g0;                      // this wave's first chunk
    const unsigned char *wq = reinterpret_cast<const unsigned char *>(packed) + ((long)cs * KSPG + kh * KS) * wstep1;
    // first parameter row of this wave: chunk / cpg, or (chunks of several groups) chunk * gpc + its share
    const long prow = GPC > 1 ? (long)cs * GPC + kh * KS / GS : (long)(cs / cpg);
    const unsigned char *sq = reinterpret_cast<const unsigned char *>(scales) + prow * N * 2;
    const unsigned char *zq = zeros + prow * N;
    int kin = cs % cpg;                                          // position of the chunk being issued in its group
    uint32_t voff_w[KS], voff_s[NQ], voff_z[NQ];                 // rows of a wave's share of a chunk
#pragma unroll
    for (int ks = 0; ks < KS; ks++) voff_w[ks] = (uint32_t)((lk + 4 * ks) * N + ncol) * 4u;
#pragma unroll
    for (int q = 0; q < NQ; q++) {
        voff_s[q] = (uint32_t)(q * N + ncol) * 2u;
        voff_z[q] = (uint32_t)(q * N + ncol);
    }
    // `i` (wave-uniform) is the wave's iteration that the loads are for; look-ahead loads past its last one
    // are issued with an empty execution mask, so they fetch nothing (with the streaming
    // hint their lines would not be cache hits) and write no register, but still take their
    // place in the in-order load queue, which keeps the wait counts below the same for every
    // iteration.  Mask change, loads and mask restore are one asm statement, so the compiler can
    // place nothing of its own under the changed mask.
    auto issue_w = [&](Stage &s, int i) {
        uint64_t saved;
#define SQP_MASKED(LOADS) "s_mov_b64 %[sv], exec\n\ts_cmp_lt_i32 %[i], %[n]\n\ts_cselect_b64 exec, exec, 0\n\t" LOADS "s_mov_b64 exec, %[sv]"
#define SQP_W(I, HINT) "global_load_dwordx4 %[w" #I "], %[vw" #I "], %[b]" HINT "\n\t"
#define SQP_Q(I, HINT) "global_load_dwordx2 %[sc" #I "], %[vs" #I "], %[sb]" HINT "\n\tglobal_load_dword %[zr" #I "], %[vz" #I "], %[zb]" HINT "\n\t"
#define SQP_OUT_W(I) [w##I] "=&v"(s.w[I])
#define SQP_OUT_Q(I) [sc##I] "=&v"(s.sc[I]), [zr##I] "=&v"(s.zr[I])
#define SQP_IN_W(I) [vw##I] "v"(voff_w[I])
#define SQP_IN_Q(I) [vs##I] "v"(voff_s[I]), [vz##I] "v"(voff_z[I])
#define SQP_BASES [i] "s"(i), [n] "s"(nown), [b] "s"(wq), [sb] "s"(sq), [zb] "s"(zq)
        if constexpr (KS == 4 && NQ == 1) {
            asm volatile(SQP_MASKED(SQP_W(0, " nt") SQP_W(1, " nt") SQP_W(2, " nt") SQP_W(3, " nt") SQP_Q(0, " nt"))
                         : SQP_OUT_W(0), SQP_OUT_W(1), SQP_OUT_W(2), SQP_OUT_W(3), SQP_OUT_Q(0), [sv] "=&s"(saved)
                         : SQP_IN_W(0), SQP_IN_W(1), SQP_IN_W(2), SQP_IN_W(3), SQP_IN_Q(0), SQP_BASES
                         : "memory", "scc");
        } else if constexpr (KS == 4 && NQ == 2) {
            asm volatile(SQP_MASKED(SQP_W(0, " nt") SQP_W(1, " nt") SQP_W(2, " nt") SQP_W(3, " nt") SQP_Q(0, " nt") SQP_Q(1, " nt"))
                         : SQP_OUT_W(0), SQP_OUT_W(1), SQP_OUT_W(2), SQP_OUT_W(3), SQP_OUT_Q(0), SQP_OUT_Q(1), [sv] "=&s"(saved)
                         : SQP_IN_W(0), SQP_IN_W(1), SQP_IN_W(2), SQP_IN_W(3), SQP_IN_Q(0), SQP_IN_Q(1), SQP_BASES
                         : "memory", "scc");
        } else if constexpr (KS == 4 && NQ == 4) {
            asm volatile(SQP_MASKED(SQP_W(0, " nt") SQP_W(1, " nt") SQP_W(2, " nt") SQP_W(3, " nt") SQP_Q(0, " nt") SQP_Q(1, " nt") SQP_Q(2, " nt")
                                        SQP_Q(3, " nt"))
                         : SQP_OUT_W(0), SQP_OUT_W(1), SQP_OUT_W(2), SQP_OUT_W(3), SQP_OUT_Q(0), SQP_OUT_Q(1), SQP_OUT_Q(2), SQP_OUT_Q(3),
                           [sv] "=&s"(saved)
                         : SQP_IN_W(0), SQP_IN_W(1), SQP_IN_W(2), SQP_IN_W(3), SQP_IN_Q(0), SQP_IN_Q(1), SQP_IN_Q(2), SQP_IN_Q(3), SQP_BASES
                         : "memory", "scc");
        } else if constexpr (KS == 2 && NQ == 1) {
#define SQP_ISSUE(HINT)                                                                                                    \
    asm volatile(SQP_MASKED(SQP_W(0, HINT) SQP_W(1, HINT) SQP_Q(0, HINT))                                                  \
                 : SQP_OUT_W(0), SQP_OUT_W(1), SQP_OUT_Q(0), [sv] "=&s"(saved)                                             \
                 : SQP_IN_W(0), SQP_IN_W(1), SQP_IN_Q(0), SQP_BASES                                                        \
                 : "memory", "scc")
            if constexpr (RB) SQP_ISSUE("");
            else SQP_ISSUE(" nt");
#undef SQP_ISSUE
        } else if constexpr (KS == 2 && NQ == 2) {
#define SQP_ISSUE(HINT)                                                                                                    \
    asm volatile(SQP_MASKED(SQP_W(0, HINT) SQP_W(1, HINT) SQP_Q(0, HINT) SQP_Q(1, HINT))                                   \
                 : SQP_OUT_W(0), SQP_OUT_W(1), SQP_OUT_Q(0), SQP_OUT_Q(1), [sv] "=&s"(saved)                               \
                 : SQP_IN_W(0), SQP_IN_W(1), SQP_IN_Q(0), SQP_IN_Q(1), SQP_BASES                                           \
                 : "memory", "scc")
            if constexpr (RB) SQP_ISSUE("");
            else SQP_ISSUE(" nt");
#undef SQP_ISSUE
        } else if constexpr (KS == 1 && NQ == 1) {
            asm volatile(SQP_MASKED(SQP_W(0, " nt") SQP_Q(0, " nt"))
                         : SQP_OUT_W(0), SQP_OUT_Q(0), [sv] "=&s"(saved)
                         : SQP_IN_W(0), SQP_IN_Q(0), SQP_BASES
                         : "memory", "scc");
        } else {
            static_assert(KS == 0, "k-steps and groups per wave and chunk");
        }
#undef SQP_MASKED
#undef SQP_W
#undef SQP_Q
#undef SQP_OUT_W
#undef SQP_OUT_Q
#undef SQP_IN_W
#undef SQP_IN_Q
#undef SQP_BASES
    };
    // wait until at most `after` loads are outstanding, then tie the stage's registers to the
    // wait so that no use of them is scheduled ahead of it
    const bool x_full = XREM == 0 || wv < XREM;  // wave-uniform: this wave issues all OX direct loads per chunk
    auto landed = [&](Stage &s) {
        if (x_full) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((P - 1) * (OX + OW)) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" ::"n"((P - 1) * (OX - 1 + OW)) : "memory");
#pragma unroll
        for (int ks = 0; ks < KS; ks++) asm volatile("" : "+v"(s.w[ks]));
#pragma unroll
        for (int q = 0; q < NQ; q++) {
            asm volatile("" : "+v"(s.sc[q]));
            asm volatile("" : "+v"(s.zr[q]));
        }
    };

    // Activations: wave w copies blocks w, w+NW, ... of the chunk straight into LDS.  Lane i
    // of a block handles row i / PP of the block and fetches piece (i % PP) ^ (row % PP) of
    // that row, so that a row's pieces (whole 128-byte lines) come from adjacent lanes, while
    // in LDS (where the hardware puts lane i at byte 16*i of the block) the pieces the 16
    // rows need for one k-step fall into 16 different bank groups.
    const int xrr = lane / PP, xpp = lane % PP;
    uint32_t xoff[OX];  // per-lane byte offset into x of each block this wave copies
#pragma unroll
    for (int i = 0; i < OX; i++) {
        const int b = ((wv + i * WAVES) % XBLOCKS) % CBLOCKS;   // block within its chunk
        const int row = b * RPB + xrr;
        const int rowc = row < M ? row : M - 1;
        xoff[i] = (uint32_t)rowc * (uint32_t)K * 2u + (uint32_t)((xpp ^ (row % PP)) * 16);
    }
    // Past the workgroup's range (look-ahead, the second chunk of an odd range's last iteration) its last chunk is fetched
    // again: cache hits, from which nothing is computed.
    const uint32_t xmost = (uint32_t)(g1 - 1) * (64 * KSPG);
    uint32_t xat = (uint32_t)g0 * (64 * KSPG);                   // byte offset in a row of the iteration whose activations are being issued
    auto issue_x = [&](int slot) {
#pragma unroll
        for (int i = 0; i < OX; i++) {
            if (i + 1 == OX && !x_full) break;
            const int b = (wv + i * WAVES) % XBLOCKS;
            // block b belongs to chunk b / CBLOCKS of the iteration
            const uint32_t at = KP > 1 ? xat + (uint32_t)(b / CBLOCKS) * (64 * KSPG) : xat;
            copy16_to_lds(x, (uint32_t)M * (uint32_t)K * 2u, xoff[i], at < xmost ? at : xmost, xring + slot * XSTAGE + b * 1024);
        }
    };
    // LDS byte address of this lane's A fragment (row lc of m-tile mt) in slot 0, piece 0
    uint32_t xrd[MT];
#pragma unroll
    for (int mt = 0; mt < MT; mt++) {
        const int row = mt * 16 + lc;
        xrd[mt] = (uint32_t)(size_t)xring + (uint32_t)(ph * CBLOCKS * 1024 + (row / RPB) * 1024 + (row % RPB) * PP * 16);
    }
    const int xsw = lc % PP;  // the row's swizzle (16 % PP == 0, so mt does not matter)

    auto compute = [&](const Stage &s, int slot) {
        f32x4 accg[MT][4];
        auto clear_g = [&]() {
#pragma unroll
            for (int mt = 0; mt < MT; mt++)
#pragma unroll
                for (int t = 0; t < 4; t++) accg[mt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
        };
        clear_g();
        h16x2 neg_hi[NQ][4], neg_lo[NQ][4], delta2[NQ][4];
        float delta[NQ][4];
#pragma unroll
        for (int q = 0; q < NQ; q++)
#pragma unroll
            for (int c = 0; c < 4; c++) {
                neg_hi[q][c] = neg_hi_at(s.zr[q], c);
                neg_lo[q][c] = neg_lo_at(s.zr[q] << 4, c);
                const h16x2 sv = __builtin_bit_cast(h16x2, (uint32_t)s.sc[q][c >> 1]);
                const h16 d16 = (c & 1) ? sv.y : sv.x;
                delta[q][c] = (float)d16;
                delta2[q][c] = h16x2{d16, d16};
            }
        // the sums of group q times its steps join the running sums
        auto scale_g = [&](int q) {
#pragma unroll
            for (int mt = 0; mt < MT; mt++)
#pragma unroll
                for (int t = 0; t < 4; t++)
#pragma unroll
                    for (int r = 0; r < 4; r++) acc[mt][t][r] = fmaf(delta[q][t], accg[mt][t][r], acc[mt][t][r]);
        };
        // The A fragments come out of the LDS ring with reads written in assembly: the
        // compiler cannot tell which ring slot a direct global->LDS load filled and would wait
        // for every outstanding load; the caller has already waited for this slot.
        auto read_x = [&](u32x4 *dst, int ks) {
#pragma unroll
            for (int mt = 0; mt < MT; mt++) {
                const uint32_t a = xrd[mt] + (uint32_t)(slot * XSTAGE) + (uint32_t)((((kh * KS + ks) * 4 + lk) ^ xsw) * 16);
                asm volatile("ds_read_b128 %0, %1" : "=&v"(dst[mt]) : "v"(a) : "memory");
            }
        };
        auto wait_x = [&](u32x4 *dst, int n) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int i = 0; i < n; i++) asm volatile("" : "+v"(dst[i]));  // no use ahead of the wait
        };
        // One word (8 k of a column per lane) after the other: a word is unpacked between the matrix instructions of the word
        // before it, and so is what is left of a k-step's activations to be permuted (the scheduler is
        // kept to that).  The first word needs no activations and is unpacked while they come from LDS; with one row tile
        // all of the wave's fragments are read in one batch, with more those of the next k-step while this one's are used.
        auto unpacked = [&](int i) {
            const int ks = i >> 2, c = i & 3, q = ks / SQ;
            if constexpr (SCALED_B) return dequant_word_scaled(s.w[ks][c], neg_hi[q][c], neg_lo[q][c], delta2[q][c], uc);
            else return dequant_word(s.w[ks][c], neg_hi[q][c], neg_lo[q][c], uc);
        };
        constexpr int XA = MT == 1 ? KS : 2;   // fragment sets
        constexpr int UNPACK = SCALED_B ? 13 : 9;
        u32x4 xa[XA][MT];
#pragma unroll
        for (int ks = 0; ks < (MT == 1 ? KS : 1); ks++) read_x(xa[ks], ks);
        h16x8 w = unpacked(0), a[MT];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < (MT == 1 ? KS : 1); ks++) wait_x(xa[ks], MT);
#pragma unroll
        for (int mt = 0; mt < MT; mt++) a[mt] = permute_x(xa[0][mt]);
#pragma unroll
        for (int i = 0; i < 4 * KS; i++) {
            const int ks = i >> 2, c = i & 3;
            if (MT > 1 && c == 0 && ks + 1 < KS) read_x(xa[(ks + 1) % XA], ks + 1);
            if (MT > 1 && c == 3 && ks + 1 < KS) wait_x(xa[(ks + 1) % XA], MT);
            const h16x8 cur = w;
            h16x8 an[MT];
            const bool turn = c == 3 && ks + 1 < KS;   // the next k-step's activations go with this word
            if (i + 1 < 4 * KS) w = unpacked(i + 1);
            if (turn) {
#pragma unroll
                for (int mt = 0; mt < MT; mt++) an[mt] = permute_x(xa[(ks + 1) % XA][mt]);
            }
#pragma unroll
            for (int mt = 0; mt < MT; mt++) {
                if constexpr (SCALED_B) acc[mt][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[mt], cur, acc[mt][c], 0, 0, 0);
                else accg[mt][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[mt], cur, accg[mt][c], 0, 0, 0);
            }
#pragma unroll
            for (int mt = 0; mt < MT; mt++) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                 // 1 MFMA
                if (turn) __builtin_amdgcn_sched_group_barrier(0x002, (UNPACK + 5 * MT - 1) / MT, 0);  // VALU
                else __builtin_amdgcn_sched_group_barrier(0x002, (UNPACK + MT - 1) / MT, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (turn) {
#pragma unroll
                for (int mt = 0; mt < MT; mt++) a[mt] = an[mt];
            }
            if constexpr (!SCALED_B)
                if (c == 3 && ks % SQ == SQ - 1) {
                    scale_g(ks / SQ);
                    if (ks + 1 < KS) clear_g();
                }
        }
    };

    // Software pipeline over the chunk range, P = D - 1 chunks ahead.  Iteration g: wait for
    // everything issued up to iteration g-P (weights and this wave's part of x of chunk g),
    // meet the other waves (now all of x(g) is in LDS and nobody reads the slot of chunk g-1 any
    // more), issue x(g+P) and the weights of chunk g+P into that slot and the stage just freed
    // (stage index static: the loop is unrolled by D), consume chunk g.  The pipeline is primed
    // by issuing chunks g0 .. g0+P-1.
    // The loading side of the loop body is free of branches: the chunk count is rounded up to a
    // multiple of D; loads past the range point at the range's last chunk (the activations: cache
    // hits) or are issued with an empty execution mask (the weight side); the arithmetic of such
    // padded iterations is skipped.  Every iteration of a wave thus issues the same number of
    // loads (OX + OW, or one fewer on the waves that copy one block less), and since loads
    // complete in issue order "at most P-1 iterations' worth of loads outstanding" means all but
    // the last P-1 iterations' have landed.
    auto advance = [&]() {
        wq += KP * KSPG * wstep1;
        if constexpr (GPC > 1) {  // several groups per chunk
            sq += (long)KP * GPC * N * 2;
            zq += (long)KP * GPC * N;
        } else if constexpr (KP == 1) {
            const bool wrap = ++kin == cpg;
            kin = wrap ? 0 : kin;
            sq += wrap ? (long)N * 2 : 0;
            zq += wrap ? (long)N : 0;
        } else {  // launched only with one chunk per group (cpg == 1)
            sq += (long)KP * N * 2;
            zq += (long)KP * N;
        }
        xat += KP * 64 * KSPG;
    };
    Stage st[D];
#pragma unroll
    for (int j = 0; j < P; j++) {
        issue_x(j);
        issue_w(st[j], j);
        advance();
    }
    const int nblk = (nsup + D - 1) / D;
    for (int b = 0; b < nblk; b++) {
#pragma unroll
        for (int d = 0; d < D; d++) {
            const int it = b * D + d;             // iteration (ring slot d); this wave's chunk in it: cs + it * KP
            landed(st[d]);
            asm volatile("s_barrier" ::: "memory");
            issue_x((d + P) % XD);
            issue_w(st[(d + P) % D], it + P);
            advance();
            if (it < nown) compute(st[d], d);     // padded iterations only keep the load counts in step
        }
    }
    // Look-ahead loads may still be in flight here (a range shorter than the pipeline issues
    // real loads it never consumes).  Their destination registers are dead by now as far as the
    // compiler can tell, but the hardware still writes them when the data arrives: `drain` waits
    // for everything outstanding and its empty uses keep every stage allocated until then, so
    // that nothing else is placed in those registers while a load is in flight.  It runs after the epilogue's stores have been issued (they only read the
    // accumulators), so that one wait covers both.
    auto drain = [&]() {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
        for (int j = 0; j < D; j++) {
#pragma unroll
            for (int ks = 0; ks < KS; ks++) asm volatile("" ::"v"(st[j].w[ks]));
#pragma unroll
            for (int q = 0; q < NQ; q++) {
                asm volatile("" ::"v"(st[j].sc[q]));
                asm volatile("" ::"v"(st[j].zr[q]));
            }
        }
    };

    // ---- epilogue.  Accumulator tile t, register r of a lane: row mt*16 + 4*(lane/16) + r,
    // column n0 + 4*(lane%16) + t.
    const int nout = n0 + 4 * lc;
    drain();
    constexpr int SW = KW * KP;            // waves per strip
    const int sid = kh + KW * ph;          // this wave among them
    // Row tile mt of a strip is finished by wave mt % SW of it: the others hand theirs over through
    // LDS (the activation ring is idle once every wave has passed the barrier), the sums are added
    // in wave order.
    auto owns = [&](int mt) { return SW == 1 || sid == mt % SW; };  // wave-uniform
    if constexpr (SW > 1) {
        static_assert((SW - 1) * NW * MT * 4096 == EXCHANGE, "the exchange fits the LDS array");
        f32x4 *ex = reinterpret_cast<f32x4 *>(xring) + (size_t)wave * (MT * (SW - 1) * 256) + lane;
        __syncthreads();
#pragma unroll
        for (int mt = 0; mt < MT; mt++)
            if (!owns(mt)) {
                const int from = sid < mt % SW ? sid : sid - 1;
#pragma unroll
                for (int t = 0; t < 4; t++) ex[(mt * (SW - 1) + from) * 256 + t * 64] = acc[mt][t];
            }
        __syncthreads();
#pragma unroll
        for (int mt = 0; mt < MT; mt++)
            if (owns(mt)) {
                const int own = mt % SW;
#pragma unroll
                for (int t = 0; t < 4; t++) {
                    const f32x4 mine = acc[mt][t];
                    f32x4 v = own == 0 ? mine : ex[mt * (SW - 1) * 256 + t * 64];
#pragma unroll
                    for (int w = 1; w < SW; w++) v += w == own ? mine : ex[(mt * (SW - 1) + (w < own ? w : w - 1)) * 256 + t * 64];
                    acc[mt][t] = v;
                }
            }
    }
    if (split == 1) {
        if (nout < N) {
#pragma unroll
            for (int mt = 0; mt < MT; mt++)
                if (owns(mt)) {
#pragma unroll
                    for (int r = 0; r < 4; r++) {
                        const int m = mt * 16 + 4 * lk + r;
                        if (m < M) store_row4(y, m, N, nout, epi, acc[mt][0][r], acc[mt][1][r], acc[mt][2][r], acc[mt][3][r]);
                    }
                }
        }
        return;
    }

    // ---- cross-workgroup: the last arrival adds the SPLIT partial tiles in split order.
    // Partials travel as device-scope (sc1) 16-byte stores and loads, written through and read
    // past the per-XCD L2, so no cache-wide write-back or invalidate is needed: each thread
    // waits for its own stores to complete, the barrier collects the workgroup, and only then
    // is the ticket taken.  Layout: [tile][split][wave][Q][lane][4] floats (each instruction
    // moves 1 KB contiguous per wave).
    {
        float *mine = ws.partial + (((size_t)tile * split + sidx) * NW + wave) * (64 * REGS) + lane * 4;
#pragma unroll
        for (int mt = 0; mt < MT; mt++)
            if (owns(mt) && mt * 16 + 4 * lk < M) {  // lanes whose four rows are all past M have nothing to hand over
#pragma unroll
                for (int t = 0; t < 4; t++)
                    // (the s_nop: a store of more than 8 bytes reads its data registers up to two wait
                    // states after issue, and the compiler, which does not look inside asm statements,
                    // may reuse them for the next copy out of the accumulator registers right away)
                    asm volatile("global_store_dwordx4 %0, %1, off offset:%2 sc1\n\ts_nop 1" ::"v"(mine + mt * 1024), "v"(acc[mt][t]), "n"(t * 1024) : "memory");
            }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __syncthreads();
    if (threadIdx.x == 0) ticket_s = __hip_atomic_fetch_add(&ws.tickets[tile * TICKET_STRIDE], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (ticket_s != (unsigned)(split - 1)) return;
    {
        const float *base = ws.partial + (((size_t)tile * split) * NW + wave) * (64 * REGS) + lane * 4;
        const size_t sstride = (size_t)NW * 64 * REGS;
        // RM row tiles at once: all of them where a strip has one wave, else the owned ones in turn
        constexpr int RM = SW == 1 ? MT : 1, Q = 4 * RM;  // Q 16-byte pieces per lane and K part
        // K parts fetched per round trip: what fits the register budget without spilling (the
        // variants with two waves per SIMD have 256 registers, so a split of 8 takes one round trip)
        constexpr int SB = RM == 1 && SW == 1 ? 6 : 8 / RM;
#pragma unroll
        for (int m1 = 0; m1 < MT; m1 += RM) {
            if (!owns(m1)) continue;
            // Lanes whose four rows are all past M stored nothing and their sums are never written:
            // they re-read the first 16 lanes' pieces (the same cache lines) instead of lines of
            // their own, which for M <= 4 cuts the bytes the last arrival pulls in to a quarter.
            // (The loads stay unconditional: every lane's destination registers must be written by
            // exactly these instructions for the wait below to cover them.  A row tile wholly past M
            // has no stored piece at all; its reads stay in the buffer and its sums are not used.)
            int dead[RM];
#pragma unroll
            for (int i = 0; i < RM; i++) dead[i] = (m1 + i) * 16 + 4 * lk < M ? 0 : -64 * lk;
            f32x4 sum[Q];
#pragma unroll
            for (int q = 0; q < Q; q++) sum[q] = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int s0 = 0; s0 < split; s0 += SB) {
                f32x4 tmp[SB][Q];
#pragma unroll
                for (int j = 0; j < SB; j++)
                    if (s0 + j < split) {
#pragma unroll
                        for (int q = 0; q < Q; q++)
                            asm volatile("global_load_dwordx4 %0, %1, off sc1" : "=v"(tmp[j][q]) : "v"(base + (size_t)(s0 + j) * sstride + (m1 * 4 + q) * 256 + dead[q / 4]) : "memory");
                    }
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
                for (int j = 0; j < SB; j++)
#pragma unroll
                    for (int q = 0; q < Q; q++) asm volatile("" : "+v"(tmp[j][q]));
#pragma unroll
                for (int j = 0; j < SB; j++)
                    if (s0 + j < split) {
#pragma unroll
                        for (int q = 0; q < Q; q++) sum[q] += tmp[j][q];
                    }
            }
            if (nout < N) {
#pragma unroll
                for (int i = 0; i < RM; i++)
#pragma unroll
                    for (int r = 0; r < 4; r++) {
                        const int m = (m1 + i) * 16 + 4 * lk + r;
                        if (m < M) store_row4(y, m, N, nout, epi, sum[i * 4 + 0][r], sum[i * 4 + 1][r], sum[i * 4 + 2][r], sum[i * 4 + 3][r]);
                    }
            }
        }
    }
    if (threadIdx.x == 0)  // ready for the next launch on this stream
        __hip_atomic_store(&ws.tickets[tile * TICKET_STRIDE], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------- launch

// Whether a launch takes the SAME variant (see the kernel; its division holds below 2^20 workgroups).
inline bool parts_together(int tiles, int split, int blocks) { return split > 1 && tiles % 8 != 0 && (long)tiles * split * blocks < (1 << 20); }

template <int MT, int NW, int KSPG, int KW, int KP, int GS>
int launch_variant(int M, int N, int K, int cpg, int tiles, int split, const h16 *x, const uint32_t *packed, const h16 *scales,
                   const uint8_t *zeros, h16 *y, int epi, const Workspace &ws, hipStream_t st)
{
    if constexpr (MT >= 2 && NW == 2 && KW == 2)
        if (parts_together(tiles, split, 1)) {
            w4a16_decode_kernel<MT, NW, KSPG, KW, KP, GS, false, true><<<dim3(tiles, split), NW * KW * KP * 64, 0, st>>>(
                M, N, K, cpg, x, packed, scales, zeros, y, ws, epi);
            return sqp_launch_status();
        }
    w4a16_decode_kernel<MT, NW, KSPG, KW, KP, GS><<<dim3(tiles, split), NW * KW * KP * 64, 0, st>>>(
        M, N, K, cpg, x, packed, scales, zeros, y, ws, epi);
    return sqp_launch_status();
}

// GS: k-steps of a chunk that belong to one group (KSPG, or fewer where a chunk holds several groups).
template <int MT, int NW, int KSPG, int GS>
int launch(int M, int N, int K, int cpg, const SqpStripPlan &plan, const h16 *x, const uint32_t *packed, const h16 *scales,
           const uint8_t *zeros, h16 *y, int epi, const SqpWorkspace &cws, hipStream_t st)
{
    constexpr int BN = 64 * NW;
    const int tiles = (N + BN - 1) / BN;
    size_t need = 0;
    const int split = sqp_strip_split(MT, NW, KSPG, 1, N, K, plan.split, &need);
    Workspace ws = {nullptr, nullptr};
    if (split > 1) {
        if (!cws.partial || !cws.tickets || need > cws.partial_bytes) return SQP_ERR_WORKSPACE;
        ws.partial = cws.partial;
        ws.tickets = cws.tickets;
    }
    if constexpr (KSPG == 4 && (NW == 2 || NW == 4)) {
        // One workgroup per compute unit: two-strip workgroups give each strip two waves (up to 32
        // rows), and both kinds take two chunks per iteration where they walk enough of them.
        int kw = plan.kw, kp = plan.kp;
        if (kw == 0) kw = NW == 2 && MT <= 2 && tiles * split <= 256 ? 2 : 1;
        if (kp == 0) kp = MT <= 2 && tiles * split <= 256 && (NW == 4 || kw == 2) && sqp_strip_two_chunks(K / 128, split) ? 2 : 1;
        if (sqp_strip_kw_hook) kw = sqp_strip_kw_hook;
        if (sqp_strip_kp_hook == 1) kp = 1;
        if (sqp_strip_kp_hook == 3) kp = 2;
        if (cpg > 1) kp = 1;  // groups of several chunks: one chunk per iteration (stepping the parameters costs 2 % otherwise)
        if constexpr (NW == 2) {
            if (kw == 2 && kp == 2) return launch_variant<MT, NW, KSPG, 2, 2, GS>(M, N, K, cpg, tiles, split, x, packed, scales, zeros, y, epi, ws, st);
            if (kw == 2) return launch_variant<MT, NW, KSPG, 2, 1, GS>(M, N, K, cpg, tiles, split, x, packed, scales, zeros, y, epi, ws, st);
        } else {
            // (several groups per chunk, or more rows: registers for two chunks' constants and sums run out,
            // and two strips are the better plan there)
            if constexpr (GS == KSPG && MT <= 2)
                if (kp == 2) return launch_variant<MT, NW, KSPG, 1, 2, GS>(M, N, K, cpg, tiles, split, x, packed, scales, zeros, y, epi, ws, st);
        }
    }
    return launch_variant<MT, NW, KSPG, 1, 1, GS>(M, N, K, cpg, tiles, split, x, packed, scales, zeros, y, epi, ws, st);
}

template <int MT, int KSPG, int GS>
int dispatch_mt(const SqpStripPlan &p, int M, int N, int K, int cpg, const h16 *x, const uint32_t *packed, const h16 *scales,
                const uint8_t *zeros, h16 *y, int epi, const SqpWorkspace &ws, hipStream_t st)
{
    if (p.nw == 2) return launch<MT, 2, KSPG, GS>(M, N, K, cpg, p, x, packed, scales, zeros, y, epi, ws, st);
    if constexpr (GS == KSPG)
        if (p.nw == 1) return launch<MT, 1, KSPG, GS>(M, N, K, cpg, p, x, packed, scales, zeros, y, epi, ws, st);
    if constexpr (GS == KSPG && MT < 3)  // eight waves of the larger variants would not fit the register file
        if (p.nw == 8) return launch<MT, 8, KSPG, GS>(M, N, K, cpg, p, x, packed, scales, zeros, y, epi, ws, st);
    return launch<MT, 4, KSPG, GS>(M, N, K, cpg, p, x, packed, scales, zeros, y, epi, ws, st);
}

}  // namespace
