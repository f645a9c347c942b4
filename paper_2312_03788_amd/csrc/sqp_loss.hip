// Quantisation loss of one linear layer, Eq. 4 of arXiv 2312.03788:
//   E = || X W - X_hat W_hat ||_F^2,   W_hat = dequantised 4-bit weights (Eq. 1),
// with X_hat = X diag(s)^-1 and the quantised W_hat of diag(s) W (Eq. 5), as the search over the
// smoothing strength alpha needs it (Sec 2.2: alpha is chosen to minimise the loss).
//
// The two products are never rounded to fp16: that would swamp their difference.  For the same reason
// they are one contraction over the concatenated inner dimension [X, X_hat] * [W; -W_hat], taken 16 k
// of the one and 16 k of the other in turn into one fp32 accumulator per output element, which
// thus stays near the difference: summed one after the other, every rounding would be relative to
// |X W| with its outlier channels (an order of magnitude more at K = 5120).  Two kernels do that:
//   loss_tile_kernel   K a multiple of 64, groups of 32 or a multiple of 64: every layer of the paper's
//                      models (loss_pair_kernel: the same for two alphas of a search at once)
//   quant_loss_kernel  any other K or group
// A workgroup owns a 128 x 128 tile, squares and sums its accumulators in fp64 and writes one
// partial; a second kernel adds the partials in a fixed order, so the result does not depend on
// scheduling.
#include "sqp_common.h"
#include "sqp_quantize_tile.h"
#include "sqp_w4_unpack.h"

namespace {

constexpr int LBM = 128, LBN = 128, LBK = 64, LPAD = 8;  // row stride 144 bytes: 16-byte reads of 32 rows spread over the banks

// ---------------------------------------------------------------- wave tiles of 64 x 64
//
// Eight waves: wave (kh, wm, wn) owns rows 64 wm .. +64 and columns 64 wn .. +64 of the tile (2 x 2
// tiles of v_mfma_f32_32x32x16_f16) for the k's of half kh of every 64-k stage; the two halves'
// sums meet in LDS.  A wave tile of 64 x 64 and not smaller, because the reads of fragments from LDS
// bound the kernel otherwise (six 16-byte reads per lane feed eight MFMAs; five feed four with 64 x 32).
// The K halves give two waves per SIMD (one unpacks while the other multiplies) without smaller tiles.
//   X, X_hat: direct global->LDS loads into a ring of three slots (rows of 128 bytes, 16-byte pieces
//     XOR-swizzled by row so that a read of 32 rows spreads over the banks).
//   W: through registers into one of two LDS buffers, transposed on the way (8 rows x 2 columns per
//     lane, v_perm_b32): fetched one stage ahead of X, written while the stage in front is multiplied.
//   W_hat: packed words straight into registers (a word is one lane's B operand).
// Two stages in flight, one barrier per stage; loads and waits in assembly as in the GEMM kernels.
// CODE: X_hat is stored with every 8 k in the order of the unpacked codes (the search does that): no
// permute here.
// Column mapping: accumulator tile t, lane l: column 64 wn + 2 (l % 32) + t (two adjacent columns
// per lane: 8-byte loads of packed words).
// What bounds it: the loads (52 KB per stage and compute unit out of L2) and the matrix cores, which
// overlap in part: 1.1 us per stage, of which the MFMAs are 0.45 (timing probes on 512 x 5120 x 5120, 92
// us complete: 74 without MFMAs, 82 without W's way, 57 without both, 90 without the unpack, 93 without
// the reads from LDS).  Measured against quant_loss_kernel: 512 x 5120 x 5120 (160 tiles) 153 -> 88 us,
// 512 x 8192 x 8192 292 -> 173, 64 x 4096 x 4096 in groups of 64 171 -> 68; rounding as there, 0.5 to 1.3
// times 2^-24 sqrt(K / 16) of a sum of 16 products.

// dequant_word_scaled with the and-ors as assembly, which the scheduler does not count among the vector instructions it
// deals out between the MFMAs but puts in front of them.  Here that is the faster place: quant_loss of 512 x 5120 x 5120
// takes 88 us with it and 94 with plain and-ors (128 x 4096 x 4096: 68 and 72), though those have 5 % fewer instructions
// (no wait states behind assembly); the strips and column slices, whose words wait for memory, are faster the other way.
struct LossConsts {
    uint32_t mask_lo = 0x000f000fu, mask_hi = 0x00f000f0u, magic_lo = 0x64006400u, magic_hi = 0x54005400u;
};
__device__ __forceinline__ h16x8 dequant_word_ahead(uint32_t w, h16x2 neg_hi, h16x2 neg_lo, h16x2 delta, const LossConsts &uc)
{
    const uint32_t w8 = w >> 8;
    uint32_t t0, t1, t2, t3;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(t0) : "v"(w), "v"(uc.mask_lo), "v"(uc.magic_lo));
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(t1) : "v"(w), "v"(uc.mask_hi), "v"(uc.magic_hi));
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(t2) : "v"(w8), "v"(uc.mask_lo), "v"(uc.magic_lo));
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(t3) : "v"(w8), "v"(uc.mask_hi), "v"(uc.magic_hi));
    u32x4 r;
    r[0] = __builtin_bit_cast(uint32_t, (__builtin_bit_cast(h16x2, t0) + neg_hi) * delta);
    r[1] = __builtin_bit_cast(uint32_t, (__builtin_bit_cast(h16x2, t1) + neg_lo) * delta);
    r[2] = __builtin_bit_cast(uint32_t, (__builtin_bit_cast(h16x2, t2) + neg_hi) * delta);
    r[3] = __builtin_bit_cast(uint32_t, (__builtin_bit_cast(h16x2, t3) + neg_lo) * delta);
    return __builtin_bit_cast(h16x8, r);
}

constexpr int SBK = 64;                       // k per stage
constexpr int SHALF = LBM * SBK * 2;          // bytes of X (and of X_hat) per stage
constexpr int SSLOT = 2 * SHALF;
constexpr int SROW = (SBK + LPAD) * 2;        // bytes per LDS row of W
constexpr int SWBUF = LBN * SROW;

// ---------------------------------------------------------------- preparation of a search's alphas

constexpr int OWN_SET = 1 << 20;               // the caller's own buffers as a set (for single losses)
struct SearchSets {                            // the prepared operands of one alpha, `stride` bytes apart
    unsigned char *base;
    size_t stride, at_scales, at_zeros, at_x;
    struct {
        uint32_t *packed;
        h16 *scales;
        uint8_t *zeros;
        h16 *x_hat;
    } own;
    // OWN: the set may be the caller's (pairs never take that one, and their kernel is spared the question)
    template <bool OWN = true> __host__ __device__ uint32_t *packed(int i) const { return OWN && i == OWN_SET ? own.packed : (uint32_t *)(base + i * stride); }
    template <bool OWN = true> __host__ __device__ h16 *scales(int i) const { return OWN && i == OWN_SET ? own.scales : (h16 *)(base + i * stride + at_scales); }
    template <bool OWN = true> __host__ __device__ uint8_t *zeros(int i) const { return OWN && i == OWN_SET ? own.zeros : base + i * stride + at_zeros; }
    template <bool OWN = true> __host__ __device__ h16 *x_hat(int i) const { return OWN && i == OWN_SET ? own.x_hat : (h16 *)(base + i * stride + at_x); }
};
struct SearchBatch {
    int set, n;                                // first set and number of alphas of the loss
    int next_set, next_n;                      // of the preparation
    const float *next_factors;                 // [next_n][K]
    int next_pieces;                           // beside single losses: of that preparation
};
constexpr int SEARCH_X_OCTS = 4096;            // 8-element pieces of x per workgroup of the preparation

// Piece `item` of the preparation of `n` alphas: weight tiles first, each for all alphas in turn (the tile then
// comes out of L2), then x.
template <int G, bool OWN>
__device__ __forceinline__ void prepare_piece(int item, int T, int N, int K, const h16 *x, const h16 *w, const SearchSets &sets, int set, int n,
                                              const float *factors, unsigned char *lds)
{
    typedef QuantizeTile<G, 512> Tile;
    const int tx = (N + 255) / 256, tiles = tx * ((K + 255) / 256);
    const int at = item / n, a = item % n;
    const float *s = factors + (size_t)a * K;
    if (at < tiles) {
        quantize_tile<G, 512, true>(at % tx, at / tx, N, K, (const uint4 *)w, s, sets.packed<OWN>(set + a), (uint16_t *)sets.scales<OWN>(set + a),
                                    sets.zeros<OWN>(set + a), *reinterpret_cast<Tile *>(lds));
        return;
    }
    const int KO = K >> 3;
    const long first = (long)(at - tiles) * SEARCH_X_OCTS, octs = (long)T * KO;
    const float4 *s4 = reinterpret_cast<const float4 *>(s);
    uint4 *out = (uint4 *)sets.x_hat<OWN>(set + a);
    for (long i = first + threadIdx.x; i < octs && i < first + SEARCH_X_OCTS; i += 512) {
        const int ko = (int)(i % KO);
        out[i] = code_order(smooth_x8(((const uint4 *)x)[i], s4[2 * ko], s4[2 * ko + 1]));
    }
}
int prepare_pieces(int T, int N, int K, int n)
{
    return n * (((N + 255) / 256) * ((K + 255) / 256) + (int)(((long)T * (K / 8) + SEARCH_X_OCTS - 1) / SEARCH_X_OCTS));
}

// PREP (0 or the group size): the workgroups behind the `losses` of the grid prepare the next alpha.
template <bool G32, bool CODE, int PREP>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
loss_tile_kernel(int M, int N, int K, int group, const h16 *__restrict__ x, const h16 *__restrict__ w,
                 const h16 *__restrict__ xh, const uint32_t *__restrict__ packed, const h16 *__restrict__ scales,
                 const uint8_t *__restrict__ zeros, double *__restrict__ partials, SearchSets sets, SearchBatch batch)
{
    constexpr int D = 3;                      // ring slots and register stages
    __shared__ __attribute__((aligned(1024))) unsigned char lds[D * SSLOT + 2 * SWBUF];
    __shared__ double red[8];
    static_assert(sizeof(lds) + sizeof(red) <= 160 * 1024, "LDS of a workgroup");
    const int tiles_x = (N + LBN - 1) / LBN, losses = tiles_x * ((M + LBM - 1) / LBM);
    if constexpr (PREP != 0) {
        static_assert(sizeof(QuantizeTile<PREP, 512>) <= sizeof(lds), "the quantiser's LDS fits the ring");
        if ((int)blockIdx.x >= losses) {
            for (int i = (int)blockIdx.x - losses; i < batch.next_pieces; i += (int)gridDim.x - losses)
                prepare_piece<PREP, true>(i, M, N, K, x, w, sets, batch.next_set, batch.next_n, batch.next_factors, lds);
            return;
        }
    }

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kh = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;
    const int l32 = lane & 31, kb = lane >> 5;
    const int m0 = (int)blockIdx.x / tiles_x * LBM, n0 = (int)blockIdx.x % tiles_x * LBN;
    const int stages = K / SBK;
    const int ncol = n0 + wn * 64 + 2 * l32;                   // this lane's two columns (N is even: both in or out)
    const bool ncol_ok = ncol < N;
    const LossConsts uc;

    f32x16 acc[2][2];
#pragma unroll
    for (int mt = 0; mt < 2; mt++)
#pragma unroll
        for (int t = 0; t < 2; t++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc[mt][t][r] = 0.f;

    struct Stage {
        u32x2 w[2];   // per k-step of 16 of this wave's half: the packed words of the lane's two columns
        uint32_t sc;  // two fp16 steps
        uint32_t zr;  // two zero points, one byte each
    };
    // Wave-uniform byte pointers, stepped per stage; past the last stage they stop and the look-ahead
    // re-reads it.  Lanes past the last column read column 0, rows past M read row M - 1: defined data
    // whose results are masked at the end.
    const int col = ncol_ok ? ncol : 0;
    const uint32_t voff_p = (uint32_t)(kb * N + col) * 4u, voff_s = (uint32_t)col * 2u, voff_z = (uint32_t)col;
    const uint32_t voff_w = n0 + 2 * lane < N ? (uint32_t)(n0 + 2 * lane) * 2u : 0u;  // W: this lane's column pair
    const long nrow = (long)N * 2;            // one row of W in bytes
    const unsigned char *pq = reinterpret_cast<const unsigned char *>(packed) + (long)kh * 8 * nrow;  // 32 k: four packed rows
    const unsigned char *xq = reinterpret_cast<const unsigned char *>(x), *hq = reinterpret_cast<const unsigned char *>(xh);
    const unsigned char *wq = reinterpret_cast<const unsigned char *>(w) + (long)wave * 8 * nrow;     // this wave's 8 rows of a stage
    const int spg = G32 ? 1 : __builtin_amdgcn_readfirstlane(group / SBK);  // stages per group (G32: two groups per stage)
    int kin = 0;                              // position of the stage being issued in its group
    int prow = G32 ? kh : 0;                  // its parameter row
    int ist = 0, wst = 0;                     // stage being issued: of X, X_hat and W_hat; of W
    // X, X_hat: wave w copies blocks w and w + 8 of the stage (a block = 8 rows x 128 bytes); lane i of a
    // block handles row i / 8 and fetches piece (i % 8) ^ ((row / 2) % 8) of it
    uint32_t xoff[2];
#pragma unroll
    for (int j = 0; j < 2; j++) {
        const int row = (wave + 8 * j) * 8 + (lane >> 3);
        const int grow = m0 + row < M ? m0 + row : M - 1;
        xoff[j] = (uint32_t)grow * (uint32_t)K * 2u + (uint32_t)(((lane & 7) ^ ((row >> 1) & 7)) * 16);
    }
    constexpr int OG = 16;                    // loads per wave and stage: X 2, X_hat 2, words 2, steps, zero points, W 8
    // A stage's loads go out in four parts, one in front of every four MFMAs of the stage in progress (in two
    // parts they hold the waves up in front of their arithmetic: 92 us against 84 on 512 x 5120 x 5120).
    auto issue_x_part = [&](Stage &st, int slot, int j) {
        unsigned char *dst = lds + slot * SSLOT + wave * 1024;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(xq + xoff[j]),
                                         (__attribute__((address_space(3))) void *)(dst + j * 8192), 16, 0, 0);
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(hq + xoff[j]),
                                         (__attribute__((address_space(3))) void *)(dst + SHALF + j * 8192), 16, 0, 0);
        if (j == 0) {
            const unsigned char *p1 = pq + 4 * nrow;
            asm volatile("global_load_dwordx2 %[w0], %[vp], %[p0]\n\t"
                         "global_load_dwordx2 %[w1], %[vp], %[p1]"
                         : [w0] "=&v"(st.w[0]), [w1] "=&v"(st.w[1])
                         : [vp] "v"(voff_p), [p0] "s"(pq), [p1] "s"(p1)
                         : "memory");
            return;
        }
        const long row = (long)__builtin_amdgcn_readfirstlane(prow) * N;
        const unsigned char *sg = reinterpret_cast<const unsigned char *>(scales) + row * 2, *zg = zeros + row;
        asm volatile("global_load_dword %[sc], %[vs], %[sg]\n\t"
                     "global_load_ushort %[zr], %[vz], %[zg]"
                     : [sc] "=&v"(st.sc), [zr] "=&v"(st.zr)
                     : [vs] "v"(voff_s), [vz] "v"(voff_z), [sg] "s"(sg), [zg] "s"(zg)
                     : "memory");
        const bool more = ist + 1 < stages;
        ist += more ? 1 : 0;
        pq += more ? 16 * nrow : 0;
        xq += more ? SBK * 2 : 0;
        hq += more ? SBK * 2 : 0;
        if constexpr (G32) {
            prow += more ? 2 : 0;
        } else {
            kin += more ? 1 : 0;
            const bool wrap = kin == spg;
            kin = wrap ? 0 : kin;
            prow += wrap ? 1 : 0;
        }
    };
    auto issue_x = [&](Stage &st, int slot) {
        issue_x_part(st, slot, 0);
        issue_x_part(st, slot, 1);
    };
    auto issue_w_part = [&](uint32_t (&r)[8], int h) {
        const unsigned char *b[4];
#pragma unroll
        for (int i = 0; i < 4; i++) b[i] = wq + (4 * h + i) * nrow;  // wave-uniform
        asm volatile("global_load_dword %[r0], %[v], %[b0]\n\t"
                     "global_load_dword %[r1], %[v], %[b1]\n\t"
                     "global_load_dword %[r2], %[v], %[b2]\n\t"
                     "global_load_dword %[r3], %[v], %[b3]"
                     : [r0] "=&v"(r[4 * h]), [r1] "=&v"(r[4 * h + 1]), [r2] "=&v"(r[4 * h + 2]), [r3] "=&v"(r[4 * h + 3])
                     : [v] "v"(voff_w), [b0] "s"(b[0]), [b1] "s"(b[1]), [b2] "s"(b[2]), [b3] "s"(b[3])
                     : "memory");
        if (h == 0) return;
        const bool more = wst + 1 < stages;
        wst += more ? 1 : 0;
        wq += more ? (long)SBK * nrow : 0;
    };
    auto issue_w = [&](uint32_t (&r)[8]) {
        issue_w_part(r, 0);
        issue_w_part(r, 1);
    };
    auto tie_w = [&](uint32_t (&r)[8]) {       // no use ahead of the wait in front
#pragma unroll
        for (int i = 0; i < 8; i++) asm volatile("" : "+v"(r[i]));
    };
    // The pair of columns of W this lane holds -> two LDS rows (column 2 c of a wave's 64 in row c, column
    // 2 c + 1 in row 32 + c), 8 k each.  Written in assembly, like every LDS access of the loop: the
    // compiler would wait for all direct loads in flight.
    const uint32_t wwr = (uint32_t)(size_t)lds + (uint32_t)(D * SSLOT + ((lane >> 5) * 64 + l32) * SROW + wave * 16);
    auto store_w = [&](const uint32_t (&r)[8], int buf) {
        u32x4 c0, c1;  // the low halves of the 8 rows; the high halves
        c0.x = __builtin_amdgcn_perm(r[1], r[0], 0x05040100u); c1.x = __builtin_amdgcn_perm(r[1], r[0], 0x07060302u);
        c0.y = __builtin_amdgcn_perm(r[3], r[2], 0x05040100u); c1.y = __builtin_amdgcn_perm(r[3], r[2], 0x07060302u);
        c0.z = __builtin_amdgcn_perm(r[5], r[4], 0x05040100u); c1.z = __builtin_amdgcn_perm(r[5], r[4], 0x07060302u);
        c0.w = __builtin_amdgcn_perm(r[7], r[6], 0x05040100u); c1.w = __builtin_amdgcn_perm(r[7], r[6], 0x07060302u);
        const uint32_t a = wwr + (uint32_t)(buf * SWBUF);
        asm volatile("ds_write_b128 %0, %1" ::"v"(a), "v"(c0) : "memory");
        asm volatile("ds_write_b128 %0, %1 offset:%2" ::"v"(a), "v"(c1), "n"(32 * SROW) : "memory");
    };

    // LDS addresses of this lane's fragments: X and X_hat (row 64 wm + l32, + 32 for the second row tile),
    // W (row 64 wn + l32, + 32 for the second column)
    const uint32_t xrd = (uint32_t)(size_t)lds + (uint32_t)((wm * 64 + l32) * 128);
    const int xkey = (l32 >> 1) & 7;
    const uint32_t wrd = (uint32_t)(size_t)lds + (uint32_t)(D * SSLOT + (wn * 64 + l32) * SROW + kh * 64 + kb * 16);

    Stage st[D];
    uint32_t wr[D][8];
    int buf = 0;                               // LDS buffer of W of the stage being consumed
    // Stage s (slot and register stage d = s % 3): its X, X_hat and W_hat, and W of stage s + 1, have landed
    // for this wave once all but the youngest group of loads have; after the barrier that holds for all
    // waves, W of stage s is in its buffer, and no wave reads the slot or the buffer of stage s - 1
    // any more, which are filled meanwhile: with W of stage s + 1 out of registers, and the loads
    // of stage s + 2 (W: s + 3, into the registers that held W of stage s).
    auto iteration = [&](Stage &cur, Stage &fill, uint32_t (&w_next)[8], uint32_t (&w_fill)[8], int slot, int fill_slot) {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(OG) : "memory");
#pragma unroll
        for (int ks = 0; ks < 2; ks++) asm volatile("" : "+v"(cur.w[ks]));
        asm volatile("" : "+v"(cur.sc));
        asm volatile("" : "+v"(cur.zr));
        tie_w(w_next);
        asm volatile("s_barrier" ::: "memory");
        u32x4 xa[2][2], xb[2][2], wb[2][2];    // fragments of X, X_hat and W: [k-step][row or column tile]
        auto read = [&](int ks) {
            const uint32_t a = xrd + (uint32_t)(slot * SSLOT) + (uint32_t)(((kh * 4 + ks * 2 + kb) ^ xkey) * 16);
            const uint32_t b = wrd + (uint32_t)(buf * SWBUF + ks * 32);
            asm volatile("ds_read_b128 %0, %1" : "=&v"(xa[ks][0]) : "v"(a) : "memory");
            asm volatile("ds_read_b128 %0, %1 offset:4096" : "=&v"(xa[ks][1]) : "v"(a) : "memory");
            asm volatile("ds_read_b128 %0, %1" : "=&v"(wb[ks][0]) : "v"(b) : "memory");
            asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(wb[ks][1]) : "v"(b), "n"(32 * SROW) : "memory");
            asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(xb[ks][0]) : "v"(a), "n"(SHALF) : "memory");
            asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(xb[ks][1]) : "v"(a), "n"(SHALF + 4096) : "memory");
        };
        read(0);
        h16x2 neg_hi[2], neg_lo[2], delta[2];
#pragma unroll
        for (int t = 0; t < 2; t++) {
            const uint32_t z = (cur.zr >> (8 * t)) & 0xffu;
            neg_hi[t] = neg_hi_of(z);
            neg_lo[t] = neg_lo_of(z);
            const uint32_t sw = cur.sc ^ 0x80008000u;  // the negated steps
            delta[t] = __builtin_bit_cast(h16x2, __builtin_amdgcn_perm(sw, sw, t ? 0x03020302u : 0x01000100u));
        }
#pragma unroll
        for (int ks = 0; ks < 2; ks++) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int i = 0; i < 2; i++) {
                asm volatile("" : "+v"(xa[ks][i]));
                asm volatile("" : "+v"(xb[ks][i]));
                asm volatile("" : "+v"(wb[ks][i]));
            }
            if (ks == 0) {
                read(1);
                issue_x_part(fill, fill_slot, 0);
            } else {
                store_w(w_next, buf ^ 1);
                issue_w_part(w_fill, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            // X W of 16 k, the words of X_hat W_hat unpacked between the MFMAs (the scheduler is told so), then
            // X_hat W_hat of the same 16 k
            h16x8 b[2], a[2];
#pragma unroll
            for (int t = 0; t < 2; t++) b[t] = dequant_word_ahead(cur.w[ks][t], neg_hi[t], neg_lo[t], delta[t], uc);
#pragma unroll
            for (int mt = 0; mt < 2; mt++) a[mt] = CODE ? __builtin_bit_cast(h16x8, xb[ks][mt]) : permute_x(xb[ks][mt]);
#pragma unroll
            for (int mt = 0; mt < 2; mt++)
#pragma unroll
                for (int t = 0; t < 2; t++)
                    acc[mt][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h16x8, xa[ks][mt]),
                                                                        __builtin_bit_cast(h16x8, wb[ks][t]), acc[mt][t], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; i++) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);            // 1 MFMA
                __builtin_amdgcn_sched_group_barrier(0x002, CODE ? 7 : 9, 0);  // VALU
            }
            __builtin_amdgcn_sched_barrier(0);
            if (ks == 0) issue_x_part(fill, fill_slot, 1);
            else issue_w_part(w_fill, 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int mt = 0; mt < 2; mt++)
#pragma unroll
                for (int t = 0; t < 2; t++)
                    acc[mt][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[mt], b[t], acc[mt][t], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        buf ^= 1;
    };
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // nothing of the compiler's own is counted below
    issue_w(wr[0]);
    issue_x(st[0], 0);
    issue_w(wr[1]);
    issue_x(st[1], 1);
    issue_w(wr[2]);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * OG) : "memory");
    tie_w(wr[0]);
    store_w(wr[0], 0);
    for (int s = 0;;) {
        iteration(st[0], st[2], wr[1], wr[0], 0, 2);
        if (++s == stages) break;
        iteration(st[1], st[0], wr[2], wr[1], 1, 0);
        if (++s == stages) break;
        iteration(st[2], st[1], wr[0], wr[2], 2, 1);
        if (++s == stages) break;
    }
    // the look-ahead loads still in flight land in registers and slots that nothing else may use before
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int j = 0; j < D; j++) {
#pragma unroll
        for (int ks = 0; ks < 2; ks++) asm volatile("" ::"v"(st[j].w[ks]));
        asm volatile("" ::"v"(st[j].sc));
        asm volatile("" ::"v"(st[j].zr));
#pragma unroll
        for (int i = 0; i < 8; i++) asm volatile("" ::"v"(wr[j][i]));
    }

    // the second half's waves (kh == 1) hand their sums to the first's: acc(kh = 0) += acc(kh = 1)
    {
        static_assert(4 * 64 * 64 * 4 <= D * SSLOT, "the exchange reuses the ring");
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
        }
    }
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
    if (tid == 0) partials[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// Whether loss_tile_kernel covers a shape.
bool loss_tile_covers(int K, int group) { return K % SBK == 0 && (group == 32 || group % SBK == 0); }

int loss_tiles(int M, int N) { return ((M + LBM - 1) / LBM) * ((N + LBN - 1) / LBN); }

template <bool CODE>
void launch_loss_tile(int M, int N, int K, int group, const void *x, const void *w, const void *x_hat, const uint32_t *packed,
                      const void *scales, const uint8_t *zeros, double *partials, hipStream_t st)
{
    if (group == 32)
        loss_tile_kernel<true, CODE, 0><<<loss_tiles(M, N), 512, 0, st>>>(M, N, K, group, (const h16 *)x, (const h16 *)w, (const h16 *)x_hat,
                                                                          packed, (const h16 *)scales, zeros, partials, SearchSets(), SearchBatch());
    else
        loss_tile_kernel<false, CODE, 0><<<loss_tiles(M, N), 512, 0, st>>>(M, N, K, group, (const h16 *)x, (const h16 *)w, (const h16 *)x_hat,
                                                                           packed, (const h16 *)scales, zeros, partials, SearchSets(), SearchBatch());
}

// The loss of one alpha (set b.set) beside the preparation of the next, whose workgroups are as many as the loss leaves
// compute units idle and take its pieces in turn (one workgroup per piece: 3 % more per alpha on
// 512 x 4096 x 4096 in groups of 64).
template <int G>
void launch_loss_and_next(int M, int N, int K, int group, const void *x, const void *w, const SearchSets &sets, SearchBatch b, double *partials,
                          hipStream_t st)
{
    const int losses = loss_tiles(M, N), idle = sqp_compute_units() - losses % sqp_compute_units();
    b.next_pieces = prepare_pieces(M, N, K, b.next_n);
    loss_tile_kernel<G == 32, true, G><<<losses + (b.next_pieces < idle ? b.next_pieces : idle), 512, 0, st>>>(
        M, N, K, group, (const h16 *)x, (const h16 *)w, sets.x_hat(b.set), sets.packed(b.set), sets.scales(b.set), sets.zeros(b.set), partials, sets, b);
}

// ---------------------------------------------------------------- two alphas of a search at once
//
// The tile, the waves and the order of every sum are loss_tile_kernel's, so each loss has its bits; but a
// workgroup accumulates the tile of TWO alphas: X and W, which do not depend on alpha, come from L2 and out of
// LDS once for both (72 KB per stage instead of 104, eight 16-byte reads per lane for 16 MFMAs instead
// of six for eight).  A stage's loads then have twice the arithmetic to hide behind, so that two
// ring slots do where one alpha needs three.  The fragments of a k-step are read where the previous
// ones have just been used up (X and W while X_hat W_hat is multiplied, X_hat while X W is): 128
// accumulator registers leave no room for two sets of them.
// What bounds it: matrix cores and loads, which overlap in part (512 x 5120 x 5120, one pair on 160 compute units:
// 147 us, twice 88 one by one; 105 without MFMAs, 118 without the direct loads, 142 without W's way or the
// unpack; bringing lines into L2 three stages ahead made it 160).  Searches, before -> now: 512 x 5120 x 5120, 21
// alphas 1907 -> 1574 us; 353 x 2304 x 2792, 6 alphas 331 -> 169; 644 x 7808 x 1328, 11 alphas 1451 -> 617;
// 64 x 4096 x 4096 in groups of 32, 21 alphas 1507 -> 480.
// A launch holds `pairs` such pairs, as many as fill the chip, and behind them one workgroup per piece of the
// next alphas' preparation (a tile of the weight smoothed and quantised, a piece of x divided), which takes what
// compute units the loss leaves idle and evens out its end.
template <int G>
__global__ void __launch_bounds__(512)
search_prepare_kernel(int T, int N, int K, const h16 *__restrict__ x, const h16 *__restrict__ w, SearchSets sets, SearchBatch batch)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[sizeof(QuantizeTile<G, 512>)];
    prepare_piece<G, false>(blockIdx.x, T, N, K, x, w, sets, batch.next_set, batch.next_n, batch.next_factors, lds);
}

template <int G>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
loss_pair_kernel(int M, int N, int K, int group, const h16 *__restrict__ x, const h16 *__restrict__ w, SearchSets sets, SearchBatch batch,
                 double *__restrict__ tile_sums)
{
    constexpr bool G32 = G == 32;
    constexpr int SLOT = 3 * SHALF;            // X, X_hat of the one alpha and of the other
    __shared__ __attribute__((aligned(1024))) unsigned char lds[2 * SLOT + 2 * SWBUF];
    __shared__ double red[2][4];
    static_assert(sizeof(lds) + sizeof(red) <= 160 * 1024, "LDS of a workgroup");
    const int rows = (M + LBM - 1) / LBM, ctiles = (N + LBN - 1) / LBN, pairs = (batch.n + 1) / 2;
    const int losses = ctiles * rows * pairs;
    if ((int)blockIdx.x >= losses) {
        static_assert(sizeof(QuantizeTile<G, 512>) <= sizeof(lds), "the quantiser's LDS fits the ring");
        prepare_piece<G, false>(blockIdx.x - losses, M, N, K, x, w, sets, batch.next_set, batch.next_n, batch.next_factors, lds);
        return;
    }
    // Workgroups go to the eight XCDs in turn: each XCD takes a run of neighbours in the order column, row, pair,
    // so that the workgroups that read the same W (and X) share it in one L2.
    const int xcd = (int)blockIdx.x & 7, run = losses >> 3, more = losses & 7;
    const int at = xcd * run + (xcd < more ? xcd : more) + ((int)blockIdx.x >> 3);
    const int pair = at % pairs, row_tile = at / pairs % rows, col_tile = at / pairs / rows;
    const bool both = 2 * pair + 1 < batch.n;   // an odd alpha out is its own partner, and only its first sums count
    const int sa = batch.set + 2 * pair, sb = sa + (both ? 1 : 0);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kh = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;
    const int l32 = lane & 31, kb = lane >> 5;
    const int m0 = row_tile * LBM, n0 = col_tile * LBN;
    const int stages = K / SBK;
    const int ncol = n0 + wn * 64 + 2 * l32;                   // this lane's two columns (N is even: both in or out)
    const bool ncol_ok = ncol < N;
    const LossConsts uc;

    f32x16 acc[2][2][2];                       // [alpha][row tile][column]
#pragma unroll
    for (int i = 0; i < 8; i++)
#pragma unroll
        for (int r = 0; r < 16; r++) acc[i >> 2][(i >> 1) & 1][i & 1][r] = 0.f;

    struct Stage {                             // per alpha
        u32x2 w[2];   // per k-step of 16 of this wave's half: the packed words of the lane's two columns
        uint32_t sc;  // two fp16 steps
        uint32_t zr;  // two zero points, one byte each
    };
    const int col = ncol_ok ? ncol : 0;
    const uint32_t voff_p = (uint32_t)(kb * N + col) * 4u, voff_s = (uint32_t)col * 2u, voff_z = (uint32_t)col;
    const uint32_t voff_w = n0 + 2 * lane < N ? (uint32_t)(n0 + 2 * lane) * 2u : 0u;  // W: this lane's column pair
    const long nrow = (long)N * 2;            // one row of W in bytes
    // Streams are buffer loads with a 32-bit scalar offset each: scalar instructions cost a wave as much as vector ones, and
    // 64-bit pointers made 171 per two stages, these 107 (search of 64 x 4096 x 4096 in groups of 32, 21 alphas: 424 -> 409 us;
    // 512 x 5120 x 5120: no more than its runs differ).  Past the last stage the offsets stop and the look-ahead re-reads it.
    // (W straight to registers, each row fetched by twice the waves, and a third slot in its room: 1578 -> 1631 us.)
    const uint32_t bytes_x = (uint32_t)M * (uint32_t)K * 2u, bytes_p = (uint32_t)(K / 8) * (uint32_t)N * 4u, rows_q = (uint32_t)(K / group) * (uint32_t)N;
    const rsrc_t buf_w = buffer_of(w, (uint32_t)K * (uint32_t)N * 2u), buf_p[2] = {buffer_of(sets.packed<false>(sa), bytes_p), buffer_of(sets.packed<false>(sb), bytes_p)};
    const rsrc_t buf_s[2] = {buffer_of(sets.scales<false>(sa), rows_q * 2u), buffer_of(sets.scales<false>(sb), rows_q * 2u)};
    const rsrc_t buf_z[2] = {buffer_of(sets.zeros<false>(sa), rows_q), buffer_of(sets.zeros<false>(sb), rows_q)};
    const h16 *const hat[2] = {sets.x_hat<false>(sa), sets.x_hat<false>(sb)};
    uint32_t p_at = (uint32_t)kh * 8u * (uint32_t)nrow, x_at = 0;  // 32 k: four packed rows
    const uint32_t p_most = p_at + (uint32_t)(stages - 1) * 16u * (uint32_t)nrow, x_most = (uint32_t)(stages - 1) * (SBK * 2);
    uint32_t w_at = (uint32_t)wave * 8u * (uint32_t)nrow;             // this wave's 8 rows of a stage
    const uint32_t w_most = w_at + (uint32_t)(stages - 1) * (uint32_t)SBK * (uint32_t)nrow;
    const int spg = G32 ? 1 : __builtin_amdgcn_readfirstlane(group / SBK);  // stages per group (G32: two groups per stage)
    int kin = 0;                               // position of the stage being issued in its group
    uint32_t z_at = G32 ? (uint32_t)(kh * N) : 0u;  // zero points of its group; the steps are at twice that
    const uint32_t z_most = (uint32_t)(__builtin_amdgcn_readfirstlane(G32 ? 2 * (stages - 1) + kh : (stages - 1) / spg) * N);
    uint32_t xoff[2];                          // as in loss_tile_kernel
#pragma unroll
    for (int j = 0; j < 2; j++) {
        const int row = (wave + 8 * j) * 8 + (lane >> 3);
        const int grow = m0 + row < M ? m0 + row : M - 1;
        xoff[j] = (uint32_t)grow * (uint32_t)K * 2u + (uint32_t)(((lane & 7) ^ ((row >> 1) & 7)) * 16);
    }
    constexpr int OX = 7, OW = 8;              // loads per wave and stage: two parts of OX (X, X_hat twice; words, steps, zero points), W
    auto issue_x_part = [&](Stage (&st)[2], int slot, int j) {
        if (j == 0) {
            auto direct = [&](const h16 *src, int at) {
#pragma unroll
                for (int i = 0; i < 2; i++) copy16_to_lds(src, bytes_x, xoff[i], x_at, lds + slot * SLOT + wave * 1024 + i * 8192 + at);
            };
            direct(x, 0);
            direct(hat[0], SHALF);
            direct(hat[1], 2 * SHALF);
            return;
        }
        const uint32_t p1 = p_at + 4u * (uint32_t)nrow, s_at = z_at * 2u;
#pragma unroll
        for (int a = 0; a < 2; a++) {
            asm volatile("buffer_load_dwordx2 %0, %1, %2, %3 offen" : "=v"(st[a].w[0]) : "v"(voff_p), "s"(buf_p[a]), "s"(p_at) : "memory");
            asm volatile("buffer_load_dwordx2 %0, %1, %2, %3 offen" : "=v"(st[a].w[1]) : "v"(voff_p), "s"(buf_p[a]), "s"(p1) : "memory");
        }
#pragma unroll
        for (int a = 0; a < 2; a++) {
            asm volatile("buffer_load_dword %0, %1, %2, %3 offen" : "=v"(st[a].sc) : "v"(voff_s), "s"(buf_s[a]), "s"(s_at) : "memory");
            asm volatile("buffer_load_ushort %0, %1, %2, %3 offen" : "=v"(st[a].zr) : "v"(voff_z), "s"(buf_z[a]), "s"(z_at) : "memory");
        }
        p_at = min(p_at + 16u * (uint32_t)nrow, p_most);
        x_at = min(x_at + SBK * 2, x_most);
        if constexpr (G32) {
            z_at = min(z_at + 2u * (uint32_t)N, z_most);
        } else {
            const bool wrap = ++kin == spg;
            kin = wrap ? 0 : kin;
            z_at = min(z_at + (wrap ? (uint32_t)N : 0u), z_most);
        }
    };
    auto issue_w_part = [&](uint32_t (&r)[8], int h) {
#pragma unroll
        for (int i = 4 * h; i < 4 * h + 4; i++)
            asm volatile("buffer_load_dword %0, %1, %2, %3 offen" : "=v"(r[i]) : "v"(voff_w), "s"(buf_w), "s"(w_at + i * (uint32_t)nrow) : "memory");
        if (h == 1) w_at = min(w_at + (uint32_t)SBK * (uint32_t)nrow, w_most);
    };
    auto tie_w = [&](uint32_t (&r)[8]) {       // no use ahead of the wait in front
#pragma unroll
        for (int i = 0; i < 8; i++) asm volatile("" : "+v"(r[i]));
    };
    const uint32_t wwr = (uint32_t)(size_t)lds + (uint32_t)(2 * SLOT + ((lane >> 5) * 64 + l32) * SROW + wave * 16);
    auto store_w = [&](const uint32_t (&r)[8], int buf) {
        u32x4 c0, c1;  // the low halves of the 8 rows; the high halves
        c0.x = __builtin_amdgcn_perm(r[1], r[0], 0x05040100u); c1.x = __builtin_amdgcn_perm(r[1], r[0], 0x07060302u);
        c0.y = __builtin_amdgcn_perm(r[3], r[2], 0x05040100u); c1.y = __builtin_amdgcn_perm(r[3], r[2], 0x07060302u);
        c0.z = __builtin_amdgcn_perm(r[5], r[4], 0x05040100u); c1.z = __builtin_amdgcn_perm(r[5], r[4], 0x07060302u);
        c0.w = __builtin_amdgcn_perm(r[7], r[6], 0x05040100u); c1.w = __builtin_amdgcn_perm(r[7], r[6], 0x07060302u);
        const uint32_t a = wwr + (uint32_t)(buf * SWBUF);
        asm volatile("ds_write_b128 %0, %1" ::"v"(a), "v"(c0) : "memory");
        asm volatile("ds_write_b128 %0, %1 offset:%2" ::"v"(a), "v"(c1), "n"(32 * SROW) : "memory");
    };
    const uint32_t xrd = (uint32_t)(size_t)lds + (uint32_t)((wm * 64 + l32) * 128);
    const int xkey = (l32 >> 1) & 7;
    const uint32_t wrd = (uint32_t)(size_t)lds + (uint32_t)(2 * SLOT + (wn * 64 + l32) * SROW + kh * 64 + kb * 16);

    u32x4 xa[2], wb[2], xb[2][2];              // fragments of X, W and X_hat (per alpha) of one k-step: [row or column tile]
    auto read_xw = [&](int slot, int ks) {
        const uint32_t a = xrd + (uint32_t)(slot * SLOT) + (uint32_t)(((kh * 4 + ks * 2 + kb) ^ xkey) * 16);
        const uint32_t b = wrd + (uint32_t)(slot * SWBUF + ks * 32);
        asm volatile("ds_read_b128 %0, %1" : "=&v"(xa[0]) : "v"(a) : "memory");
        asm volatile("ds_read_b128 %0, %1 offset:4096" : "=&v"(xa[1]) : "v"(a) : "memory");
        asm volatile("ds_read_b128 %0, %1" : "=&v"(wb[0]) : "v"(b) : "memory");
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(wb[1]) : "v"(b), "n"(32 * SROW) : "memory");
    };
    auto read_xh = [&](int slot, int ks) {
        const uint32_t a = xrd + (uint32_t)(slot * SLOT) + (uint32_t)(((kh * 4 + ks * 2 + kb) ^ xkey) * 16);
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(xb[0][0]) : "v"(a), "n"(SHALF) : "memory");
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(xb[0][1]) : "v"(a), "n"(SHALF + 4096) : "memory");
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(xb[1][0]) : "v"(a), "n"(2 * SHALF) : "memory");
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(xb[1][1]) : "v"(a), "n"(2 * SHALF + 4096) : "memory");
    };
    auto tie_xw = [&]() {                      // no use ahead of the wait in front
#pragma unroll
        for (int i = 0; i < 2; i++) {
            asm volatile("" : "+v"(xa[i]));
            asm volatile("" : "+v"(wb[i]));
        }
    };
    auto tie_xh = [&]() {
#pragma unroll
        for (int a = 0; a < 2; a++)
#pragma unroll
            for (int i = 0; i < 2; i++) asm volatile("" : "+v"(xb[a][i]));
    };
    auto tie_stage = [&](Stage (&cur)[2]) {
#pragma unroll
        for (int a = 0; a < 2; a++) {
#pragma unroll
            for (int ks = 0; ks < 2; ks++) asm volatile("" : "+v"(cur[a].w[ks]));
            asm volatile("" : "+v"(cur[a].sc));
            asm volatile("" : "+v"(cur[a].zr));
        }
    };
    // Stage s (slot, LDS buffer of W and registers by its parity).  On entry its X, X_hat, W and words have landed
    // for all waves, the first fragments are on their way, and no wave reads the other slot and buffer
    // any more, which are filled meanwhile: with the loads of stage s + 1 and, once it has landed, W of that
    // stage; W of stage s + 2 follows into the registers that held W of stage s.  The hand-over to stage
    // s + 1 (wait for its loads, barrier) sits between the last MFMAs of the two alphas, when all fragments
    // have been read: the barrier's wait and the next fragments' way hide behind those MFMAs.
    auto iteration = [&](Stage (&cur)[2], Stage (&fill)[2], uint32_t (&w_next)[8], uint32_t (&w_fill)[8], int slot) {
        h16x2 neg_hi[2][2], neg_lo[2][2], delta[2][2];
#pragma unroll
        for (int a = 0; a < 2; a++)
#pragma unroll
            for (int t = 0; t < 2; t++) {
                const uint32_t z = (cur[a].zr >> (8 * t)) & 0xffu;
                neg_hi[a][t] = neg_hi_of(z);
                neg_lo[a][t] = neg_lo_of(z);
                const uint32_t sw = cur[a].sc ^ 0x80008000u;  // the negated steps
                delta[a][t] = __builtin_bit_cast(h16x2, __builtin_amdgcn_perm(sw, sw, t ? 0x03020302u : 0x01000100u));
            }
#pragma unroll
        for (int ks = 0; ks < 2; ks++) {
            asm volatile("s_waitcnt lgkmcnt(4)" ::: "memory");  // X and W (the reads of X_hat are younger)
            tie_xw();
            if (ks == 0) {
                issue_x_part(fill, slot ^ 1, 0);
            } else {
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * OX) : "memory");  // W of the next stage, issued in the last iteration
                tie_w(w_next);
                store_w(w_next, slot ^ 1);
                issue_w_part(w_fill, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            // X W of 16 k for both alphas, the words of the first unpacked between the MFMAs (the scheduler is told so)
            h16x8 b[2];
#pragma unroll
            for (int t = 0; t < 2; t++) b[t] = dequant_word_ahead(cur[0].w[ks][t], neg_hi[0][t], neg_lo[0][t], delta[0][t], uc);
#pragma unroll
            for (int a = 0; a < 2; a++)
#pragma unroll
                for (int mt = 0; mt < 2; mt++)
#pragma unroll
                    for (int t = 0; t < 2; t++)
                        acc[a][mt][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h16x8, xa[mt]), __builtin_bit_cast(h16x8, wb[t]),
                                                                               acc[a][mt][t], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 8; i++) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // 1 MFMA
                __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);  // VALU
            }
            __builtin_amdgcn_sched_barrier(0);
            if (ks == 0) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            else asm volatile("s_waitcnt lgkmcnt(2)" ::: "memory");  // (the two writes of W are younger)
            tie_xh();
            if (ks == 0) {
                read_xw(slot, 1);
                issue_x_part(fill, slot ^ 1, 1);
            } else {
                issue_w_part(w_fill, 1);
            }
            __builtin_amdgcn_sched_barrier(0);
            // X_hat W_hat of the same 16 k, the words of the second alpha unpacked between the MFMAs of the first
            h16x8 c[2];
#pragma unroll
            for (int t = 0; t < 2; t++) c[t] = dequant_word_ahead(cur[1].w[ks][t], neg_hi[1][t], neg_lo[1][t], delta[1][t], uc);
#pragma unroll
            for (int mt = 0; mt < 2; mt++)
#pragma unroll
                for (int t = 0; t < 2; t++)
                    acc[0][mt][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h16x8, xb[0][mt]), b[t], acc[0][mt][t], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; i++) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (ks == 1) {
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(OW) : "memory");  // all of stage s + 1 (W of the one behind it is younger)
                tie_stage(fill);
                asm volatile("s_barrier" ::: "memory");
                read_xw(slot ^ 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int mt = 0; mt < 2; mt++)
#pragma unroll
                for (int t = 0; t < 2; t++)
                    acc[1][mt][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h16x8, xb[1][mt]), c[t], acc[1][mt][t], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (ks == 0) read_xh(slot, 1);
            else read_xh(slot ^ 1, 0);
        }
    };
    Stage st[2][2];                            // [parity of the stage][alpha]
    uint32_t wr[2][8];                         // W of a stage of that parity
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // nothing of the compiler's own is counted below
    issue_w_part(wr[0], 0);
    issue_w_part(wr[0], 1);
    issue_x_part(st[0], 0, 0);
    issue_x_part(st[0], 0, 1);
    issue_w_part(wr[1], 0);
    issue_w_part(wr[1], 1);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * OX + OW) : "memory");
    tie_w(wr[0]);
    store_w(wr[0], 0);
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(OW) : "memory");
    tie_stage(st[0]);
    asm volatile("s_barrier" ::: "memory");
    read_xw(0, 0);
    read_xh(0, 0);
    for (int s = 0;;) {
        iteration(st[0], st[1], wr[1], wr[0], 0);
        if (++s == stages) break;
        iteration(st[1], st[0], wr[0], wr[1], 1);
        if (++s == stages) break;
    }
    // the look-ahead loads still in flight land in registers and slots that nothing else may use before
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int j = 0; j < 2; j++) {
#pragma unroll
        for (int a = 0; a < 2; a++) {
            asm volatile("" ::"v"(st[j][a].w[0]), "v"(st[j][a].w[1]));
            asm volatile("" ::"v"(st[j][a].sc), "v"(st[j][a].zr));
        }
#pragma unroll
        for (int i = 0; i < 8; i++) asm volatile("" ::"v"(wr[j][i]));
        asm volatile("" ::"v"(xa[j]), "v"(wb[j]), "v"(xb[j][0]), "v"(xb[j][1]));
    }

    // the second half's waves (kh == 1) hand their sums to the first's, then the squares of the tile: as in loss_tile_kernel
    static_assert(4 * 64 * 64 * 4 <= 2 * SLOT, "the exchange reuses the ring");
#pragma unroll
    for (int al = 0; al < 2; al++) {
        f32x4 *ex = reinterpret_cast<f32x4 *>(lds) + (size_t)(wave & 3) * 16 * 64 + lane;
        __syncthreads();
        if (kh == 1) {
#pragma unroll
            for (int q = 0; q < 16; q++) {
                const f32x16 &a = acc[al][q >> 3][(q >> 2) & 1];
                ex[q * 64] = f32x4{a[(q & 3) * 4], a[(q & 3) * 4 + 1], a[(q & 3) * 4 + 2], a[(q & 3) * 4 + 3]};
            }
        }
        __syncthreads();
        if (kh == 0) {
            double ss = 0.0;
#pragma unroll
            for (int q = 0; q < 16; q++) {
                const f32x4 v = ex[q * 64];
#pragma unroll
                for (int r = 0; r < 4; r++) acc[al][q >> 3][(q >> 2) & 1][(q & 3) * 4 + r] += v[r];
            }
#pragma unroll
            for (int mt = 0; mt < 2; mt++)
#pragma unroll
                for (int t = 0; t < 2; t++)
#pragma unroll
                    for (int r = 0; r < 16; r++) {
                        const int row = m0 + wm * 64 + mt * 32 + 8 * (r >> 2) + 4 * kb + (r & 3);
                        if (row < M && ncol_ok) ss += (double)acc[al][mt][t][r] * (double)acc[al][mt][t][r];
                    }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) ss += __shfl_xor(ss, off, 64);
            if (lane == 0) red[al][wave] = ss;
        }
    }
    __syncthreads();
    if (tid < (both ? 2 : 1))
        tile_sums[((size_t)2 * pair + tid) * ctiles * rows + (size_t)row_tile * ctiles + col_tile] =
            (red[tid][0] + red[tid][1]) + (red[tid][2] + red[tid][3]);
}

// The weight of set `i` in the caller's own buffers.
__global__ void __launch_bounds__(256) copy_to_own_kernel(SearchSets sets, int i, long packed16, long scales16, long zeros8)
{
    const long at = (long)blockIdx.x * 256 + threadIdx.x;
    if (at < packed16) reinterpret_cast<uint4 *>(sets.own.packed)[at] = reinterpret_cast<const uint4 *>(sets.packed(i))[at];
    if (at < scales16) reinterpret_cast<uint4 *>(sets.own.scales)[at] = reinterpret_cast<const uint4 *>(sets.scales(i))[at];
    if (at < zeros8) reinterpret_cast<uint2 *>(sets.own.zeros)[at] = reinterpret_cast<const uint2 *>(sets.zeros(i))[at];
}

// Preparation of batch.next_n alphas; the losses of batch.n alphas beside the preparation of next_n others.
template <int G>
void launch_prepare(int T, int N, int K, const void *x, const void *w, const SearchSets &sets, const SearchBatch &b, hipStream_t st)
{
    search_prepare_kernel<G><<<prepare_pieces(T, N, K, b.next_n), 512, 0, st>>>(T, N, K, (const h16 *)x, (const h16 *)w, sets, b);
}
template <int G>
void launch_loss_pairs(int T, int N, int K, int group, const void *x, const void *w, const SearchSets &sets, const SearchBatch &b, double *tile_sums,
                       hipStream_t st)
{
    const int grid = loss_tiles(T, N) * ((b.n + 1) / 2) + (b.next_n ? prepare_pieces(T, N, K, b.next_n) : 0);
    loss_pair_kernel<G><<<grid, 512, 0, st>>>(T, N, K, group, (const h16 *)x, (const h16 *)w, sets, b, tile_sums);
}
#define SQP_BY_GROUP(CALL)               \
    switch (group) {                     \
        case 32: CALL(32); break;        \
        case 64: CALL(64); break;        \
        case 128: CALL(128); break;      \
        default: CALL(256); break;       \
    }

// ---------------------------------------------------------------- any K and group
//
// Eight waves with tiles of 64 x 32, all tiles through registers into LDS, packed words unpacked in
// registers.  The global loads of the next k-step are issued before the current one is multiplied.

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
    const LossConsts uc;

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
            bq[ks] = dequant_word_ahead(rword[ks], neg_hi_of(rz[ks]), neg_lo_of(rz[ks]),
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
    if (loss_tile_covers(K, group))
        launch_loss_tile<false>(M, N, K, group, x, w, x_hat, packed, scales, zeros, scratch, st);
    else if (M % LBM == 0 && N % LBN == 0 && K % LBK == 0)
        quant_loss_kernel<true><<<dim3(gx, gy), 512, 0, st>>>(M, N, K, group, (const h16 *)x, (const h16 *)w, (const h16 *)x_hat,
                                                             packed, (const h16 *)scales, zeros, scratch);
    else
        quant_loss_kernel<false><<<dim3(gx, gy), 512, 0, st>>>(M, N, K, group, (const h16 *)x, (const h16 *)w, (const h16 *)x_hat,
                                                              packed, (const h16 *)scales, zeros, scratch);
    sum_partials_kernel<<<1, 256, 0, st>>>(scratch, (long)gx * gy, loss);
    return sqp_launch_status();
}

// ---------------------------------------------------------------- search over alpha

static size_t up256(size_t v) { return (v + 255) & ~(size_t)255; }

// How a buffer holds a search: factors [n_alpha][K], tile sums [n_alpha][tiles], then `sets` sets of prepared operands.
struct SearchRoom {
    int sets;                                  // 0: not even one set fits
    size_t at_sums, at_sets;
    SearchSets layout;                         // base not set
};

static SearchRoom search_room(int T, int N, int K, int group, int n_alpha, size_t bytes)
{
    SearchRoom r = {};
    if (!loss_tile_covers(K, group)) return r;
    const size_t rows = (size_t)(K / group), blocks = (size_t)sqp_quant_loss_scratch_doubles(T, N);
    r.at_sums = up256((size_t)n_alpha * K * sizeof(float));
    r.at_sets = r.at_sums + up256(n_alpha * blocks * sizeof(double));
    r.layout.at_scales = up256((size_t)K / 8 * N * 4);
    r.layout.at_zeros = r.layout.at_scales + up256(rows * N * 2);
    r.layout.at_x = r.layout.at_zeros + up256(rows * N);
    r.layout.stride = r.layout.at_x + up256((size_t)T * K * sizeof(h16));
    if (bytes >= r.at_sets + r.layout.stride) {
        const size_t n = (bytes - r.at_sets) / r.layout.stride;
        r.sets = n < 4096 ? (int)n : 4096;
    }
    return r;
}

static size_t search_bytes(int T, int N, int K, int group, int n_alpha, int sets)
{
    const SearchRoom r = search_room(T, N, K, group, n_alpha, 0);
    return r.at_sets + sets * r.layout.stride;
}

// Alphas per launch: the number of pairs for which an estimate of the whole search is shortest, in units of
// a loss workgroup's time.  A launch takes at least as many rounds of the chip (one workgroup per compute
// unit) as its losses need, and at least its work spread evenly: losses and the next batch's preparation
// (0.45 of the losses' work: 21 us on the whole chip against 147 us on 160 compute units per pair,
// 512 x 5120 x 5120).  The first batch is prepared alone, a last single alpha takes 0.6.
// Measured against the estimate, 512 x 5120 x 5120, 21 alphas, 1 to 6 pairs: 1796, 1860, 1749, 1686, 1717,
// 1793 us (10.9, 11.2, 10.6, 10.0, 10.9, 10.7); 644 x 7808 x 1328, 11 alphas: 1234, 758, 619 (3, taken), 821.
static int search_batch(int T, int N, int n_alpha)
{
    const double tiles = (double)sqp_quant_loss_scratch_doubles(T, N), cus = sqp_compute_units();
    constexpr double PREPARE = 0.45, SINGLE = 0.6;
    int best = 1;
    double shortest = 0;
    for (int p = 1; p <= (n_alpha + 1) / 2 && p <= 16; p++) {
        double t = 0;
        for (int i = 0; i < n_alpha; i += 2 * p) {
            const int n = n_alpha - i < 2 * p ? n_alpha - i : 2 * p, next = n_alpha - i - n < 2 * p ? n_alpha - i - n : 2 * p;
            if (i == 0) t += PREPARE * n / 2 * tiles / cus;
            const double losses = n == 1 ? SINGLE * tiles : (n + 1) / 2 * tiles, even = (losses + PREPARE * next / 2 * tiles) / cus;
            const double rounds = (n == 1 ? SINGLE : 1.0) * (double)(long)(((n + 1) / 2 * tiles + cus - 1) / cus);
            t += rounds > even ? rounds : even;
        }
        if (p == 1 || t < shortest * 0.999) shortest = t, best = p;
    }
    return 2 * best;
}

static bool prepares_in_tiles(int group) { return group == 32 || group == 64 || group == 128 || group == 256; }

// Two batches of sets, one being used and one being prepared.
static int search_sets_wanted(int T, int N, int K, int group, int n_alpha)
{
    const int batch = search_batch(T, N, n_alpha);
    const size_t most = ((size_t)1 << 30) / search_room(T, N, K, group, n_alpha, 0).layout.stride;  // 1 GB of them, or two batches of one pair
    const int want = n_alpha <= batch ? n_alpha : 2 * batch;
    return (size_t)want <= most ? want : (most > 4 ? (int)most : (want < 4 ? want : 4));
}

// Alphas per launch, and whether the next ones are prepared beside their losses; own: the caller's buffers serve as a
// set beside the `sets` of the region.
struct SearchPlan {
    int batch;
    bool beside;
};
static SearchPlan search_plan(int T, int N, int K, int group, int n_alpha, int sets, bool own)
{
    // Sets for two batches: the next one is prepared beside the losses.  With two or three sets, single losses beside
    // the next alpha's preparation where the tiles leave room for that (90 us per alpha on 512 x 5120 x 5120),
    // pairs behind the preparation of both otherwise (95 there, but 113 against 135 with 66 tiles and K = 7808).
    // One set, or one alpha: the kernel for one.  One set and the caller's own: single losses beside the next
    // alpha's preparation where the loss leaves at least a quarter of the chip idle (88 us per alpha on 512 x 5120 x
    // 5120 against 108 one after the other); no set: the caller's own, one alpha after the other.
    SearchPlan p = {search_batch(T, N, n_alpha), false};
    const bool tiled = prepares_in_tiles(group);
    const long tiles = loss_tiles(T, N), cus = sqp_compute_units();
    p.beside = tiled && p.batch < n_alpha && sets >= 4;
    if (p.beside) {
        p.batch = 2 * p.batch <= sets ? p.batch : sets / 4 * 2;
    } else {
        p.batch = p.batch <= sets ? p.batch : sets;
        if (tiled && p.batch < n_alpha && sets >= 2 && 16 * tiles > 7 * cus && 16 * tiles <= 13 * cus) p.batch = 1, p.beside = true;
    }
    // (Two sets: pairs in turn lose with short K, 1.06 times on 128 x 1024 x 1024.)
    const bool idle = 4 * (cus - tiles) >= cus;
    if (own && (p.batch <= 1 || n_alpha == 1 || (tiled && idle && sets == 2 && K <= 2048))) {
        p.beside = tiled && n_alpha > 1 && (p.beside || (sets >= 1 && idle));
        p.batch = 1;
    }
    return p;
}

// Whether the region holds the factors and the tile sums.
static bool search_fits(int T, int N, int n_alpha, const SearchRoom &room, size_t bytes)
{
    return room.at_sets > 0 && room.at_sums + (size_t)n_alpha * sqp_quant_loss_scratch_doubles(T, N) * sizeof(double) <= bytes;
}

// Test hook: sets that fit a region of this size (-1: not even the factors and sums), alphas per launch (0: none) and
// whether the next ones are prepared beside them; bytes 0: sqp_alpha_search's own region.  Host arithmetic only.
extern "C" void sqp_debug_search_plan(int T, int N, int K, int group, int n_alpha, size_t bytes, int *out3)
{
    const bool own = bytes == 0;
    if (own) bytes = (size_t)K * N * sizeof(h16);
    const SearchRoom room = search_room(T, N, K, group, n_alpha, bytes);
    const bool fits = search_fits(T, N, n_alpha, room, bytes);
    const SearchPlan p = fits && (own || room.sets) ? search_plan(T, N, K, group, n_alpha, room.sets, own) : SearchPlan{0, false};
    out3[0] = fits ? room.sets : -1;
    out3[1] = p.batch;
    out3[2] = p.beside;
}

// The losses of all alphas and the argmin, everything in `region` (amax is given).  With sets.own (sqp_alpha_search) its
// weight is the last alpha's at the end, and it serves as a set where the losses are computed one by one.
static int search_all(int T, int N, int K, int group, int n_alpha, const float *alphas, const void *x_cal, const void *w, const float *amax,
                      void *region, const SearchRoom &room, SearchSets sets, double *loss, int *best, hipStream_t st)
{
    unsigned char *const base = (unsigned char *)region;
    const size_t blocks = (size_t)sqp_quant_loss_scratch_doubles(T, N);
    const bool own = sets.own.packed != nullptr;
    float *factors = (float *)base;
    double *tile_sums = (double *)(base + room.at_sums);
    sets.base = base + room.at_sets;
    int rc = sqp_smooth_factors(K, n_alpha, alphas, amax, factors, st);
    if (rc != SQP_OK) return rc;
    const SearchPlan plan = search_plan(T, N, K, group, n_alpha, room.sets, own);
    const int batch = plan.batch;
    const bool beside = plan.beside;
    const bool tiled = prepares_in_tiles(group);
    // the first set of the batch that starts with alpha i (single losses: the last alpha gets the caller's set)
    auto set_of = [&](int i) {
        if (own && batch == 1) return beside && (n_alpha - 1 - i) % 2 ? 0 : OWN_SET;
        return beside && i / batch % 2 ? batch : 0;
    };
    auto prepare = [&](int first, int n, int set) {
        if (tiled && n > 1) {
            const SearchBatch b = {0, 0, set, n, factors + (size_t)first * K, 0};
#define SQP_PREPARE(G) launch_prepare<G>(T, N, K, x_cal, w, sets, b, st)
            SQP_BY_GROUP(SQP_PREPARE)
#undef SQP_PREPARE
            return sqp_launch_status();
        }
        int e = SQP_OK;
        for (int i = 0; i < n && e == SQP_OK; i++)
            e = sqp_smooth_quantize(T, N, K, group, x_cal, w, factors + (size_t)(first + i) * K, sets.x_hat(set + i), sets.packed(set + i),
                                    sets.scales(set + i), sets.zeros(set + i), st);
        return e;
    };
    for (int i = 0; i < n_alpha && rc == SQP_OK; i += batch) {
        const int n = n_alpha - i < batch ? n_alpha - i : batch, after = n_alpha - i - n < batch ? n_alpha - i - n : batch;
        const int set = set_of(i), next = set_of(i + n);
        if (!beside || i == 0) rc = prepare(i, n, set);
        if (rc != SQP_OK) break;
        if (n == 1 && beside && after > 0) {
            const SearchBatch b = {set, 1, next, after, factors + (size_t)(i + n) * K, 0};
#define SQP_LOSS_NEXT(G) launch_loss_and_next<G>(T, N, K, group, x_cal, w, sets, b, tile_sums + i * blocks, st)
            SQP_BY_GROUP(SQP_LOSS_NEXT)
#undef SQP_LOSS_NEXT
        } else if (n == 1) {
            launch_loss_tile<true>(T, N, K, group, x_cal, w, sets.x_hat(set), sets.packed(set), sets.scales(set), sets.zeros(set), tile_sums + i * blocks, st);
        } else {
            const SearchBatch b = {set, n, beside ? next : 0, beside ? after : 0, factors + (size_t)(i + n) * K, 0};
#define SQP_PAIRS(G) launch_loss_pairs<G>(T, N, K, group, x_cal, w, sets, b, tile_sums + i * blocks, st)
            SQP_BY_GROUP(SQP_PAIRS)
#undef SQP_PAIRS
        }
    }
    if (rc != SQP_OK) return rc;
    sum_partials_kernel<<<n_alpha, 256, 0, st>>>(tile_sums, (long)blocks, loss);
    argmin_kernel<<<1, 64, 0, st>>>(loss, n_alpha, best);
    if (own && batch > 1) {  // (a copy: 6 us on 5120 x 5120, where preparing the weight takes 21)
        const long packed16 = (long)K / 32 * N, scales16 = (long)(K / group) * (N / 8);  // (N % 8 == 0, K % 64 == 0)
        copy_to_own_kernel<<<(unsigned)((packed16 + 255) / 256), 256, 0, st>>>(sets, set_of((n_alpha - 1) / batch * batch) + (n_alpha - 1) % batch,
                                                                                packed16, scales16, scales16);
    }
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
    if (rc != SQP_OK) return rc;
    // The factors, the tile sums and as many sets of prepared operands as fit beside them live in w_s, which the search
    // otherwise fills with the smoothed weight: here the quantisation smooths the weight as it reads it, and x_hat
    // and w_s get the last alpha's values at the end.  Layers too narrow for the factors and sums run the
    // single calls in turn.
    const size_t bytes = (size_t)K * N * sizeof(h16);
    const SearchRoom room = search_room(T, N, K, group, n_alpha, bytes);
    if (search_fits(T, N, n_alpha, room, bytes)) {
        SearchSets sets = room.layout;
        sets.own = {packed, (h16 *)scales, zeros, (h16 *)x_hat};
        rc = search_all(T, N, K, group, n_alpha, alphas, x_cal, w, amax, w_s, room, sets, loss, best, st);
        if (rc == SQP_OK) rc = sqp_smooth_factor(K, alphas[n_alpha - 1], amax, s, st);
        if (rc == SQP_OK) rc = sqp_smooth_apply_x(T, K, x_cal, s, x_hat, stream);  // (not in code order)
        if (rc == SQP_OK) rc = sqp_smooth_apply_w(K, N, w, s, w_s, stream);
        return rc;
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

// The buffers of a search in one scratch buffer: what the single calls need, or what the fused search wants.
static size_t single_calls_bytes(int T, int N, int K, int group)
{
    return up256((size_t)2 * K * 4) + up256((size_t)K * 4) + up256((size_t)T * K * 2) + up256((size_t)K * N * 2) + up256((size_t)K / 8 * N * 4) +
           up256((size_t)(K / group) * N * 2) + up256((size_t)(K / group) * N) + up256((size_t)sqp_quant_loss_scratch_doubles(T, N) * 8);
}

static int check_search(int T, int N, int K, int group, int n_alpha)
{
    if (T <= 0 || n_alpha <= 0 || n_alpha > 4096) return SQP_ERR_SHAPE;
    const int rc = sqp_check_quant_shape(N, K, group);
    if (rc) return rc;
    if (sqp_too_big(T, K) || sqp_too_big(T, N)) return SQP_ERR_SHAPE;
    if ((T + LBM - 1) / LBM > 65535 || K / group > 65535) return SQP_ERR_SHAPE;
    return SQP_OK;
}

extern "C" size_t sqp_alpha_search_scratch_bytes(int T, int N, int K, int group, int n_alpha)
{
    if (check_search(T, N, K, group, n_alpha) != SQP_OK) return 0;
    if (!loss_tile_covers(K, group)) return single_calls_bytes(T, N, K, group);
    const size_t head = up256((size_t)2 * K * sizeof(float));
    return head + search_bytes(T, N, K, group, n_alpha, search_sets_wanted(T, N, K, group, n_alpha));
}

extern "C" size_t sqp_alpha_search_scratch_least_bytes(int T, int N, int K, int group, int n_alpha)
{
    if (check_search(T, N, K, group, n_alpha) != SQP_OK) return 0;
    if (!loss_tile_covers(K, group)) return single_calls_bytes(T, N, K, group);
    return up256((size_t)2 * K * sizeof(float)) + search_bytes(T, N, K, group, n_alpha, 1);
}

extern "C" int sqp_alpha_search_scratch(int T, int N, int K, int group, int n_alpha, const float *alphas, const void *x_cal, const void *w,
                                        void *scratch, size_t scratch_bytes, double *loss, int *best, void *stream)
{
    if (!alphas || !x_cal || !w || !scratch || !loss || !best) return SQP_ERR_NULL;
    const int rc = check_search(T, N, K, group, n_alpha);
    if (rc) return rc;
    for (int i = 0; i < n_alpha; i++)
        if (!(alphas[i] >= 0.0f && alphas[i] <= 1.0f)) return SQP_ERR_ARG;
    if (sqp_misaligned(x_cal) || sqp_misaligned(w) || sqp_misaligned(scratch)) return SQP_ERR_ALIGN;
    if ((reinterpret_cast<uintptr_t>(loss) & 7u) || (reinterpret_cast<uintptr_t>(best) & 3u)) return SQP_ERR_ALIGN;
    unsigned char *const base = (unsigned char *)scratch;
    const size_t head = up256((size_t)2 * K * sizeof(float));
    if (loss_tile_covers(K, group)) {
        const SearchRoom room = search_room(T, N, K, group, n_alpha, scratch_bytes < head ? 0 : scratch_bytes - head);
        if (room.sets == 0) return SQP_ERR_WORKSPACE;
        const int e = sqp_channel_absmax(T, K, N, x_cal, w, (float *)base, (hipStream_t)stream);
        return e != SQP_OK ? e : search_all(T, N, K, group, n_alpha, alphas, x_cal, w, (float *)base, base + head, room, room.layout, loss, best, (hipStream_t)stream);
    }
    if (scratch_bytes < single_calls_bytes(T, N, K, group)) return SQP_ERR_WORKSPACE;
    size_t at = 0;
    auto take = [&](size_t bytes) {
        void *p = base + at;
        at += up256(bytes);
        return p;
    };
    float *amax = (float *)take((size_t)2 * K * 4), *s = (float *)take((size_t)K * 4);
    void *x_hat = take((size_t)T * K * 2), *w_s = take((size_t)K * N * 2), *packed = take((size_t)K / 8 * N * 4);
    void *scales = take((size_t)(K / group) * N * 2), *zeros = take((size_t)(K / group) * N);
    void *sums = take((size_t)sqp_quant_loss_scratch_doubles(T, N) * 8);
    return sqp_alpha_search(T, N, K, group, n_alpha, alphas, x_cal, w, amax, s, x_hat, w_s, (uint32_t *)packed, scales, (uint8_t *)zeros,
                            (double *)sums, loss, best, stream);
}
