// Companion kernels of the W4A16 layer: smoothing factors (Eq. 6), smoothing of
// activations and weights (Eq. 5), group-wise 4-bit quantise + pack and dequantise
// (Eq. 1, Sec 2.2) of arXiv 2312.03788.  All are single streaming passes, bound by HBM
// bandwidth; every result here is defined bit-exactly (IEEE fp32 divide/multiply, one
// round-to-nearest-even to fp16), so no fast-math and no FMA contraction in this file.
#include "sqp_common.h"
#include "sqp_quantize_tile.h"

#pragma clang fp contract(off)

namespace {

// ------------------------------------------------------------------ Eq. 6

__global__ void fill_zero_u32(uint32_t *p, int n)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// max_t |x[t][j]|, accumulated into ax_bits[j] as the bit pattern of a non-negative
// float (unsigned order == float order there), so the atomic max is order-independent.
// Block: 32 column-octets x 8 row lanes.
__global__ void __launch_bounds__(256) absmax_x_kernel(int T, int K, const uint4 *x, uint32_t *ax_bits)
{
    __shared__ float red[8][256];
    const int oct = threadIdx.x & 31, rl = threadIdx.x >> 5;
    const int koct = blockIdx.x * 32 + oct;  // column octet
    const int KO = K >> 3;
    float m[8];
#pragma unroll
    for (int i = 0; i < 8; i++) m[i] = 0.0f;
    if (koct < KO) {
        for (int t = blockIdx.y * 8 + rl; t < T; t += 8 * gridDim.y) {
            uint4 v = x[(size_t)t * KO + koct];
            uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int i = 0; i < 4; i++) {
                m[2 * i] = fmaxf(m[2 * i], fabsf(h2f_lo(w[i])));
                m[2 * i + 1] = fmaxf(m[2 * i + 1], fabsf(h2f_hi(w[i])));
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 8; i++) red[rl][oct * 8 + i] = m[i];
    __syncthreads();
    const int col = blockIdx.x * 256 + threadIdx.x;
    if (col < K) {
        float r = 0.0f;
#pragma unroll
        for (int i = 0; i < 8; i++) r = fmaxf(r, red[i][threadIdx.x]);
        atomicMax(&ax_bits[col], __builtin_bit_cast(uint32_t, r));
    }
}

// The same for up to ABSMAX_DIRECT_ROWS rows: a workgroup takes 64 columns over all of T (8 column octets x
// 64 row lanes), so nothing has to be zeroed before and no atomics are needed.  512 x 22016: 5 + 9 us
// (fill, then atomics) -> 10.5; with many more rows the K / 64 workgroups would walk them too long.
constexpr int ABSMAX_DIRECT_ROWS = 1024;
__global__ void __launch_bounds__(512) absmax_x_direct_kernel(int T, int K, const uint4 *__restrict__ x, float *__restrict__ ax)
{
    __shared__ float red[8][8][9];  // [wave][octet][column], padded
    const int oct = threadIdx.x & 7, rl = threadIdx.x >> 3;
    const int KO = K >> 3, koct = blockIdx.x * 8 + oct;
    float m[8];
#pragma unroll
    for (int i = 0; i < 8; i++) m[i] = 0.0f;
    if (koct < KO) {
#pragma unroll 4
        for (int t = rl; t < T; t += 64) {
            const uint4 v = x[(size_t)t * KO + koct];
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int i = 0; i < 4; i++) {
                m[2 * i] = fmaxf(m[2 * i], fabsf(h2f_lo(w[i])));
                m[2 * i + 1] = fmaxf(m[2 * i + 1], fabsf(h2f_hi(w[i])));
            }
        }
    }
    // lanes l, l + 8, ... of a wave hold the same octet; then the eight waves meet in LDS
#pragma unroll
    for (int i = 0; i < 8; i++)
#pragma unroll
        for (int off = 8; off <= 32; off <<= 1) m[i] = fmaxf(m[i], __shfl_xor(m[i], off, 64));
    if ((threadIdx.x & 63) < 8) {
#pragma unroll
        for (int i = 0; i < 8; i++) red[threadIdx.x >> 6][oct][i] = m[i];
    }
    __syncthreads();
    const int col = blockIdx.x * 64 + threadIdx.x;
    if (threadIdx.x < 64 && col < K) {
        float r = 0.0f;
#pragma unroll
        for (int w = 0; w < 8; w++) r = fmaxf(r, red[w][threadIdx.x >> 3][threadIdx.x & 7]);
        ax[col] = r;
    }
}

__device__ __forceinline__ float smooth_factor_of(float ax, float aw, float alpha)
{
    ax = ax > 1e-5f ? ax : 1e-5f;
    aw = aw > 1e-5f ? aw : 1e-5f;
    const double a = (double)alpha;
    return (float)(pow((double)ax, a) / pow((double)aw, 1.0 - a));
}

// One block per input channel j: aw = max_n |w[j][n]|.  FACTOR: then Eq. 6 with ax read from
// s[j] (left there by absmax_x_kernel) and s[j] overwritten with the factor; otherwise aw is
// stored to s[j].
template <bool FACTOR>
__global__ void __launch_bounds__(256) absmax_w_kernel(int N, float alpha, const uint4 *w, float *s)
{
    __shared__ float red[4];
    const int j = blockIdx.x;
    const int NO = N >> 3;
    const uint4 *row = w + (size_t)j * NO;
    float m = 0.0f;
#pragma unroll 4  // four loads in flight per thread: 65 -> 61 us on 22016 x 8192
    for (int o = threadIdx.x; o < NO; o += 256) {
        const uint4 v = load_stream(row + o);
        uint32_t q[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; i++) m = fmaxf(m, fmaxf(fabsf(h2f_lo(q[i])), fabsf(h2f_hi(q[i]))));
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        const float aw = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
        s[j] = FACTOR ? smooth_factor_of(s[j], aw, alpha) : aw;
    }
}

// Eq. 6 from stored maxima: amax = [ax (K) | aw (K)].
__global__ void __launch_bounds__(256) smooth_factor_kernel(int K, float alpha, const float *amax, float *s)
{
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j < K) s[j] = smooth_factor_of(amax[j], amax[K + j], alpha);
}

// The same for a batch of alphas: factors[i][j] (one grid row per alpha).
struct AlphaBatch {
    float a[64];
};
__global__ void __launch_bounds__(256) smooth_factors_kernel(int K, AlphaBatch alphas, const float *amax, float *factors)
{
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j < K) factors[(size_t)blockIdx.y * K + j] = smooth_factor_of(amax[j], amax[K + j], alphas.a[blockIdx.y]);
}

// ------------------------------------------------------------------ Eq. 5

template <bool CODE_ORDER>
__global__ void __launch_bounds__(256) apply_x_kernel(long total_oct, int KO, const uint4 *x, const float4 *s, uint4 *out)
{
    long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= total_oct) return;
    const int ko = (int)(i % KO);
    const uint4 r = smooth_x8(x[i], s[2 * ko], s[2 * ko + 1]);
    out[i] = CODE_ORDER ? code_order(r) : r;
}

__global__ void __launch_bounds__(256) apply_w_kernel(long total_oct, int NO, const uint4 *w, const float *s, uint4 *out)
{
    long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= total_oct) return;
    out[i] = smooth_w8(load_stream(w + i), s[i / NO]);
}

// ------------------------------------------------------------------ Eq. 1
// The quantiser on its own.  SMOOTH: with the smoothing factors applied as the weight is read, and the
// workgroups past the last group of rows (blockIdx.y >= qrows) divide the activations: one launch for
// what the search needs per alpha.  Measured, per alpha on 512 x 5120 x 5120: three launches of 5.3 +
// 15.9 + 18.6 us become one of 25.
// Groups of 64 on 5120 x 27648: 83 us with one column pair per thread (4-byte loads) -> 65 us
// (5.7 TB/s of bytes read and written).
struct SmoothArgs {
    const float *s;      // [K] smoothing factors
    const uint4 *x;      // [T][K] activations
    uint4 *x_hat;
    long x_octs;         // T * K / 8
    int KO;              // K / 8
    int qrows;           // grid rows that quantise
};
template <int G, bool SMOOTH>
__global__ void __launch_bounds__(G == 256 ? 512 : 256)
quantize_pack_tile_kernel(int N, int K, const uint4 *__restrict__ w, uint32_t *__restrict__ packed,
                          uint16_t *__restrict__ scales, uint8_t *__restrict__ zeros, SmoothArgs sm)
{
    constexpr int THREADS = G == 256 ? 512 : 256;
    __shared__ QuantizeTile<G, THREADS> sh;
    if constexpr (SMOOTH) {
        if ((int)blockIdx.y >= sm.qrows) {
            const long stride = (long)(gridDim.y - sm.qrows) * gridDim.x * THREADS;
            for (long i = ((long)(blockIdx.y - sm.qrows) * gridDim.x + blockIdx.x) * THREADS + threadIdx.x; i < sm.x_octs; i += stride) {
                const int ko = (int)(i % sm.KO);
                const float4 *s4 = reinterpret_cast<const float4 *>(sm.s);
                sm.x_hat[i] = code_order(smooth_x8(sm.x[i], s4[2 * ko], s4[2 * ko + 1]));
            }
            return;
        }
    }
    quantize_tile<G, THREADS, SMOOTH>(blockIdx.x, blockIdx.y, N, K, w, sm.s, packed, scales, zeros, sh);
}

// Any other group size (multiple of 8): the group is read twice.  SMOOTH: rows times s as above.
template <bool SMOOTH>
__global__ void __launch_bounds__(256) quantize_pack_any_kernel(int N, int G, const uint32_t *w, uint2 *packed, uint32_t *scales, uint16_t *zeros,
                                                                const float *s)
{
    const int n2 = blockIdx.x * 256 + threadIdx.x;
    const int N2 = N >> 1;
    if (n2 >= N2) return;
    const int t = blockIdx.y;
    const uint32_t *wp = w + (size_t)t * G * N2 + n2;
    auto load = [&](int i) {
        const uint32_t v = wp[(size_t)i * N2];
        if constexpr (!SMOOTH) return v;
        return smooth_w2(v, s[(size_t)t * G + i]);
    };
    uint32_t v0 = load(0);
    float mn0 = h2f_lo(v0), mx0 = mn0, mn1 = h2f_hi(v0), mx1 = mn1;
    for (int i = 1; i < G; i++) {
        uint32_t v = load(i);
        float a = h2f_lo(v), b = h2f_hi(v);
        mn0 = fminf(mn0, a);
        mx0 = fmaxf(mx0, a);
        mn1 = fminf(mn1, b);
        mx1 = fmaxf(mx1, b);
    }
    GroupParams p0 = group_params(mn0, mx0), p1 = group_params(mn1, mx1);
    scales[(size_t)t * N2 + n2] = (uint32_t)p0.d16 | ((uint32_t)p1.d16 << 16);
    zeros[(size_t)t * N2 + n2] = (uint16_t)(p0.z | (p1.z << 8));
    uint2 *pp = packed + (size_t)t * (G / 8) * N2 + n2;
    for (int j = 0; j < G / 8; j++) {
        uint32_t w0 = 0, w1 = 0;
#pragma unroll
        for (int i = 0; i < 8; i++) {
            uint32_t v = load(8 * j + i);
            w0 |= code_of(h2f_lo(v), p0) << (4 * i);
            w1 |= code_of(h2f_hi(v), p1) << (4 * i);
        }
        pp[(size_t)j * N2] = make_uint2(w0, w1);
    }
}

// One thread expands one packed word of two adjacent columns into 8 rows.
// grid: (ceil(N/512), K/8), block 256.
__global__ void __launch_bounds__(256) dequantize_kernel(int N, int words_per_group, const uint2 *packed, const uint32_t *scales, const uint16_t *zeros, uint32_t *w_hat)
{
    const int n2 = blockIdx.x * 256 + threadIdx.x;
    const int N2 = N >> 1;
    if (n2 >= N2) return;
    const int j = blockIdx.y;
    const int t = j / words_per_group;
    uint2 pw = packed[(size_t)j * N2 + n2];
    uint32_t sc = scales[(size_t)t * N2 + n2];
    uint16_t zz = zeros[(size_t)t * N2 + n2];
    float d0 = h2f_lo(sc), d1 = h2f_hi(sc);
    int z0 = zz & 0xff, z1 = zz >> 8;
    uint32_t *out = w_hat + (size_t)j * 8 * N2 + n2;
#pragma unroll
    for (int i = 0; i < 8; i++) {
        int q0 = (int)((pw.x >> (4 * i)) & 15u), q1 = (int)((pw.y >> (4 * i)) & 15u);
        out[(size_t)i * N2] = pack_h2((float)(q0 - z0) * d0, (float)(q1 - z1) * d1);
    }
}

}  // namespace

// max_t |x[t][j]| to ax [K].
static void absmax_x(int T, int K, const void *x, float *ax, hipStream_t st)
{
    if (T <= ABSMAX_DIRECT_ROWS) {
        absmax_x_direct_kernel<<<(K + 63) / 64, 512, 0, st>>>(T, K, (const uint4 *)x, ax);
        return;
    }
    fill_zero_u32<<<(K + 255) / 256, 256, 0, st>>>((uint32_t *)ax, K);
    absmax_x_kernel<<<dim3((K + 255) / 256, 64), 256, 0, st>>>(T, K, (const uint4 *)x, (uint32_t *)ax);
}

extern "C" int sqp_smooth_scales(int T, int K, int N, float alpha, const void *x_cal, const void *w, float *s, void *stream)
{
    if (!x_cal || !w || !s) return SQP_ERR_NULL;
    if (T <= 0 || K <= 0 || N <= 0 || (K % 8) || (N % 8)) return SQP_ERR_SHAPE;
    if (sqp_too_big(T, K) || sqp_too_big(K, N)) return SQP_ERR_SHAPE;
    if (sqp_misaligned(x_cal) || sqp_misaligned(w) || sqp_misaligned(s)) return SQP_ERR_ALIGN;
    if (!(alpha >= 0.0f && alpha <= 1.0f)) return SQP_ERR_ARG;
    hipStream_t st = (hipStream_t)stream;
    absmax_x(T, K, x_cal, s, st);
    absmax_w_kernel<true><<<K, 256, 0, st>>>(N, alpha, (const uint4 *)w, s);
    return sqp_launch_status();
}

// The two halves of sqp_smooth_scales as separate steps (the per-channel maxima do not depend on
// alpha, so a search over alpha computes them once): amax = [max_t|x_cal[t][j]| (K) | max_n|w[j][n]| (K)].
int sqp_channel_absmax(int T, int K, int N, const void *x_cal, const void *w, float *amax, hipStream_t st)
{
    absmax_x(T, K, x_cal, amax, st);
    absmax_w_kernel<false><<<K, 256, 0, st>>>(N, 0.0f, (const uint4 *)w, amax + K);
    return sqp_launch_status();
}

int sqp_smooth_factor(int K, float alpha, const float *amax, float *s, hipStream_t st)
{
    smooth_factor_kernel<<<(K + 255) / 256, 256, 0, st>>>(K, alpha, amax, s);
    return sqp_launch_status();
}

int sqp_smooth_factors(int K, int n_alpha, const float *alphas, const float *amax, float *factors, hipStream_t st)
{
    for (int i0 = 0; i0 < n_alpha; i0 += 64) {
        AlphaBatch b;
        const int n = n_alpha - i0 < 64 ? n_alpha - i0 : 64;
        for (int i = 0; i < 64; i++) b.a[i] = alphas[i0 + (i < n ? i : 0)];
        smooth_factors_kernel<<<dim3((K + 255) / 256, n), 256, 0, st>>>(K, b, amax, factors + (size_t)i0 * K);
    }
    return sqp_launch_status();
}

extern "C" int sqp_smooth_apply_x(int M, int K, const void *x, const float *s, void *x_out, void *stream)
{
    if (!x || !s || !x_out) return SQP_ERR_NULL;
    if (M <= 0 || K <= 0 || (K % 8) || sqp_too_big(M, K)) return SQP_ERR_SHAPE;
    if (sqp_misaligned(x) || sqp_misaligned(s) || sqp_misaligned(x_out)) return SQP_ERR_ALIGN;
    long total = (long)M * (K / 8);
    apply_x_kernel<false><<<(unsigned)((total + 255) / 256), 256, 0, (hipStream_t)stream>>>(total, K / 8, (const uint4 *)x, (const float4 *)s, (uint4 *)x_out);
    return sqp_launch_status();
}

extern "C" int sqp_smooth_apply_w(int K, int N, const void *w, const float *s, void *w_out, void *stream)
{
    if (!w || !s || !w_out) return SQP_ERR_NULL;
    if (K <= 0 || N <= 0 || (N % 8) || sqp_too_big(K, N)) return SQP_ERR_SHAPE;
    if (sqp_misaligned(w) || sqp_misaligned(s) || sqp_misaligned(w_out)) return SQP_ERR_ALIGN;
    long total = (long)K * (N / 8);
    apply_w_kernel<<<(unsigned)((total + 255) / 256), 256, 0, (hipStream_t)stream>>>(total, N / 8, (const uint4 *)w, s, (uint4 *)w_out);
    return sqp_launch_status();
}

// fp16 [N][K] (one row per output feature, the orientation checkpoints store) -> [K][N] (the
// orientation of Eq. 2 that every other entry point takes).  128 x 128 tile per workgroup.  A thread
// loads an 8 x 8 block (eight pieces of 16 bytes; 16 lanes cover 256 bytes of a row), transposes it
// in registers (v_perm_b32) and hands its octets over through LDS in pieces of 16 bytes, so that it can
// store 256 bytes of a row with 16 lanes too.  LDS holds [k][n] with the octets of a row XOR-ed by the
// k block: 16 lanes touch 16 different octet columns both ways.  Measured on 8192 x 22016: 158 us with
// 64 x 64 tiles whose halves crossed LDS one by one -> 125 us (5.8 TB/s read and written).
// Workgroups take the tiles with n fastest: the rows of the result are finished front to back.
__global__ void __launch_bounds__(256) transpose_nk_kernel(int N, int K, const uint4 *__restrict__ in, uint4 *__restrict__ out)
{
    __shared__ uint4 tile[128][16];
    const int hi = threadIdx.x >> 4, lo = threadIdx.x & 15;
    const int NO = N >> 3, KO = K >> 3;                        // N % 8 == 0, K % 8 == 0: a block is in or out as a whole
    const int tn = (N + 127) / 128;
    const int nb = (int)(blockIdx.x % tn) * 16, kb = (int)(blockIdx.x / tn) * 16;  // first octets of the tile
    uint4 v[8];
    if (nb + hi < NO && kb + lo < KO) {
#pragma unroll
        for (int i = 0; i < 8; i++) v[i] = load_stream(in + (size_t)((nb + hi) * 8 + i) * KO + kb + lo);
    } else {
#pragma unroll
        for (int i = 0; i < 8; i++) v[i] = make_uint4(0, 0, 0, 0);
    }
    // v[i] = row n = i, k = 0..7  ->  t[k] = n 0..7 of column k: pairs of rows, then halves of the pairs
#pragma unroll
    for (int d = 0; d < 4; d++) {
        auto word = [&](int i) { return d == 0 ? v[i].x : (d == 1 ? v[i].y : (d == 2 ? v[i].z : v[i].w)); };
        uint4 even, odd;  // columns k = 2 d and 2 d + 1
        even.x = __builtin_amdgcn_perm(word(1), word(0), 0x05040100u); odd.x = __builtin_amdgcn_perm(word(1), word(0), 0x07060302u);
        even.y = __builtin_amdgcn_perm(word(3), word(2), 0x05040100u); odd.y = __builtin_amdgcn_perm(word(3), word(2), 0x07060302u);
        even.z = __builtin_amdgcn_perm(word(5), word(4), 0x05040100u); odd.z = __builtin_amdgcn_perm(word(5), word(4), 0x07060302u);
        even.w = __builtin_amdgcn_perm(word(7), word(6), 0x05040100u); odd.w = __builtin_amdgcn_perm(word(7), word(6), 0x07060302u);
        tile[lo * 8 + 2 * d][hi ^ lo] = even;
        tile[lo * 8 + 2 * d + 1][hi ^ lo] = odd;
    }
    __syncthreads();
    // now hi is the k block, lo the n octet
    if (nb + lo < NO && kb + hi < KO) {
#pragma unroll
        for (int i = 0; i < 8; i++) out[(size_t)((kb + hi) * 8 + i) * NO + nb + lo] = tile[hi * 8 + i][lo ^ hi];
    }
}

extern "C" int sqp_transpose_nk(int N, int K, const void *w_nk, void *w_kn, void *stream)
{
    if (!w_nk || !w_kn) return SQP_ERR_NULL;
    if (N <= 0 || K <= 0 || (N % 8) || (K % 8) || sqp_too_big(K, N)) return SQP_ERR_SHAPE;
    if (sqp_misaligned(w_nk) || sqp_misaligned(w_kn)) return SQP_ERR_ALIGN;
    if ((N + 63) / 64 > 65535) return SQP_ERR_SHAPE;
    transpose_nk_kernel<<<(unsigned)((long)((N + 127) / 128) * ((K + 127) / 128)), 256, 0, (hipStream_t)stream>>>(N, K, (const uint4 *)w_nk, (uint4 *)w_kn);
    return sqp_launch_status();
}

template <int G, bool SMOOTH>
static void launch_quantize_tile(int N, int K, const void *w, uint32_t *packed, void *scales, uint8_t *zeros, SmoothArgs sm, hipStream_t st)
{
    constexpr int THREADS = G == 256 ? 512 : 256, ROWS = THREADS / 2;
    const int gx = (N + 255) / 256, rows = (K + ROWS - 1) / ROWS;
    int extra = 0;
    if (SMOOTH) {
        // activations: about eight octets per thread
        sm.qrows = rows;
        extra = (int)((sm.x_octs + 8L * THREADS * gx - 1) / (8L * THREADS * gx));
        if (extra > 65535 - rows) extra = 65535 - rows;  // (a grid row covers any share of them)
        if (extra == 0)
            apply_x_kernel<true><<<(unsigned)((sm.x_octs + 255) / 256), 256, 0, st>>>(sm.x_octs, sm.KO, sm.x, (const float4 *)sm.s, sm.x_hat);
    }
    quantize_pack_tile_kernel<G, SMOOTH><<<dim3(gx, rows + extra), THREADS, 0, st>>>(N, K, (const uint4 *)w, packed, (uint16_t *)scales, zeros, sm);
}

// Groups of 32, 64, 128 and 256 rows read the weight once, others twice.
template <bool SMOOTH>
static int launch_quantize(int N, int K, int group, const void *w, uint32_t *packed, void *scales, uint8_t *zeros, const SmoothArgs &sm,
                           hipStream_t st)
{
    switch (group) {
        case 32: launch_quantize_tile<32, SMOOTH>(N, K, w, packed, scales, zeros, sm, st); break;
        case 64: launch_quantize_tile<64, SMOOTH>(N, K, w, packed, scales, zeros, sm, st); break;
        case 128: launch_quantize_tile<128, SMOOTH>(N, K, w, packed, scales, zeros, sm, st); break;
        case 256: launch_quantize_tile<256, SMOOTH>(N, K, w, packed, scales, zeros, sm, st); break;
        default:
            quantize_pack_any_kernel<SMOOTH><<<dim3((N / 2 + 255) / 256, K / group), 256, 0, st>>>(
                N, group, (const uint32_t *)w, (uint2 *)packed, (uint32_t *)scales, (uint16_t *)zeros, sm.s);
            if (SMOOTH)
                apply_x_kernel<true><<<(unsigned)((sm.x_octs + 255) / 256), 256, 0, st>>>(sm.x_octs, sm.KO, sm.x, (const float4 *)sm.s, sm.x_hat);
            break;
    }
    return sqp_launch_status();
}

extern "C" int sqp_quantize_pack(int N, int K, int group, const void *w, uint32_t *packed, void *scales, uint8_t *zeros, void *stream)
{
    if (!w || !packed || !scales || !zeros) return SQP_ERR_NULL;
    int rc = sqp_check_quant_shape(N, K, group);
    if (rc) return rc;
    if (K / group > 65535) return SQP_ERR_SHAPE;
    if (sqp_misaligned(w) || sqp_misaligned(packed) || sqp_misaligned(scales) || sqp_misaligned(zeros)) return SQP_ERR_ALIGN;
    return launch_quantize<false>(N, K, group, w, packed, scales, zeros, SmoothArgs(), (hipStream_t)stream);
}

// s * w quantised and x / s, as sqp_smooth_apply_w, sqp_quantize_pack and sqp_smooth_apply_x give
// them, without the smoothed weight in between and with x / s in code order.  Arguments are
// already validated.
int sqp_smooth_quantize(int T, int N, int K, int group, const void *x, const void *w, const float *s, void *x_hat,
                        uint32_t *packed, void *scales, uint8_t *zeros, hipStream_t st)
{
    SmoothArgs sm;
    sm.s = s;
    sm.x = (const uint4 *)x;
    sm.x_hat = (uint4 *)x_hat;
    sm.x_octs = (long)T * (K / 8);
    sm.KO = K / 8;
    sm.qrows = 0;
    return launch_quantize<true>(N, K, group, w, packed, scales, zeros, sm, st);
}

extern "C" int sqp_dequantize(int N, int K, int group, const uint32_t *packed, const void *scales, const uint8_t *zeros, void *w_hat, void *stream)
{
    if (!packed || !scales || !zeros || !w_hat) return SQP_ERR_NULL;
    int rc = sqp_check_quant_shape(N, K, group);
    if (rc) return rc;
    if (K / 8 > 65535) return SQP_ERR_SHAPE;
    if (sqp_misaligned(packed) || sqp_misaligned(scales) || sqp_misaligned(zeros) || sqp_misaligned(w_hat)) return SQP_ERR_ALIGN;
    dim3 grid((N / 2 + 255) / 256, K / 8);
    dequantize_kernel<<<grid, 256, 0, (hipStream_t)stream>>>(N, group / 8, (const uint2 *)packed, (const uint32_t *)scales, (const uint16_t *)zeros, (uint32_t *)w_hat);
    return sqp_launch_status();
}
