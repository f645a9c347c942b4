// Device code of the quantiser (Eq. 1, Sec 2.2 of arXiv 2312.03788) and of smoothing (Eq. 5), shared by
// the stand-alone kernels and by the loss kernel, which prepares the next alpha of a search beside
// its own work.  Every result is defined bit-exactly: no FMA contraction.
#pragma once
#include "sqp_common.h"

namespace {

__device__ __forceinline__ float h2f_lo(uint32_t v) { return (float)__builtin_bit_cast(h16x2, v).x; }
__device__ __forceinline__ float h2f_hi(uint32_t v) { return (float)__builtin_bit_cast(h16x2, v).y; }
__device__ __forceinline__ uint32_t pack_h2(float a, float b)
{
    h16x2 r;
    r.x = (h16)a;
    r.y = (h16)b;
    return __builtin_bit_cast(uint32_t, r);
}

// (k0 .. k7) -> (k0, k4, k1, k5, k2, k6, k3, k7): the order in which the GEMM kernels unpack a word.
__device__ __forceinline__ uint4 code_order(const uint4 &v)
{
    return make_uint4(__builtin_amdgcn_perm(v.z, v.x, 0x05040100u), __builtin_amdgcn_perm(v.z, v.x, 0x07060302u),
                      __builtin_amdgcn_perm(v.w, v.y, 0x05040100u), __builtin_amdgcn_perm(v.w, v.y, 0x07060302u));
}

__device__ __forceinline__ uint4 smooth_x8(const uint4 &v, const float4 &s0, const float4 &s1)
{
    uint4 r;
    r.x = pack_h2(h2f_lo(v.x) / s0.x, h2f_hi(v.x) / s0.y);
    r.y = pack_h2(h2f_lo(v.y) / s0.z, h2f_hi(v.y) / s0.w);
    r.z = pack_h2(h2f_lo(v.z) / s1.x, h2f_hi(v.z) / s1.y);
    r.w = pack_h2(h2f_lo(v.w) / s1.z, h2f_hi(v.w) / s1.w);
    return r;
}
// The product is rounded to fp32 and then to fp16, as Eq. 5's kernel is defined.  The empty asm keeps
// the compiler from folding the two into a mixed-precision multiply-add with one rounding, which
// gave another fp16 value in about one product of ten million where the result feeds arithmetic.
__device__ __forceinline__ float mul_f32(float a, float b)
{
    float p = a * b;
    asm("" : "+v"(p));
    return p;
}
__device__ __forceinline__ uint32_t smooth_w2(uint32_t v, float sj) { return pack_h2(mul_f32(sj, h2f_lo(v)), mul_f32(sj, h2f_hi(v))); }
__device__ __forceinline__ uint4 smooth_w8(const uint4 &v, float sj)
{
    return make_uint4(smooth_w2(v.x, sj), smooth_w2(v.y, sj), smooth_w2(v.z, sj), smooth_w2(v.w, sj));
}

struct GroupParams {
    float d;     // the fp16-rounded step, as float
    uint16_t d16;
    int z;
};

__device__ __forceinline__ GroupParams group_params(float wmin, float wmax)
{
    float lo = wmin < 0.0f ? wmin : 0.0f;
    float hi = wmax > 0.0f ? wmax : 0.0f;
    float d32 = (hi - lo) / 15.0f;
    h16 dh = (h16)d32;
    uint16_t bits = __builtin_bit_cast(uint16_t, dh);
    if ((bits & 0x7fffu) == 0) bits = 0x0001u;
    GroupParams p;
    p.d16 = bits;
    p.d = (float)__builtin_bit_cast(h16, bits);
    int z = (int)rintf(-lo / p.d);
    p.z = z < 0 ? 0 : (z > 15 ? 15 : z);
    return p;
}

__device__ __forceinline__ uint32_t code_of(float v, const GroupParams &p)
{
    int q = (int)rintf(v / p.d) + p.z;
    q = q < 0 ? 0 : (q > 15 ? 15 : q);
    return (uint32_t)q;
}

// The code of Eq. 1 needs rint(v / d) with the correctly rounded quotient.  A full IEEE
// division per weight makes the kernel ALU-bound, so the quotient is first formed as
// t = v * (1 / d): |t - v/d| <= 2^-23 * |v/d| <= 1.8e-6 (|v/d| <= 15.01 because the group's
// range contains 0), and the rounded quotient lies within 0.9e-6 of v/d.  Unless t is within
// NEAR_TIE of a half-integer, rint(t) is therefore rint of the exact quotient; the rare
// words with such a value are redone with the division (a wave-uniform branch).
constexpr float NEAR_TIE = 4.0e-6f;

// Groups of 32, 64, 128 or 256 rows: a workgroup of 256 threads (512 for groups of 256) quantises
// 128 (256) rows x 256 columns, i.e. 128 / G groups at once.  Thread (part = tid / 32, oct = tid % 32)
// holds rows 16 part .. 16 part + 15 of columns 8 oct .. 8 oct + 7 in registers (16 loads of 16
// bytes; a wave's load covers two rows x 512 contiguous bytes).  Column minima and maxima (exact
// packed fp16 min / max) meet in LDS; the step, the zero point and the reciprocal step of a column
// and group are then computed by one thread alone (three IEEE divisions per column and group, not
// per thread and column) and handed to the others through LDS.  Coding pass, per weight:
// t = fma(w, 1 / Delta, Z) -- within 1.9e-6 of (correctly rounded w / Delta) + Z wherever the code
// is not clamped, see NEAR_TIE -- then round, clamp to [0, 15] as a float, and the eight codes of a
// word are assembled by a fused multiply-add chain (sum c_i 16^i per half word is exact in fp32).
// A word containing a value within NEAR_TIE of a rounding tie is redone with the division of the
// definition (wave-uniform branch, about 0.4 % of the words), and so is one with a NaN among its t (from a
// NaN or an infinity), which the clamp would turn into code 0: a NaN gets code Z, as a weight of 0 does,
// whatever its neighbours hold.  The maximum over |t - rint(t)| propagates NaNs (v_maximum3_f32), which
// costs nothing over one that does not.
// SMOOTH: the weight is multiplied by the smoothing factor of its row as it is read (one rounding to
// fp16, as sqp_smooth_apply_w does it), which saves the smoothed weight's way out and back.
// (bx, by): the workgroup's tile of 256 columns and 16 PARTS rows.  All threads take part; a caller that
// does several tiles in turn needs no barrier between them.
template <int G, int THREADS>
struct QuantizeTile {
    static constexpr int PARTS = THREADS / 32;       // 16-row parts of a workgroup
    static constexpr int GP = G / 16;                // parts of a group
    static constexpr int GB = PARTS / GP;            // groups of a workgroup
    uint4 red[PARTS][2][32];                         // [part][min | max][oct]
    float par_d[GB][256], par_inv[GB][256], par_z[GB][256];  // per group and column of the workgroup
};
template <int G, int THREADS, bool SMOOTH>
__device__ __forceinline__ void quantize_tile(int bx, int by, int N, int K, const uint4 *__restrict__ w, const float *__restrict__ s,
                                              uint32_t *__restrict__ packed, uint16_t *__restrict__ scales, uint8_t *__restrict__ zeros,
                                              QuantizeTile<G, THREADS> &sh)
{
#pragma clang fp contract(off)
    constexpr int PARTS = THREADS / 32, GP = G / 16, GB = PARTS / GP;
    const int oct = threadIdx.x & 31, part = threadIdx.x >> 5;
    const int NO = N >> 3;
    const int o = bx * 32 + oct;
    const int row0 = by * (PARTS * 16) + part * 16;   // a group ends inside K or not at all, so a part does as well
    const bool in = o < NO && row0 < K;
    const int grp = part / GP;                                 // this thread's group in the workgroup
    const uint4 *wp = w + (size_t)(row0 < K ? row0 : 0) * NO + (o < NO ? o : 0);
    uint4 v[16];
#pragma unroll
    for (int i = 0; i < 16; i++) v[i] = SMOOTH ? wp[(size_t)i * NO] : load_stream(wp + (size_t)i * NO);
    if constexpr (SMOOTH) {  // (no streaming hint on these loads: the next alpha reads the same weight again)
        const float *sp = s + (row0 < K ? row0 : 0);
#pragma unroll
        for (int i = 0; i < 16; i++) {
            v[i] = smooth_w8(v[i], sp[i]);
            // (kept as packed fp16: the compiler would hold the 128 fp32 values otherwise)
            asm volatile("" : "+v"(v[i].x), "+v"(v[i].y), "+v"(v[i].z), "+v"(v[i].w));
        }
    }
    h16x2 mn[4], mx[4];
    {
        const uint32_t q[4] = {v[0].x, v[0].y, v[0].z, v[0].w};
#pragma unroll
        for (int c = 0; c < 4; c++) mn[c] = mx[c] = __builtin_bit_cast(h16x2, q[c]);
    }
#pragma unroll
    for (int i = 1; i < 16; i++) {
        const uint32_t q[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
        for (int c = 0; c < 4; c++) {
            const h16x2 e = __builtin_bit_cast(h16x2, q[c]);
            mn[c] = __builtin_elementwise_min(mn[c], e);
            mx[c] = __builtin_elementwise_max(mx[c], e);
        }
    }
    auto as_u4 = [](const h16x2 (&a)[4]) {
        return make_uint4(__builtin_bit_cast(uint32_t, a[0]), __builtin_bit_cast(uint32_t, a[1]),
                          __builtin_bit_cast(uint32_t, a[2]), __builtin_bit_cast(uint32_t, a[3]));
    };
    sh.red[part][0][oct] = as_u4(mn);
    sh.red[part][1][oct] = as_u4(mx);
    __syncthreads();
    // THREADS threads, 256 columns x GB groups: column 8 oct + c of a group, i.e. half (c & 1) of
    // dword (c >> 1) of the octet
    for (int u = part; u < 8 * GB; u += PARTS) {
        const int c = u & 7, g = u >> 3;
        const uint32_t *rmn = reinterpret_cast<const uint32_t *>(&sh.red[g * GP][0][oct]) + (c >> 1);
        const uint32_t *rmx = reinterpret_cast<const uint32_t *>(&sh.red[g * GP][1][oct]) + (c >> 1);
        constexpr int PSTRIDE = 2 * 32 * 4;  // dwords between parts
        float lo = 0.f, hi = 0.f;
#pragma unroll
        for (int pp = 0; pp < GP; pp++) {
            const h16x2 a = __builtin_bit_cast(h16x2, rmn[pp * PSTRIDE]), b = __builtin_bit_cast(h16x2, rmx[pp * PSTRIDE]);
            const float fa = (c & 1) ? (float)a.y : (float)a.x, fb = (c & 1) ? (float)b.y : (float)b.x;
            lo = pp == 0 ? fa : fminf(lo, fa);
            hi = pp == 0 ? fb : fmaxf(hi, fb);
        }
        const GroupParams gp = group_params(lo, hi);
        const int col = oct * 8 + c;
        sh.par_d[g][col] = gp.d;
        sh.par_inv[g][col] = 1.0f / gp.d;
        sh.par_z[g][col] = (float)gp.z;
        const int n = bx * 256 + col;
        const int t = by * GB + g;
        if (n < N && t * G < K) {
            scales[(size_t)t * N + n] = gp.d16;
            zeros[(size_t)t * N + n] = (uint8_t)gp.z;
        }
    }
    __syncthreads();
    if (!in) return;  // (no barrier below)
    uint32_t *pp0 = packed + (size_t)(row0 >> 3) * N + (size_t)o * 8;
#pragma unroll
    for (int j = 0; j < 2; j++) {
        uint32_t word[8];
#pragma unroll
        for (int c = 0; c < 8; c++) {
            const float inv = sh.par_inv[grp][oct * 8 + c], zf = sh.par_z[grp][oct * 8 + c];
            float code[8], worst = 0.f;
#pragma unroll
            for (int i = 0; i < 8; i++) {
                const uint4 &row = v[8 * j + i];
                const uint32_t dw = (c >> 1) == 0 ? row.x : ((c >> 1) == 1 ? row.y : ((c >> 1) == 2 ? row.z : row.w));
                const float x = (c & 1) ? h2f_hi(dw) : h2f_lo(dw);
                const float tq = fmaf(x, inv, zf);
                const float r = rintf(tq);
                worst = __builtin_elementwise_maximum(worst, fabsf(tq - r));
                code[i] = fminf(fmaxf(r, 0.0f), 15.0f);
            }
            const float lo4 = fmaf(fmaf(fmaf(code[3], 16.0f, code[2]), 16.0f, code[1]), 16.0f, code[0]);
            const float hi4 = fmaf(fmaf(fmaf(code[7], 16.0f, code[6]), 16.0f, code[5]), 16.0f, code[4]);
            word[c] = (uint32_t)lo4 | ((uint32_t)hi4 << 16);
            if (__builtin_amdgcn_ballot_w64(!(worst < 0.5f - NEAR_TIE)) != 0ull) {
                GroupParams gp;
                gp.d = sh.par_d[grp][oct * 8 + c];
                gp.z = (int)zf;
                gp.d16 = 0;
                uint32_t wd = 0;
#pragma unroll
                for (int i = 0; i < 8; i++) {
                    const uint4 &row = v[8 * j + i];
                    const uint32_t dw = (c >> 1) == 0 ? row.x : ((c >> 1) == 1 ? row.y : ((c >> 1) == 2 ? row.z : row.w));
                    wd |= code_of((c & 1) ? h2f_hi(dw) : h2f_lo(dw), gp) << (4 * i);
                }
                word[c] = wd;
            }
        }
        uint4 *dst = reinterpret_cast<uint4 *>(pp0 + (size_t)j * N);
        dst[0] = make_uint4(word[0], word[1], word[2], word[3]);
        dst[1] = make_uint4(word[4], word[5], word[6], word[7]);
    }
}

}  // namespace
