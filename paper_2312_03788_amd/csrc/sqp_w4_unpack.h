// Device helpers shared by the W4A16 GEMM kernels: loads with a scalar offset, 4-bit code unpack and the matching
// permutation of activations (Eq. 1 of arXiv 2312.03788, second line: (code - Z) * Delta).
#pragma once
#include "sqp_common.h"

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// A buffer's descriptor for loads written in assembly.
typedef int rsrc_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ rsrc_t buffer_of(const void *p, uint32_t bytes)
{
    const uint64_t at = reinterpret_cast<uint64_t>(p);
    return rsrc_t{(int)(uint32_t)at, (int)(uint32_t)(at >> 32), (int)bytes, 0x00020000};
}

// Direct global -> LDS load of 16 bytes per lane: lane i's from base + lane_offset + offset to dst + 16 i (dst and offset
// wave-uniform).  A buffer load: neither a 64-bit address per lane nor one per call; bytes: size of the buffer.
__device__ __forceinline__ void copy16_to_lds(const void *base, uint32_t bytes, uint32_t lane_offset, uint32_t offset, void *dst)
{
    const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(src, (__attribute__((address_space(3))) void *)dst, 16, lane_offset, offset, 0, 0);
}

// Constants of the nibble unpack, held in registers (v_and_or_b32 takes no literals, and one scalar).  (The empty asm hides their
// values, so the compiler keeps them there and makes one instruction of each and-or below.  Those were asm statements
// themselves; behind one of them it puts a wait state wherever the next instruction reads the result, 10 % of
// the instructions of the column slices' loop.)
struct UnpackConsts {
    uint32_t mask_lo, mask_hi, magic_lo, magic_hi;
};
__device__ __forceinline__ UnpackConsts unpack_consts()
{
    UnpackConsts uc = {0x000f000fu, 0x00f000f0u, 0x64006400u, 0x54005400u};
    asm("" : "+s"(uc.mask_lo), "+s"(uc.mask_hi), "+v"(uc.magic_lo), "+v"(uc.magic_hi));
    return uc;
}

// fp16 bit patterns of -(1024 + Z) and -(64 + Z), replicated into both halves:
// 1024 + Z is 0x6400 + Z and 64 + Z is 0x5400 + 16 Z for Z <= 15.
__device__ __forceinline__ h16x2 neg_hi_of(uint32_t z) { return __builtin_bit_cast(h16x2, z * 0x00010001u + 0xe400e400u); }
__device__ __forceinline__ h16x2 neg_lo_of(uint32_t z) { return __builtin_bit_cast(h16x2, z * 0x00100010u + 0xd400d400u); }

// The same from byte c of four zero points, one v_perm_b32 each: the byte (for the second one z16 = the four zero points
// << 4, which stay within their bytes) under the high bytes.
__device__ __forceinline__ h16x2 neg_hi_at(uint32_t z, int c)
{
    return __builtin_bit_cast(h16x2, __builtin_amdgcn_perm(0xe400e400u, z, 0x07000500u + 0x00010001u * c));
}
__device__ __forceinline__ h16x2 neg_lo_at(uint32_t z16, int c)
{
    return __builtin_bit_cast(h16x2, __builtin_amdgcn_perm(0xd400d400u, z16, 0x07000500u + 0x00010001u * c));
}

// packed word (8 codes of one column) -> 8 exact fp16 values (code - Z), in the order
// (k0,k4),(k1,k5),(k2,k6),(k3,k7): the nibbles are OR-ed into the mantissa of 1024.0
// (bits 3:0) or 64.0 (bits 7:4) and the offset is removed by an exact packed fp16 add.
// 1 shift + 4 and-or + 4 packed adds.
__device__ __forceinline__ h16x8 dequant_word(uint32_t w, h16x2 neg_hi, h16x2 neg_lo, const UnpackConsts &uc)
{
    const uint32_t w8 = w >> 8;
    const uint32_t t0 = (w & uc.mask_lo) | uc.magic_lo, t1 = (w & uc.mask_hi) | uc.magic_hi;
    const uint32_t t2 = (w8 & uc.mask_lo) | uc.magic_lo, t3 = (w8 & uc.mask_hi) | uc.magic_hi;
    h16x2 b0 = __builtin_bit_cast(h16x2, t0) + neg_hi;
    h16x2 b1 = __builtin_bit_cast(h16x2, t1) + neg_lo;
    h16x2 b2 = __builtin_bit_cast(h16x2, t2) + neg_hi;
    h16x2 b3 = __builtin_bit_cast(h16x2, t3) + neg_lo;
    h16x8 r;
    r.s0 = b0.x; r.s1 = b0.y; r.s2 = b1.x; r.s3 = b1.y;
    r.s4 = b2.x; r.s5 = b2.y; r.s6 = b3.x; r.s7 = b3.y;
    return r;
}

// The same, times the step: the fp16 dequantised weights w_hat = fp16((code - Z) * Delta)
// themselves (one rounding, as Eq. 1 defines them).  4 more packed multiplies.
__device__ __forceinline__ h16x8 dequant_word_scaled(uint32_t w, h16x2 neg_hi, h16x2 neg_lo, h16x2 delta, const UnpackConsts &uc)
{
    const uint32_t w8 = w >> 8;
    const uint32_t t0 = (w & uc.mask_lo) | uc.magic_lo, t1 = (w & uc.mask_hi) | uc.magic_hi;
    const uint32_t t2 = (w8 & uc.mask_lo) | uc.magic_lo, t3 = (w8 & uc.mask_hi) | uc.magic_hi;
    h16x2 b0 = (__builtin_bit_cast(h16x2, t0) + neg_hi) * delta;
    h16x2 b1 = (__builtin_bit_cast(h16x2, t1) + neg_lo) * delta;
    h16x2 b2 = (__builtin_bit_cast(h16x2, t2) + neg_hi) * delta;
    h16x2 b3 = (__builtin_bit_cast(h16x2, t3) + neg_lo) * delta;
    h16x8 r;
    r.s0 = b0.x; r.s1 = b0.y; r.s2 = b1.x; r.s3 = b1.y;
    r.s4 = b2.x; r.s5 = b2.y; r.s6 = b3.x; r.s7 = b3.y;
    return r;
}

// 8 consecutive-k activations (x0..x7 as four dwords) -> the nibble order above.
__device__ __forceinline__ h16x8 permute_x(const u32x4 &v)
{
    u32x4 p;
    p.x = __builtin_amdgcn_perm(v.z, v.x, 0x05040100u);  // (x0, x4)
    p.y = __builtin_amdgcn_perm(v.z, v.x, 0x07060302u);  // (x1, x5)
    p.z = __builtin_amdgcn_perm(v.w, v.y, 0x05040100u);  // (x2, x6)
    p.w = __builtin_amdgcn_perm(v.w, v.y, 0x07060302u);  // (x3, x7)
    return __builtin_bit_cast(h16x8, p);
}

// The unpack in the order of k, for kernels in which many waves read the same activations (those then need no
// permutation): byte i of a word holds the codes of k = 2 i and 2 i + 1.  v_perm_b32 puts it under the high bytes of
// 1024.0 and 64.0, one AND clears the other nibble of each half, and the offsets 1024 + Z and 64 + Z go with one exact
// packed add.
constexpr uint32_t PAIR_HIGH_BYTES = 0x54006400u, PAIR_MASK = 0xfff0ff0fu;
constexpr uint32_t PAIR_SELECT = 0x07000500u;  // + 0x00010001 i: (byte i of the word, its high byte), twice
__device__ __forceinline__ h16x2 neg_pair_of(uint32_t z) { return __builtin_bit_cast(h16x2, z * 0x00100001u + 0xd400e400u); }

// packed word -> the fp16 dequantised weights fp16((code - Z) * Delta) of k = 0 .. 7, neg = neg_pair_of(Z).
__device__ __forceinline__ h16x8 dequant_word_pairs(uint32_t w, h16x2 neg, h16x2 delta)
{
    u32x4 r;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const uint32_t t = __builtin_amdgcn_perm(PAIR_HIGH_BYTES, w, PAIR_SELECT + 0x00010001u * i) & PAIR_MASK;
        r[i] = __builtin_bit_cast(uint32_t, (__builtin_bit_cast(h16x2, t) + neg) * delta);
    }
    return __builtin_bit_cast(h16x8, r);
}
