// Shared host-side helpers of the sqp library (argument checks, launch status).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sqp.h"
#include "sqp_test_hooks.h"

typedef _Float16 h16;
typedef _Float16 h16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 h16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 h16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

static inline bool sqp_misaligned(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

// Size limit of every entry point: a tensor has fewer than 2^31 elements (the kernels keep
// per-lane offsets in 32 bits).
static inline bool sqp_too_big(long rows, long cols) { return rows * cols >= (1L << 31); }

static inline int sqp_check_quant_shape(int N, int K, int group)
{
    if (N <= 0 || K <= 0 || group < 8) return SQP_ERR_SHAPE;
    if (sqp_too_big(K, N)) return SQP_ERR_SHAPE;
    if ((N % 8) || (K % 8) || (group % 8) || (K % group)) return SQP_ERR_SHAPE;
    return SQP_OK;
}

static inline int sqp_launch_status()
{
    return hipGetLastError() == hipSuccess ? SQP_OK : SQP_ERR_LAUNCH;
}

// The device buffer the GEMM paths may use for fp32 partial sums when they split the inner
// dimension across workgroups: a ticket area (one counter per output tile, zero between
// launches: the last workgroup of a tile to arrive resets it) followed by the partial sums.
// It is never allocated here: it is the caller's buffer (sqp_set_workspace) or the library's
// static device array (sqp_w4a16_gemm_static).  partial == nullptr: none, plans do not split.
// own: scratch that belongs to this call alone (sqp_w4a16_gemm_scratch), for plans that split tiles of
// a grid that fills the chip by itself.  Those never go through the shared buffer: such calls may
// overlap with any other call.
constexpr size_t SQP_WS_TICKETS = (size_t)1 << 17;                       // counters
constexpr size_t SQP_WS_TICKET_BYTES = SQP_WS_TICKETS * sizeof(unsigned);  // 512 KB
struct SqpWorkspace {
    unsigned *tickets;
    float *partial;
    size_t partial_bytes;
    float *own;
    size_t own_bytes;
};
// The workspace the caller has set for the current device (partial == nullptr if none; own == nullptr).
SqpWorkspace sqp_caller_workspace();
// Enqueue a kernel that zeroes the ticket area.
int sqp_zero_tickets(unsigned *tickets, hipStream_t stream);

// Decode (weight-streaming) and prefill (tiled matrix-core) back ends of sqp_w4a16_gemm.
// Arguments are already validated.
// epi: 0 = y [M][N] fp16; 1 = SiLU(gate) * up of interleaved (gate, up) column pairs, y [M][N/2].
// A plan that splits K needs ws; without one (partial == nullptr) a plan that does not split runs; with one below
// the least size (see below) the call fails with SQP_ERR_WORKSPACE and enqueues nothing.
int sqp_gemm_decode(int M, int N, int K, int group, const h16 *x, const uint32_t *packed,
                    const h16 *scales, const uint8_t *zeros, h16 *y, int epi, const SqpWorkspace &ws, hipStream_t stream);
int sqp_gemm_prefill(int M, int N, int K, int group, const h16 *x, const uint32_t *packed,
                     const h16 *scales, const uint8_t *zeros, h16 *y, int epi, const SqpWorkspace &ws, hipStream_t stream);
// Shared by every GEMM entry point: argument checks and the choice between the two paths.
int sqp_gemm_entry(int M, int N, int K, int group, const void *x, const uint32_t *packed, const void *scales,
                   const uint8_t *zeros, void *y, int epi, const SqpWorkspace &ws, void *stream);
// Bytes of partial sums the preferred plan of a shape needs (0: it does not split K).
size_t sqp_gemm_decode_partial_bytes(int M, int N, int K, int group);
size_t sqp_gemm_prefill_partial_bytes(int M, int N, int K, int group);
// Bytes of the call's own scratch the preferred plan uses (0: none, or the workspace serves it).
size_t sqp_gemm_prefill_scratch_bytes(int M, int N, int K, int group);
// Bytes below which a call with a workspace is refused; between the two a plan that fits runs.
size_t sqp_gemm_decode_least_bytes(int M, int N, int K, int group);
size_t sqp_gemm_prefill_least_bytes(int M, int N, int K, int group);

// Compute units of the current device.
int sqp_compute_units();

// Eq. 6 in two steps: per-channel maxima amax = [max_t|x_cal[t][j]| (K) | max_n|w[j][n]| (K)],
// then the factor for one alpha.  Arguments are already validated.
int sqp_channel_absmax(int T, int K, int N, const void *x_cal, const void *w, float *amax, hipStream_t stream);
int sqp_smooth_factor(int K, float alpha, const float *amax, float *s, hipStream_t stream);
// The factors of n_alpha alphas (host array) at once: factors [n_alpha][K].
int sqp_smooth_factors(int K, int n_alpha, const float *alphas, const float *amax, float *factors, hipStream_t stream);
// x_hat = x / s (Eq. 5) and s * w quantised and packed (Eq. 5, Eq. 1), the smoothed weight kept in
// registers only: the same values as sqp_smooth_apply_x, sqp_smooth_apply_w and sqp_quantize_pack
// give, but every 8 k of x_hat in the order of the unpacked codes (k0, k4, k1, k5, k2, k6, k3, k7).
int sqp_smooth_quantize(int T, int N, int K, int group, const void *x, const void *w, const float *s, void *x_hat,
                        uint32_t *packed, void *scales, uint8_t *zeros, hipStream_t stream);

#ifdef __HIPCC__
// Streaming reads of a weight, every byte of which is touched once per call: the non-temporal
// hint lets them pass through the caches (a plain read probe streams 12-15 % faster with it on this
// chip; interleaving 5120 x 13824 twice 97 -> 89 us, and the maximum over its result that follows 65 ->
// 59).  Stores go without it: with hinted loads, plain stores are faster (weight scaling on
// 22016 x 8192 115 -> 105 us, transpose 147 -> 125 us), and so is the activation tensor's pass, which
// fits the Infinity Cache.
__device__ __forceinline__ uint4 load_stream(const uint4 *p)
{
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}

// SiLU(g) = g / (1 + exp(-g)) in fp32 (the hardware exponential: about 1 ulp of fp32).
__device__ __forceinline__ float sqp_silu(float g) { return g / (1.0f + __expf(-g)); }
#endif
