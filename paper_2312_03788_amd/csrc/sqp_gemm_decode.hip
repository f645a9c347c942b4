// Launch plans of the weight-streaming W4A16 GEMM (up to 64 rows) and its fallback kernel.  The
// kernels themselves: sqp_strip_kernel.h, sqp_slice_kernel.h.
#include <limits.h>

#include "sqp_slice.h"
#include "sqp_strip.h"

namespace {

constexpr size_t SQP_TICKET_STRIDE = 32;  // one ticket per 128-byte line, as the strip kernel lays them out

// Any group size that is a multiple of 8 and any M: one thread per output element.
// Correctness path for group sizes the matrix-core kernels do not cover.
__global__ void __launch_bounds__(256)
w4a16_generic_kernel(int M, int N, int K, int group, const h16 *__restrict__ x, const uint32_t *__restrict__ packed,
                     const h16 *__restrict__ scales, const uint8_t *__restrict__ zeros, h16 *__restrict__ y)
{
    const int n = blockIdx.x * 256 + threadIdx.x;
    const int m = blockIdx.y;
    if (n >= N) return;
    const h16 *xr = x + (size_t)m * K;
    float acc = 0.f;
    for (int g = 0; g < K / group; g++) {
        const float d = (float)scales[(size_t)g * N + n];
        const int z = zeros[(size_t)g * N + n];
        float accg = 0.f;
        for (int j = 0; j < group / 8; j++) {
            const int row = g * (group / 8) + j;
            const uint32_t w = packed[(size_t)row * N + n];
#pragma unroll
            for (int i = 0; i < 8; i++)
                accg = fmaf((float)xr[row * 8 + i], (float)((int)((w >> (4 * i)) & 15u) - z), accg);
        }
        acc = fmaf(d, accg, acc);
    }
    y[(size_t)m * N + n] = (h16)acc;
}

}  // namespace

// ---------------------------------------------------------------- launch

// Test/benchmark hooks: 1 = never two waves per strip; two chunks per iteration: 0 = automatic,
// 1 = never, 2 = wherever built.
int sqp_strip_kw_hook = 0;
int sqp_strip_kp_hook = 0;

// Two chunks per iteration (the kernel's KP = 2, twice the waves: two per SIMD where the launch
// has one workgroup per compute unit) pays once a workgroup walks at least 10 chunks: 5-10 %
// on the narrow 34B layers and on 11008->4096 / 13824->5120, a loss on ranges of 4 to 7 chunks
// (4096->4096, 5120->5120), where the pipeline is mostly ramp.
bool sqp_strip_two_chunks(int chunks, int split)
{
    if (sqp_strip_kp_hook == 1) return false;
    if (sqp_strip_kp_hook == 2) return true;
    return chunks / split >= 10;
}

// The split a launch really runs with (at most one part per chunk; none when the layer has
// more tiles than the workspace has tickets: such a layer fills the chip anyway) and the
// bytes of fp32 partial tiles it then leaves in the workspace.  blocks: row blocks of 16 mt rows.
int sqp_strip_split(int mt, int nw, int kspg, int blocks, int N, int K, int split, size_t *partial_bytes)
{
    const int tiles = (N + 64 * nw - 1) / (64 * nw) * blocks;
    const int chunks = K / (32 * kspg);
    if (split > chunks) split = chunks;
    if (split < 1) split = 1;
    if ((size_t)tiles * SQP_TICKET_STRIDE > SQP_WS_TICKETS) split = 1;
    *partial_bytes = split > 1 ? (size_t)tiles * split * nw * mt * 16 * 64 * sizeof(float) : 0;
    return split;
}

namespace {

typedef SqpStripPlan Plan;

// Test/benchmark hooks: force the K split, or strips and K split (0 = automatic).
int g_force_split = 0;
Plan g_force_plan = {0, 0, 0, 0};

// Strips per workgroup and K split, from sweeps on Code Llama shapes.  Four strips per
// workgroup share one copy of the activations.  Narrow layers (up to 128 column tiles) run
// best with at most one workgroup per compute unit (256 in all; one more than that and a
// second round of workgroups starts, which costs 20 % and more), each walking a long K
// range; wider ones with two to three workgroups per unit.  More splits than that cost
// more in fp32 partial tiles than the extra parallelism brings.
// Two strips per workgroup with half the split: the same number of waves when each strip
// has two (KW = 2: up to 32 rows, chunks of four k-steps), with half as many partial tiles to
// hand over but the activations fetched by twice as many workgroups.  That wins on the
// narrowest layers (up to 32 four-strip tiles) unless K is long (more than 24 chunks per
// workgroup), where the streaming phase outweighs the hand-over; with 17 to 32 rows the
// partial tiles are twice as large and it wins up to 40 tiles whatever K.  Without the two-wave
// variant, two strips only pay where 256 four-strip workgroups would get fewer than eight
// chunks each.
// kp_ok: the launch can take two chunks per iteration (up to 16 rows, groups of 128); then a
// layer of up to 40 four-strip tiles runs best in two-strip workgroups with half the split
// whatever K (8192->10240: 80 tiles x 3 instead of 40 x 6; 22016->8192: 64 x 4 instead of
// 32 x 8: half the partial tiles), if that leaves each workgroup at least 16 chunks.
Plan make_plan(int M, int N, int K, int chunk, bool kp_ok)
{
    const int chunks = K / chunk;
    int max_split = chunks / 4;  // at least four chunks per workgroup
    if (max_split < 1) max_split = 1;
    auto split_for = [&](int tiles) {
        int want = tiles <= 128 ? 256 / tiles : (704 + tiles / 2) / tiles;
        if (want > max_split) want = max_split;
        return want < 1 ? 1 : want;
    };
    Plan p = {4, 1, 0, 0};
    const int tiles4 = (N + 255) / 256;
    p.split = split_for(tiles4);
    const int split2 = split_for((N + 127) / 128);
    const bool two_waves = M <= 32 && chunk == 128;  // the launch will give each strip two waves
    bool two_strips;
    if (two_waves && M <= 16)
        two_strips = (tiles4 <= 32 && chunks <= 24 * split2) || (kp_ok && sqp_strip_kp_hook != 1 && tiles4 <= 40 && chunks / split2 >= 16);
    else if (two_waves) two_strips = tiles4 <= 40;  // 17..32 rows: partial tiles twice as large, so also with a long K
    else two_strips = tiles4 <= 24 && chunks < 8 * (256 / tiles4);
    if (two_strips) {
        p.nw = 2;
        p.split = split2;
    }
    // More than 32 rows: the fp32 partial tiles are four times as large and the last arrival's
    // fetch of them is bound by its one compute unit, so the same waves are grouped into twice as
    // many workgroups of two strips (half the bytes per fetching unit; 1-6 % faster at M = 64).
    if (M > 32 && p.nw == 4 && p.split > 1) p.nw = 2;
    return p;
}

// The plan of calls with 17 to 64 rows, and of groups of 32 and 64 at any of these row counts: two
// strips per workgroup, two waves per strip, and eight waves (two chunks per iteration) wherever a
// workgroup walks at least eight chunks.  With that many rows a wave alone on its SIMD runs unpack
// and MFMAs one after the other (2500 cycles per chunk at 48 rows, of which the MFMAs are 770), two
// overlap; and two strips with the K split in the workgroup leave half the partial tiles that four
// strips leave.  One workgroup per compute unit (256), at least four chunks each (two on layers
// too small to fill half the chip otherwise).
// Exceptions, from sweeps over strips, waves and parts (us per launch, before -> plan taken):
//   - one part would leave the chip emptier than two four-wave workgroups per unit by a quarter of the
//     work (129 to 170 tiles): those (5120->18432, 48 rows: 28.4 with eight waves, 23.7);
//   - more than 256 tiles: two four-wave workgroups per unit in turn (8192->44032, 48 rows: 77.5 ->
//     66.8; 24 rows, groups of 64: 59 -> 54); four strips with one wave each up to 32 rows in groups
//     of 128 (20 rows: 52.7 against 57.2) and up to 16 rows (groups of 64: 44.5 against 46.5);
//   - up to 32 rows and more than 32 chunks per workgroup: four strips with half the K range each
//     (22016->8192, 20 rows: 27.3 against 29.8), the activations then cost more than the hand-over.
// Plain cases: 48 rows 5120->15360 24.1 -> 21.3, 5120->5120 18.3 -> 13.6, 13824->5120 26.8 -> 19.1,
// 5120->27648 36 -> 30; 20 rows, groups of 64: 4096->4096 11.4 -> 8.7, 11008->4096 18.7 -> 12.6,
// 4096->22016 28 -> 20.3.
Plan wide_plan(int M, int N, int K, int group)
{
    const int chunks = K / 128, tiles2 = (N + 127) / 128, tiles4 = (N + 255) / 256;
    auto capped = [&](int want, int least) {  // at least `least` chunks per workgroup
        const int most = chunks / least;
        return want > most ? (most < 1 ? 1 : most) : (want < 1 ? 1 : want);
    };
    if (tiles2 > 256) {
        if (M <= 16 || (M <= 32 && group % 128 == 0)) return Plan{4, capped((704 + tiles4 / 2) / tiles4, 4), 1, 1};
        return Plan{2, capped((704 + tiles2 / 2) / tiles2, 4), 2, 1};
    }
    int split = capped(256 / tiles2, 4);
    if (2 * tiles2 * split < 256) split = capped(256 / tiles2, 2);
    if (M <= 32 && group % 128 == 0 && chunks > 32 * split) return Plan{4, capped(256 / tiles4, 4), 1, 2};
    const int split4w = capped(512 / tiles2, 4);
    if (chunks >= 8 * split && 10 * tiles2 * split4w > 26 * tiles2 * split) return Plan{2, split4w, 2, 1};
    return Plan{2, split, 2, chunks >= 8 * split ? 2 : 1};
}

// k-steps per chunk of the kernel a group size takes (0: the generic kernel): four, i.e. 128 k, also
// for groups of 32 and 64 (several groups per chunk); those with K not a multiple of 128 take
// chunks of one group, and so do the plans of one or eight strips that a test hook can force.
int chunk_ksteps(int K, int group)
{
    const bool odd_strips = g_force_plan.nw == 1 || g_force_plan.nw == 8;
    if (group % 128 == 0 || ((group == 32 || group == 64) && K % 128 == 0 && !odd_strips)) return 4;
    return group == 32 ? 1 : (group == 64 ? 2 : 0);
}

// A test hook that forces a plan by strips keeps a call from the column slices.
bool strips_forced() { return g_force_plan.nw > 0 || g_force_split > 0; }

}  // namespace

extern "C" void sqp_debug_set_decode_split(int split) { g_force_split = split; }
extern "C" void sqp_debug_set_decode_plan(int nw, int split) { g_force_plan = Plan{nw, split, 0, 0}; }
extern "C" void sqp_debug_set_decode_kw(int kw) { sqp_strip_kw_hook = kw; }
extern "C" void sqp_debug_set_decode_kp(int kp) { sqp_strip_kp_hook = kp; }
static int g_slice_mode = 0;
extern "C" void sqp_debug_set_decode_slice(int mode) { g_slice_mode = mode; }

// Layers that fill the chip with slices of 32 (0) or 64 (1) columns and take them whatever the rule of
// slice_plan below says (-1: none; up to 16 rows, groups of 128).  The slice kernel has no
// hand-over between workgroups, but every workgroup fetches all of x from L2, and that traffic
// (workgroups x fetched rows x K) is what it costs.  It wins up to 8 rows (a third to a half of
// the activation traffic of 16 rows at K = 8192) and beyond that where x is small (short K) and
// the strip kernel is furthest from its roofline (narrow layers): 64-column slices from 150
// slices on (more than 8 rows: up to 128 KB of x per workgroup, or up to 192 KB and at most 400
// slices); below that 32-column slices, unless K is long and the slices are few (then the
// activations dominate again; 5 to 12 rows: only with K up to 8192, 13 to 16: up to 4096).
static int slice_variant(int M, int N, int K, int group)
{
    if (M > 16 || group != 128) return -1;
    const long xbytes = 4L * ((M + 3) / 4) * K * 2;  // activations a workgroup fetches
    const int slices64 = (N + 63) / 64, slices32 = (N + 31) / 32;
    if (slices64 >= 150) return (M <= 8 || xbytes <= (128L << 10) || (xbytes <= (192L << 10) && slices64 <= 400)) ? 1 : -1;
    if (slices32 >= 96 && (slices32 >= 200 || K <= 8192)) return (M <= 4 || (M <= 12 && K <= 8192) || K <= 4096) ? 0 : -1;
    return -1;
}
extern "C" int sqp_debug_decode_slice_choice(int M, int N, int K, int group) { return slice_variant(M, N, K, group); }
static SqpSlicePlan g_slice_plan = {0, 0, false};
extern "C" void sqp_debug_set_slice_plan(int tb, int wv, int grouped) { g_slice_plan = SqpSlicePlan{tb, wv, grouped != 0}; }

// Whether a call of up to 32 rows takes the column-slice kernel, and how wide its slices are.
//   Width: the narrowest that fits the chip in one round, i.e. 16 columns up to 4096, 32 up to 8192, 64 from
//   there on (one workgroup too many costs a round: 4352 columns in 16s 10.8 us, in 32s 8.7 at one row and
//   K = 8192).  Above 16384 columns 64, or 32 in groups of 32 up to 16 rows and 32768 columns (their unpack
//   is the longer one: 22016 columns, K = 2112, 6 rows 12.3 -> 9.8 us).
//   Waves: eight; 16 for one to four rows on narrow layers with long K (4096->1024 at one row 4.7 -> 4.4 us);
//   four with 64 columns, up to 8 rows and two slices per compute unit (4096->22016 at one row 12.8 -> 11.6).
//   K: the strip kernel's hand-over costs about the same whatever K, the slices' latency and activations grow
//   with K, so K above `longest` goes to the strips: us at 1 / 8 / 16 / 32 rows, strips against slices, N = 1024:
//   K = 4096 7.1 / 7.2 / 7.3 / 9.2 against 4.4 / 5.0 / 5.9 / 7.3, K = 12288 9.4 / 9.5 / 9.9 / 11.9 against
//   8.5 / 10.5 / 13.0 / 17.4.  From 257 to 320 and from 513 to 576 slices of 64 columns the chip is a round or two
//   and a little full, and short K only is worth it (17904 columns, K = 9984, 5 rows: 30.3 against 24.2).  K not
//   a multiple of 128: the strips take chunks of one group there, so slices pay up to 1.6 times that K, from
//   8192 columns on with any.  Above 8192 columns groups of several chunks hold out longer (the strip kernel
//   takes one chunk per iteration there).  Rows of packed words that are not whole 128-byte lines (N % 32) cost
//   slices more lines than strips: 20840 columns, K = 13952, one row 41.5 against 32.6, 21920 columns, K = 12032
//   30.9 against 35.5.
//   The lengths have the least time over 10430 calls (1 to 32 rows, N 512 to 44032, K 512 to 22016, groups of 32 to
//   384, most of them drawn over these ranges, weights from HBM), what is slower than before slices took these
//   calls counted several times.  On 3223 other calls drawn likewise: 1.28 times faster than before in the
//   geometric mean, 1.3 % behind the best variant of each; 1.5 % of them more than 3 % slower than before, at
//   worst 15 % (the sweep is among the profiles).
//   Without a workspace the strips cannot split K: slices are taken wherever they would, but for 17 and more rows
//   and K below 3072 above 16384 columns (0.86 to 1.1 there).  1 to 32 rows without one, strips against slices: 3.9 times their time in the mean of 263 such
//   calls up to 4096 columns, 3.6 (54) up to 8192, 2.5 (18) up to 16384, 1.6 (60) from there on.
static Plan plan_for(int M, int N, int K, int group, bool have_workspace);
static SqpSlicePlan slice_plan(int M, int N, int K, int group, bool have_workspace)
{
    const SqpSlicePlan none = {0, 0, false};
    if (g_slice_mode < 0 || M > 32 || (group != 32 && group != 64 && group % 128 != 0)) return none;
    if (g_slice_plan.tb > 0) return g_slice_plan;
    if (g_slice_mode > 0) return SqpSlicePlan{2 * g_slice_mode, 8, false};
    if (strips_forced()) return none;
    const int blocks = M > 16 ? 4 : (M + 3) / 4 - 1;  // blocks of four rows less one; 17 to 32 rows
    constexpr int ANY = 1 << 28;
    static const struct { int columns, longest[5]; } lengths[9] = {
        {2048, {12288, 8192, 7168, 6144, 6144}},
        {4096, {13312, 9728, 8704, 6144, 5632}},
        {8192, {13312, 12288, 9728, 6656, 6144}},
        {12288, {16384, 13312, 12288, 7168, 7168}},
        {16384, {ANY, ANY, 20480, 11264, 13312}},
        {20480, {4096, 2560, 2560, 2048, 0}},
        {32768, {16384, 8192, 7680, 4096, 0}},
        {36864, {3072, 2816, 2048, 1536, 0}},
        {INT_MAX, {9728, 9216, 8192, 4096, 2048}},
    };
    int row = 0;
    while (N > lengths[row].columns) row++;
    double most = lengths[row].longest[blocks];
    if (N > 16384) most *= group == 32 ? 0.85 : (group > 128 ? 2.0 : 1.0);
    else if (N > 8192 && group == 32) most = 11264;
    else if (N > 8192 && M > 12 && group > 128) most *= 1.6;
    if (N > 32768 && M > 16 && K < 1024) most = 0;
    if (N % 32 != 0) most *= group <= 64 ? 0.8 : (N > 8192 ? 0.9 : 1.0);
    if (K % 128 != 0) {
        if (N <= 8192) most *= 1.6;
        else if (N > 16384 && N <= 20480 && group == 64 && M > 8) most = 2048;
        else if (N <= 32768 || M > 16) most = ANY;
        else most *= group == 32 && M > 8 ? 0.0 : 0.75;
    }
    if (K > most && slice_variant(M, N, K, group) < 0 && (have_workspace || (N > 16384 && M > 16 && K < 3072) || plan_for(M, N, K, group, true).split < 2)) return none;
    const int width = N <= 4096 ? 0 : (N <= 8192 ? 1 : (N <= 16384 ? 2 : 3));
    SqpSlicePlan p = {width == 0 ? 1 : (width == 1 ? 2 : 4), 8, width < 2};
    if (group == 32 && width == 3 && N <= 32768 && M <= 16) p.tb = 2, p.grouped = true;
    if (M <= 16 && width < 2 && K > 2048 && M <= (width == 0 ? 4 : 2)) p.wv = 16;
    if (M <= 8 && p.tb == 4 && width == 3 && N <= 32768 && group >= 64) p.wv = 4;
    return p;
}

// Calls that take slices and report no workspace.  The others that take them, since the rule above, go on
// reporting what the strip kernel would use, and are refused with less: sizes that callers have
// stored, and what they were told about too small a buffer, stay true.
static bool slices_alone(int M, int N, int K, int group)
{
    if (g_slice_mode < 0) return false;
    return g_slice_plan.tb > 0 || g_slice_mode > 0 || strips_forced() ? slice_plan(M, N, K, group, true).tb > 0 : slice_variant(M, N, K, group) >= 0;
}

extern "C" void sqp_debug_decode_slice_plan(int M, int N, int K, int group, int *tb, int *wv)
{
    const SqpSlicePlan p = slice_plan(M, N, K, group, true);
    *tb = p.tb;
    *wv = p.wv;
}

int sqp_gemm_generic(int M, int N, int K, int group, const h16 *x, const uint32_t *packed, const h16 *scales,
                     const uint8_t *zeros, h16 *y, hipStream_t stream)
{
    if (M > 65535) return SQP_ERR_SHAPE;
    w4a16_generic_kernel<<<dim3((N + 255) / 256, M), 256, 0, stream>>>(M, N, K, group, x, packed, scales, zeros, y);
    return sqp_launch_status();
}

// Test hook: the launch plan by strips (no launch, no GPU needed): strips per workgroup, K split as
// requested by the heuristic, and the kernel family (0 = generic, else k-steps of one group).  Calls
// with up to 16 rows and groups of 128 run it, and so do chunks of one group of 32 or 64; the others
// run wide_plan.
extern "C" void sqp_debug_decode_plan(int M, int N, int K, int group, int *nw, int *split, int *kspg)
{
    const int chunk = group % 128 == 0 ? 128 : group;
    const Plan p = make_plan(M, N, K, chunk, M <= 16 && group == 128);
    *nw = p.nw;
    *split = p.split;
    *kspg = group == 32 ? 1 : (group == 64 ? 2 : (group % 128 == 0 ? 4 : 0));
}

// Bytes of partial tiles a plan leaves (kspg: k-steps per chunk, mt: 16-row tiles of the kernel).
static size_t plan_bytes(const Plan &p, int N, int K, int group, int kspg, int mt)
{
    const bool one_group = kspg < 4 || group % 128 == 0;  // one and eight strips (test hooks) exist there only
    int nw = p.nw;
    if (nw != 2 && !(nw == 1 && one_group) && !(nw == 8 && one_group && mt < 3)) nw = 4;
    size_t bytes = 0;
    sqp_strip_split(mt, nw, kspg, 1, N, K, p.split, &bytes);
    return bytes;
}

// Fewer K parts where the partial tiles would not fit `room` bytes (one part needs none).
static void fit_split(Plan &p, int N, int K, int group, int kspg, int mt, size_t room)
{
    while (p.split > 1 && plan_bytes(p, N, K, group, kspg, mt) > room) p.split--;
}

// The same for the plan by strips: one group per chunk, row tiles in steps of 16, 32 and 64.
static size_t strips_bytes(int M, int N, int K, int group)
{
    const int kspg = group == 32 ? 1 : (group == 64 ? 2 : 4), mt = M <= 16 ? 1 : (M <= 32 ? 2 : 4);
    Plan p = make_plan(M, N, K, kspg == 4 ? 128 : group, M <= 16 && group == 128);
    fit_split(p, N, K, group, kspg, mt, SQP_STATIC_PARTIAL_BYTES);
    return plan_bytes(p, N, K, group, kspg, mt);
}

// The plan a call runs with: the heuristic's, overridden by the test hooks, without a split
// when there is no workspace to put partial sums in.
static Plan plan_for(int M, int N, int K, int group, bool have_workspace)
{
    const int chunk = 32 * chunk_ksteps(K, group);
    Plan p;
    if (chunk == 128 && (M > 16 || group < 128)) {
        p = wide_plan(M, N, K, group);
        // Where the plan by strips does not split (fewer than eight chunks of K, or 470 and more four-strip
        // tiles) nothing is split: such a shape reports no workspace, and callers run it beside calls
        // that use theirs.
        if (strips_bytes(M, N, K, group) == 0) p.split = 1;
    } else {
        p = make_plan(M, N, K, chunk, M <= 16 && group == 128);
    }
    // No plan of the library's own needs more than the static array holds.  (Rounding can take one past it:
    // 623 two-strip tiles x 5 parts x 16 KB, 6976 -> 39816 in groups of 64.)
    if (chunk) fit_split(p, N, K, group, chunk / 32, sqp_strip_row_tiles(M), SQP_STATIC_PARTIAL_BYTES);
    if (g_force_plan.nw > 0) p = g_force_plan;
    if (g_force_split > 0) p.split = g_force_split;
    if (!have_workspace) p.split = 1;
    return p;
}

// Test hook: what a call launches if it takes the strip kernel (kw, kp 0: by the rules at the launch).
extern "C" void sqp_debug_decode_launch(int M, int N, int K, int group, int *nw, int *split, int *kw, int *kp)
{
    const Plan p = chunk_ksteps(K, group) ? plan_for(M, N, K, group, true) : Plan{0, 0, 0, 0};
    *nw = p.nw;
    *split = p.split;
    *kw = p.kw;
    *kp = p.kp;
}

size_t sqp_gemm_decode_partial_bytes(int M, int N, int K, int group)
{
    const int kspg = chunk_ksteps(K, group);
    if (kspg == 0) return 0;  // generic kernel
    if (slices_alone(M, N, K, group)) return 0;
    return plan_bytes(plan_for(M, N, K, group, true), N, K, group, kspg, sqp_strip_row_tiles(M));
}

// What a workspace has to hold at least for a call not to be refused: the partial tiles of the plan
// by strips, where wide_plan asks for more.
// Callers with a buffer of that size are served with fewer K parts.
size_t sqp_gemm_decode_least_bytes(int M, int N, int K, int group)
{
    const size_t want = sqp_gemm_decode_partial_bytes(M, N, K, group);
    if (want == 0 || g_force_plan.nw > 0 || g_force_split > 0) return want;
    const size_t strips = strips_bytes(M, N, K, group);
    return strips < want ? strips : want;
}

int sqp_gemm_decode(int M, int N, int K, int group, const h16 *x, const uint32_t *packed, const h16 *scales,
                    const uint8_t *zeros, h16 *y, int epi, const SqpWorkspace &ws, hipStream_t stream)
{
    SqpSlicePlan sp = slice_plan(M, N, K, group, ws.partial != nullptr);
    if (sp.tb) {
        if (ws.partial != nullptr && ws.partial_bytes < sqp_gemm_decode_least_bytes(M, N, K, group)) return SQP_ERR_WORKSPACE;
        if (epi != 0 && sp.tb == 1) sp.tb = 2;  // a lane's columns are whole (gate, up) pairs
        if (group == 32) return sqp_slice_g32(sp, M, N, K, 1, x, packed, scales, zeros, y, epi, stream);
        if (group == 64) return sqp_slice_g64(sp, M, N, K, 1, x, packed, scales, zeros, y, epi, stream);
        if (group == 128) return sqp_slice_g128(sp, M, N, K, 1, x, packed, scales, zeros, y, epi, stream);
        return sqp_slice_g256(sp, M, N, K, group / 128, x, packed, scales, zeros, y, epi, stream);
    }
    const int kspg = chunk_ksteps(K, group);
    if (kspg == 0) {
        if (epi != 0) return SQP_ERR_SHAPE;  // the fused activation needs a group size the matrix-core kernels cover
        return sqp_gemm_generic(M, N, K, group, x, packed, scales, zeros, y, stream);
    }
    Plan p = plan_for(M, N, K, group, ws.partial != nullptr);
    if (ws.partial != nullptr && ws.partial_bytes >= sqp_gemm_decode_least_bytes(M, N, K, group))
        fit_split(p, N, K, group, kspg, sqp_strip_row_tiles(M), ws.partial_bytes);
    if (kspg < 4) return sqp_strip_one_group(group, p, M, N, K, 1, x, packed, scales, zeros, y, epi, ws, stream);
    if (group == 32) return sqp_strip_g32(p, M, N, K, 1, x, packed, scales, zeros, y, epi, ws, stream);
    if (group == 64) return sqp_strip_g64(p, M, N, K, 1, x, packed, scales, zeros, y, epi, ws, stream);
    if (M <= 32) return sqp_strip_g128_rows32(p, M, N, K, group / 128, x, packed, scales, zeros, y, epi, ws, stream);
    return sqp_strip_g128_rows64(p, M, N, K, group / 128, x, packed, scales, zeros, y, epi, ws, stream);
}
