"""GPU parity for the W4A16 GEMM (Eq. 3) against the oracle's fp64 definition:
|y_gpu - y_ref| <= 1e-3 * sum_k|x_k w_hat_k| + 1 fp16 ulp per element."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as wl
from gpu_util import dev, gemm_tolerance_ok, host, silu_tolerance

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sqp():
    import paper_2312_03788_amd as m
    m.lib()
    return m


def _layer(orc, M, K, N, group, shape_idx=0):
    """Smoothed + quantised layer operands from the oracle (numpy)."""
    x, xcal, w = wl.layer_inputs(M, K, N, shape_idx=shape_idx)
    s = orc.smooth_scales(xcal, w, wl.ALPHA)
    xs = orc.smooth_apply_x(x, s)
    ws = orc.smooth_apply_w(w, s)
    p, sc, z = orc.quantize_pack(ws, group)
    return xs, p, sc, z


def _check(orc, sqp, xs, p, sc, z, group):
    y_ref, t_ref = orc.w4a16_gemm_ref(xs, p, sc, z, group)
    y = host(sqp.w4a16_gemm(dev(xs), dev(p), dev(sc), dev(z), group))
    torch.cuda.synchronize()
    ok, worst, nbad = gemm_tolerance_ok(orc, y, y_ref, t_ref)
    assert ok, "worst err/tol %.3f, %d elements out of tolerance" % (worst, nbad)
    return y


def test_cfg1_single_layer(orc, sqp):
    """M=4, K=N=1024, group 128, alpha=0.5, outlier channels."""
    print("case cfg1", flush=True)
    xs, p, sc, z = _layer(orc, 4, 1024, 1024, 128)
    _check(orc, sqp, xs, p, sc, z, 128)


@pytest.mark.parametrize("M", [1, 2, 7, 8, 15, 16, 17, 31, 32, 33, 48, 63, 64])
def test_decode_row_counts(orc, sqp, M):
    print("case rows", M, flush=True)
    xs, p, sc, z = _layer(orc, M, 512, 192, 128)
    _check(orc, sqp, xs, p, sc, z, 128)


@pytest.mark.parametrize("group", [32, 64, 128, 256])
@pytest.mark.parametrize("M", [33, 47, 48, 49, 64])
def test_rows_33_to_64_take_the_rounded_weight(sqp, M, group):
    """33 to 64 rows multiply w_hat = fp16((code - Z) Delta), the value sqp_dequantize gives: a row of
    x with two ones is the fp16 rounding of a sum of two such values, which fp32 holds exactly (steps
    within a factor of 8 and codes up to 15, so exponents less than 13 apart)."""
    print("case rounded weight", M, group, flush=True)
    K, N = 768, 72
    rng = np.random.Generator(np.random.PCG64(1000 * group + M))
    p = rng.integers(0, 2**32, size=(K // 8, N), dtype=np.uint32)
    sc = rng.uniform(0.01, 0.08, size=(K // group, N)).astype(np.float16)
    z = rng.integers(0, 16, size=(K // group, N), dtype=np.uint8)
    x = np.zeros((M, K), np.float16)
    at = np.stack([rng.choice(K, 2, replace=False) for _ in range(M)])
    x[np.arange(M)[:, None], at] = 1.0
    dp, dsc, dz = dev(p), dev(sc), dev(z)
    w_hat = host(sqp.dequantize(dp, dsc, dz, group)).astype(np.float32)
    y = host(sqp.w4a16_gemm(dev(x), dp, dsc, dz, group))
    assert np.array_equal(y, (w_hat[at[:, 0]] + w_hat[at[:, 1]]).astype(np.float16))


@pytest.mark.parametrize("M,K,N,group", [
    (3, 128, 8, 128), (5, 256, 72, 128), (16, 384, 520, 128), (9, 1152, 200, 128), (4, 256, 64, 32),
    (16, 320, 136, 64), (33, 1024, 264, 256), (2, 48, 24, 24), (6, 64, 16, 8), (64, 2048, 1000, 128),
    (8, 1024, 264, 1024), (16, 2048, 136, 2048), (40, 1536, 72, 512)])  # the last three: one group per column / long groups
def test_decode_ragged_shapes(orc, sqp, M, K, N, group):
    print("case ragged", M, K, N, group, flush=True)
    xs, p, sc, z = _layer(orc, M, K, N, group)
    _check(orc, sqp, xs, p, sc, z, group)


@pytest.mark.parametrize("split", [1, 2, 3, 5, 8])
def test_decode_split_k_deterministic(orc, sqp, split):
    """Every K split gives an in-tolerance result, and repeated runs are bit-identical."""
    print("case split", split, flush=True)
    L = sqp.lib()
    xs, p, sc, z = _layer(orc, 16, 2048, 328, 128)
    L.sqp_debug_set_decode_split(split)
    try:
        y0 = _check(orc, sqp, xs, p, sc, z, 128)
        for _ in range(3):
            y1 = _check(orc, sqp, xs, p, sc, z, 128)
            assert np.array_equal(y0.view(np.uint16), y1.view(np.uint16))
    finally:
        L.sqp_debug_set_decode_split(0)


def test_integer_exact(orc, sqp):
    """step = 1, Z = 0, small integer activations: every partial sum is an exact integer in
    fp32, so the GPU result must equal the integer product exactly."""
    rng = np.random.Generator(np.random.PCG64(3))
    M, N, K, g = 16, 96, 512, 128
    q = rng.integers(0, 16, size=(K, N))
    x = rng.integers(-4, 5, size=(M, K))
    p = np.zeros((K // 8, N), np.uint32)
    for i in range(8):
        p |= q[i::8].astype(np.uint32) << np.uint32(4 * i)
    ones = np.ones((K // g, N), np.float16)
    zz = np.zeros((K // g, N), np.uint8)
    y = host(sqp.w4a16_gemm(dev(x.astype(np.float16)), dev(p), dev(ones), dev(zz), g))
    assert np.array_equal(y.astype(np.int64), x @ q)


def test_tiny_activations(orc, sqp):
    """Activations in the fp16 subnormal range still meet the tolerance."""
    xs, p, sc, z = _layer(orc, 8, 512, 128, 128)
    xs = (xs.astype(np.float32) * 2.0 ** -16).astype(np.float16)
    _check(orc, sqp, xs, p, sc, z, 128)


@pytest.mark.parametrize("shape_idx", [0, 1, 2, 3])
@pytest.mark.parametrize("M", [1, 8, 12, 16])
def test_cfg2_7b_shapes(orc, sqp, shape_idx, M):
    """Code Llama-7B layer shapes at decode row counts, full-output parity (the library's own
    plan: column slices of 64 or 32 columns up to 12 rows on three of the shapes, strips
    otherwise)."""
    K, N = wl.MODEL_SHAPES["7b"][shape_idx]
    print("case 7b", K, N, M, flush=True)
    xs, p, sc, z = _layer_cached(orc, M, K, N, shape_idx)
    _check(orc, sqp, xs, p, sc, z, 128)


@pytest.mark.parametrize("shape_idx", [0, 1, 2, 3])
def test_cfg4_34b_decode_shapes(orc, sqp, shape_idx):
    """The four Code Llama-34B layer shapes at M = 16 with the library's own launch plan:
    the configuration the benchmark times.  Full-output parity against the oracle."""
    K, N = wl.MODEL_SHAPES["34b"][shape_idx]
    print("case 34b", K, N, 16, flush=True)
    xs, p, sc, z = _layer_cached(orc, 16, K, N, shape_idx)
    _check(orc, sqp, xs, p, sc, z, 128)


_cache = {}


def _layer_cached(orc, M, K, N, shape_idx):
    """Quantise each big weight once per session (the oracle quantiser is slow)."""
    key = (K, N, shape_idx)
    if key not in _cache:
        _, xcal, w = wl.layer_inputs(1, K, N, shape_idx=shape_idx)
        s = orc.smooth_scales(xcal, w, wl.ALPHA)
        ws = orc.smooth_apply_w(w, s)
        _cache.clear()
        _cache[key] = (s,) + orc.quantize_pack(ws, 128)
    s, p, sc, z = _cache[key]
    x = wl.activation(M, K, seed=2000 + M)
    return orc.smooth_apply_x(x, s), p, sc, z


# ---------------------------------------------------------------- prefill (M > 64)

@pytest.mark.parametrize("M,K,N,group", [
    (65, 256, 264, 128), (256, 512, 256, 64), (300, 1024, 520, 128), (130, 384, 72, 64),
    (129, 512, 136, 256), (100, 128, 64, 32), (257, 192, 8, 64), (512, 2048, 1000, 128),
    (130, 1024, 264, 1024), (300, 1024, 520, 32), (257, 192, 72, 32), (140, 96, 136, 32)])
@pytest.mark.parametrize("tiles", [0, 1, 2])
@pytest.mark.parametrize("shape", [1, 2])
def test_prefill_shapes(orc, sqp, M, K, N, group, tiles, shape):
    """Tiled matrix-core path: full-output parity on shapes spanning several tiles with
    ragged edges in M and N, several group sizes (32 takes the fallback path); with the
    automatic tile choice, with full tiles only and with half-width tiles only; for both
    full-tile shapes (1: 128 x 512, 2: 256 x 256)."""
    print("case prefill", M, K, N, group, tiles, shape, flush=True)
    xs, p, sc, z = _layer(orc, M, K, N, group)
    L = sqp.lib()
    L.sqp_debug_set_prefill_tiles(tiles)
    L.sqp_debug_set_prefill_shape(shape)
    try:
        _check(orc, sqp, xs, p, sc, z, group)
    finally:
        L.sqp_debug_set_prefill_tiles(0)
        L.sqp_debug_set_prefill_shape(0)


@pytest.mark.parametrize("M,K,N,group,ksplit", [
    (300, 1024, 520, 128, 2), (300, 1024, 520, 128, 3), (65, 256, 264, 128, 2), (130, 384, 72, 64, 3),
    (129, 512, 136, 256, 4), (257, 1024, 264, 128, 16), (300, 1024, 520, 1024, 3), (300, 1024, 520, 32, 3), (130, 512, 72, 32, 8)])
@pytest.mark.parametrize("shape", [1, 2])
def test_prefill_k_split(orc, sqp, M, K, N, group, ksplit, shape):
    """Tiled path with K split across workgroups (fp32 partial matrices added in part order):
    parts that start inside a quantisation group, ragged M and N; twice, bit-identical."""
    print("case prefill ksplit", M, K, N, group, ksplit, shape, flush=True)
    xs, p, sc, z = _layer(orc, M, K, N, group)
    L = sqp.lib()
    L.sqp_debug_set_prefill_ksplit(ksplit)
    L.sqp_debug_set_prefill_shape(shape)
    try:
        y_ref, t_ref = orc.w4a16_gemm_ref(xs, p, sc, z, group)
        args = (dev(xs), dev(p), dev(sc), dev(z), group)
        y = host(sqp.w4a16_gemm(*args))
        y2 = host(sqp.w4a16_gemm(*args))
    finally:
        L.sqp_debug_set_prefill_ksplit(-1)
        L.sqp_debug_set_prefill_shape(0)
    assert np.array_equal(y.view(np.uint16), y2.view(np.uint16))
    ok, worst, nbad = gemm_tolerance_ok(orc, y, y_ref, t_ref)
    assert ok, "worst err/tol %.3f, %d elements out of tolerance" % (worst, nbad)


@pytest.mark.parametrize("rt,nt,parts", [(3, 2, 1), (3, 2, 4), (4, 2, 2), (4, 4, 1), (5, 2, 1), (5, 2, 3), (6, 2, 1), (6, 2, 5)])
@pytest.mark.parametrize("M,K,N,group", [
    (65, 64, 8, 64), (96, 320, 264, 64), (97, 1024, 520, 128), (160, 640, 256, 128), (161, 384, 776, 192),
    (192, 512, 248, 512), (193, 768, 264, 256), (321, 448, 1032, 64)])
def test_prefill_tile_heights(orc, sqp, M, K, N, group, rt, nt, parts):
    """Tiles of 96, 128, 160 and 192 rows with and without K parts, and of 512 columns: one row or column
    past a tile and one short of it, one stage, parts that start inside a group; plain and with
    the fused activation; repeated runs are bit-identical."""
    print("case tile heights", M, K, N, group, rt, nt, parts, flush=True)
    xs, p, sc, z = _layer(orc, M, K, N, group)
    L = sqp.lib()
    L.sqp_debug_set_prefill_variant(rt, nt, parts)
    try:
        y0 = _check(orc, sqp, xs, p, sc, z, group)
        y1 = _check(orc, sqp, xs, p, sc, z, group)
    finally:
        L.sqp_debug_set_prefill_variant(0, 0, 0)
    assert np.array_equal(y0.view(np.uint16), y1.view(np.uint16))


@pytest.mark.parametrize("rt,nt", [(3, 2), (4, 2), (4, 4), (5, 2), (6, 2)])
@pytest.mark.parametrize("stages", [1, 2, 3, 4, 5, 7])
def test_prefill_few_stages(orc, sqp, rt, nt, stages):
    """Every remainder of the loop over three stages of 64 k, and calls of fewer, at each tile size, on grids of tiles
    that do not divide among the eight XCDs nor into equal groups of tile rows (9 or more rows of tiles)."""
    M, K, N = 9 * 32 * rt - 5, 64 * stages, 392
    print("case few stages", M, K, N, rt, nt, flush=True)
    xs, p, sc, z = _layer(orc, M, K, N, 64)
    L = sqp.lib()
    L.sqp_debug_set_prefill_variant(rt, nt, 1)
    try:
        _check(orc, sqp, xs, p, sc, z, 64)
    finally:
        L.sqp_debug_set_prefill_variant(0, 0, 0)


@pytest.mark.parametrize("tiles", [1, 2])
@pytest.mark.parametrize("stages", [1, 2, 3, 4, 5, 7])
def test_prefill_few_stages_groups_of_32(orc, sqp, tiles, stages):
    """The same in groups of 32, whose full and half-width tiles have two groups per stage."""
    M, K, N = 2 * 128 - 5, 64 * stages, 520
    print("case few stages, groups of 32", M, K, N, tiles, flush=True)
    xs, p, sc, z = _layer(orc, M, K, N, 32)
    L = sqp.lib()
    L.sqp_debug_set_prefill_tiles(tiles)
    L.sqp_debug_set_prefill_ksplit(0)
    try:
        _check(orc, sqp, xs, p, sc, z, 32)
    finally:
        L.sqp_debug_set_prefill_tiles(0)
        L.sqp_debug_set_prefill_ksplit(-1)


@pytest.mark.parametrize("rt", [4, 5])
@pytest.mark.parametrize("M_off,K,N,group", [(0, 64, 8, 64), (-1, 448, 384, 64), (1, 320, 392, 320), (70, 1024, 760, 256), (-40, 640, 96, 128)])
def test_prefill_three_columns_per_lane(orc, sqp, M_off, K, N, group, rt):
    """Tiles of 384 columns: rows and columns at the edges of a tile, of a wave's 96 columns and of a lane's three (the
    last columns of a row end in the middle of a lane's), plain and with the fused activation."""
    M = 32 * rt + M_off
    print("case three columns", M, K, N, group, rt, flush=True)
    xs, p, sc, z = _layer(orc, M, K, N, group)
    L = sqp.lib()
    L.sqp_debug_set_prefill_variant(rt, 3, 1)
    try:
        y0 = _check(orc, sqp, xs, p, sc, z, group)
        h = host(sqp.w4a16_gemm_silu_mul(dev(xs), dev(p), dev(sc), dev(z), group)) if N % 16 == 0 else None
    finally:
        L.sqp_debug_set_prefill_variant(0, 0, 0)
    L.sqp_debug_set_prefill_variant(4, 4, 1)
    try:  # the same products in the same order
        y1 = host(sqp.w4a16_gemm(dev(xs), dev(p), dev(sc), dev(z), group))
        h1 = host(sqp.w4a16_gemm_silu_mul(dev(xs), dev(p), dev(sc), dev(z), group)) if N % 16 == 0 else None
    finally:
        L.sqp_debug_set_prefill_variant(0, 0, 0)
    assert np.array_equal(y0.view(np.uint16), y1.view(np.uint16))
    if h is not None:
        assert np.array_equal(h.view(np.uint16), h1.view(np.uint16))


@pytest.mark.parametrize("rt", [3, 4, 5, 6])
@pytest.mark.parametrize("M_off,K,N,group,parts", [
    (0, 128, 8, 64, 1), (-1, 256, 136, 128, 1), (1, 384, 120, 192, 1), (33, 640, 264, 64, 1), (-17, 1024, 392, 512, 4), (5, 1920, 248, 320, 3),
    (64, 1792, 128, 256, 2), (-1, 256, 144, 128, 1), (5, 1920, 240, 640, 3)])
def test_prefill_waves_halve_k(orc, sqp, M_off, K, N, group, parts, rt):
    """Tiles of 128 columns whose waves halve every stage of 128 k between them: one row or column past a tile and
    short of it, one to fifteen stages, groups that end in the middle of a stage or span several, with and without K
    parts; plain and with the fused activation (N a multiple of 16); repeated runs are bit-identical, and equal to whole-K
    tiles within the fp32 accumulation."""
    M = max(1, 64 * rt + M_off)
    print("case halved k", M, K, N, group, rt, parts, flush=True)
    xs, p, sc, z = _layer(orc, M, K, N, group)
    xs = xs * np.float16(0.25)                             # (the fused products stay below fp16's largest value)
    d = (dev(xs), dev(p), dev(sc), dev(z), group)
    fused = N % 16 == 0
    L = sqp.lib()
    L.sqp_debug_set_prefill_variant(rt, 2 + 16, parts)
    try:
        y0 = _check(orc, sqp, xs, p, sc, z, group)
        y1 = _check(orc, sqp, xs, p, sc, z, group)
        h = host(sqp.w4a16_gemm_silu_mul(*d)).astype(np.float64) if fused else None
    finally:
        L.sqp_debug_set_prefill_variant(0, 0, 0)
    assert np.array_equal(y0.view(np.uint16), y1.view(np.uint16))
    L.sqp_debug_set_prefill_variant(rt, 2, parts)
    try:
        whole = host(sqp.w4a16_gemm(*d)).astype(np.float64)
    finally:
        L.sqp_debug_set_prefill_variant(0, 0, 0)
    y_ref, t_ref = orc.w4a16_gemm_ref(xs, p, sc, z, group)
    # The same products in two orders: each sum is within K roundings of 2^-23 (cut off, not rounded) of its terms' sizes,
    # and rounded once to fp16.
    assert np.all(np.abs(y0.astype(np.float64) - whole) <= 2 * K * 2.0 ** -23 * t_ref + orc.ulp16(y_ref))
    if fused:
        h_ref, tol = silu_tolerance(orc, y_ref, t_ref)
        assert h.shape == (M, N // 2) and np.abs(h_ref).max() < 60000
        assert np.all(np.abs(h - h_ref) <= tol), "worst err/tol %.3f" % float((np.abs(h - h_ref) / tol).max())


def test_prefill_left_over_k_parts(orc, sqp):
    """A grid of one full round and a few tiles, K long enough that the left-over half-width tiles are
    split in K too (M = 2050, N = 8144: 17 x 16 = 272 tiles).  Sampled rows against the oracle, from
    the whole rounds and the left-over tiles; every element against full tiles only, within
    the fp32 accumulation of both (K 2^-23 of the sum of magnitudes) and one fp16 ulp; the fused
    activation likewise through its own pair of launches."""
    import ctypes
    K, N, M = 2048, 8144, 2050
    print("case prefill left over", M, K, N, flush=True)
    out = (ctypes.c_int * 8)()
    L = sqp.lib()
    assert L.sqp_debug_prefill_launches(M, N, K, 128, 256, out) == 2 and out[3] == 1 and out[7] >= 2, list(out)
    xs, p, sc, z = _layer(orc, M, K, N, 128)
    args = (dev(xs), dev(p), dev(sc), dev(z), 128)
    rng = np.random.Generator(np.random.PCG64(22))
    rows = np.unique(np.concatenate([[0, M - 1, 2047, 2048], rng.choice(M, 20, replace=False)]))
    y_ref, t_ref = orc.w4a16_gemm_ref(np.ascontiguousarray(xs[rows]), p, sc, z, 128)
    y, h = sqp.w4a16_gemm(*args), sqp.w4a16_gemm_silu_mul(*args)
    ok, worst, nbad = gemm_tolerance_ok(orc, host(y)[rows], y_ref, t_ref)
    assert ok, "worst err/tol %.3f, %d elements out of tolerance" % (worst, nbad)
    L.sqp_debug_set_prefill_tiles(1)
    try:
        y1, h1 = sqp.w4a16_gemm(*args), sqp.w4a16_gemm_silu_mul(*args)
    finally:
        L.sqp_debug_set_prefill_tiles(0)
    mags = args[0].float().abs() @ sqp.dequantize(*args[1:4], 128).float().abs()
    ulp = torch.exp2(torch.floor(torch.log2(y1.float().abs().clamp(min=2.0 ** -14))) - 10)
    assert bool(((y.float() - y1.float()).abs() <= K * 2.0 ** -23 * mags + ulp).all())
    e = K * 2.0 ** -23 * torch.maximum(mags[:, 0::2], mags[:, 1::2])      # |SiLU'| <= 1.1, |SiLU(g)| <= |g|
    g, u = y1[:, 0::2].float().abs() + ulp[:, 0::2], y1[:, 1::2].float().abs() + ulp[:, 1::2]
    ulp_h = torch.exp2(torch.floor(torch.log2(h1.float().abs().clamp(min=2.0 ** -14))) - 10)
    assert bool(((h.float() - h1.float()).abs() <= e * (1.1 * u + g + e) + ulp_h).all())


def test_cfg4_34b_m256_sampled(orc, sqp):
    """34B-shaped 8192 -> 8192 at M = 256 with the library's own plan (half-width tiles and a
    K split): 24 sampled rows plus the first and last against the oracle."""
    K, N, M = 8192, 8192, 256
    print("case prefill 34b m256", M, K, N, flush=True)
    xs, p, sc, z = _layer_cached(orc, M, K, N, 1)
    rng = np.random.Generator(np.random.PCG64(13))
    rows = np.unique(np.concatenate([[0, M - 1, 127, 128], rng.choice(M, 24, replace=False)]))
    y_ref, t_ref = orc.w4a16_gemm_ref(np.ascontiguousarray(xs[rows]), p, sc, z, 128)
    y = host(sqp.w4a16_gemm(dev(xs), dev(p), dev(sc), dev(z), 128))
    ok, worst, nbad = gemm_tolerance_ok(orc, y[rows], y_ref, t_ref)
    assert ok, "worst err/tol %.3f, %d elements out of tolerance" % (worst, nbad)


def test_prefill_mixed_launch(orc, sqp):
    """A tile grid of one full round of 256 plus a remainder (N = 4352, M = 3968: 17 x 16 =
    272 tiles): the automatic choice runs 256 wide tiles and 32 narrow ones.  Sampled rows
    against the oracle, among them rows of the last row of tiles."""
    K, N, M = 256, 4352, 3968
    print("case prefill mixed", M, K, N, flush=True)
    xs, p, sc, z = _layer(orc, M, K, N, 128)
    rng = np.random.Generator(np.random.PCG64(21))
    rows = np.unique(np.concatenate([[0, M - 1, 3839, 3840, 3841], rng.choice(M, 40, replace=False)]))
    y_ref, t_ref = orc.w4a16_gemm_ref(np.ascontiguousarray(xs[rows]), p, sc, z, 128)
    y = host(sqp.w4a16_gemm(dev(xs), dev(p), dev(sc), dev(z), 128))
    ok, worst, nbad = gemm_tolerance_ok(orc, y[rows], y_ref, t_ref)
    assert ok, "worst err/tol %.3f, %d elements out of tolerance" % (worst, nbad)


def _random_shapes(seed, count, m_lo, m_hi):
    """Seeded random (M, K, N, group): K a multiple of the group, N a multiple of 8, sizes the
    oracle finishes in a fraction of a second, spanning every kernel variant of the range."""
    rng = np.random.Generator(np.random.PCG64(seed))
    out = []
    for _ in range(count):
        group = int(rng.choice([32, 64, 128, 128, 128, 256]))
        K = group * int(rng.integers(1, max(2, 3072 // group)))
        N = 8 * int(rng.integers(1, 160))
        M = int(rng.integers(m_lo, m_hi + 1))
        out.append((M, K, N, group))
    return out


@pytest.mark.parametrize("M,K,N,group", _random_shapes(101, 16, 1, 64))
def test_decode_random_shapes(orc, sqp, M, K, N, group):
    """Random small shapes through the streaming kernel with the library's own launch plan and
    with a forced deep K split (where the chunk count allows it), against the oracle."""
    print("case random decode", M, K, N, group, flush=True)
    xs, p, sc, z = _layer(orc, M, K, N, group)
    _check(orc, sqp, xs, p, sc, z, group)
    L = sqp.lib()
    L.sqp_debug_set_decode_plan(2, 5)
    try:
        _check(orc, sqp, xs, p, sc, z, group)
    finally:
        L.sqp_debug_set_decode_plan(0, 0)


@pytest.mark.parametrize("nw,split", [(1, 1), (1, 3), (8, 1), (8, 2)])
@pytest.mark.parametrize("M,K,N,group", [(7, 1024, 1032, 128), (20, 512, 264, 64), (50, 768, 200, 32), (16, 1536, 520, 256)])
def test_decode_other_strip_counts(orc, sqp, M, K, N, group, nw, split):
    """The one- and eight-strip workgroups (which the launch plan does not pick by itself, but
    which the library builds and the plan hook can select) through every row-tile variant."""
    print("case strips", M, K, N, group, nw, split, flush=True)
    xs, p, sc, z = _layer(orc, M, K, N, group)
    L = sqp.lib()
    L.sqp_debug_set_decode_plan(nw, split)
    try:
        _check(orc, sqp, xs, p, sc, z, group)
    finally:
        L.sqp_debug_set_decode_plan(0, 0)


@pytest.mark.parametrize("nw,split", [(2, 1), (2, 3), (2, 5), (4, 1), (4, 2), (4, 3)])
@pytest.mark.parametrize("M,K,N", [(16, 2048, 328), (7, 1152, 1032), (1, 128 * 13, 520), (16, 128, 264), (32, 2048, 328), (19, 1152, 520)])
def test_decode_two_chunks_per_iteration(orc, sqp, M, K, N, nw, split):
    """The strip kernel with two chunks per iteration (twice the waves, each half of them taking
    every other chunk; the 16- and the 32-row variant): even and odd chunk ranges, ranges shorter than the pipeline, a single
    chunk (the second half of the waves has nothing to do); repeated runs are bit-identical."""
    print("case two chunks", M, K, N, nw, split, flush=True)
    xs, p, sc, z = _layer(orc, M, K, N, 128)
    L = sqp.lib()
    L.sqp_debug_set_decode_plan(nw, split)
    L.sqp_debug_set_decode_kp(2)
    L.sqp_debug_set_decode_slice(-1)
    try:
        y0 = _check(orc, sqp, xs, p, sc, z, 128)
        y1 = _check(orc, sqp, xs, p, sc, z, 128)
        assert np.array_equal(y0.view(np.uint16), y1.view(np.uint16))
    finally:
        L.sqp_debug_set_decode_plan(0, 0)
        L.sqp_debug_set_decode_kp(0)
        L.sqp_debug_set_decode_slice(0)


@pytest.mark.parametrize("nw,kw,kp", [(2, 2, 1), (2, 2, 3), (4, 1, 3)])
@pytest.mark.parametrize("M,K,N,group,split", [
    (17, 128, 136, 128, 1), (33, 640, 264, 128, 2), (48, 1152, 520, 384, 3), (49, 1280, 200, 256, 1), (64, 128 * 13, 328, 128, 5),
    (1, 256, 72, 64, 1), (16, 1152, 264, 64, 4), (20, 640, 136, 64, 1), (47, 896, 392, 64, 3), (64, 384, 8, 64, 1),
    (3, 128, 264, 32, 1), (32, 1408, 136, 32, 2), (40, 640, 520, 32, 1), (61, 768, 264, 32, 6)])
def test_decode_wide_variants(orc, sqp, M, K, N, group, split, nw, kw, kp):
    """The eight-wave and two-wave-per-strip variants of every row-tile count, with one and several
    groups per chunk and several chunks per group: row tiles finished by different waves, chunk
    ranges shorter than the pipeline, odd ranges, ragged columns; repeated runs are bit-identical."""
    print("case wide", M, K, N, group, split, nw, kw, kp, flush=True)
    xs, p, sc, z = _layer(orc, M, K, N, group)
    L = sqp.lib()
    L.sqp_debug_set_decode_plan(nw, split)
    L.sqp_debug_set_decode_kw(kw)
    L.sqp_debug_set_decode_kp(kp)
    L.sqp_debug_set_decode_slice(-1)
    try:
        y0 = _check(orc, sqp, xs, p, sc, z, group)
        y1 = _check(orc, sqp, xs, p, sc, z, group)
        assert np.array_equal(y0.view(np.uint16), y1.view(np.uint16))
    finally:
        L.sqp_debug_set_decode_plan(0, 0)
        L.sqp_debug_set_decode_kw(0)
        L.sqp_debug_set_decode_kp(0)
        L.sqp_debug_set_decode_slice(0)


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("M,K,N", [
    (1, 128, 8), (3, 256, 40), (5, 1152, 72), (16, 384, 520), (7, 1024, 1032), (16, 1536, 2056), (9, 128 * 7, 200),
    (16, 4096, 1024), (2, 128 * 19, 264)])
def test_decode_slice_kernel(orc, sqp, M, K, N, mode):
    """The column-slice kernel (a workgroup owns 32 columns over all of K, its waves take every
    WV-th chunk and add up through LDS), both variants, forced through the hook: fewer chunks
    than waves, chunk counts that do not divide among the waves, ragged column counts; repeated
    runs are bit-identical."""
    print("case slice", M, K, N, mode, flush=True)
    xs, p, sc, z = _layer(orc, M, K, N, 128)
    L = sqp.lib()
    L.sqp_debug_set_decode_slice(mode)
    try:
        y0 = _check(orc, sqp, xs, p, sc, z, 128)
        y1 = _check(orc, sqp, xs, p, sc, z, 128)
        assert np.array_equal(y0.view(np.uint16), y1.view(np.uint16))
    finally:
        L.sqp_debug_set_decode_slice(0)


@pytest.mark.parametrize("mode", [1, 2])
def test_decode_slice_integer_exact(orc, sqp, mode):
    """Integer operands (step 1, Z = 0): every partial sum is an exact integer in fp32, so the
    slice kernel's result is the integer product rounded once to fp16."""
    rng = np.random.Generator(np.random.PCG64(5))
    M, N, K, g = 16, 104, 128 * 11, 128
    q = rng.integers(0, 16, size=(K, N))
    x = rng.integers(-4, 5, size=(M, K))
    p = np.zeros((K // 8, N), np.uint32)
    for i in range(8):
        p |= q[i::8].astype(np.uint32) << np.uint32(4 * i)
    ones = np.ones((K // g, N), np.float16)
    zz = np.zeros((K // g, N), np.uint8)
    L = sqp.lib()
    L.sqp_debug_set_decode_slice(mode)
    try:
        y = host(sqp.w4a16_gemm(dev(x.astype(np.float16)), dev(p), dev(ones), dev(zz), g))
    finally:
        L.sqp_debug_set_decode_slice(0)
    assert np.array_equal(y, (x @ q).astype(np.float16))


@pytest.mark.parametrize("tb,wv,grouped", [(1, 8, 0), (1, 16, 1), (2, 8, 1), (2, 16, 0), (4, 4, 0), (4, 8, 1)])
@pytest.mark.parametrize("M,K,N,group", [
    (1, 128, 8, 128), (4, 1152, 520, 128), (5, 128 * 17, 40, 128), (8, 2304, 1032, 768), (9, 512, 2056, 256), (16, 128 * 19, 264, 128),
    (2, 64, 24, 64), (7, 192, 520, 64), (12, 64 * 33, 1032, 64), (3, 32, 16, 32), (6, 1120, 264, 32), (13, 1056, 72, 32), (16, 992, 2056, 32),
    (17, 384, 136, 128), (24, 768, 520, 384), (31, 1088, 1032, 64), (32, 1248, 264, 32)])
def test_decode_slice_variants(orc, sqp, M, K, N, group, tb, wv, grouped):
    """Every slice width and wave count of the column-slice kernel, forced: fewer chunks than waves and chunk
    counts that do not divide among them, a last chunk of one to three k-steps, several groups per
    chunk and several chunks per group (also with a group boundary inside a wave's stride), ragged
    columns, slices mapped to XCDs in fours with and without a remainder; bit-identical repeats."""
    print("case slice variants", M, K, N, group, tb, wv, grouped, flush=True)
    xs, p, sc, z = _layer(orc, M, K, N, group)
    L = sqp.lib()
    L.sqp_debug_set_slice_plan(tb, wv, grouped)
    try:
        y0 = _check(orc, sqp, xs, p, sc, z, group)
        y1 = _check(orc, sqp, xs, p, sc, z, group)
        assert np.array_equal(y0.view(np.uint16), y1.view(np.uint16))
    finally:
        L.sqp_debug_set_slice_plan(0, 0, 0)


@pytest.mark.parametrize("mt,split,kp", [(3, 1, 1), (3, 3, 2), (4, 1, 2), (4, 2, 1)])
@pytest.mark.parametrize("M,K,N,group", [(65, 768, 8, 128), (96, 1024, 144, 64), (97, 896, 520, 32), (128, 2304, 272, 768), (145, 1280, 392, 128), (193, 768, 1040, 256)])
def test_row_blocks(orc, sqp, M, K, N, group, mt, split, kp):
    """More than 64 rows by the strip kernel in row blocks of 48 and 64, forced: whole last blocks and last
    blocks of 1 to 33 rows, ragged columns, parts of unequal length, several groups per chunk and
    several chunks per group; the fused activation; bit-identical repeats; nothing written past y."""
    print("case row blocks", M, K, N, group, mt, split, kp, flush=True)
    xs, p, sc, z = _layer(orc, M, K, N, group)
    L = sqp.lib()
    L.sqp_debug_set_row_blocks(mt, split, kp)
    try:
        y0 = _check(orc, sqp, xs, p, sc, z, group)
        buf = torch.full((M * N + 4096,), -7.0, dtype=torch.half, device="cuda")
        sqp.w4a16_gemm(dev(xs), dev(p), dev(sc), dev(z), group, out=buf[:M * N].view(M, N))
        assert np.array_equal(host(buf[:M * N]).view(np.uint16), y0.reshape(-1).view(np.uint16))
        assert bool((buf[M * N:] == -7.0).all())
        if N % 16:
            return
        act = host(sqp.w4a16_gemm_silu_mul(dev(xs), dev(p), dev(sc), dev(z), group)).astype(np.float64)
    finally:
        L.sqp_debug_set_row_blocks(0, 0, 0)
    y = orc.w4a16_gemm_ref(xs, p, sc, z, group)
    gate, up, tg, tu = y[0][:, 0::2], y[0][:, 1::2], y[1][:, 0::2], y[1][:, 1::2]
    sig = 1 / (1 + np.exp(-gate))
    # the tolerances of the two sums (1e-3 of their terms) through silu (|silu'| < 1.1) and the product, half an ulp
    # of fp16 at the result (2^-11 of it, or of its smallest normal) and of silu itself
    tol = 1e-3 * (1.1 * tg * (np.abs(up) + 1e-3 * tu) + np.abs(gate * sig) * tu) + 2.0 ** -10 * np.abs(gate * sig * up) + 2.0 ** -24
    assert (np.abs(act - gate * sig * up) <= tol).all()


@pytest.mark.parametrize("M,K,N,group", [(161, 384, 776, 192), (65, 768, 1024, 192), (100, 1920, 520, 320), (70, 128, 264, 128)])
def test_more_than_64_rows_by_the_rule(orc, sqp, M, K, N, group):
    """Small layers above 64 rows with groups whose ends lie inside a chunk of 128 k (and one that is a chunk),
    nothing forced."""
    print("case rows by rule", M, K, N, group, flush=True)
    xs, p, sc, z = _layer(orc, M, K, N, group)
    _check(orc, sqp, xs, p, sc, z, group)


@pytest.mark.parametrize("M,K,N,group,blocks", [(65, 1024, 1024, 128, True), (160, 4096, 1024, 64, True), (160, 8192, 8192, 128, False), (700, 512, 2056, 32, True)])
def test_row_blocks_workspace(sqp, M, K, N, group, blocks):
    """Row blocks by the rule and the tiles agree to the roundings of their sums; a shape that reports no
    workspace takes no K parts, and one that does takes them within what it reports."""
    print("case row blocks rule", M, K, N, group, flush=True)
    L = sqp.lib()
    out = (ctypes.c_int * 3)()
    reported = sqp.workspace_bytes(M, N, K, group)
    L.sqp_debug_row_blocks(M, N, K, group, 256, int(reported > 0), out)
    assert (out[0] > 0) == blocks
    if blocks:
        assert out[1] == 1 or (512 << 10) + out[1] * -(-M // (16 * out[0])) * 16 * out[0] * -(-N // 128) * 128 * 4 <= reported
    gen = torch.Generator(device="cuda").manual_seed(M + N)
    w = torch.randn(K, N, generator=gen, device="cuda").half() * 0.02
    p, sc, z = sqp.quantize_pack(w, group)
    x = torch.randn(M, K, generator=gen, device="cuda").half()
    y = sqp.w4a16_gemm(x, p, sc, z, group)
    L.sqp_debug_set_row_blocks(-1, 0, 0)
    try:
        t = sqp.w4a16_gemm(x, p, sc, z, group)
    finally:
        L.sqp_debug_set_row_blocks(0, 0, 0)
    # both multiply the same rounded weights: K fp32 additions of terms with absolute sum A (error K 2^-24 A), one fp16 ulp
    a = x.abs().float() @ sqp.dequantize(p, sc, z, group).abs().float()
    assert bool(((y - t).abs().float() <= K * 2.0 ** -23 * a + 2.0 ** -10 * t.abs().float() + 2.0 ** -24).all())


@pytest.mark.parametrize("M,group,tb,wv", [(1, 128, 1, 8), (6, 64, 2, 8), (16, 256, 2, 16), (3, 128, 4, 8), (20, 64, 2, 8)])
def test_decode_slice_nonfinite_activations(orc, sqp, M, group, tb, wv):
    """An infinity or a NaN among the activations gives what the strip kernel gives for it (sums over the
    differences code - Z: an infinity times a code above, below or at the zero point), and the other rows
    keep every bit."""
    K, N = 1024, 264
    xs, p, sc, z = _layer(orc, M, K, N, group)
    clean = xs.copy()
    xs[0, 333] = np.inf
    if M > 2:
        xs[2, 100], xs[2, 900] = -np.inf, np.nan
    L = sqp.lib()
    run = lambda a: host(sqp.w4a16_gemm(dev(a), dev(p), dev(sc), dev(z), group))
    try:
        L.sqp_debug_set_decode_slice(-1)
        want = run(xs)
        L.sqp_debug_set_decode_slice(0)
        L.sqp_debug_set_slice_plan(tb, wv, 0)
        got, ref = run(xs), run(clean)
    finally:
        L.sqp_debug_set_decode_slice(0)
        L.sqp_debug_set_slice_plan(0, 0, 0)
    hit = [0] if M <= 2 else [0, 2]
    assert np.isinf(want[0]).any()
    assert np.array_equal(np.isnan(got[hit]), np.isnan(want[hit]))
    inf = np.isinf(want[hit])
    assert np.array_equal(got[hit][inf], want[hit][inf])
    rest = [m for m in range(M) if m not in hit]
    assert np.array_equal(got[rest].view(np.uint16), ref[rest].view(np.uint16))


@pytest.mark.parametrize("M,K,N,group,tb,wv", [(1, 1056, 264, 32, 1, 8), (7, 1088, 136, 32, 2, 8), (20, 1120, 136, 32, 4, 8), (3, 1088, 264, 64, 1, 16), (16, 192, 72, 64, 4, 8)])
def test_decode_slice_infinite_step_of_the_last_group(orc, sqp, M, K, N, group, tb, wv):
    """A last chunk of one to three k-steps: its last group has a step of infinity in every second column, and the
    results are the strip kernel's infinities (an infinite step counts once, with its own group's sum)."""
    print("case infinite step", M, K, N, group, tb, wv, flush=True)
    xs, p, sc, z = _layer(orc, M, K, N, group)
    sc[-1, 0::2] = np.inf
    L = sqp.lib()
    run = lambda: host(sqp.w4a16_gemm(dev(xs), dev(p), dev(sc), dev(z), group))
    try:
        L.sqp_debug_set_decode_slice(-1)
        want = run()
        L.sqp_debug_set_decode_slice(0)
        L.sqp_debug_set_slice_plan(tb, wv, 0)
        got = run()
    finally:
        L.sqp_debug_set_decode_slice(0)
        L.sqp_debug_set_slice_plan(0, 0, 0)
    assert np.isinf(want[:, 0::2]).all()
    assert np.array_equal(got[:, 0::2], want[:, 0::2]) and np.isfinite(got[:, 1::2]).all()


_ZERO_CODE_SHAPES = [(1, 4096, 1024, 128), (3, 1024, 264, 64), (8, 1024, 520, 128), (13, 1152, 136, 32), (16, 1024, 264, 256), (20, 1024, 264, 64)]


@pytest.mark.parametrize("M,K,N,group,tb,wv", [(*s, *v) for s in _ZERO_CODE_SHAPES for v in [(0, 0), (1, 8), (1, 16), (2, 8), (4, 4), (4, 8)]] +
                         [(40, 1024, 264, 128, 0, 0), (70, 1024, 264, 128, 0, 0)])
def test_codes_at_the_zero_point_count_nothing(orc, sqp, M, K, N, group, tb, wv):
    """A weight whose code is the zero point is exactly 0: whatever finite activations meet such weights only, also next
    to the largest fp16 value, their sum is exactly 0, by the rule and in every slice variant; one other code in
    the column then gives its own product alone, rounded as the plain product is."""
    print("case zero codes", M, K, N, group, tb, wv, flush=True)
    rng = np.random.Generator(np.random.PCG64(M + K))
    z = rng.integers(0, 16, size=(K // group, N)).astype(np.uint8)
    q = np.repeat(z, group, 0).astype(np.uint32)
    single = rng.integers(0, K, size=N // 2)   # the even columns get one other code, a step of 1 / 64
    q[single, np.arange(0, N, 2)] ^= 1
    p = np.zeros((K // 8, N), np.uint32)
    for i in range(8):
        p |= q[i::8] << np.uint32(4 * i)
    sc = np.full((K // group, N), 1 / 64, np.float16)
    x = (rng.standard_normal((M, K)) * np.where(rng.random(K) < 0.05, 20000, 1)).clip(-60000, 60000).astype(np.float16)
    want = np.zeros((M, N), np.float16)
    sign = (q[single, np.arange(0, N, 2)].astype(np.int64) - z[single // group, np.arange(0, N, 2)])
    want[:, 0::2] = (x[:, single].astype(np.float64) * sign / 64).astype(np.float16)
    L = sqp.lib()
    L.sqp_debug_set_slice_plan(tb, wv, 0)
    try:
        y = host(sqp.w4a16_gemm(dev(x), dev(p), dev(sc), dev(z), group))
    finally:
        L.sqp_debug_set_slice_plan(0, 0, 0)
    assert np.array_equal(y, want)  # (0 == -0)


@pytest.mark.parametrize("M,K,N,group", _random_shapes(202, 8, 65, 700))
def test_prefill_random_shapes(orc, sqp, M, K, N, group):
    """Random shapes above 64 rows (tiled kernel: wide and narrow tiles, K parts; groups of 32
    take the row-block fallback), against the oracle."""
    print("case random prefill", M, K, N, group, flush=True)
    xs, p, sc, z = _layer(orc, M, K, N, group)
    _check(orc, sqp, xs, p, sc, z, group)


def test_prefill_integer_exact(orc, sqp):
    """step = 1, Z = 0, small integer activations: exact integer product."""
    rng = np.random.Generator(np.random.PCG64(4))
    M, N, K, g = 300, 320, 256, 128
    q = rng.integers(0, 16, size=(K, N))
    x = rng.integers(-4, 5, size=(M, K))
    p = np.zeros((K // 8, N), np.uint32)
    for i in range(8):
        p |= q[i::8].astype(np.uint32) << np.uint32(4 * i)
    ones = np.ones((K // g, N), np.float16)
    zz = np.zeros((K // g, N), np.uint8)
    y = host(sqp.w4a16_gemm(dev(x.astype(np.float16)), dev(p), dev(ones), dev(zz), g))
    assert np.array_equal(y.astype(np.int64), x @ q)


def test_prefill_full_size_sampled(orc, sqp):
    """34B-shaped 8192 -> 8192 at M = 2048 (the launch configuration the benchmark times):
    the oracle evaluates 24 seeded rows plus the first and last row over all N; every sampled
    element is the full-K definition.  Run twice: the result must be bit-identical."""
    K, N, M = 8192, 8192, 2048
    print("case prefill full", M, K, N, flush=True)
    xs, p, sc, z = _layer_cached(orc, M, K, N, 1)
    rng = np.random.Generator(np.random.PCG64(12))
    rows = np.unique(np.concatenate([[0, M - 1, 255, 256], rng.choice(M, 24, replace=False)]))
    y_ref, t_ref = orc.w4a16_gemm_ref(np.ascontiguousarray(xs[rows]), p, sc, z, 128)
    dp, dsc, dz, dx = dev(p), dev(sc), dev(z), dev(xs)
    y = host(sqp.w4a16_gemm(dx, dp, dsc, dz, 128))
    y2 = host(sqp.w4a16_gemm(dx, dp, dsc, dz, 128))
    assert np.array_equal(y.view(np.uint16), y2.view(np.uint16))
    ok, worst, nbad = gemm_tolerance_ok(orc, y[rows], y_ref, t_ref)
    assert ok, "worst err/tol %.3f, %d elements out of tolerance" % (worst, nbad)
