"""Host logic that needs no GPU: the launch plans the library derives from a shape (the
decode path's strips and K split, the tiled path's tile mix and K parts) and the argument
checks of the loss entry point."""
import ctypes
import random

import pytest

import workloads as wl


@pytest.fixture(scope="module")
def L():
    import paper_2312_03788_amd as sqp
    return sqp.lib()


def _decode_plan(L, M, N, K, group):
    nw, split, kspg = ctypes.c_int(), ctypes.c_int(), ctypes.c_int()
    L.sqp_debug_decode_plan(M, N, K, group, ctypes.byref(nw), ctypes.byref(split), ctypes.byref(kspg))
    return nw.value, split.value, kspg.value


def _tile_plan(L, M, N, K, cus=256):
    full, half, ks = ctypes.c_long(), ctypes.c_long(), ctypes.c_int()
    L.sqp_debug_prefill_plan(M, N, K, cus, ctypes.byref(full), ctypes.byref(half), ctypes.byref(ks))
    return full.value, half.value, ks.value


def test_decode_plan_invariants(L):
    shapes = [s for m in ("7b", "13b", "34b") for s in wl.MODEL_SHAPES[m]] + [(128, 8), (1024, 264), (65536, 64)]
    for (K, N) in shapes:
        for group in (32, 64, 128, 256):
            if K % group:
                continue
            nw, split, kspg = _decode_plan(L, 16, N, K, group)
            chunk = 128 if group % 128 == 0 else group
            chunks = K // chunk
            assert nw in (2, 4) and kspg == {32: 1, 64: 2}.get(group, 4)
            assert 1 <= split <= max(1, chunks // 4)          # at least four chunks per workgroup
            tiles = -(-N // (64 * nw))
            if tiles <= 128:
                # narrow layers: never more than one workgroup per compute unit, and as many as
                # the chunk bound allows below that
                assert tiles * split <= 256
                if split < max(1, chunks // 4):
                    assert tiles * (split + 1) > 256
            elif split < max(1, chunks // 4):
                assert abs(tiles * split - 704) <= tiles
            if nw == 2:                                        # only narrow layers, and not with a long K range
                # (groups of 128, where a launch can take two chunks per iteration: up to 40 tiles
                # if each workgroup then still walks 16 chunks)
                assert -(-N // 256) <= ((40 if group == 128 else 32) if group % 128 == 0 else 24)
                if -(-N // 256) > 32:
                    assert chunks // split >= 16
                if group % 128 == 0 and not (group == 128 and chunks // split >= 16):
                    assert chunks <= 24 * split
    assert _decode_plan(L, 16, 1024, 1024, 24)[2] == 0        # other group sizes: generic kernel


def test_decode_plan_34b_values(L):
    """The plans the benchmark's launches run with (they are part of its configuration)."""
    got = {(K, N): _decode_plan(L, 16, N, K, 128)[:2] for (K, N) in wl.MODEL_SHAPES["34b"]}
    assert got == {(8192, 10240): (2, 3), (8192, 8192): (2, 4), (8192, 44032): (4, 4), (22016, 8192): (2, 4)}


def test_decode_slice_choice(L):
    """Which calls take the column-slice kernel: groups of 128 only; up to 8 rows, 64-column
    slices on the wide layers, 32-column slices on the narrow ones unless K is long and the
    slices are few; more than 8 rows only where x is small enough (short K) and the layer not
    too wide; the 16-row calls of the benchmark sweep (K = 8192 and 22016) keep the strip kernel."""
    L.sqp_debug_decode_slice_choice.restype = ctypes.c_int
    ch = lambda M, K, N, g=128: L.sqp_debug_decode_slice_choice(M, N, K, g)
    assert [ch(1, K, N) for (K, N) in wl.MODEL_SHAPES["34b"]] == [1, 0, 1, 0]
    assert [ch(4, K, N) for (K, N) in wl.MODEL_SHAPES["34b"]] == [1, 0, 1, 0]
    assert [ch(8, K, N) for (K, N) in wl.MODEL_SHAPES["34b"]] == [1, 0, 1, -1]     # K = 22016: two blocks of x are too many
    assert [ch(1, K, N) for (K, N) in wl.MODEL_SHAPES["13b"]] == [1, 0, 1, -1]
    assert [ch(4, K, N) for (K, N) in wl.MODEL_SHAPES["7b"]] == [1, 0, 1, -1]
    assert [ch(12, K, N) for (K, N) in wl.MODEL_SHAPES["34b"]] == [1, 0, -1, -1]
    assert [ch(9, K, N) for (K, N) in wl.MODEL_SHAPES["13b"]] == [1, 0, 1, -1]
    assert [ch(12, K, N) for (K, N) in wl.MODEL_SHAPES["7b"]] == [1, 0, 1, -1]
    assert [ch(16, K, N) for (K, N) in wl.MODEL_SHAPES["7b"]] == [1, 0, 1, -1]      # short K: x is small
    assert [ch(16, K, N) for (K, N) in wl.MODEL_SHAPES["13b"]] == [1, -1, -1, -1]
    for (K, N) in wl.MODEL_SHAPES["34b"]:
        assert ch(13, K, N) == -1 and ch(16, K, N) == -1 and ch(64, K, N) == -1
        assert ch(1, K, N, 64) == -1 and ch(1, K, N, 256) == -1
    assert ch(1, 4096, 1024) == -1 and ch(1, 128, 8) == -1      # few slices: the strip kernel and its K split


def test_slice_calls_need_no_workspace(L):
    """A call that takes the column-slice kernel reports no workspace; the 16-row calls of the
    34B sweep (strip kernel, K split across workgroups) report tickets plus partial sums."""
    L.sqp_debug_decode_slice_choice.restype = ctypes.c_int
    L.sqp_w4a16_gemm_workspace_bytes.restype = ctypes.c_size_t
    for model in ("7b", "13b", "34b"):
        for (K, N) in wl.MODEL_SHAPES[model]:
            for M in (1, 4, 8, 12, 16):
                need = L.sqp_w4a16_gemm_workspace_bytes(M, N, K, 128)
                if L.sqp_debug_decode_slice_choice(M, N, K, 128) >= 0:
                    assert need == 0
    for (K, N) in wl.MODEL_SHAPES["34b"]:
        assert L.sqp_w4a16_gemm_workspace_bytes(16, N, K, 128) > 512 << 10


def test_slice_plan_values(L):
    """Widths and waves at the edges of the rule: one round of 16, 32 and 64 columns, the K from which the
    strip kernel takes over, groups and K that it covers badly."""
    def plan(M, N, K, g):
        tb, wv = ctypes.c_int(), ctypes.c_int()
        L.sqp_debug_decode_slice_plan(M, N, K, g, ctypes.byref(tb), ctypes.byref(wv))
        return tb.value, wv.value
    assert plan(1, 4096, 4096, 128) == (1, 16) and plan(1, 4104, 4096, 128)[0] == 2
    assert plan(8, 8192, 4096, 128) == (2, 8) and plan(8, 8200, 4096, 128) == (4, 8)
    assert plan(1, 1024, 12288, 128) == (1, 16) and plan(1, 1024, 12416, 128) == (0, 0)
    assert plan(16, 1024, 6144, 64) == (1, 8) and plan(16, 1024, 6208, 64) == (1, 8) and plan(16, 1024, 6272, 64) == (0, 0)
    assert plan(32, 16384, 9216, 128)[0] == 4 and plan(33, 16384, 1024, 128) == (0, 0)
    assert plan(4, 22016, 4096, 128) == (4, 4) and plan(4, 22016, 4096, 32) == (2, 8) and plan(1, 4096, 4096, 24) == (0, 0)


def test_slice_plan_between_model_shapes(L):
    """Layers between the models' shapes that run up to 1.4 times slower in slices than in strips take strips (a little
    more than 256 slices and long K; K not a multiple of 128, narrow and long; short K and many columns at 17
    and more rows), and their neighbours that run faster in slices keep them."""
    def sliced(M, N, K, g):
        tb, wv = ctypes.c_int(), ctypes.c_int()
        L.sqp_debug_decode_slice_plan(M, N, K, g, ctypes.byref(tb), ctypes.byref(wv))
        return tb.value > 0
    for call in [(7, 17816, 6784, 64), (5, 17904, 9984, 64), (22, 21128, 5888, 256), (19, 20808, 2816, 256), (11, 888, 19648, 64), (31, 888, 19648, 64),
                 (12, 9848, 17024, 32), (22, 33104, 512, 64), (30, 39936, 512, 128), (15, 35624, 2848, 32), (32, 4016, 6144, 32), (29, 952, 13600, 32)]:
        assert not sliced(*call), call
    for call in [(5, 17904, 1024, 64), (17, 23296, 6336, 32), (32, 22016, 2112, 32), (11, 888, 8640, 64), (12, 9848, 8192, 32), (32, 39936, 1024, 128), (6, 22016, 2112, 32)]:
        assert sliced(*call), call


def test_decode_plan_many_rows(L):
    """More than 32 rows: two strips per workgroup, the split of the 16-row plan."""
    for (K, N) in wl.MODEL_SHAPES["34b"]:
        tiles4, chunks = -(-N // 256), K // 128
        four_strip_split = min(256 // tiles4 if tiles4 <= 128 else (704 + tiles4 // 2) // tiles4, max(1, chunks // 4))
        assert _decode_plan(L, 48, N, K, 128)[:2] == (2, four_strip_split)
    assert _decode_plan(L, 64, 512, 256, 128)[:2] == (2, 1)            # short K: no split
    assert _decode_plan(L, 64, 65536, 256, 128)[:2] == (4, 1)


def test_decode_plan_small_model_values(L):
    """Shapes where the sweeps found the four-strip, rounded-up plan 10-25 % off the best."""
    assert _decode_plan(L, 16, 4096, 4096, 128)[:2] == (2, 8)      # narrow and short: two strips
    assert _decode_plan(L, 16, 5120, 5120, 128)[:2] == (2, 6)
    assert _decode_plan(L, 16, 4096, 11008, 128)[:2] == (2, 8)
    assert _decode_plan(L, 16, 5120, 13824, 128)[:2] == (2, 6)     # 40 two-strip tiles x 6 = 240 workgroups
    assert _decode_plan(L, 32, 5120, 13824, 128)[:2] == (2, 6)
    assert _decode_plan(L, 32, 8192, 22016, 128)[:2] == (2, 4)     # 17..32 rows: also with a long K
    assert _decode_plan(L, 16, 8192, 22016, 128)[:2] == (2, 4)     # up to 16 rows, groups of 128: two chunks per iteration, so too
    assert _decode_plan(L, 16, 8192, 22016, 256)[:2] == (4, 8)     # other groups: a long K keeps four strips
    assert _decode_plan(L, 32, 12288, 4096, 128)[:2] == (4, 5)     # 48 tiles: four strips
    assert _decode_plan(L, 16, 22016, 4096, 128)[:2] == (4, 2)     # 86 tiles: 172 workgroups, not 258


def test_wide_plan_invariants(L):
    """17 to 64 rows, and groups of 32 and 64: at most one eight-wave or two four-wave workgroups per
    compute unit while the column tiles allow it, chunks for every workgroup, partial sums below
    the static array's size."""
    def launch(M, N, K, group):
        v = [ctypes.c_int() for _ in range(4)]
        L.sqp_debug_decode_launch(M, N, K, group, *[ctypes.byref(x) for x in v])
        return tuple(x.value for x in v)
    L.sqp_w4a16_gemm_workspace_bytes.restype = ctypes.c_size_t
    shapes = [s for m in ("7b", "13b", "34b") for s in wl.MODEL_SHAPES[m]] + [(128, 8), (1024, 264), (65536, 64), (5120, 18432), (768, 262144)]
    for (K, N) in shapes:
        for group in (32, 64, 128, 256):
            for M in (1, 16, 17, 32, 33, 64):
                if M <= 16 and group >= 128:
                    continue
                nw, split, kw, kp = launch(M, N, K, group)
                tiles, chunks = -(-N // (64 * nw)), K // 128
                assert nw in (2, 4) and kw in (1, 2) and kp in (1, 2) and not (nw == 4 and kw == 2)
                assert 1 <= split <= max(1, chunks // 2)
                if -(-N // 128) <= 256:
                    assert split == 1 or tiles * split <= (256 if kp == 2 else 512)
                assert kp == 1 or chunks >= 8 * split
                assert L.sqp_w4a16_gemm_workspace_bytes(M, N, K, group) <= (512 << 10) + (48 << 20)
    assert launch(48, 15360, 5120, 128) == (2, 2, 2, 2)      # 120 tiles x 2 parts
    assert launch(20, 4096, 4096, 64) == (2, 8, 2, 1)        # four chunks each: one per iteration
    assert launch(48, 18432, 5120, 128) == (2, 3, 2, 1)      # 144 tiles: three parts, two workgroups per unit
    assert launch(48, 44032, 8192, 128) == (2, 2, 2, 1)
    assert launch(20, 8192, 22016, 128) == (4, 8, 1, 2)


@pytest.mark.parametrize("shape", [1, 2])
def test_tile_plan_invariants(L, shape):
    """Both full-tile shapes (1: 128 x 512, 2: 256 x 256)."""
    bm, bn = (128, 512) if shape == 1 else (256, 256)
    L.sqp_debug_set_prefill_shape(shape)
    try:
        for M in (65, 128, 256, 300, 512, 1024, 2048, 4096):
            for (K, N) in wl.MODEL_SHAPES["34b"] + [(1024, 264), (256, 8), (8192, 256)]:
                for cus in (256, 304, 64):
                    full, half, ks = _tile_plan(L, M, N, K, cus)
                    tiles = -(-N // bn) * -(-M // bm)
                    assert full >= 0 and half >= 0 and ks >= 1
                    assert full + half // 2 == tiles and half % 2 == 0   # every tile exactly once
                    if ks >= 2:
                        assert full == 0 and 4 * tiles <= cus
                        assert half * ks <= cus                          # one round
                        assert K // 64 // ks >= 8                        # at least 8 stages per part
                    else:
                        assert full % cus == 0 or half == 0              # first launch: whole rounds only
                        assert half <= cus                               # the remainder is one round
    finally:
        L.sqp_debug_set_prefill_shape(0)


def test_tile_plan_bench_shapes(L):
    """The tile counts of the benchmark's M = 2048 launches are the same for both shapes."""
    for shape in (0, 1, 2):
        L.sqp_debug_set_prefill_shape(shape)
        try:
            assert _tile_plan(L, 2048, 8192, 8192) == (256, 0, 1)
            assert _tile_plan(L, 2048, 10240, 8192) == (256, 128, 1)
            assert _tile_plan(L, 2048, 44032, 8192) == (1280, 192, 1)
            assert _tile_plan(L, 4096, 8192, 22016) == (512, 0, 1)
            assert _tile_plan(L, 256, 8192, 8192) == (0, 64, 4)
        finally:
            L.sqp_debug_set_prefill_shape(0)


def test_prefill_launches_invariants(L):
    """The launches of the tiled path cover every tile once, one-round plans stay within the chip, K
    parts keep at least eight stages each and their partial sums fit the static array."""
    out = (ctypes.c_int * 8)()
    L.sqp_w4a16_gemm_workspace_bytes.restype = ctypes.c_size_t
    for M in (65, 96, 97, 128, 160, 161, 192, 300, 512, 700, 1024, 2048, 3001, 4096):
        for (K, N) in [s for m in ("7b", "13b", "34b") for s in wl.MODEL_SHAPES[m]] + [(1024, 264), (256, 8), (8192, 256)]:
            for group in (64, 128, 32):
                n = L.sqp_debug_prefill_launches(M, N, K, group, 256, out)
                v = [tuple(out[4 * i:4 * i + 4]) for i in range(n)]
                assert n in (1, 2)
                if n == 1:
                    rt, nt, tiles, parts = v[0]
                    assert tiles >= -(-N // (128 * nt)) * -(-M // (32 * rt))
                    assert parts == 1 or tiles * parts <= 256
                else:
                    assert v[0][:2] == (4, 4) and v[1][:2] == (4, 2) and v[0][2] % 256 == 0 and v[0][3] == 1
                    assert v[0][2] + v[1][2] // 2 == -(-N // 512) * -(-M // 128) and v[1][2] * v[1][3] <= 256
                for rt, nt, tiles, parts in v:
                    assert parts >= 1 and (parts == 1 or (nt == 2 and K // 64 // parts >= 8))
                assert L.sqp_w4a16_gemm_workspace_bytes(M, N, K, group) <= (512 << 10) + (48 << 20)
    one = lambda M, N, K: (L.sqp_debug_prefill_launches(M, N, K, 128, 256, out), tuple(out[:4]))
    assert one(160, 10240, 8192) == (1, (5, 2, 40, 6))       # one tile of 160 rows
    assert one(190, 8192, 8192) == (1, (3, 2, 64, 4))        # two of 96
    assert one(512, 22016, 4096) == (1, (4, 4, 172, 1))
    assert L.sqp_debug_prefill_launches(3001, 44032, 8192, 128, 256, out) == 2 and tuple(out[4:8]) == (4, 2, 32, 8)


def test_prefill_choice_stays_in_its_room(L):
    """What a call launches with some room for its K parts: every tile once, one launch of 256 or 384 columns at most one
    workgroup per compute unit (two of the variants with half the registers), left-over tiles in K parts at most one, at
    least eight stages of 64 k per part, parts within the room given, waves that halve K only where K is whole
    stages of 128 and groups are not of 32."""
    out, seen, drawn = (ctypes.c_int * 10)(), set(), [0, 0, 0]
    L.sqp_debug_prefill_choice.argtypes = [ctypes.c_int] * 5 + [ctypes.c_size_t, ctypes.POINTER(ctypes.c_int)]
    rng = random.Random(19)
    for _ in range(4000):
        group = rng.choice([128, 128, 64, 32, 192, 256])
        M, N, K = int(2 ** rng.uniform(6.1, 11.5)), 8 * int(2 ** rng.uniform(5, 12.4)), group * int(2 ** rng.uniform(0, 7))
        if K % 64:
            continue
        room = rng.choice([0, 1 << 20, 8 << 20, 48 << 20])
        n = L.sqp_debug_prefill_choice(M, N, K, group, 256, room, out)
        for i in range(n):
            rt, nt, tiles, parts, kh = out[5 * i:5 * i + 5]
            seen.add((rt, nt, kh, tiles * parts > 256))
            assert kh == 1 or (kh == 2 and nt == 2 and K % 128 == 0 and group % 64 == 0)
            assert nt != 3 or (rt in (4, 5) and n == 1 and tiles <= 256 and group != 32)
            assert parts == 1 or (nt == 2 and K // 64 >= 8 * parts and parts * tiles * 32 * rt * (256 // kh) * 4 <= room)
            if nt < 4 and (n == 1 or parts > 1):
                assert tiles * parts <= (512 if n == 1 and group != 32 and nt == 2 and kh == 1 and rt <= 4 else 256)
        whole = -(-N // 512) * -(-M // 128)   # tiles of 128 x 512: left and right half of each where they are halved
        if n == 1:
            rt, nt, tiles, parts, kh = out[:5]
            assert tiles == -(-N // (128 * nt // kh)) * -(-M // (32 * rt)) or ((rt, nt, kh) == (4, 2, 1) and tiles == 2 * whole)
        elif n == 2:
            assert tuple(out[:2]) == (4, 4) and tuple(out[3:5]) == (1, 1) and tuple(out[5:7]) == (4, 2) and out[9] == 1
            assert out[2] % 256 == 0 and 2 * out[2] + out[7] == 2 * whole
        drawn[n] += 1
    assert {(rt, 2, kh, False) for rt in (3, 4, 5, 6) for kh in (1, 2)} <= seen
    assert {(3, 2, 1, True), (4, 3, 1, False), (5, 3, 1, False)} <= seen
    assert drawn[1] > 1000 and drawn[2] > 50, drawn


@pytest.mark.parametrize("M,K,N,group", [(308, 9088, 136, 64), (95, 11520, 152, 64), (113, 6784, 376, 64), (79, 10496, 584, 64),
                                         (188, 6144, 104, 128), (82, 10496, 96, 128), (200, 8320, 224, 64)])
def test_few_columns_and_long_k_stay_with_the_row_blocks(L, M, K, N, group):
    """Tiles in 9 to 12 K parts of a few hundred KB, whose reduction waits for one part after the other, took 13 to 18 %
    longer than the strip kernel's row blocks on these."""
    rows = (ctypes.c_int * 3)()
    L.sqp_debug_row_blocks(M, N, K, group, 256, 1, rows)
    assert rows[0] in (3, 4) and rows[1] > 4


def test_every_sufficient_buffer_gives_the_same_launches(L):
    """A buffer larger than the size reported for a shape (the static array, a workspace that has grown for other shapes)
    changes nothing: neither the tiled launches nor the row blocks.  Drawn shapes, and some on which an estimate with more
    room would choose differently."""
    out, rows = (ctypes.c_int * 10)(), (ctypes.c_int * 3)()
    L.sqp_debug_prefill_choice.argtypes = [ctypes.c_int] * 5 + [ctypes.c_size_t, ctypes.POINTER(ctypes.c_int)]
    L.sqp_w4a16_gemm_scratch_bytes.restype = ctypes.c_size_t
    shapes = [(314, 2456, 16128, 128), (75, 25128, 14848, 128), (569, 6128, 15104, 128), (319, 6992, 10240, 128),
              (89, 16584, 28928, 256), (71, 25416, 21888, 128), (1434, 1632, 17280, 128), (77, 21872, 9664, 64)]
    rng = random.Random(23)
    for _ in range(20000):
        group = rng.choice([128, 128, 64, 192, 256])
        shapes.append((int(2 ** rng.uniform(6.05, 11.5)), 8 * int(2 ** rng.uniform(5, 12.5)), group * int(2 ** rng.uniform(0, 7.5)), group))
    used = 0
    for (M, N, K, group) in shapes:
        if max(M * K, K * N, M * N) >= 1 << 31:
            continue
        want = L.sqp_w4a16_gemm_workspace_bytes(M, N, K, group)
        got, blocks = set(), set()
        # (no scratch is ever reported beside a workspace: the one room is that of whichever the shape uses)
        need = want - (512 << 10) if want else L.sqp_w4a16_gemm_scratch_bytes(M, N, K, group)
        for room in (need, max(need, 48 << 20), max(need, 64 << 20), 1 << 40):
            n = L.sqp_debug_prefill_choice(M, N, K, group, 256, room, out)
            got.add(tuple(out[:5 * n]))
        for ws in (1, 2):
            L.sqp_debug_row_blocks(M, N, K, group, 256, ws, rows)
            blocks.add(tuple(rows))
        assert len(got) == 1 and len(blocks) == 1, (M, N, K, group, got, blocks)
        launches = got.pop()
        used += want > 0 and any(launches[3::5][i] > 1 for i in range(len(launches) // 5))
        if need == 0:  # neither buffer: nothing may be left in a shared one
            assert all(parts == 1 for parts in launches[3::5]), (M, N, K, group, launches)
    assert used > 4000


def test_plans_fit_the_static_array(L):
    """No shape's own plan needs more partial sums than the static array of sqp_w4a16_gemm_static holds, the
    least size of a workspace is at most the preferred one, and a call in blocks of 64 rows reports what
    its last block of fewer rows needs too.  Shapes at random, K mostly not a multiple
    of 128, and some that rounding would take past the limit."""
    limit = (512 << 10) + (48 << 20)
    rng = random.Random(7)
    shapes = [(64, 39816, 6976, 64), (64, 39816, 7008, 32), (2815, 39816, 6944, 32), (85, 71504, 6880, 32), (426, 118528, 2592, 32),
              (95, 110360, 3360, 32), (1346, 8192, 2048, 128), (1152, 8192, 22016, 64)]
    for _ in range(20000):
        group = rng.choice([8, 24, 32, 32, 64, 64, 96, 128, 192, 256])
        shapes.append((int(2 ** rng.uniform(0, 12.5)), 8 * int(2 ** rng.uniform(0, 14.5)), group * int(2 ** rng.uniform(0, 8.5)), group))
    for (M, N, K, group) in shapes:
        if max(M * K, K * N, M * N) >= 1 << 31:
            continue
        want, least = L.sqp_w4a16_gemm_workspace_bytes(M, N, K, group), L.sqp_w4a16_gemm_workspace_least_bytes(M, N, K, group)
        assert least <= want <= limit, (M, N, K, group, want)
        if M > 64 and M % 64 and group % 64 and (group != 32 or K % 64):
            assert L.sqp_w4a16_gemm_workspace_least_bytes(M % 64, N, K, group) <= least, (M, N, K, group)
            assert L.sqp_w4a16_gemm_workspace_bytes(M % 64, N, K, group) <= want, (M, N, K, group)


def test_calls_that_touch_no_workspace(L):
    """Shapes with work for the whole chip never split through the workspace, which all calls of a device
    share: callers run them beside calls that use it.  More tiles of 128 x 512 than a quarter of the
    compute units (256 where there is no GPU), or at most 64 rows and fewer than eight chunks of K."""
    for (M, N, K, group) in [(2048, 10240, 8192, 128), (3001, 44032, 8192, 128), (320, 44032, 8192, 128), (2050, 8144, 2048, 128),
                             (640, 8192, 8192, 128), (700, 8200, 1024, 64), (700, 8200, 1024, 32)]:
        assert -(-M // 128) * -(-N // 512) > 64
        assert L.sqp_w4a16_gemm_workspace_bytes(M, N, K, group) == L.sqp_w4a16_gemm_workspace_least_bytes(M, N, K, group) == 0
        assert L.sqp_w4a16_gemm_scratch_bytes(M, N, K, group) <= 48 << 20
    assert L.sqp_w4a16_gemm_scratch_bytes(2048, 10240, 8192, 128) > 0
    for group in (64, 128, 256):
        for M in (17, 33, 48, 49, 64):
            for (K, N) in [(512, 8), (512, 264), (768, 10240), (768, 1024), (256, 22016)]:
                if group >= 128:
                    assert L.sqp_w4a16_gemm_workspace_bytes(M, N, K, group) == 0, (M, N, K, group)
                assert L.sqp_w4a16_gemm_scratch_bytes(M, N, K, group) == 0
    # few tiles: the workspace serves them, and they need no scratch
    for (M, N, K, group) in [(160, 8192, 8192, 128), (256, 2056, 4096, 64), (65, 520, 2048, 128)]:
        assert L.sqp_w4a16_gemm_workspace_bytes(M, N, K, group) > 0 and L.sqp_w4a16_gemm_scratch_bytes(M, N, K, group) == 0


def test_quant_loss_argument_errors(L):
    P = ctypes.c_void_p
    good, odd, null = P(0x1000), P(0x1008), P(0)
    q = L.sqp_quant_loss
    assert q(4, 1024, 1024, 128, good, good, good, good, good, good, null, good, null) == -1
    assert q(0, 1024, 1024, 128, good, good, good, good, good, good, good, good, null) == -2
    assert q(4, 1024, 1024, 100, good, good, good, good, good, good, good, good, null) == -2
    assert q(4, 1024, 1024, 128, good, odd, good, good, good, good, good, good, null) == -3
    assert L.sqp_quant_loss_scratch_doubles(512, 8192) == 4 * 64
    assert L.sqp_quant_loss_scratch_doubles(129, 130) == 4
    assert L.sqp_quant_loss_scratch_doubles(0, 8) == 0


def test_mlp_entry_argument_errors(L):
    P = ctypes.c_void_p
    good, odd, null = P(0x1000), P(0x1008), P(0)
    f = ctypes.c_float
    assert L.sqp_rmsnorm(4, 1024, null, good, f(1e-5), good, null) == -1
    assert L.sqp_rmsnorm(4, 1020, good, good, f(1e-5), good, null) == -2
    assert L.sqp_rmsnorm(4, 1024, good, good, f(-1.0), good, null) == -4
    assert L.sqp_rmsnorm(4, 1024, good, good, f(float("nan")), good, null) == -4
    assert L.sqp_rmsnorm(4, 1024, good, odd, f(1e-5), good, null) == -3
    assert L.sqp_scale_columns(8, 1020, good, good, good, null) == -2
    assert L.sqp_scale_columns(8, 1024, good, null, good, null) == -1
    assert L.sqp_interleave_gate_up(8, 1024, good, good, odd, null) == -3
    assert L.sqp_interleave_gate_up(0, 1024, good, good, good, null) == -2
    g = L.sqp_w4a16_gemm_silu_mul
    assert g(4, 1032, 1024, 128, good, good, good, good, good, null) == -2   # N % 16
    assert g(4, 1024, 1024, 24, good, good, good, good, good, null) == -2    # group not covered by the fused store
    assert g(4, 1024, 1152, 192, good, good, good, good, good, null) == -2
    assert g(4, 1024, 1024, 128, good, good, null, good, good, null) == -1
    assert L.sqp_transpose_nk(1024, 1020, good, good, null) == -2
    assert L.sqp_transpose_nk(1024, 1024, good, odd, null) == -3


def test_row_blocks_take_whole_groups_only(L):
    """The strip kernel's chunks of 128 k hold whole groups or are parts of one: calls of more than 64 rows with other
    multiples of 64 (192, 320, ...) keep the tiled kernel, by the rule and with forced row blocks; the
    same shapes with a group that divides into chunks do take row blocks."""
    out = (ctypes.c_int * 3)()

    def rows(M, K, N, group, ws):
        L.sqp_debug_row_blocks(M, N, K, group, 256, ws, out)
        return out[0]
    rng = random.Random(17)
    shapes = [(161, 384, 776, 192), (65, 768, 1024, 192), (128, 1920, 1024, 320), (100, 4992, 4096, 192), (128, 3840, 2048, 192)]
    shapes += [(rng.randint(65, 1024), 128 * g // 64 * rng.randint(1, 8), 8 * rng.randint(96, 1024), g) for g in (192, 320, 448, 576) for _ in range(100)]
    taken = 0
    for force in (0, 3):
        L.sqp_debug_set_row_blocks(force, 1, 1)
        try:
            for M, K, N, g in shapes:
                assert K % g == 0 and K % 128 == 0
                for ws in (0, 1):
                    assert rows(M, K, N, g, ws) == 0, (M, K, N, g, ws, force)
                    taken += rows(M, K, N, 128, ws) > 0
        finally:
            L.sqp_debug_set_row_blocks(0, 0, 0)
    assert taken > len(shapes)


@pytest.mark.parametrize("T,K,N,group,n,plan", [
    (512, 4096, 2048, 128, 21, (1, 1, 1)),   # one set beside the caller's own: the next alpha prepared beside the loss
    (512, 4096, 640, 128, 21, (0, 1, 0)),    # none: the fused search one alpha after the other in the caller's own buffers
    (1024, 128, 4096, 128, 3, (1, 1, 0)),    # 256 tiles leave no room beside them
    (512, 5120, 5120, 128, 1, (2, 1, 0)),    # one alpha
    (512, 5120, 5120, 128, 21, (2, 1, 1)),   # two sets, 160 tiles: singles beside
    (64, 4096, 4096, 32, 21, (3, 3, 0)), (33, 2304, 520, 128, 4, (3, 3, 0)), (33, 2304, 2304, 64, 4, (3, 3, 0)),  # pairs in turn
    (128, 1024, 1024, 128, 21, (2, 1, 1)), (512, 2048, 4096, 64, 3, (2, 1, 1)),  # short K: singles
    (130, 384, 8, 32, 4, (-1, 0, 0)), (70, 240, 72, 40, 3, (-1, 0, 0))])  # single calls in turn
def test_alpha_search_plan_in_its_own_buffers(L, T, K, N, group, n, plan):
    """What sqp_alpha_search makes of the buffers that its callers have handed over since before it kept several sets."""
    out = (ctypes.c_int * 3)()
    L.sqp_debug_search_plan(T, N, K, group, n, ctypes.c_size_t(0), out)
    assert tuple(out) == plan


def test_forced_strips_are_strips(L):
    """A forced plan by strips, or a forced split, is what a call launches and reports, also where the rule takes column
    slices: tests that force one mean the strip kernel."""
    tb, wv = ctypes.c_int(), ctypes.c_int()
    for M, N, K, g in [(16, 328, 2048, 128), (7, 1032, 1024, 128), (20, 264, 512, 64), (1, 12288, 4096, 128)]:
        L.sqp_debug_decode_slice_plan(M, N, K, g, ctypes.byref(tb), ctypes.byref(wv))
        assert tb.value > 0
        for force, reset in ((lambda: L.sqp_debug_set_decode_plan(2, 2), lambda: L.sqp_debug_set_decode_plan(0, 0)),
                             (lambda: L.sqp_debug_set_decode_split(2), lambda: L.sqp_debug_set_decode_split(0))):
            force()
            try:
                L.sqp_debug_decode_slice_plan(M, N, K, g, ctypes.byref(tb), ctypes.byref(wv))
                assert tb.value == 0 and L.sqp_w4a16_gemm_workspace_bytes(M, N, K, g) > 512 << 10
            finally:
                reset()


def test_alpha_search_scratch_sizes(L):
    """The preferred scratch holds two batches of alphas, all of them where one batch does, within 1 GB (or four alphas'
    operands, where those are more); the least holds one alpha's; both 0 for invalid arguments."""
    sizes = []
    for f in (L.sqp_alpha_search_scratch_bytes, L.sqp_alpha_search_scratch_least_bytes):
        f.restype = ctypes.c_size_t
        sizes.append(f)
    up = lambda v: (v + 255) // 256 * 256

    def sets(T, N, K, group, n):
        head = up(8 * K) + up(4 * n * K) + up(8 * n * (-(-T // 128) * -(-N // 128)))
        one = up(K // 2 * N) + up(K // group * N * 2) + up(K // group * N) + up(2 * T * K)
        most, least = (f(T, N, K, group, n) for f in sizes)
        assert least == head + one and (most - head) % one == 0
        assert most - head <= max(1 << 30, 4 * one)
        return (most - head) // one
    assert sets(512, 5120, 5120, 128, 1) == 1         # one alpha
    assert sets(512, 5120, 5120, 128, 21) == 16       # two batches of four pairs
    assert sets(64, 1024, 1024, 128, 4) == 4          # all alphas in one batch
    big = sets(512, 44032, 8192, 128, 21)             # 198 MB each: the cap
    assert big in (4, 5)
    assert sets(4096, 65536, 16384, 128, 21) == 4     # 705 MB each: four all the same
    for bad in [(0, 8, 8, 8, 1), (8, 8, 64, 64, 0), (8, 12, 64, 64, 1), (8, 8, 64, 48, 1)]:
        assert [f(*bad) for f in sizes] == [0, 0]
    assert sizes[0](70, 72, 240, 40, 3) == sizes[1](70, 72, 240, 40, 3) > 0   # single calls


def test_slice_plans_are_built(L):
    """The rule asks for 16 waves up to four rows and for four up to eight in groups of 64 and more: the only rows that those
    variants exist for (the dispatch takes eight waves otherwise, which the rule did not mean)."""
    rng, seen, tb, wv = random.Random(23), set(), ctypes.c_int(), ctypes.c_int()
    for _ in range(30000):
        g = rng.choice([32, 64, 128, 256, 384])
        M, N, K = rng.randint(1, 32), 8 * int(2 ** rng.uniform(4, 12.5)), g * rng.randint(1, 22016 // g)
        L.sqp_debug_decode_slice_plan(M, N, K, g, ctypes.byref(tb), ctypes.byref(wv))
        seen.add((tb.value, wv.value))
        assert (tb.value, wv.value) in ((0, 0), (1, 8), (2, 8), (4, 8), (1, 16), (2, 16), (4, 4))
        assert wv.value != 16 or M <= 4
        assert wv.value != 4 or (M <= 8 and g >= 64)
    assert len(seen) == 7
