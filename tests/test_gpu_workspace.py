"""The GEMM's caller-owned workspace (sqp_set_workspace) and guard regions around every output.

Calls go straight through the C ABI (ctypes), with buffers this test owns:
  * split launches on a caller buffer, recorded into a HIP graph on a side stream with no eager
    call before the capture, replayed several times with eager work in between;
  * a workspace that is too small gives SQP_ERR_WORKSPACE and enqueues nothing; none at all
    runs the plan without a split;
  * every output buffer of every entry point (and the partial sums in the workspace) sits
    between guard regions that must still hold their fill pattern after the call.
"""
import ctypes

import numpy as np
import pytest
import torch

import workloads as wl
from gpu_util import dev, gemm_tolerance_ok

pytestmark = pytest.mark.gpu

GUARD = 4096
FILL = 0xA5
TICKET_BYTES = 512 << 10


@pytest.fixture(scope="module")
def sqp():
    import paper_2312_03788_amd as m
    m.lib()
    return m


class Guarded:
    """A device buffer of `nbytes` between two guard regions filled with a pattern."""

    def __init__(self, nbytes, dtype=torch.uint8, shape=None):
        self.nbytes = int(nbytes)
        pad = (-self.nbytes) % 16
        self.raw = torch.full((self.nbytes + pad + 2 * GUARD,), FILL, dtype=torch.uint8, device="cuda")
        self.body = self.raw[GUARD:GUARD + self.nbytes]
        self.dtype, self.shape = dtype, shape

    @property
    def ptr(self):
        return ctypes.c_void_p(self.raw.data_ptr() + GUARD)

    def view(self):
        t = self.body.view(self.dtype)
        return t.reshape(self.shape) if self.shape is not None else t

    def numpy(self):
        return self.view().cpu().numpy()

    def check(self, what):
        torch.cuda.synchronize()
        lo = self.raw[:GUARD].cpu().numpy()
        hi = self.raw[GUARD + self.nbytes:].cpu().numpy()
        assert (lo == FILL).all(), "%s: bytes before the buffer were written" % what
        assert (hi == FILL).all(), "%s: bytes after the buffer were written" % what


def _ptr(t):
    return ctypes.c_void_p(t.data_ptr())


def _dev(a):
    if a.dtype == np.uint32:
        a = a.view(np.int32)
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _layer(orc, M, K, N, group, shape_idx=0):
    x, xcal, w = wl.layer_inputs(M, K, N, shape_idx=shape_idx)
    s = orc.smooth_scales(xcal, w, wl.ALPHA)
    p, sc, z = orc.quantize_pack(orc.smooth_apply_w(w, s), group)
    return orc.smooth_apply_x(x, s), p, sc, z


def _gemm(L, M, N, K, group, dx, dp, dsc, dz, y_ptr, stream=None):
    st = ctypes.c_void_p(stream if stream is not None else torch.cuda.current_stream().cuda_stream)
    return L.sqp_w4a16_gemm(M, N, K, group, _ptr(dx), _ptr(dp), _ptr(dsc), _ptr(dz), y_ptr, st)


def _set_ws(L, ptr, nbytes):
    rc = L.sqp_set_workspace(ptr, ctypes.c_size_t(nbytes), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0, rc


# shapes whose own plan splits K: the streaming kernel (16 and 64 rows) and the tiled kernel's K parts
SPLIT_CASES = [(16, 2048, 328, 128), (64, 4096, 512, 128), (7, 1024, 200, 64), (256, 2048, 520, 128), (130, 1024, 264, 64)]


def test_workspace_graph_capture_side_stream(orc, sqp):
    """Split launches on a caller-owned workspace recorded into a graph on a non-default
    stream; no eager GEMM call has used this workspace or these shapes before the capture."""
    L = sqp.lib()
    need = max(sqp.workspace_bytes(M, N, K, g) for (M, K, N, g) in SPLIT_CASES)
    assert need > TICKET_BYTES
    ws = Guarded(need)
    cases = []
    for (M, K, N, g) in SPLIT_CASES:
        assert sqp.workspace_bytes(M, N, K, g) > 0, (M, K, N, g)
        xs, p, sc, z = _layer(orc, M, K, N, g)
        cases.append((M, K, N, g, xs, p, sc, z, _dev(xs), _dev(p), _dev(sc), _dev(z), Guarded(2 * M * N, torch.float16, (M, N))))
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    try:
        with torch.cuda.stream(side):
            _set_ws(L, ws.ptr, need)     # enqueues the ticket-zeroing kernel on the side stream
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                for (M, K, N, g, xs, p, sc, z, dx, dp, dsc, dz, y) in cases:
                    rc = _gemm(L, M, N, K, g, dx, dp, dsc, dz, y.ptr, torch.cuda.current_stream().cuda_stream)
                    assert rc == 0, rc
        torch.cuda.synchronize()
        first = None
        for replay in range(3):
            for c in cases:
                c[-1].view().zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            outs = [c[-1].numpy().copy() for c in cases]
            if first is None:
                first = outs
                for (M, K, N, g, xs, p, sc, z, *_), y in zip(cases, outs):
                    y_ref, t_ref = orc.w4a16_gemm_ref(xs, p, sc, z, g)
                    ok, worst, nbad = gemm_tolerance_ok(orc, y, y_ref, t_ref)
                    assert ok, "(%d,%d,%d,%d): worst err/tol %.3f, %d out of tolerance" % (M, K, N, g, worst, nbad)
            else:
                for a, b in zip(first, outs):
                    assert np.array_equal(a.view(np.uint16), b.view(np.uint16)), "replay %d differs" % replay
            # eager work of the same kind between the replays (same workspace, default stream)
            M, K, N, g, xs, p, sc, z, dx, dp, dsc, dz, y = cases[replay % len(cases)]
            assert _gemm(L, M, N, K, g, dx, dp, dsc, dz, y.ptr) == 0
            torch.cuda.synchronize()
            assert np.array_equal(y.numpy().view(np.uint16), first[replay % len(cases)].view(np.uint16))
        for c in cases:
            c[-1].check("y of %s" % (c[:4],))
        ws.check("workspace")
    finally:
        torch.cuda.synchronize()
        sqp.set_workspace(0)   # through the binding, so that it knows no workspace is set any more


def test_workspace_too_small_or_absent(orc, sqp):
    L = sqp.lib()
    M, K, N, g = 16, 2048, 328, 128
    xs, p, sc, z = _layer(orc, M, K, N, g)
    dx, dp, dsc, dz = _dev(xs), _dev(p), _dev(sc), _dev(z)
    y_ref, t_ref = orc.w4a16_gemm_ref(xs, p, sc, z, g)
    need = sqp.workspace_bytes(M, N, K, g)
    ws = Guarded(need)
    y = Guarded(2 * M * N, torch.float16, (M, N))
    try:
        # 16 bytes short of what the plan needs: refused, nothing written
        _set_ws(L, ws.ptr, need - 16)
        assert _gemm(L, M, N, K, g, dx, dp, dsc, dz, y.ptr) == -6
        torch.cuda.synchronize()
        assert (y.body.cpu().numpy() == FILL).all()
        # exactly enough
        _set_ws(L, ws.ptr, need)
        assert _gemm(L, M, N, K, g, dx, dp, dsc, dz, y.ptr) == 0
        torch.cuda.synchronize()
        ok, worst, nbad = gemm_tolerance_ok(orc, y.numpy(), y_ref, t_ref)
        assert ok, (worst, nbad)
        ws.check("workspace")
        # none: the plan without a split
        assert L.sqp_set_workspace(None, ctypes.c_size_t(0), None) == 0
        y.view().zero_()
        assert _gemm(L, M, N, K, g, dx, dp, dsc, dz, y.ptr) == 0
        torch.cuda.synchronize()
        ok, worst, nbad = gemm_tolerance_ok(orc, y.numpy(), y_ref, t_ref)
        assert ok, (worst, nbad)
        y.check("y")
        # argument errors of the setter
        assert L.sqp_set_workspace(ctypes.c_void_p(ws.raw.data_ptr() + GUARD + 8), ctypes.c_size_t(need), None) == -3
        assert L.sqp_set_workspace(ws.ptr, ctypes.c_size_t(TICKET_BYTES), None) == -6
    finally:
        torch.cuda.synchronize()
        sqp.set_workspace(0)   # through the binding, so that it knows no workspace is set any more


@pytest.mark.parametrize("M,K,N,group", [
    (1, 256, 8, 128), (5, 512, 72, 128), (16, 2048, 328, 128), (17, 1024, 200, 64), (33, 512, 136, 32), (64, 1024, 264, 128),
    (3, 48, 24, 24), (65, 256, 264, 128), (130, 384, 72, 64), (257, 1024, 264, 128), (300, 1024, 520, 128), (100, 128, 64, 32)])
@pytest.mark.parametrize("with_ws", [True, False])
def test_gemm_outputs_between_guards(orc, sqp, M, K, N, group, with_ws):
    """Ragged M and N through every kernel family, with and without a workspace: y and the
    partial sums stay inside their buffers, and the result meets the tolerance."""
    print("case guard gemm", M, K, N, group, with_ws, flush=True)
    L = sqp.lib()
    xs, p, sc, z = _layer(orc, M, K, N, group)
    dx, dp, dsc, dz = _dev(xs), _dev(p), _dev(sc), _dev(z)
    y = Guarded(2 * M * N, torch.float16, (M, N))
    need = sqp.workspace_bytes(M, N, K, group)
    ws = Guarded(need) if (with_ws and need) else None
    try:
        if ws is not None:
            _set_ws(L, ws.ptr, need)
        else:
            assert L.sqp_set_workspace(None, ctypes.c_size_t(0), None) == 0
        assert _gemm(L, M, N, K, group, dx, dp, dsc, dz, y.ptr) == 0
        y.check("y")
        if ws is not None:
            ws.check("workspace")
        y_ref, t_ref = orc.w4a16_gemm_ref(xs, p, sc, z, group)
        ok, worst, nbad = gemm_tolerance_ok(orc, y.numpy(), y_ref, t_ref)
        assert ok, "worst err/tol %.3f, %d elements out of tolerance" % (worst, nbad)
        if N % 16 == 0 and group in (32, 64, 128):
            h = Guarded(2 * M * (N // 2), torch.float16, (M, N // 2))
            st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
            assert L.sqp_w4a16_gemm_silu_mul(M, N, K, group, _ptr(dx), _ptr(dp), _ptr(dsc), _ptr(dz), h.ptr, st) == 0
            h.check("silu_mul y")
            if ws is not None:
                ws.check("workspace after silu_mul")
    finally:
        torch.cuda.synchronize()
        sqp.set_workspace(0)   # through the binding, so that it knows no workspace is set any more


@pytest.mark.parametrize("M,K,N,group", [(65, 256, 264, 128), (130, 384, 72, 64), (300, 1024, 520, 128), (100, 128, 64, 32)])
@pytest.mark.parametrize("with_ws", [True, False])
def test_tiled_gemm_outputs_between_guards(orc, sqp, M, K, N, group, with_ws):
    """The same in the tiled kernel, on shapes that the rule gives to the strip kernel's row blocks."""
    sqp.lib().sqp_debug_set_row_blocks(-1, 0, 0)
    try:
        test_gemm_outputs_between_guards(orc, sqp, M, K, N, group, with_ws)
    finally:
        sqp.lib().sqp_debug_set_row_blocks(0, 0, 0)


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("M,K,N", [(1, 256, 8), (5, 512, 72), (9, 1152, 200), (16, 2048, 328), (13, 128, 1032), (4, 128 * 9, 48)])
def test_slice_kernel_outputs_between_guards(orc, sqp, M, K, N, mode):
    """The column-slice kernel (forced, both slice widths, no workspace set) on ragged M and N:
    y of the plain and of the fused call stay inside their buffers and meet the tolerance."""
    print("case guard slice", M, K, N, mode, flush=True)
    L = sqp.lib()
    group = 128
    xs, p, sc, z = _layer(orc, M, K, N, group)
    dx, dp, dsc, dz = _dev(xs), _dev(p), _dev(sc), _dev(z)
    y = Guarded(2 * M * N, torch.float16, (M, N))
    L.sqp_debug_set_decode_slice(mode)
    try:
        assert L.sqp_set_workspace(None, ctypes.c_size_t(0), None) == 0
        assert sqp.workspace_bytes(M, N, K, group) == 0
        assert _gemm(L, M, N, K, group, dx, dp, dsc, dz, y.ptr) == 0
        y.check("y")
        y_ref, t_ref = orc.w4a16_gemm_ref(xs, p, sc, z, group)
        ok, worst, nbad = gemm_tolerance_ok(orc, y.numpy(), y_ref, t_ref)
        assert ok, "worst err/tol %.3f, %d elements out of tolerance" % (worst, nbad)
        if N % 16 == 0:
            h = Guarded(2 * M * (N // 2), torch.float16, (M, N // 2))
            st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
            assert L.sqp_w4a16_gemm_silu_mul(M, N, K, group, _ptr(dx), _ptr(dp), _ptr(dsc), _ptr(dz), h.ptr, st) == 0
            h.check("silu_mul y")
    finally:
        torch.cuda.synchronize()
        L.sqp_debug_set_decode_slice(0)
        sqp.set_workspace(0)


@pytest.mark.parametrize("K,N,group", [(256, 8, 128), (384, 72, 64), (1024, 520, 128), (96, 24, 24), (512, 136, 32), (2048, 1000, 256)])
def test_companion_outputs_between_guards(orc, sqp, K, N, group):
    """Every output of the companion entry points between guard regions, on ragged shapes;
    the contents are compared with the oracle as in the bit-exact tests."""
    print("case guard companion", K, N, group, flush=True)
    L = sqp.lib()
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    T, M = 37, 5
    xcal = wl.activation(T, K, seed=3000)
    x = wl.activation(M, K, seed=2000 + M)
    w = wl.weight(K, N, seed=1000)
    dxcal, dx, dw = _dev(xcal), _dev(x), _dev(w)
    s = Guarded(4 * K, torch.float32, (K,))
    assert L.sqp_smooth_scales(T, K, N, ctypes.c_float(0.5), _ptr(dxcal), _ptr(dw), s.ptr, st) == 0
    s.check("s")
    s_ref = orc.smooth_scales(xcal, w, 0.5)
    assert np.abs(s.numpy().view(np.int32).astype(np.int64) - s_ref.view(np.int32).astype(np.int64)).max() <= 1
    ds = _dev(s_ref)
    xo = Guarded(2 * M * K, torch.float16, (M, K))
    wo = Guarded(2 * K * N, torch.float16, (K, N))
    assert L.sqp_smooth_apply_x(M, K, _ptr(dx), _ptr(ds), xo.ptr, st) == 0
    assert L.sqp_smooth_apply_w(K, N, _ptr(dw), _ptr(ds), wo.ptr, st) == 0
    xo.check("x_out")
    wo.check("w_out")
    ws_ref = orc.smooth_apply_w(w, s_ref)
    assert np.array_equal(xo.numpy().view(np.uint16), orc.smooth_apply_x(x, s_ref).view(np.uint16))
    assert np.array_equal(wo.numpy().view(np.uint16), ws_ref.view(np.uint16))
    pk = Guarded(4 * (K // 8) * N, torch.int32, (K // 8, N))
    sc = Guarded(2 * (K // group) * N, torch.float16, (K // group, N))
    zr = Guarded((K // group) * N, torch.uint8, (K // group, N))
    assert L.sqp_quantize_pack(N, K, group, wo.ptr, pk.ptr, sc.ptr, zr.ptr, st) == 0
    for b, name in ((pk, "packed"), (sc, "scales"), (zr, "zeros")):
        b.check(name)
    p_ref, sc_ref, z_ref = orc.quantize_pack(ws_ref, group)
    assert np.array_equal(pk.numpy().view(np.uint32), p_ref)
    assert np.array_equal(sc.numpy().view(np.uint16), sc_ref.view(np.uint16))
    assert np.array_equal(zr.numpy(), z_ref)
    wh = Guarded(2 * K * N, torch.float16, (K, N))
    assert L.sqp_dequantize(N, K, group, pk.ptr, sc.ptr, zr.ptr, wh.ptr, st) == 0
    wh.check("w_hat")
    assert np.array_equal(wh.numpy().view(np.uint16), orc.dequantize(p_ref, sc_ref, z_ref, group).view(np.uint16))
    # Eq. 4: scratch and the one-double result
    L.sqp_quant_loss_scratch_doubles.restype = ctypes.c_long
    nd = int(L.sqp_quant_loss_scratch_doubles(T, N))
    scr = Guarded(8 * nd, torch.float64, (nd,))
    loss = Guarded(8, torch.float64, (1,))
    dxh = _dev(orc.smooth_apply_x(xcal, s_ref))
    assert L.sqp_quant_loss(T, N, K, group, _ptr(dxcal), _ptr(dw), _ptr(dxh), pk.ptr, sc.ptr, zr.ptr, scr.ptr, loss.ptr, st) == 0
    scr.check("loss scratch")
    loss.check("loss")
    e_ref = orc.quant_loss(xcal, w, orc.smooth_apply_x(xcal, s_ref), orc.dequantize(p_ref, sc_ref, z_ref, group))
    assert abs(float(loss.numpy()[0]) - e_ref) <= 2e-3 * e_ref
    # transposed input and the LlamaMLP helpers
    wt = Guarded(2 * K * N, torch.float16, (K, N))
    dwn = _dev(np.ascontiguousarray(w.T))
    assert L.sqp_transpose_nk(N, K, _ptr(dwn), wt.ptr, st) == 0
    wt.check("w_kn")
    assert np.array_equal(wt.numpy().view(np.uint16), w.view(np.uint16))
    yn = Guarded(2 * M * K, torch.float16, (M, K))
    gamma = _dev(np.ones(K, np.float16))
    assert L.sqp_rmsnorm(M, K, _ptr(dx), _ptr(gamma), ctypes.c_float(1e-5), yn.ptr, st) == 0
    yn.check("rmsnorm y")
    wc = Guarded(2 * K * N, torch.float16, (K, N))
    dsn = _dev(np.linspace(0.5, 2.0, N).astype(np.float32))
    assert L.sqp_scale_columns(K, N, _ptr(dw), _ptr(dsn), wc.ptr, st) == 0
    wc.check("scale_columns out")
    wi = Guarded(2 * K * 2 * N, torch.float16, (K, 2 * N))
    assert L.sqp_interleave_gate_up(K, N, _ptr(dw), _ptr(dw), wi.ptr, st) == 0
    wi.check("interleave out")
    assert np.array_equal(wi.numpy()[:, 0::2].view(np.uint16), w.view(np.uint16))


@pytest.mark.parametrize("M,K,N,group", [(56, 1024, 2056, 128), (40, 1024, 520, 64), (65, 2048, 520, 128), (130, 1024, 264, 32),
                                         (150, 1536, 1032, 256)])
def test_workspace_between_least_and_preferred(orc, sqp, M, K, N, group):
    """Buffers from the least size (nothing beside the tickets, where that is 0) to the preferred one: a
    plan that fits runs, inside its buffer; 16 bytes below the least size the call is refused."""
    print("case least workspace", M, K, N, group, flush=True)
    L = sqp.lib()
    least, want = int(L.sqp_w4a16_gemm_workspace_least_bytes(M, N, K, group)), sqp.workspace_bytes(M, N, K, group)
    assert 0 <= least <= want and want > 0
    xs, p, sc, z = _layer(orc, M, K, N, group)
    dx, dp, dsc, dz = _dev(xs), _dev(p), _dev(sc), _dev(z)
    rows = np.unique(np.linspace(0, M - 1, min(M, 48)).astype(int))
    y_ref, t_ref = orc.w4a16_gemm_ref(np.ascontiguousarray(xs[rows]), p, sc, z, group)
    y = Guarded(2 * M * N, torch.float16, (M, N))
    try:
        lo = max(least, TICKET_BYTES + 16)
        for size in sorted({lo, lo + (want - lo) // 3 // 16 * 16, max(lo, want - 16), want}):
            ws = Guarded(size)
            _set_ws(L, ws.ptr, size)
            y.view().zero_()
            assert _gemm(L, M, N, K, group, dx, dp, dsc, dz, y.ptr) == 0, size
            torch.cuda.synchronize()
            ok, worst, nbad = gemm_tolerance_ok(orc, y.numpy()[rows], y_ref, t_ref)
            assert ok, (size, worst, nbad)
            ws.check("workspace")
            y.check("y")
        if least > TICKET_BYTES + 16:
            ws = Guarded(least)
            _set_ws(L, ws.ptr, least - 16)
            assert _gemm(L, M, N, K, group, dx, dp, dsc, dz, y.ptr) == -6
    finally:
        torch.cuda.synchronize()
        sqp.set_workspace(0)


@pytest.mark.parametrize("M,K,N,group", [(65, 2048, 520, 128), (130, 1024, 264, 32), (150, 1536, 1032, 256)])
def test_workspace_between_least_and_preferred_in_tiles(orc, sqp, M, K, N, group):
    """The same for the tiled kernel's parts, on shapes that the rule gives to the strip kernel's row blocks."""
    sqp.lib().sqp_debug_set_row_blocks(-1, 0, 0)
    try:
        test_workspace_between_least_and_preferred(orc, sqp, M, K, N, group)
    finally:
        sqp.lib().sqp_debug_set_row_blocks(0, 0, 0)


@pytest.mark.parametrize("M,K,N,group", [(11, 16448, 136, 64), (2, 14080, 264, 128), (20, 7168, 520, 256), (32, 9216, 72, 32)])
def test_without_a_workspace_long_k_takes_slices(orc, sqp, M, K, N, group):
    """K so long that the strip kernel is faster where it can split: without a workspace it cannot, and the column slices
    run (the bits of the forced ones); with one the strips do."""
    print("case no workspace", M, K, N, group, flush=True)
    L = sqp.lib()
    tb, wv = ctypes.c_int(), ctypes.c_int()
    L.sqp_debug_decode_slice_plan(M, N, K, group, ctypes.byref(tb), ctypes.byref(wv))
    assert tb.value == 0
    xs, p, sc, z = _layer(orc, M, K, N, group)
    dx, dp, dsc, dz = _dev(xs), _dev(p), _dev(sc), _dev(z)
    y, forced = Guarded(2 * M * N, torch.float16, (M, N)), Guarded(2 * M * N, torch.float16, (M, N))
    assert L.sqp_set_workspace(None, ctypes.c_size_t(0), None) == 0
    try:
        assert _gemm(L, M, N, K, group, dx, dp, dsc, dz, y.ptr) == 0
        L.sqp_debug_set_slice_plan(1, 16 if M <= 4 else 8, 1)
        assert _gemm(L, M, N, K, group, dx, dp, dsc, dz, forced.ptr) == 0
    finally:
        L.sqp_debug_set_slice_plan(0, 0, 0)
        torch.cuda.synchronize()
        sqp.set_workspace(0)
    y.check("y")
    ok, worst, nbad = gemm_tolerance_ok(orc, y.numpy(), *orc.w4a16_gemm_ref(xs, p, sc, z, group))
    assert ok, (worst, nbad)
    assert np.array_equal(y.numpy().view(np.uint16), forced.numpy().view(np.uint16))


@pytest.mark.parametrize("M,K,N,group,fused", [(2050, 2048, 8144, 128, 0), (660, 2048, 5184, 64, 1)])
def test_scratch_of_one_call(orc, sqp, M, K, N, group, fused):
    """Grids that fill the chip: no workspace asked for and none touched; with a scratch buffer of the
    call's own the K parts stay inside it, whatever its size; a misaligned one is refused.  (Without row
    blocks, which one of the shapes takes and which leave the scratch untouched.)"""
    print("case scratch", M, K, N, group, fused, flush=True)
    L = sqp.lib()
    want = int(L.sqp_w4a16_gemm_scratch_bytes(M, N, K, group))
    assert sqp.workspace_bytes(M, N, K, group) == 0 and want > 0
    xs, p, sc, z = _layer(orc, M, K, N, group)
    dx, dp, dsc, dz = _dev(xs), _dev(p), _dev(sc), _dev(z)
    rows = np.unique(np.linspace(0, M - 1, 24).astype(int))
    y_ref, t_ref = orc.w4a16_gemm_ref(np.ascontiguousarray(xs[rows]), p, sc, z, group)
    NY = N // 2 if fused else N
    y, ws = Guarded(2 * M * NY, torch.float16, (M, NY)), Guarded(1 << 20)
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    call = lambda own, size: L.sqp_w4a16_gemm_scratch(M, N, K, group, fused, _ptr(dx), _ptr(dp), _ptr(dsc), _ptr(dz), y.ptr, own,
                                                      ctypes.c_size_t(size), st)
    outs = []
    L.sqp_debug_set_row_blocks(-1, 0, 0)
    try:
        _set_ws(L, ws.ptr, 1 << 20)
        torch.cuda.synchronize()
        ws.body[TICKET_BYTES:] = FILL
        for size in (0, 16, want // 3 // 16 * 16, want - 16, want):
            own = Guarded(size)
            y.view().zero_()
            assert call(own.ptr if size else None, size) == 0, size
            torch.cuda.synchronize()
            if not fused:
                ok, worst, nbad = gemm_tolerance_ok(orc, y.numpy()[rows], y_ref, t_ref)
                assert ok, (size, worst, nbad)
            outs.append(y.numpy().copy())
            own.check("scratch")
            y.check("y")
        assert (ws.body.cpu().numpy()[TICKET_BYTES:] == FILL).all(), "the shared workspace was written"
        # the binding passes a buffer of the preferred size, with and without an output
        fn = sqp.w4a16_gemm_silu_mul if fused else sqp.w4a16_gemm
        out = torch.empty((M, NY), dtype=torch.float16, device="cuda")
        for got in (fn(dx, dp, dsc, dz, group), fn(dx, dp, dsc, dz, group, out=out)):
            assert np.array_equal(got.cpu().numpy().view(np.uint16), outs[-1].view(np.uint16))
        if fused:  # the plain product's gate and up, each fp16-rounded (2^-11) and summed in another order
            gu = sqp.w4a16_gemm(dx, dp, dsc, dz, group).double()
            h = torch.nn.functional.silu(gu[:, 0::2]) * gu[:, 1::2]
            for o in outs:
                d = (torch.from_numpy(o).cuda().double() - h).abs()
                assert bool((d <= 4 * 2.0 ** -11 * h.abs() + 2.0 ** -10 * gu[:, 1::2].abs() * gu[:, 0::2].abs() + 1e-3).all())
        assert call(ctypes.c_void_p(own.raw.data_ptr() + GUARD + 8), want) == -3
    finally:
        L.sqp_debug_set_row_blocks(0, 0, 0)
        torch.cuda.synchronize()
        sqp.set_workspace(0)


def test_prefill_beside_decode_on_another_stream(orc, sqp):
    """A prompt whose tiles fill the chip on one stream beside split decode calls on another, through the
    binding: each gives the bits it gives alone.  (The prompt's shape reports no workspace, so the
    two need no ordering.)"""
    print("case two streams", flush=True)
    pre, dec = (2050, 2048, 8144, 128), (16, 2048, 328, 128)
    assert sqp.workspace_bytes(pre[0], pre[2], pre[1], pre[3]) == 0 and sqp.workspace_bytes(dec[0], dec[2], dec[1], dec[3]) > 0
    args = []
    for (M, K, N, g) in (pre, dec):
        xs, p, sc, z = _layer(orc, M, K, N, g)
        args.append((_dev(xs), _dev(p), _dev(sc), _dev(z), g))
    sqp.set_workspace(32 << 20)
    try:
        alone = [sqp.w4a16_gemm(*a) for a in args]
        torch.cuda.synchronize()
        streams = [torch.cuda.Stream(), torch.cuda.Stream()]
        outs = [[], []]
        for _ in range(12):
            for i, reps in ((0, 1), (1, 8)):
                with torch.cuda.stream(streams[i]):
                    outs[i] += [sqp.w4a16_gemm(*args[i]) for _ in range(reps)]
        torch.cuda.synchronize()
        for i in (0, 1):
            for y in outs[i]:
                assert torch.equal(y, alone[i])
    finally:
        torch.cuda.synchronize()
        sqp.set_workspace(0)


def test_scratch_under_capture(orc, sqp):
    """Under graph capture a call that is given its output allocates nothing and takes the plan without K
    parts; one that is not takes scratch from the graph's pool, as its output.  Replays are bit-identical
    to the eager calls, with eager work in between."""
    M, K, N, g = 2050, 2048, 8144, 128
    xs, p, sc, z = _layer(orc, M, K, N, g)
    dx, dp, dsc, dz = _dev(xs), _dev(p), _dev(sc), _dev(z)
    y_ref, t_ref = orc.w4a16_gemm_ref(np.ascontiguousarray(xs[-4:]), p, sc, z, g)
    eager = sqp.w4a16_gemm(dx, dp, dsc, dz, g)
    given = torch.empty_like(eager)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        own = sqp.w4a16_gemm(dx, dp, dsc, dz, g)
        sqp.w4a16_gemm(dx, dp, dsc, dz, g, out=given)
    first = None
    for _ in range(3):
        own.zero_(), given.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(own, eager)
        ok, worst, nbad = gemm_tolerance_ok(orc, given[-4:].cpu().numpy(), y_ref, t_ref)
        assert ok, (worst, nbad)
        first = given.clone() if first is None else first
        assert torch.equal(given, first) and torch.equal(sqp.w4a16_gemm(dx, dp, dsc, dz, g), eager)


def test_native_marshalling_equals_general_path(orc, sqp):
    """The serving calls through the native marshalling give the general path's bits, with and without
    an output; what the general path refuses is refused with the same error, and what it takes
    (a flat output of the right size, a tensor subclass) is still taken."""
    import paper_2312_03788_amd.binding as b
    _, xcal, w = wl.layer_inputs(1, 512, 272)
    p, sc, z = (dev(a) for a in orc.quantize_pack(w, 128))
    x, s = dev(np.ascontiguousarray(xcal[:5])), dev(orc.smooth_scales(xcal, w, 0.5))
    gamma = torch.ones(512, dtype=torch.float16, device="cuda")
    new = lambda n: torch.empty((5, n), dtype=torch.float16, device="cuda")
    calls = [(sqp.w4a16_gemm, (x, p, sc, z, 128), 272), (sqp.w4a16_gemm_static, (x, p, sc, z, 128), 272),
             (sqp.w4a16_gemm_silu_mul, (x, p, sc, z, 128), 136), (sqp.rmsnorm, (x, gamma, 1e-5), 512), (sqp.smooth_apply_x, (x, s), 512)]

    class Tagged(torch.Tensor):
        pass

    def general(fn, *args, **kw):
        held, b._fast = b._fast, None
        try:
            return fn(*args, **kw)
        finally:
            b._fast = held

    for fn, args, n in calls:
        want = general(fn, *args)
        assert b._native(x) and fn(*args).shape == want.shape == (5, n)
        for out in (None, new(n), torch.empty(5 * n, dtype=torch.float16, device="cuda")):
            got = fn(*args, out=out)
            assert out is None or got is out
            assert torch.equal(got.reshape(5, n), want) and got.dtype == torch.float16
        tagged = (args[0].as_subclass(Tagged),) + args[1:]
        got, seen = fn(*tagged), general(fn, *tagged)
        assert type(got) is type(seen) and torch.equal(got.as_subclass(torch.Tensor), want)
        kept = torch.nn.Parameter(args[0], requires_grad=False)
        assert type(fn(kept, *args[1:])) is type(general(fn, kept, *args[1:])) is torch.Tensor
        bad = [(x.float(),) + args[1:], (x.cpu(),) + args[1:], (torch.cat([x, x], 1)[:, ::2],) + args[1:],
               (x.reshape(-1)[:5 * 512 - 5].reshape(5, 511),) + args[1:], args[:1] + (args[1].double(),) + args[2:]]
        for a in bad:
            messages = []
            for run in (fn, lambda *v: general(fn, *v)):
                with pytest.raises((b.SqpError, RuntimeError)) as e:
                    run(*a)
                messages.append(str(e.value))
            assert messages[0] == messages[1], messages
    torch.cuda.synchronize()


def test_native_marshalling_of_preparation_equals_the_general_path(orc, sqp):
    """The calls that prepare a weight: the general path's bits with and without outputs (also a flat one and,
    where that path takes one, a larger one), its types for subclasses and parameters, its errors."""
    import paper_2312_03788_amd.binding as b
    _, xcal, wn = wl.layer_inputs(1, 512, 272)
    x, w = dev(np.ascontiguousarray(xcal[:7])), dev(wn)
    s, cols = dev(orc.smooth_scales(xcal, wn, 0.5)), torch.rand(272, device="cuda") + 0.5
    pk = sqp.quantize_pack(w, 64)

    class Tagged(torch.Tensor):
        pass

    def general(fn, *args, **kw):
        held, b._fast = b._fast, None
        try:
            return fn(*args, **kw)
        finally:
            b._fast = held

    tup = lambda o: o if isinstance(o, tuple) else (o,)
    calls = [(sqp.smooth_scales, (x, w, 0.5), 1), (sqp.smooth_apply_w, (w, s), 0), (sqp.scale_columns, (w, cols), 0), (sqp.transpose_nk, (w,), 0),
             (sqp.interleave_gate_up, (w, w * 2), 0), (sqp.quantize_pack, (w, 64), 0), (sqp.dequantize, (*pk, 64), 0)]
    for fn, args, where in calls:
        want = tup(general(fn, *args))
        outs = [None, tuple(torch.empty_like(o) for o in want)]
        if len(want) == 1:
            outs += [(torch.empty(want[0].numel(), dtype=want[0].dtype, device="cuda"),), (torch.zeros(want[0].numel() + 8, dtype=want[0].dtype, device="cuda"),)]
        for out in outs:
            got = tup(fn(*args) if out is None else fn(*args, out=out if len(out) > 1 else out[0]))
            assert out is None or all(g is o for g, o in zip(got, out))
            for g, o in zip(got, want):
                assert g.dtype == o.dtype and torch.equal(g.reshape(-1)[:o.numel()], o.reshape(-1)), fn.__name__
                assert out is not None or g.shape == o.shape
        for cast in (lambda t: t.as_subclass(Tagged), lambda t: torch.nn.Parameter(t, requires_grad=False)):
            odd = args[:where] + (cast(args[where]),) + args[where + 1:]
            for g, o, v in zip(tup(fn(*odd)), tup(general(fn, *odd)), want):
                assert type(g) is type(o) and torch.equal(g.as_subclass(torch.Tensor), v)
        first = args[where]
        for v in (first.double(), first.cpu(), torch.cat([first, first], 1)[:, ::2], first[:0]):
            a = args[:where] + (v,) + args[where + 1:]
            messages = []
            for run in (fn, lambda *q: general(fn, *q)):
                with pytest.raises((b.SqpError, RuntimeError)) as e:
                    run(*a)
                messages.append(str(e.value))
            assert messages[0] == messages[1], (fn.__name__, messages)
    for bad in (lambda: sqp.quantize_pack(w, 0), lambda: sqp.quantize_pack(w, 100), lambda: sqp.smooth_scales(x[:, :508].contiguous(), w, 0.5)):
        with pytest.raises(b.SqpError):
            bad()
    torch.cuda.synchronize()


def test_native_outputs_under_dispatch_modes(orc, sqp):
    """Outputs are allocated through the dispatcher wherever a mode or the inference mode wants to know of them."""
    from torch.utils._python_dispatch import TorchDispatchMode
    seen = []

    class Watch(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            seen.append(str(func))
            return func(*args, **(kwargs or {}))

    w = torch.randn((512, 272), device="cuda").half()
    x = torch.randn((3, 512), device="cuda").half()
    p = sqp.quantize_pack(w, 128)
    want = sqp.w4a16_gemm(x, *p, 128)
    with Watch():
        got = sqp.w4a16_gemm(x, *p, 128)
    assert any("empty" in f for f in seen) and torch.equal(got, want)
    with torch.inference_mode():
        got = sqp.w4a16_gemm(x, *p, 128)
        assert got.is_inference() and torch.equal(got, want)
    with torch.no_grad():
        got = sqp.w4a16_gemm(x, *p, 128)
    assert not got.is_inference() and not got.requires_grad and torch.equal(got, want)


def test_native_outputs_under_a_profiler(sqp):
    """A profiler's operator records show the allocation of a native call's output, as they show any other operator's."""
    w = torch.randn((512, 272), device="cuda").half()
    x = torch.randn((3, 512), device="cuda").half()
    p, ones = sqp.quantize_pack(w, 128), torch.ones(512, device="cuda")
    sqp.w4a16_gemm(x, *p, 128)
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CPU]) as prof:
        sqp.w4a16_gemm(x, *p, 128)
        sqp.smooth_apply_w(w, ones)
    seen = {e.key: e.count for e in prof.key_averages()}
    assert seen.get("aten::empty", 0) >= 2, seen


def test_native_marshalling_reports_the_librarys_code(sqp):
    """A code that the library returns ends in the general path's error after one call: a launch error may
    stem from earlier work while this call's kernels were enqueued, so it neither disappears nor is
    the call made again (in place, smooth_apply_x would divide twice).  The library's entry points are
    replaced by counting stubs."""
    import paper_2312_03788_amd.binding as b
    L = sqp.lib()
    c, vp = ctypes.c_int, ctypes.c_void_p
    calls = []

    def stub(nargs, types):
        def run(*a):
            calls.append(len(a))
            return -5
        return ctypes.CFUNCTYPE(*types)(run)

    gemm = [c] + [c] * 4 + [vp] * 6
    entries = [stub(10, gemm) for _ in range(3)] + [L.sqp_w4a16_gemm_workspace_bytes]
    entries += [stub(7, [c, c, c, vp, vp, ctypes.c_float, vp, vp]), stub(6, [c, c, c, vp, vp, vp, vp])]
    entries += [stub(13, [c] * 6 + [vp] * 6 + [ctypes.c_size_t, vp]), L.sqp_w4a16_gemm_scratch_bytes]
    address = lambda f: ctypes.cast(f, vp).value
    x, s = torch.randn((5, 512), device="cuda").half(), torch.full((512,), 2.0, device="cuda")
    p = torch.zeros((64, 272), dtype=torch.int32, device="cuda")
    sc = torch.zeros((4, 272), dtype=torch.float16, device="cuda")
    z = torch.zeros((4, 272), dtype=torch.uint8, device="cuda")
    gamma, before = torch.ones(512, dtype=torch.float16, device="cuda"), x.clone()
    sqp.set_workspace(1 << 20)
    real = [L.sqp_w4a16_gemm, L.sqp_w4a16_gemm_silu_mul, L.sqp_w4a16_gemm_static, L.sqp_w4a16_gemm_workspace_bytes, L.sqp_rmsnorm,
            L.sqp_smooth_apply_x, L.sqp_w4a16_gemm_scratch, L.sqp_w4a16_gemm_scratch_bytes]
    try:
        b._fast.bind(*[address(f) for f in entries])
        for name, call in (("sqp_smooth_apply_x", lambda: sqp.smooth_apply_x(x, s, out=x)),
                           ("sqp_rmsnorm", lambda: sqp.rmsnorm(x, gamma, 1e-5, out=x)),
                           ("sqp_w4a16_gemm", lambda: sqp.w4a16_gemm(x, p, sc, z, 128)),
                           ("sqp_w4a16_gemm_silu_mul", lambda: sqp.w4a16_gemm_silu_mul(x, p, sc, z, 128)),
                           ("sqp_w4a16_gemm_static", lambda: sqp.w4a16_gemm_static(x, p, sc, z, 128))):
            calls.clear()
            with pytest.raises(b.SqpError, match=name + r" failed: HIP launch error \(-5\)"):
                call()
            assert len(calls) == 1, name
        torch.cuda.synchronize()
        assert torch.equal(x, before)
    finally:
        b._fast.bind(*[address(f) for f in real])
        sqp.set_workspace(0)


def test_native_marshalling_declines_without_aborting(sqp):
    """Tensor methods that throw (a nested tensor has no size in its ragged dimension) end in
    the general path's exception, never in an abort."""
    ragged = torch.nested.nested_tensor([torch.zeros(512), torch.zeros(256)], dtype=torch.float16, device="cuda")
    x = torch.zeros((2, 512), dtype=torch.float16, device="cuda")
    p = torch.zeros((64, 272), dtype=torch.int32, device="cuda")
    sc = torch.zeros((4, 272), dtype=torch.float16, device="cuda")
    z = torch.zeros((4, 272), dtype=torch.uint8, device="cuda")
    for fn in (sqp.w4a16_gemm, sqp.w4a16_gemm_static, sqp.w4a16_gemm_silu_mul):
        fn(x, p, sc, z, 128)
        with pytest.raises(RuntimeError):
            fn(ragged, p, sc, z, 128)
    with pytest.raises(RuntimeError):
        sqp.rmsnorm(ragged, sc[0, :], 1e-5)
    with pytest.raises(RuntimeError):
        sqp.smooth_apply_x(ragged, torch.ones(512, device="cuda"))
    torch.cuda.synchronize()
