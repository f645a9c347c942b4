// Argument marshalling of the serving calls (GEMM, RMSNorm, activation smoothing) and of the calls that
// prepare a weight for torch tensors, in C++: a decode launch takes 5 to 15 us on the GPU, the same checks and
// the ctypes conversion in Python 11 us per GEMM call; the calls on a 1024 x 1024 weight take 9 to 14 us of
// host time in Python and 4 to 7 here.  Holds no arithmetic and no state but the addresses of the
// library's entry points, which the Python binding hands over (so that it always calls the library
// that the binding loaded).
//
// Every function returns the output tensor, or None for anything but the plain case (wrong type,
// device, layout or shape, tensor subclasses, a workspace that has to grow): nothing has been enqueued
// then, and the binding takes its general path, which reports the error.  Once the library has been
// called its code is the result: an error comes back as an integer, never as None, because the call
// may have been enqueued all the same (the status also carries errors of earlier work) and must not run
// twice.  Tensor methods may throw (nested tensors have no size in every dimension), so all of
// them are called inside a try block.  The library's
// calls run without the GIL, as under ctypes: a launch may have to wait for room in the queue.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ops/empty.h>
#include <ATen/ops/empty_cuda_dispatch.h>
#include <ATen/record_function.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>

namespace {

typedef int (*GemmFn)(int, int, int, int, const void *, const uint32_t *, const void *, const uint8_t *, void *, void *);
typedef size_t (*WorkspaceFn)(int, int, int, int);
typedef int (*ScratchGemmFn)(int, int, int, int, int, const void *, const uint32_t *, const void *, const uint8_t *, void *, void *, size_t, void *);
typedef int (*RmsnormFn)(int, int, const void *, const void *, float, void *, void *);
typedef int (*ApplyFn)(int, int, const void *, const float *, void *, void *);

typedef int (*ScalesFn)(int, int, int, float, const void *, const void *, float *, void *);
typedef int (*PackFn)(int, int, int, const void *, uint32_t *, void *, uint8_t *, void *);
typedef int (*UnpackFn)(int, int, int, const uint32_t *, const void *, const uint8_t *, void *, void *);
typedef int (*TransposeFn)(int, int, const void *, void *, void *);
typedef int (*InterleaveFn)(int, int, const void *, const void *, void *, void *);

GemmFn g_gemm[3];  // plain, fused activation, static scratch
WorkspaceFn g_workspace_bytes, g_scratch_bytes;
ScratchGemmFn g_gemm_scratch;
RmsnormFn g_rmsnorm;
ApplyFn g_apply[3];  // x / s and s * w per row of w, w / s per column
ScalesFn g_scales;
PackFn g_pack;
UnpackFn g_unpack;
TransposeFn g_transpose;
InterleaveFn g_interleave;

// The tensor behind an argument if it is a dense GPU tensor of this type on device `dev`, else null.  A
// subclass other than torch.nn.Parameter has semantics of its own (__torch_function__, the type of
// what torch.empty_like makes of it), with or without a dispatch key that tells.
const at::Tensor *plain(PyObject *o, at::ScalarType type, long dev)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || t.key_set().has(c10::DispatchKey::Python) || t.layout() != at::kStrided || !t.is_cuda()) return nullptr;
    if (t.scalar_type() != type || t.get_device() != dev || !t.is_contiguous()) return nullptr;
    return &t;
}

// A new tensor on the device of `like`.  Without dispatch modes, transforms, inference or grad modes that change the
// thread's dispatch keys the dispatcher ends at the GPU's own `empty`: that is called straight away then
// (0.7 us of a call of 4 to 5 instead of 0.8), unless a profiler or another observer records the operators.
at::Tensor fresh(at::IntArrayRef size, at::ScalarType type, const at::Tensor &like)
{
    const c10::impl::LocalDispatchKeySet tls = c10::impl::tls_local_dispatch_key_set();
    if (tls.included_ == c10::default_included_set && tls.excluded_ == c10::default_excluded_set && !at::hasCallbacks())
        return at::cuda::empty(size, type, at::kStrided, like.device(), false, c10::nullopt);
    return at::empty(size, like.options().dtype(type));
}

// `out` as given, or a new tensor like `like` with rows x cols elements (a given one is only taken
// if it has exactly that many).
bool output(PyObject *out, const at::Tensor &like, long rows, long cols, long dev, at::Tensor &y, at::ScalarType type = at::kHalf)
{
    if (out == Py_None) {
        y = fresh({rows, cols}, type, like);
        return true;
    }
    const at::Tensor *t = plain(out, type, dev);
    if (!t || t->numel() != rows * cols) return false;
    y = *t;
    return true;
}

PyObject *result(int rc, PyObject *out, const at::Tensor &y)
{
    if (rc != 0) return PyLong_FromLong(rc);
    if (out == Py_None) return THPVariable_Wrap(y);
    Py_INCREF(out);
    return out;
}

bool fits(long v) { return v > 0 && v <= INT_MAX; }

// gemm(which, x, packed, scales, zeros, group, out, device, stream, workspace bytes held)
PyObject *gemm(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 10) Py_RETURN_NONE;
    const long which = PyLong_AsLong(a[0]), group = PyLong_AsLong(a[5]), dev = PyLong_AsLong(a[7]);
    void *stream = PyLong_AsVoidPtr(a[8]);
    const size_t held = PyLong_AsSize_t(a[9]);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    if (which < 0 || which > 2 || !g_gemm[which]) Py_RETURN_NONE;
    try {
        const at::Tensor *x = plain(a[1], at::kHalf, dev), *packed = plain(a[2], at::kInt, dev);
        const at::Tensor *scales = plain(a[3], at::kHalf, dev), *zeros = plain(a[4], at::kByte, dev);
        if (!x || !packed || !scales || !zeros || x->dim() != 2 || packed->dim() != 2) Py_RETURN_NONE;
        const long M = x->size(0), K = x->size(1), N = packed->size(1);
        if (!fits(M) || !fits(K) || !fits(N) || !fits(group) || packed->size(0) * 8 != K) Py_RETURN_NONE;
        if (which != 2 && g_workspace_bytes((int)M, (int)N, (int)K, (int)group) > held) Py_RETURN_NONE;
        // scratch of this call alone: freed to the allocator's pool of this stream when the call returns, so
        // whatever takes it next is ordered behind the kernels (with `out` the general path looks
        // whether the caller may not allocate)
        const size_t own = which == 2 ? 0 : g_scratch_bytes((int)M, (int)N, (int)K, (int)group);
        if (own > 0 && a[6] != Py_None) Py_RETURN_NONE;
        at::Tensor y, scratch;
        if (!output(a[6], *x, M, which == 1 ? N / 2 : N, dev, y)) Py_RETURN_NONE;
        const void *xp = x->data_ptr(), *pp = packed->data_ptr(), *sp = scales->data_ptr(), *zp = zeros->data_ptr();
        void *yp = y.data_ptr();
        if (own > 0) scratch = fresh({(long)own}, at::kByte, *x);
        void *op = own > 0 ? scratch.data_ptr() : nullptr;
        int rc;
        Py_BEGIN_ALLOW_THREADS
        if (own > 0)
            rc = g_gemm_scratch((int)M, (int)N, (int)K, (int)group, which, xp, (const uint32_t *)pp, sp, (const uint8_t *)zp, yp, op, own, stream);
        else
            rc = g_gemm[which]((int)M, (int)N, (int)K, (int)group, xp, (const uint32_t *)pp, sp, (const uint8_t *)zp, yp, stream);
        Py_END_ALLOW_THREADS
        return result(rc, a[6], y);
    } catch (...) {  // e.g. out of memory: the general path raises it as Python does
        Py_RETURN_NONE;
    }
}

// rmsnorm(x, gamma, eps, out, device, stream)
PyObject *rmsnorm(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 6) Py_RETURN_NONE;
    const double eps = PyFloat_AsDouble(a[2]);
    const long dev = PyLong_AsLong(a[4]);
    void *stream = PyLong_AsVoidPtr(a[5]);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    try {
        const at::Tensor *x = plain(a[0], at::kHalf, dev), *gamma = plain(a[1], at::kHalf, dev);
        if (!x || !gamma || x->dim() != 2 || !fits(x->size(0)) || !fits(x->size(1))) Py_RETURN_NONE;
        const long M = x->size(0), H = x->size(1);
        at::Tensor y;
        if (!output(a[3], *x, M, H, dev, y)) Py_RETURN_NONE;
        const void *xp = x->data_ptr(), *gp = gamma->data_ptr();
        void *yp = y.data_ptr();
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = g_rmsnorm((int)M, (int)H, xp, gp, (float)eps, yp, stream);
        Py_END_ALLOW_THREADS
        return result(rc, a[3], y);
    } catch (...) {
        Py_RETURN_NONE;
    }
}

// The last two arguments of the calls below; false: not whole numbers.
bool place(PyObject *const *a, Py_ssize_t n, long &dev, void *&stream)
{
    dev = PyLong_AsLong(a[n - 2]);
    stream = PyLong_AsVoidPtr(a[n - 1]);
    if (!PyErr_Occurred()) return true;
    PyErr_Clear();
    return false;
}

// apply(which, x, s, out, device, stream): x / s (0), s * x (1: per row), x / s (2: per column)
PyObject *apply(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    long dev;
    void *stream;
    if (n != 6 || !place(a, n, dev, stream)) Py_RETURN_NONE;
    const long which = PyLong_AsLong(a[0]);
    if (which < 0 || which > 2 || !g_apply[which]) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    try {
        const at::Tensor *x = plain(a[1], at::kHalf, dev), *s = plain(a[2], at::kFloat, dev);
        if (!x || !s || x->dim() != 2 || !fits(x->size(0)) || !fits(x->size(1))) Py_RETURN_NONE;
        const long rows = x->size(0), cols = x->size(1);
        at::Tensor y;
        if (!output(a[3], *x, rows, cols, dev, y)) Py_RETURN_NONE;
        const void *xp = x->data_ptr(), *sp = s->data_ptr();
        void *yp = y.data_ptr();
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = g_apply[which]((int)rows, (int)cols, xp, (const float *)sp, yp, stream);
        Py_END_ALLOW_THREADS
        return result(rc, a[3], y);
    } catch (...) {
        Py_RETURN_NONE;
    }
}

// smooth_scales(x_cal, w, alpha, out, device, stream)
PyObject *smooth_scales(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    long dev;
    void *stream;
    if (n != 6 || !g_scales || !place(a, n, dev, stream)) Py_RETURN_NONE;
    const double alpha = PyFloat_AsDouble(a[2]);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    try {
        const at::Tensor *x = plain(a[0], at::kHalf, dev), *w = plain(a[1], at::kHalf, dev);
        if (!x || !w || x->dim() != 2 || w->dim() != 2 || x->size(1) != w->size(0)) Py_RETURN_NONE;
        const long T = x->size(0), K = x->size(1), N = w->size(1);
        if (!fits(T) || !fits(K) || !fits(N)) Py_RETURN_NONE;
        at::Tensor s;
        if (a[3] == Py_None) s = fresh({K}, at::kFloat, *w);
        else if (!output(a[3], *w, K, 1, dev, s, at::kFloat)) Py_RETURN_NONE;
        const void *xp = x->data_ptr(), *wp = w->data_ptr();
        void *sp = s.data_ptr();
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = g_scales((int)T, (int)K, (int)N, (float)alpha, xp, wp, (float *)sp, stream);
        Py_END_ALLOW_THREADS
        return result(rc, a[3], s);
    } catch (...) {
        Py_RETURN_NONE;
    }
}

// quantize_pack(w, group, device, stream): new (packed, scales, zeros)
PyObject *quantize_pack(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    long dev;
    void *stream;
    if (n != 4 || !g_pack || !place(a, n, dev, stream)) Py_RETURN_NONE;
    const long group = PyLong_AsLong(a[1]);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    try {
        const at::Tensor *w = plain(a[0], at::kHalf, dev);
        if (!w || w->dim() != 2 || !fits(group)) Py_RETURN_NONE;
        const long K = w->size(0), N = w->size(1);
        if (!fits(K) || !fits(N) || K % group || K % 8) Py_RETURN_NONE;
        const at::Tensor packed = fresh({K / 8, N}, at::kInt, *w), scales = fresh({K / group, N}, at::kHalf, *w),
                         zeros = fresh({K / group, N}, at::kByte, *w);
        const void *wp = w->data_ptr();
        void *pp = packed.data_ptr(), *sp = scales.data_ptr(), *zp = zeros.data_ptr();
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = g_pack((int)N, (int)K, (int)group, wp, (uint32_t *)pp, sp, (uint8_t *)zp, stream);
        Py_END_ALLOW_THREADS
        if (rc != 0) return PyLong_FromLong(rc);
        return Py_BuildValue("(NNN)", THPVariable_Wrap(packed), THPVariable_Wrap(scales), THPVariable_Wrap(zeros));
    } catch (...) {
        Py_RETURN_NONE;
    }
}

// dequantize(packed, scales, zeros, group, out, device, stream)
PyObject *dequantize(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    long dev;
    void *stream;
    if (n != 7 || !g_unpack || !place(a, n, dev, stream)) Py_RETURN_NONE;
    const long group = PyLong_AsLong(a[3]);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    try {
        const at::Tensor *packed = plain(a[0], at::kInt, dev), *scales = plain(a[1], at::kHalf, dev), *zeros = plain(a[2], at::kByte, dev);
        if (!packed || !scales || !zeros || packed->dim() != 2 || !fits(group)) Py_RETURN_NONE;
        const long K = packed->size(0) * 8, N = packed->size(1);
        if (!fits(K) || !fits(N)) Py_RETURN_NONE;
        at::Tensor y;
        if (!output(a[4], *scales, K, N, dev, y)) Py_RETURN_NONE;
        const void *pp = packed->data_ptr(), *sp = scales->data_ptr(), *zp = zeros->data_ptr();
        void *yp = y.data_ptr();
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = g_unpack((int)N, (int)K, (int)group, (const uint32_t *)pp, sp, (const uint8_t *)zp, yp, stream);
        Py_END_ALLOW_THREADS
        return result(rc, a[4], y);
    } catch (...) {
        Py_RETURN_NONE;
    }
}

// transpose_nk(w_nk, out, device, stream)
PyObject *transpose_nk(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    long dev;
    void *stream;
    if (n != 4 || !g_transpose || !place(a, n, dev, stream)) Py_RETURN_NONE;
    try {
        const at::Tensor *w = plain(a[0], at::kHalf, dev);
        if (!w || w->dim() != 2 || !fits(w->size(0)) || !fits(w->size(1))) Py_RETURN_NONE;
        const long N = w->size(0), K = w->size(1);
        at::Tensor y;
        if (!output(a[1], *w, K, N, dev, y)) Py_RETURN_NONE;
        const void *wp = w->data_ptr();
        void *yp = y.data_ptr();
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = g_transpose((int)N, (int)K, wp, yp, stream);
        Py_END_ALLOW_THREADS
        return result(rc, a[1], y);
    } catch (...) {
        Py_RETURN_NONE;
    }
}

// interleave_gate_up(w_gate, w_up, out, device, stream): two tensors of one shape
PyObject *interleave_gate_up(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    long dev;
    void *stream;
    if (n != 5 || !g_interleave || !place(a, n, dev, stream)) Py_RETURN_NONE;
    try {
        const at::Tensor *gate = plain(a[0], at::kHalf, dev), *up = plain(a[1], at::kHalf, dev);
        if (!gate || !up || gate->dim() != 2 || !up->sizes().equals(gate->sizes())) Py_RETURN_NONE;
        const long K = gate->size(0), I = gate->size(1);
        if (!fits(K) || !fits(2 * I)) Py_RETURN_NONE;
        at::Tensor y;
        if (!output(a[2], *gate, K, 2 * I, dev, y)) Py_RETURN_NONE;
        const void *gp = gate->data_ptr(), *upp = up->data_ptr();
        void *yp = y.data_ptr();
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = g_interleave((int)K, (int)I, gp, upp, yp, stream);
        Py_END_ALLOW_THREADS
        return result(rc, a[2], y);
    } catch (...) {
        Py_RETURN_NONE;
    }
}

// bind(addresses of sqp_w4a16_gemm, _silu_mul, _static, _workspace_bytes, sqp_rmsnorm, sqp_smooth_apply_x,
//      sqp_w4a16_gemm_scratch, _scratch_bytes)
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    void *p[8];
    if (n != 8) {
        PyErr_SetString(PyExc_TypeError, "bind takes eight addresses");
        return nullptr;
    }
    for (int i = 0; i < 8; i++) p[i] = PyLong_AsVoidPtr(a[i]);
    if (PyErr_Occurred()) return nullptr;
    for (int i = 0; i < 3; i++) g_gemm[i] = (GemmFn)p[i];
    g_workspace_bytes = (WorkspaceFn)p[3];
    g_rmsnorm = (RmsnormFn)p[4];
    g_apply[0] = (ApplyFn)p[5];
    g_gemm_scratch = (ScratchGemmFn)p[6];
    g_scratch_bytes = (WorkspaceFn)p[7];
    Py_RETURN_NONE;
}

// bind_preparation(addresses of sqp_smooth_apply_w, sqp_scale_columns, sqp_smooth_scales, sqp_quantize_pack, sqp_dequantize,
//      sqp_transpose_nk, sqp_interleave_gate_up)
PyObject *bind_preparation(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    void *p[7];
    if (n != 7) {
        PyErr_SetString(PyExc_TypeError, "bind_preparation takes seven addresses");
        return nullptr;
    }
    for (int i = 0; i < 7; i++) p[i] = PyLong_AsVoidPtr(a[i]);
    if (PyErr_Occurred()) return nullptr;
    g_apply[1] = (ApplyFn)p[0];
    g_apply[2] = (ApplyFn)p[1];
    g_scales = (ScalesFn)p[2];
    g_pack = (PackFn)p[3];
    g_unpack = (UnpackFn)p[4];
    g_transpose = (TransposeFn)p[5];
    g_interleave = (InterleaveFn)p[6];
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, nullptr},
    {"gemm", (PyCFunction)(void (*)(void))gemm, METH_FASTCALL, nullptr},
    {"rmsnorm", (PyCFunction)(void (*)(void))rmsnorm, METH_FASTCALL, nullptr},
    {"bind_preparation", (PyCFunction)(void (*)(void))bind_preparation, METH_FASTCALL, nullptr},
    {"apply", (PyCFunction)(void (*)(void))apply, METH_FASTCALL, nullptr},
    {"smooth_scales", (PyCFunction)(void (*)(void))smooth_scales, METH_FASTCALL, nullptr},
    {"quantize_pack", (PyCFunction)(void (*)(void))quantize_pack, METH_FASTCALL, nullptr},
    {"dequantize", (PyCFunction)(void (*)(void))dequantize, METH_FASTCALL, nullptr},
    {"transpose_nk", (PyCFunction)(void (*)(void))transpose_nk, METH_FASTCALL, nullptr},
    {"interleave_gate_up", (PyCFunction)(void (*)(void))interleave_gate_up, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_sqp_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject *PyInit__sqp_torch() { return PyModule_Create(&module); }
