// Argument marshalling of the linear calls in native code.  A call hands over up to 2 q + 3 tensors;
// looking each of them over from Python costs about 1 us apiece and made the host the slower side of
// every call below some 30 us.
//
// Each function takes the address of the descriptor, or None where the caller was handed anything
// but a TessDesc, and the tensors as the Python caller has them.
// It returns the library's status when everything is plain (torch.Tensor and Parameter objects on the device,
// the descriptor's types and shapes, contiguous rows, lists or tuples of q panels with one leading
// dimension) and -1, with no call made, when anything is not: the Python code of binding.py then
// takes the call and says what is wrong, or serves the rarer forms.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/device_lazy_init.h>

#include "tesseract.h"

namespace {

struct Entry {
    decltype(&tess_linear_fwd) fwd;
    decltype(&tess_linear_bwd_dx) dx;
    decltype(&tess_linear_bwd_dx_act) dx_act;
    decltype(&tess_linear_bwd_dw) dw;
    decltype(&tess_linear_bwd_dw_bias) dw_bias;
} entry;

struct NotPlain {};      // thrown where the Python code has to take the call

void need(bool ok)
{
    if (!ok) throw NotPlain{};
}

struct Dims {
    const tess_desc* d;
    int64_t m, kb, n;
};

Dims dims_of(PyObject* address)
{
    const auto* d = static_cast<const tess_desc*>(PyLong_AsVoidPtr(address));
    if (PyErr_Occurred()) PyErr_Clear();
    need(d && d->q >= 1 && d->q <= TESS_MAX_Q && d->d >= 1 && d->d <= d->q && d->a > 0 && d->b > 0 && d->c > 0);
    need(d->a % ((int64_t)d->q * d->d) == 0 && d->b % d->q == 0 && d->c % d->q == 0);
    need((d->in_dtype == TESS_F32 || d->in_dtype == TESS_BF16) && (d->out_dtype == TESS_F32 || d->out_dtype == TESS_BF16));
    return {d, d->a / ((int64_t)d->q * d->d), d->b / d->q, d->c / d->q};
}

at::ScalarType scalar(int code) { return code == TESS_F32 ? at::kFloat : at::kBFloat16; }

const at::Tensor& tensor(PyObject* o)
{
    need(THPVariable_CheckExact(o));
    const at::Tensor& t = THPVariable_Unpack(o);
    need(t.defined() && t.layout() == at::kStrided && t.is_cuda() && t.has_storage());
    return t;
}

// pointer and leading dimension of a [rows, cols] block
void* block(PyObject* o, int code, int64_t rows, int64_t cols, int64_t& ld)
{
    const at::Tensor& t = tensor(o);
    need(t.scalar_type() == scalar(code) && t.dim() == 2 && t.size(0) == rows && t.size(1) == cols);
    need(t.stride(1) == 1 || cols == 1);
    ld = t.stride(0);
    if (rows == 1 && ld < cols) ld = cols;
    return t.data_ptr();
}

struct Panels {
    const void* p[TESS_MAX_Q];
    int64_t ld;
};

Panels panels(PyObject* seq, int q, int code, int64_t rows, int64_t cols)
{
    need(PyList_CheckExact(seq) || PyTuple_CheckExact(seq));
    need(PySequence_Fast_GET_SIZE(seq) == q);
    PyObject** items = PySequence_Fast_ITEMS(seq);
    Panels out;
    for (int t = 0; t < q; ++t) {
        int64_t ld;
        out.p[t] = block(items[t], code, rows, cols, ld);
        if (t == 0) out.ld = ld;
        need(ld == out.ld);
    }
    return out;
}

// a contiguous vector of n elements, or null for None
void* vec(PyObject* o, at::ScalarType type, int64_t n)
{
    if (o == Py_None) return nullptr;
    const at::Tensor& t = tensor(o);
    need(t.scalar_type() == type && t.dim() == 1 && t.size(0) == n && t.is_contiguous());
    return t.data_ptr();
}

struct Scratch {
    void* p = nullptr;
    size_t bytes = 0;
};

Scratch scratch(PyObject* o)
{
    if (o == Py_None) return {};
    const at::Tensor& t = tensor(o);
    need(t.is_contiguous());
    return {t.data_ptr(), (size_t)t.numel() * t.element_size()};
}

void* current_stream()
{
    need(!torch::utils::is_device_in_bad_fork(at::kCUDA));      // Python refuses: no device call in a forked child
    return c10::hip::getCurrentHIPStream().stream();
}

int integer(PyObject* o)
{
    const long v = PyLong_AsLong(o);
    if (v == -1 && PyErr_Occurred()) { PyErr_Clear(); throw NotPlain{}; }
    need(v >= 0 && v < (1 << 30));
    return (int)v;
}

int truth(PyObject* o)
{
    const int v = PyObject_IsTrue(o);
    if (v < 0) { PyErr_Clear(); throw NotPlain{}; }
    return v;
}

// Runs `body`; no C++ exception leaves it.
template <typename F>
PyObject* guarded(Py_ssize_t got, Py_ssize_t want, F&& body)
{
    if (got != want) {
        PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, got);
        return nullptr;
    }
    int status = -1;
    try {
        status = body();
    } catch (...) {
        status = -1;
    }
    return PyLong_FromLong(status);
}

// The interpreter runs on while the library enqueues its kernels.
template <typename F>
int released(F&& call)
{
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = call();
    Py_END_ALLOW_THREADS
    return status;
}

// (desc, a_panels, b_panels, bias, act, c_out, preact_out, workspace, stream)
PyObject* fwd(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded(n, 9, [&] {
        if (a[8] != Py_None) return -1;      // a stream object: its handle is read in Python
        const Dims s = dims_of(a[0]);
        const Panels x = panels(a[1], s.d->q, s.d->in_dtype, s.m, s.kb), w = panels(a[2], s.d->q, s.d->in_dtype, s.kb, s.n);
        const void* bias = vec(a[3], scalar(s.d->in_dtype), s.n);
        const int act = integer(a[4]);
        int64_t ldc, ldp;
        void* out = block(a[5], s.d->out_dtype, s.m, s.n, ldc);
        void* pre = a[6] == Py_None ? nullptr : block(a[6], s.d->out_dtype, s.m, s.n, ldp);
        need(!pre || ldp == ldc);
        const Scratch ws = scratch(a[7]);
        void* st = current_stream();
        return released([&] { return (int)entry.fwd(s.d, x.p, x.ld, w.p, w.ld, bias, act, out, ldc, pre, ws.p, ws.bytes, st); });
    });
}

// (desc, dy_panels, w_panels, dx_out, workspace, stream)
PyObject* dx(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded(n, 6, [&] {
        if (a[5] != Py_None) return -1;      // a stream object: its handle is read in Python
        const Dims s = dims_of(a[0]);
        const Panels dy = panels(a[1], s.d->q, s.d->in_dtype, s.m, s.n), w = panels(a[2], s.d->q, s.d->in_dtype, s.kb, s.n);
        int64_t ldo;
        void* out = block(a[3], s.d->out_dtype, s.m, s.kb, ldo);
        const Scratch ws = scratch(a[4]);
        void* st = current_stream();
        return released([&] { return (int)entry.dx(s.d, dy.p, dy.ld, w.p, w.ld, out, ldo, ws.p, ws.bytes, st); });
    });
}

// (desc, dy_panels, w_panels, preact, act, dz_out, workspace, stream)
PyObject* dx_act(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded(n, 8, [&] {
        if (a[7] != Py_None) return -1;      // a stream object: its handle is read in Python
        const Dims s = dims_of(a[0]);
        const Panels dy = panels(a[1], s.d->q, s.d->in_dtype, s.m, s.n), w = panels(a[2], s.d->q, s.d->in_dtype, s.kb, s.n);
        int64_t ldz, ldo;
        const void* z = block(a[3], s.d->in_dtype, s.m, s.kb, ldz);
        const int act = integer(a[4]);
        void* out = block(a[5], s.d->out_dtype, s.m, s.kb, ldo);
        const Scratch ws = scratch(a[6]);
        void* st = current_stream();
        return released([&] { return (int)entry.dx_act(s.d, dy.p, dy.ld, w.p, w.ld, z, ldz, act, out, ldo, ws.p, ws.bytes, st); });
    });
}

struct DwArgs {
    Dims s;
    Panels x, dy;
    void* out;
    int64_t ldo;
    int accumulate;
};

// desc, x_panels, dy_panels, dw_out, accumulate
DwArgs dw_args(PyObject* const* a)
{
    DwArgs r;
    r.s = dims_of(a[0]);
    const tess_desc* d = r.s.d;
    r.x = panels(a[1], d->q, d->in_dtype, r.s.m, r.s.kb);
    r.dy = panels(a[2], d->q, d->in_dtype, r.s.m, r.s.n);
    r.accumulate = truth(a[4]);
    r.out = block(a[3], r.accumulate ? TESS_F32 : d->out_dtype, r.s.kb, r.s.n, r.ldo);
    return r;
}

// (desc, x_panels, dy_panels, dw_out, accumulate, workspace, stream)
PyObject* dw(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded(n, 7, [&] {
        if (a[6] != Py_None) return -1;      // a stream object: its handle is read in Python
        const DwArgs r = dw_args(a);
        const Scratch ws = scratch(a[5]);
        void* st = current_stream();
        return released([&] { return (int)entry.dw(r.s.d, r.x.p, r.x.ld, r.dy.p, r.dy.ld, r.out, r.ldo, r.accumulate, ws.p, ws.bytes, st); });
    });
}

// (desc, x_panels, dy_panels, dw_out, accumulate, dbias_out, workspace, stream)
PyObject* dw_bias(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return guarded(n, 8, [&] {
        if (a[7] != Py_None) return -1;      // a stream object: its handle is read in Python
        const DwArgs r = dw_args(a);
        void* db = vec(a[5], at::kFloat, r.s.n);
        const Scratch ws = scratch(a[6]);
        void* st = current_stream();
        return released([&] { return (int)entry.dw_bias(r.s.d, r.x.p, r.x.ld, r.dy.p, r.dy.ld, r.out, r.ldo, db, r.accumulate, ws.p, ws.bytes, st); });
    });
}

// (addresses of the five library functions)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    if (n != 5) {
        PyErr_SetString(PyExc_TypeError, "expected 5 addresses");
        return nullptr;
    }
    void* f[5];
    for (int i = 0; i < 5; ++i) {
        f[i] = PyLong_AsVoidPtr(a[i]);
        if (PyErr_Occurred()) return nullptr;
    }
    entry = {reinterpret_cast<decltype(entry.fwd)>(f[0]), reinterpret_cast<decltype(entry.dx)>(f[1]),
             reinterpret_cast<decltype(entry.dx_act)>(f[2]), reinterpret_cast<decltype(entry.dw)>(f[3]),
             reinterpret_cast<decltype(entry.dw_bias)>(f[4])};
    Py_RETURN_NONE;
}

#define METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(bind), METHOD(fwd), METHOD(dx), METHOD(dx_act), METHOD(dw), METHOD(dw_bias),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tess_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__tess_call(void) { return PyModule_Create(&module); }
