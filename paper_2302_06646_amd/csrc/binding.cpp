// The usual call of the Python binding, marshalled natively.  A function here looks its tensors over as the binding does
// (contiguous device tensors of the right type and shape), takes torch's current stream and calls the C ABI with the GIL
// released; it returns the library's status, or None for anything it does not know (another argument type, a tensor that is a
// wrapper of some transform, a mismatch), which the binding then looks at in Python and refuses or serves as before.
// Bound by nothing but its own length: a training step of three calls spent 32 us on the host in Python and ctypes, two
// thirds of them in attribute look-ups and conversions, and small layers ran at that speed.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>
#include <new>

#include "../../include/longconv.h"

namespace {

struct Api {
    decltype(&longconv_kspec_compute) kspec_compute;
    decltype(&longconv_fwd) fwd;
    decltype(&longconv_bwd) bwd;
    decltype(&longconv_fwd_gated) fwd_gated;
    decltype(&longconv_bwd_gated) bwd_gated;
    decltype(&longconv2d_fwd) fwd2d;
    decltype(&longconv2d_bwd) bwd2d;
    decltype(&longconv_kreg_fwd) kreg_fwd;
    decltype(&longconv_kreg_bwd) kreg_bwd;
    decltype(&longconv_lbfly_spectrum) lbfly_spectrum;
    decltype(&longconv_lbfly_spectrum_bwd) lbfly_spectrum_bwd;
    decltype(&longconv_lbfly_fwd) lbfly_fwd;
    decltype(&longconv_lbfly_bwd) lbfly_bwd;
} g_api = {};

// a plain device tensor: torch.Tensor or Parameter, strided, its own storage, no functional transform around it
const at::Tensor* plain(PyObject* o)
{
    if (!THPVariable_CheckTypeExact(Py_TYPE(o))) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != c10::kStrided || !t.has_storage()) return nullptr;
    const c10::DispatchKeySet usual = c10::autograd_dispatch_keyset_with_ADInplaceOrView | c10::autocast_dispatch_keyset;
    if ((t.key_set() - usual) != c10::DispatchKeySet(c10::DispatchKey::CUDA)) return nullptr;
    return &t;
}

// Arguments of one call: `ok` stays true while everything is what the binding's checks let pass.
struct Args {
    PyObject* const* a;
    bool ok = true;
    const at::Tensor* first(int i, int dims)       // the tensor that names the shape
    {
        const at::Tensor* t = plain(a[i]);
        if (!t || t->dim() != dims) { ok = false; return nullptr; }
        return t;
    }
    void* ptr(int i, c10::ScalarType dt, c10::IntArrayRef shape, bool may_be_none = true)
    {
        if (!ok) return nullptr;
        if (may_be_none && a[i] == Py_None) return nullptr;
        const at::Tensor* t = plain(a[i]);
        if (!t || t->scalar_type() != dt || t->sizes() != shape || !t->is_contiguous()) { ok = false; return nullptr; }
        return t->data_ptr();
    }
    // workspace or stored spectrum: any device tensor, taken by its address (and its number of elements)
    void* raw(int i, size_t* n = nullptr, bool may_be_none = true)
    {
        if (n) *n = 0;
        if (!ok) return nullptr;
        if (may_be_none && a[i] == Py_None) return nullptr;
        const at::Tensor* t = plain(a[i]);
        if (!t) { ok = false; return nullptr; }
        if (n) *n = (size_t)t->numel();
        return t->data_ptr();
    }
    long number(int i)
    {
        if (!ok) return 0;
        const long v = PyLong_CheckExact(a[i]) ? PyLong_AsLong(a[i]) : -1;
        if (v < 0 || v > 0x7fffffffL) { PyErr_Clear(); ok = false; }
        return v;
    }
    double real(int i)
    {
        if (!ok) return 0;
        if (!PyFloat_CheckExact(a[i])) { ok = false; return 0; }
        return PyFloat_AS_DOUBLE(a[i]);
    }
    void* stream(int i)
    {
        if (!ok) return nullptr;
        if (a[i] == Py_None) return c10::hip::getCurrentHIPStream().stream();
        PyObject* v = PyObject_GetAttrString(a[i], "cuda_stream");
        void* p = nullptr;
        if (v && PyLong_CheckExact(v)) p = PyLong_AsVoidPtr(v);
        else ok = false;
        Py_XDECREF(v);
        if (PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        return p;
    }
};

int io_code(c10::ScalarType dt)
{
    return dt == at::kFloat ? LONGCONV_F32 : dt == at::kHalf ? LONGCONV_F16 : dt == at::kBFloat16 ? LONGCONV_BF16 : -1;
}

struct WithoutGil {
    PyThreadState* state = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(state); }
};

// `body` fills the call in and returns its status through `call`; nothing that Python could see happens before `ok` is known.
// What is thrown before the library is entered leaves the call to Python; what the library throws is a Python error, since work
// may have been launched.
template <class F>
PyObject* guarded(PyObject* const* a, Py_ssize_t n, Py_ssize_t want, bool bound, F&& body)
{
    if (n != want || !bound) Py_RETURN_NONE;
    bool entered = false;
    try {
        Args A{a};
        int status = 0;
        const auto call = [&](auto&& f) {
            if (!A.ok) return;
            entered = true;
            const WithoutGil scope;
            status = f();
        };
        body(A, call);
        if (A.ok) return PyLong_FromLong(status);
    } catch (const std::bad_alloc&) {
        if (entered) return PyErr_NoMemory();
    } catch (const std::exception& e) {
        if (entered) return PyErr_Format(PyExc_RuntimeError, "longconv: %s", e.what());
    } catch (...) {
        if (entered) return PyErr_Format(PyExc_RuntimeError, "longconv: unknown C++ exception");
    }
    PyErr_Clear();
    Py_RETURN_NONE;
}

const c10::ScalarType F = at::kFloat;

PyObject* kspec_compute(PyObject*, PyObject* const* a, Py_ssize_t n)     // k, D, kspec, io, workspace, stream
{
    return guarded(a, n, 6, g_api.kspec_compute, [&](Args& A, auto& call) {
        const at::Tensor* t = A.first(0, 2);
        if (!t) return;
        const int64_t H = t->size(0), N = t->size(1);
        size_t wb;
        const auto k = (const float*)A.ptr(0, F, {H, N}), D = (const float*)A.ptr(1, F, {H});
        void *ks = A.raw(2), *ws = A.raw(4, &wb), *st = A.stream(5);
        const int io = (int)A.number(3);
        call([&] { return g_api.kspec_compute(k, D, ks, H, N, io, ws, wb, st); });
    });
}

// shape and I/O type of the rows in argument i
struct Rows {
    int64_t B = 0, H = 0, N = 0, M = 0;
    c10::ScalarType dt = at::kFloat;
    int io = -1;
    Rows(Args& A, int i, int dims)
    {
        const at::Tensor* t = A.first(i, dims);
        if (!t) return;
        dt = t->scalar_type();
        io = io_code(dt);
        if (io < 0) { A.ok = false; return; }
        B = t->size(0);
        H = t->size(1);
        N = t->size(2);
        M = dims == 4 ? t->size(3) : 0;
    }
};

PyObject* fwd(PyObject*, PyObject* const* a, Py_ssize_t n)               // u, k, D, y, workspace, kspec, stream
{
    return guarded(a, n, 7, g_api.fwd, [&](Args& A, auto& call) {
        const Rows r(A, 0, 3);
        size_t wb;
        const void* u = A.ptr(0, r.dt, {r.B, r.H, r.N});
        const auto k = (const float*)A.ptr(1, F, {r.H, r.N}), D = (const float*)A.ptr(2, F, {r.H});
        void *y = A.ptr(3, r.dt, {r.B, r.H, r.N}), *ws = A.raw(4, &wb, false), *ks = A.raw(5), *st = A.stream(6);
        call([&] { return g_api.fwd(u, k, D, ks, y, r.B, r.H, r.N, r.io, ws, wb, st); });
    });
}

PyObject* bwd(PyObject*, PyObject* const* a, Py_ssize_t n)               // dy, u, k, D, du, dk, dD, workspace, kspec, stream
{
    return guarded(a, n, 10, g_api.bwd, [&](Args& A, auto& call) {
        const Rows r(A, 0, 3);
        size_t wb;
        const void *dy = A.ptr(0, r.dt, {r.B, r.H, r.N}), *u = A.ptr(1, r.dt, {r.B, r.H, r.N});
        const auto k = (const float*)A.ptr(2, F, {r.H, r.N}), D = (const float*)A.ptr(3, F, {r.H});
        void* du = A.ptr(4, r.dt, {r.B, r.H, r.N});
        const auto dk = (float*)A.ptr(5, F, {r.H, r.N}), dD = (float*)A.ptr(6, F, {r.H});
        void *ws = A.raw(7, &wb, false), *ks = A.raw(8), *st = A.stream(9);
        call([&] { return g_api.bwd(dy, u, k, D, ks, du, dk, dD, r.B, r.H, r.N, r.io, ws, wb, st); });
    });
}

PyObject* fwd_gated(PyObject*, PyObject* const* a, Py_ssize_t n)         // u, k, D, g, y, workspace, kspec, stream
{
    return guarded(a, n, 8, g_api.fwd_gated, [&](Args& A, auto& call) {
        const Rows r(A, 0, 3);
        size_t wb;
        const void *u = A.ptr(0, r.dt, {r.B, r.H, r.N}), *g = A.ptr(3, r.dt, {r.B, r.H, r.N});
        const auto k = (const float*)A.ptr(1, F, {r.H, r.N}), D = (const float*)A.ptr(2, F, {r.H});
        void *y = A.ptr(4, r.dt, {r.B, r.H, r.N}), *ws = A.raw(5, &wb, false), *ks = A.raw(6), *st = A.stream(7);
        call([&] { return g_api.fwd_gated(u, k, D, ks, g, y, r.B, r.H, r.N, r.io, ws, wb, st); });
    });
}

PyObject* bwd_gated(PyObject*, PyObject* const* a, Py_ssize_t n)   // dy, g, u, k, D, du, dk, dD, dg, workspace, kspec, stream
{
    return guarded(a, n, 12, g_api.bwd_gated, [&](Args& A, auto& call) {
        const Rows r(A, 0, 3);
        size_t wb;
        const void *dy = A.ptr(0, r.dt, {r.B, r.H, r.N}), *g = A.ptr(1, r.dt, {r.B, r.H, r.N});
        const void* u = A.ptr(2, r.dt, {r.B, r.H, r.N});
        const auto k = (const float*)A.ptr(3, F, {r.H, r.N}), D = (const float*)A.ptr(4, F, {r.H});
        void *du = A.ptr(5, r.dt, {r.B, r.H, r.N}), *dg = A.ptr(8, r.dt, {r.B, r.H, r.N});
        const auto dk = (float*)A.ptr(6, F, {r.H, r.N}), dD = (float*)A.ptr(7, F, {r.H});
        void *ws = A.raw(9, &wb, false), *ks = A.raw(10), *st = A.stream(11);
        call([&] { return g_api.bwd_gated(dy, g, u, k, D, ks, du, dk, dD, dg, r.B, r.H, r.N, r.io, ws, wb, st); });
    });
}

PyObject* fwd2d(PyObject*, PyObject* const* a, Py_ssize_t n)             // u, k, D, y, workspace, stream
{
    return guarded(a, n, 6, g_api.fwd2d, [&](Args& A, auto& call) {
        const Rows r(A, 0, 4);
        size_t wb;
        const void* u = A.ptr(0, r.dt, {r.B, r.H, r.N, r.M});
        const auto k = (const float*)A.ptr(1, F, {r.H, r.N, r.M}), D = (const float*)A.ptr(2, F, {r.H});
        void *y = A.ptr(3, r.dt, {r.B, r.H, r.N, r.M}), *ws = A.raw(4, &wb, false), *st = A.stream(5);
        call([&] { return g_api.fwd2d(u, k, D, y, r.B, r.H, r.N, r.M, r.io, ws, wb, st); });
    });
}

PyObject* bwd2d(PyObject*, PyObject* const* a, Py_ssize_t n)             // dy, u, k, D, du, dk, dD, workspace, stream
{
    return guarded(a, n, 9, g_api.bwd2d, [&](Args& A, auto& call) {
        const Rows r(A, 0, 4);
        size_t wb;
        const void *dy = A.ptr(0, r.dt, {r.B, r.H, r.N, r.M}), *u = A.ptr(1, r.dt, {r.B, r.H, r.N, r.M});
        const auto k = (const float*)A.ptr(2, F, {r.H, r.N, r.M}), D = (const float*)A.ptr(3, F, {r.H});
        void* du = A.ptr(4, r.dt, {r.B, r.H, r.N, r.M});
        const auto dk = (float*)A.ptr(5, F, {r.H, r.N, r.M}), dD = (float*)A.ptr(6, F, {r.H});
        void *ws = A.raw(7, &wb, false), *st = A.stream(8);
        call([&] { return g_api.bwd2d(dy, u, k, D, du, dk, dD, r.B, r.H, r.N, r.M, r.io, ws, wb, st); });
    });
}

PyObject* kreg_fwd(PyObject*, PyObject* const* a, Py_ssize_t n)          // k, drop_mask, kbar, p, lam, stream
{
    return guarded(a, n, 6, g_api.kreg_fwd, [&](Args& A, auto& call) {
        const at::Tensor* t = A.first(0, 2);
        if (!t) return;
        const int64_t H = t->size(0), N = t->size(1);
        const auto k = (const float*)A.ptr(0, F, {H, N}), m = (const float*)A.ptr(1, F, {H, N});
        const auto kbar = (float*)A.ptr(2, F, {H, N});
        const int p = (int)A.number(3);
        const float lam = (float)A.real(4);
        void* st = A.stream(5);
        call([&] { return g_api.kreg_fwd(k, m, kbar, H, N, p, lam, st); });
    });
}

PyObject* kreg_bwd(PyObject*, PyObject* const* a, Py_ssize_t n)          // k, drop_mask, dkbar, dk, p, lam, stream
{
    return guarded(a, n, 7, g_api.kreg_bwd, [&](Args& A, auto& call) {
        const at::Tensor* t = A.first(0, 2);
        if (!t) return;
        const int64_t H = t->size(0), N = t->size(1);
        const auto k = (const float*)A.ptr(0, F, {H, N}), m = (const float*)A.ptr(1, F, {H, N});
        const auto dkbar = (const float*)A.ptr(2, F, {H, N});
        const auto dk = (float*)A.ptr(3, F, {H, N});
        const int p = (int)A.number(4);
        const float lam = (float)A.real(5);
        void* st = A.stream(6);
        call([&] { return g_api.kreg_bwd(k, m, dkbar, dk, H, N, p, lam, st); });
    });
}

PyObject* lbfly_spectrum(PyObject*, PyObject* const* a, Py_ssize_t n)    // k, D, shat, stream
{
    return guarded(a, n, 4, g_api.lbfly_spectrum, [&](Args& A, auto& call) {
        const at::Tensor* t = A.first(0, 2);
        if (!t) return;
        const int64_t H = t->size(0), N = t->size(1);
        const auto k = (const float*)A.ptr(0, F, {H, N}), D = (const float*)A.ptr(1, F, {H});
        const auto s = (float*)A.ptr(2, F, {H, 2 * N, 2});
        void* st = A.stream(3);
        call([&] { return g_api.lbfly_spectrum(k, D, s, H, N, st); });
    });
}

PyObject* lbfly_spectrum_bwd(PyObject*, PyObject* const* a, Py_ssize_t n)     // dshat, dk, dD, stream
{
    return guarded(a, n, 4, g_api.lbfly_spectrum_bwd, [&](Args& A, auto& call) {
        const at::Tensor* t = A.first(0, 3);
        if (!t) return;
        const int64_t H = t->size(0), L = t->size(1), N = L / 2;
        const auto s = (const float*)A.ptr(0, F, {H, L, 2});
        const auto dk = (float*)A.ptr(1, F, {H, N}), dD = (float*)A.ptr(2, F, {H});
        void* st = A.stream(3);
        call([&] { return g_api.lbfly_spectrum_bwd(s, dk, dD, H, N, st); });
    });
}

PyObject* lbfly_fwd(PyObject*, PyObject* const* a, Py_ssize_t n)         // u, shat, Af, Ai, y, stream
{
    return guarded(a, n, 6, g_api.lbfly_fwd, [&](Args& A, auto& call) {
        const Rows r(A, 0, 3);
        const void* u = A.ptr(0, r.dt, {r.B, r.H, r.N});
        const auto s = (const float*)A.ptr(1, F, {r.H, 2 * r.N, 2});
        const auto f = (const float*)A.ptr(2, F, {r.H, 3, 16, 16, 2}), i = (const float*)A.ptr(3, F, {r.H, 3, 16, 16, 2});
        void *y = A.ptr(4, r.dt, {r.B, r.H, r.N}), *st = A.stream(5);
        call([&] { return g_api.lbfly_fwd(u, s, f, i, y, r.B, r.H, r.N, r.io, st); });
    });
}

PyObject* lbfly_bwd(PyObject*, PyObject* const* a, Py_ssize_t n)  // dy, u, shat, Af, Ai, du, dshat, dAf, dAi, workspace, stream
{
    return guarded(a, n, 11, g_api.lbfly_bwd, [&](Args& A, auto& call) {
        const Rows r(A, 0, 3);
        size_t wb;
        const void *dy = A.ptr(0, r.dt, {r.B, r.H, r.N}), *u = A.ptr(1, r.dt, {r.B, r.H, r.N});
        const auto s = (const float*)A.ptr(2, F, {r.H, 2 * r.N, 2});
        const auto f = (const float*)A.ptr(3, F, {r.H, 3, 16, 16, 2}), i = (const float*)A.ptr(4, F, {r.H, 3, 16, 16, 2});
        void* du = A.ptr(5, r.dt, {r.B, r.H, r.N});
        const auto ds = (float*)A.ptr(6, F, {r.H, 2 * r.N, 2});
        const auto df = (float*)A.ptr(7, F, {r.H, 3, 16, 16, 2}), di = (float*)A.ptr(8, F, {r.H, 3, 16, 16, 2});
        void *ws = A.raw(9, &wb, false), *st = A.stream(10);
        call([&] { return g_api.lbfly_bwd(dy, u, s, f, i, du, ds, df, di, r.B, r.H, r.N, r.io, ws, wb, st); });
    });
}

// bind({name: address}): the entry points of the library that the binding has loaded
PyObject* bind(PyObject*, PyObject* arg)
{
    if (!PyDict_Check(arg)) {
        PyErr_SetString(PyExc_TypeError, "bind() takes a dict of addresses");
        return nullptr;
    }
    bool ok = true;
    const auto set = [&](auto& slot, const char* name) {
        PyObject* v = PyDict_GetItemString(arg, name);
        void* p = v ? PyLong_AsVoidPtr(v) : nullptr;
        if (!p) ok = false;
        slot = reinterpret_cast<std::remove_reference_t<decltype(slot)>>(p);
    };
    set(g_api.kspec_compute, "longconv_kspec_compute");
    set(g_api.fwd, "longconv_fwd");
    set(g_api.bwd, "longconv_bwd");
    set(g_api.fwd_gated, "longconv_fwd_gated");
    set(g_api.bwd_gated, "longconv_bwd_gated");
    set(g_api.fwd2d, "longconv2d_fwd");
    set(g_api.bwd2d, "longconv2d_bwd");
    set(g_api.kreg_fwd, "longconv_kreg_fwd");
    set(g_api.kreg_bwd, "longconv_kreg_bwd");
    set(g_api.lbfly_spectrum, "longconv_lbfly_spectrum");
    set(g_api.lbfly_spectrum_bwd, "longconv_lbfly_spectrum_bwd");
    set(g_api.lbfly_fwd, "longconv_lbfly_fwd");
    set(g_api.lbfly_bwd, "longconv_lbfly_bwd");
    if (!ok) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_KeyError, "an entry point is missing");
        return nullptr;
    }
    Py_RETURN_NONE;
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"bind", bind, METH_O, nullptr}, FAST(kspec_compute), FAST(fwd), FAST(bwd), FAST(fwd_gated), FAST(bwd_gated), FAST(fwd2d),
    FAST(bwd2d), FAST(kreg_fwd), FAST(kreg_bwd), FAST(lbfly_spectrum), FAST(lbfly_spectrum_bwd), FAST(lbfly_fwd),
    FAST(lbfly_bwd), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
