// Argument marshalling of the hot entry points in native code (host only): checks the tensors, fills the shape struct, finds the
// current stream and calls the C ABI.  The ctypes way through Python attributes took 8 us a call, as long as the launches of a
// small decode step; this takes about one.
//
// Every function returns the moc_status of the call, or kNotTaken without having called anything when an argument is not
// exactly what the entry point wants; binding.py then goes its own way, which reports the error.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <dlfcn.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/moc.h"

namespace {

constexpr long kNotTaken = -1000;

decltype(&moc_ffn_fwd) p_fwd;
decltype(&moc_ffn_bwd) p_bwd;
decltype(&moc_ffn_decode) p_decode;
decltype(&moc_ffn_fwd_grouped) p_fwd_grouped;
decltype(&moc_ffn_decode_grouped) p_decode_grouped;
decltype(&moc_ffn_fwd_experts) p_fwd_experts;
decltype(&moc_ffn_bwd_experts) p_bwd_experts;
decltype(&moc_rmsnorm) p_rmsnorm;
decltype(&moc_residual_add) p_residual;

// The arguments of one call: `ok` stays true as long as everything fits.
struct Args {
    PyObject* const* v;
    bool ok = true;
    at::ScalarType dt = at::kFloat;
    moc_shape s{};
    int64_t experts = 0;

    const at::Tensor* tensor(int i) {
        if (!ok || !THPVariable_Check(v[i])) { ok = false; return nullptr; }
        const at::Tensor& t = THPVariable_Unpack(v[i]);
        ok = t.is_cuda() && t.is_contiguous();
        return ok ? &t : nullptr;
    }
    void* ptr(int i, at::ScalarType want, int64_t r, int64_t c) {
        const at::Tensor* t = tensor(i);
        if (!t) return nullptr;
        const auto sz = t->sizes();
        ok = t->scalar_type() == want && sz.size() == 2 && sz[0] == r && sz[1] == c;
        return t->data_ptr();
    }
    void* act(int i) { return ptr(i, dt, s.T, s.d); }
    void* sel(int i) { return ptr(i, dt, s.T, s.K); }
    void* weight(int i) {                                // [F, d], or [experts, F, d]
        if (experts == 0) return ptr(i, dt, s.F, s.d);
        const at::Tensor* t = tensor(i);
        if (!t) return nullptr;
        const auto sz = t->sizes();
        ok = t->scalar_type() == dt && sz.size() == 3 && sz[0] == experts && sz[1] == s.F && sz[2] == s.d;
        return t->data_ptr();
    }
    int32_t* idx(int i) { return static_cast<int32_t*>(ptr(i, at::kInt, s.T, s.K)); }
    void* bytes(int i, size_t* n) {
        const at::Tensor* t = tensor(i);
        if (!t) return nullptr;
        *n = t->numel() * t->element_size();
        return t->data_ptr();
    }
    long number(int i) {
        if (!ok || !PyLong_CheckExact(v[i])) { ok = false; return 0; }
        int over = 0;
        const long n = PyLong_AsLongAndOverflow(v[i], &over);
        ok = !over && n >= INT32_MIN && n <= INT32_MAX;
        return n;
    }
    // x is argument ix, W_gate (or the experts' W_gates) iw
    void* shape(int ix, int iw, bool with_experts = false) {
        const at::Tensor* x = tensor(ix);
        const at::Tensor* w = x ? tensor(iw) : nullptr;
        if (!w) return nullptr;
        dt = x->scalar_type();
        const int64_t nd = with_experts ? 3 : 2;
        ok = (dt == at::kFloat || dt == at::kBFloat16) && x->dim() == 2 && w->dim() == nd && x->size(0) <= INT32_MAX &&
             x->size(1) <= INT32_MAX && w->size(nd - 2) <= INT32_MAX;
        if (!ok) return nullptr;
        s.T = (int32_t)x->size(0);
        s.d = (int32_t)x->size(1);
        s.F = (int32_t)w->size(nd - 2);
        s.dtype = dt == at::kFloat ? MOC_F32 : MOC_BF16;
        experts = with_experts ? w->size(0) : 0;
        return x->data_ptr();
    }
    // experts + 1 row offsets from a list or tuple of integers
    int32_t* offsets(int i, int32_t* buf, int cap) {
        if (!ok || !(PyList_CheckExact(v[i]) || PyTuple_CheckExact(v[i])) || experts + 1 > cap || PySequence_Fast_GET_SIZE(v[i]) != experts + 1) {
            ok = false;
            return nullptr;
        }
        PyObject** items = PySequence_Fast_ITEMS(v[i]);
        for (int64_t e = 0; e <= experts; ++e) {
            if (!PyLong_CheckExact(items[e])) { ok = false; return nullptr; }
            int over = 0;
            const long n = PyLong_AsLongAndOverflow(items[e], &over);
            if (over || n < INT32_MIN || n > INT32_MAX) { ok = false; return nullptr; }
            buf[e] = (int32_t)n;
        }
        return buf;
    }
};

void* stream() { return static_cast<void*>(c10::hip::getCurrentHIPStream().stream()); }

template <class F> PyObject* finish(Args& a, const F& call) {
    if (!a.ok) return PyLong_FromLong(kNotTaken);
    void* st = stream();
    long r;
    Py_BEGIN_ALLOW_THREADS
    r = call(st);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(r);
}

#define NEED(n_) \
    if (nargs != (n_)) return PyLong_FromLong(kNotTaken)

// decode(x, wg, wu, wd, K, y, idx or None, ws)
PyObject* f_decode(PyObject*, PyObject* const* v, Py_ssize_t nargs) {
    NEED(8);
    Args a{v};
    void* x = a.shape(0, 1);
    a.s.K = (int32_t)a.number(4);
    void *wg = a.weight(1), *wu = a.weight(2), *wd = a.weight(3), *y = a.act(5);
    int32_t* idx = v[6] == Py_None ? nullptr : a.idx(6);
    size_t n = 0;
    void* ws = a.bytes(7, &n);
    return finish(a, [&](void* st) { return p_decode(&a.s, x, wg, wu, wd, y, idx, ws, n, st); });
}

// decode_grouped(x, wg, wu, wd, K, a, b, y, idx or None, ws)
PyObject* f_decode_grouped(PyObject*, PyObject* const* v, Py_ssize_t nargs) {
    NEED(10);
    Args a{v};
    void* x = a.shape(0, 1);
    a.s.K = (int32_t)a.number(4);
    const int32_t ga = (int32_t)a.number(5), gb = (int32_t)a.number(6);
    void *wg = a.weight(1), *wu = a.weight(2), *wd = a.weight(3), *y = a.act(7);
    int32_t* idx = v[8] == Py_None ? nullptr : a.idx(8);
    size_t n = 0;
    void* ws = a.bytes(9, &n);
    return finish(a, [&](void* st) { return p_decode_grouped(&a.s, ga, gb, x, wg, wu, wd, y, idx, ws, n, st); });
}

// fwd(x, wg, wu, wd, K, y, idx, gvals, uvals, ws)
PyObject* f_fwd(PyObject*, PyObject* const* v, Py_ssize_t nargs) {
    NEED(10);
    Args a{v};
    void* x = a.shape(0, 1);
    a.s.K = (int32_t)a.number(4);
    void *wg = a.weight(1), *wu = a.weight(2), *wd = a.weight(3), *y = a.act(5);
    int32_t* idx = a.idx(6);
    void *gv = a.sel(7), *uv = a.sel(8);
    size_t n = 0;
    void* ws = a.bytes(9, &n);
    return finish(a, [&](void* st) { return p_fwd(&a.s, x, wg, wu, wd, y, idx, gv, uv, ws, n, st); });
}

// fwd_grouped(x, wg, wu, wd, K, a, b, y, idx, gvals, uvals, ws)
PyObject* f_fwd_grouped(PyObject*, PyObject* const* v, Py_ssize_t nargs) {
    NEED(12);
    Args a{v};
    void* x = a.shape(0, 1);
    a.s.K = (int32_t)a.number(4);
    const int32_t ga = (int32_t)a.number(5), gb = (int32_t)a.number(6);
    void *wg = a.weight(1), *wu = a.weight(2), *wd = a.weight(3), *y = a.act(7);
    int32_t* idx = a.idx(8);
    void *gv = a.sel(9), *uv = a.sel(10);
    size_t n = 0;
    void* ws = a.bytes(11, &n);
    return finish(a, [&](void* st) { return p_fwd_grouped(&a.s, ga, gb, x, wg, wu, wd, y, idx, gv, uv, ws, n, st); });
}

// bwd(x, wg, wu, wd, idx, gvals, uvals, dy, dx, dwg, dwu, dwd, ws, K)
PyObject* f_bwd(PyObject*, PyObject* const* v, Py_ssize_t nargs) {
    NEED(14);
    Args a{v};
    void* x = a.shape(0, 1);
    a.s.K = (int32_t)a.number(13);
    void *wg = a.weight(1), *wu = a.weight(2), *wd = a.weight(3);
    int32_t* idx = a.idx(4);
    void *gv = a.sel(5), *uv = a.sel(6), *dy = a.act(7), *dx = a.act(8), *dwg = a.weight(9), *dwu = a.weight(10), *dwd = a.weight(11);
    size_t n = 0;
    void* ws = a.bytes(12, &n);
    return finish(a, [&](void* st) { return p_bwd(&a.s, x, wg, wu, wd, idx, gv, uv, dy, dx, dwg, dwu, dwd, ws, n, st); });
}

constexpr int kMaxOffsets = 65;

// fwd_experts(x, offsets, wg, wu, wd, K, y, idx, gvals, uvals, ws)
PyObject* f_fwd_experts(PyObject*, PyObject* const* v, Py_ssize_t nargs) {
    NEED(11);
    Args a{v};
    int32_t buf[kMaxOffsets];
    void* x = a.shape(0, 2, true);
    const int32_t* off = a.offsets(1, buf, kMaxOffsets);
    a.s.K = (int32_t)a.number(5);
    void *wg = a.weight(2), *wu = a.weight(3), *wd = a.weight(4), *y = a.act(6);
    int32_t* idx = a.idx(7);
    void *gv = a.sel(8), *uv = a.sel(9);
    size_t n = 0;
    void* ws = a.bytes(10, &n);
    return finish(a, [&](void* st) { return p_fwd_experts(&a.s, (int32_t)a.experts, off, x, wg, wu, wd, y, idx, gv, uv, ws, n, st); });
}

// bwd_experts(x, offsets, wg, wu, wd, idx, gvals, uvals, dy, dx, dwg, dwu, dwd, ws, K)
PyObject* f_bwd_experts(PyObject*, PyObject* const* v, Py_ssize_t nargs) {
    NEED(15);
    Args a{v};
    int32_t buf[kMaxOffsets];
    void* x = a.shape(0, 2, true);
    const int32_t* off = a.offsets(1, buf, kMaxOffsets);
    a.s.K = (int32_t)a.number(14);
    void *wg = a.weight(2), *wu = a.weight(3), *wd = a.weight(4);
    int32_t* idx = a.idx(5);
    void *gv = a.sel(6), *uv = a.sel(7), *dy = a.act(8), *dx = a.act(9), *dwg = a.weight(10), *dwu = a.weight(11), *dwd = a.weight(12);
    size_t n = 0;
    void* ws = a.bytes(13, &n);
    return finish(a, [&](void* st) {
        return p_bwd_experts(&a.s, (int32_t)a.experts, off, x, wg, wu, wd, idx, gv, uv, dy, dx, dwg, dwu, dwd, ws, n, st);
    });
}

// h (argument i) gives T, d and the dtype
void* plain_shape(Args& a, int i) {
    const at::Tensor* h = a.tensor(i);
    if (!h) return nullptr;
    a.dt = h->scalar_type();
    a.ok = (a.dt == at::kFloat || a.dt == at::kBFloat16) && h->dim() == 2 && h->size(0) <= INT32_MAX && h->size(1) <= INT32_MAX;
    if (!a.ok) return nullptr;
    a.s.T = (int32_t)h->size(0);
    a.s.d = (int32_t)h->size(1);
    a.s.dtype = a.dt == at::kFloat ? MOC_F32 : MOC_BF16;
    return h->data_ptr();
}

// rmsnorm(h, gain, eps, out)
PyObject* f_rmsnorm(PyObject*, PyObject* const* v, Py_ssize_t nargs) {
    NEED(4);
    Args a{v};
    void* h = plain_shape(a, 0);
    const at::Tensor* gain = a.tensor(1);
    if (gain) a.ok = gain->scalar_type() == a.dt && gain->dim() == 1 && gain->size(0) == a.s.d;
    a.ok = a.ok && PyFloat_CheckExact(v[2]);
    void* out = a.act(3);
    if (!a.ok) return PyLong_FromLong(kNotTaken);
    const void* gp = gain->data_ptr();
    const float eps = (float)PyFloat_AS_DOUBLE(v[2]);
    return finish(a, [&](void* st) { return p_rmsnorm(a.s.T, a.s.d, a.s.dtype, h, gp, eps, out, st); });
}

// residual_add(h, y)
PyObject* f_residual_add(PyObject*, PyObject* const* v, Py_ssize_t nargs) {
    NEED(2);
    Args a{v};
    void* h = plain_shape(a, 0);
    void* y = a.act(1);
    return finish(a, [&](void* st) { return p_residual(a.s.T, a.s.d, a.s.dtype, h, y, st); });
}

// bind(path of the loaded library): resolves the entry points; False if one is missing
PyObject* f_bind(PyObject*, PyObject* arg) {
    const char* path = PyUnicode_AsUTF8(arg);
    if (!path) return nullptr;
    void* lib = dlopen(path, RTLD_NOW | RTLD_LOCAL);
    if (!lib) Py_RETURN_FALSE;
    bool ok = true;
    auto get = [&](auto& fn, const char* name) {
        fn = reinterpret_cast<std::remove_reference_t<decltype(fn)>>(dlsym(lib, name));
        ok = ok && fn;
    };
    get(p_fwd, "moc_ffn_fwd");
    get(p_bwd, "moc_ffn_bwd");
    get(p_decode, "moc_ffn_decode");
    get(p_fwd_grouped, "moc_ffn_fwd_grouped");
    get(p_decode_grouped, "moc_ffn_decode_grouped");
    get(p_fwd_experts, "moc_ffn_fwd_experts");
    get(p_bwd_experts, "moc_ffn_bwd_experts");
    get(p_rmsnorm, "moc_rmsnorm");
    get(p_residual, "moc_residual_add");
    return PyBool_FromLong(ok);
}

// torch throws where a tensor has no memory of its own (fake tensors and other subclasses under tracing): not taken.  The calls
// into the library, made without the interpreter's lock, do not throw.
template <PyObject* (*Fn)(PyObject*, PyObject* const*, Py_ssize_t)> PyObject* guarded(PyObject* self, PyObject* const* v, Py_ssize_t nargs) {
    try {
        return Fn(self, v, nargs);
    } catch (...) {
        return PyLong_FromLong(kNotTaken);
    }
}

#define FAST(name_, fn_) {name_, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(guarded<fn_>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"bind", f_bind, METH_O, nullptr},
                         FAST("decode", f_decode),
                         FAST("decode_grouped", f_decode_grouped),
                         FAST("fwd", f_fwd),
                         FAST("fwd_grouped", f_fwd_grouped),
                         FAST("bwd", f_bwd),
                         FAST("fwd_experts", f_fwd_experts),
                         FAST("bwd_experts", f_bwd_experts),
                         FAST("rmsnorm", f_rmsnorm),
                         FAST("residual_add", f_residual_add),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&module); }
