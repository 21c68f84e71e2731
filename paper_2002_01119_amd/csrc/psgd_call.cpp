// The Python binding's short way into libpsgd: the calls of a training loop with plain device tensors, checked and passed on
// without building Python objects for every shape and pointer (psgd.py's own way takes 2.5 to 3 us of a 5.5 to 10 us call).
// A call that is not plainly in order is not answered here: NOT_MINE sends it psgd.py's way, which checks it argument by argument
// and raises what there is to raise, as it does for the library's refusals of an argument; other failures psgd.py raises at once.  Nothing is kept between calls but the addresses of the library's functions.
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include <c10/hip/HIPStream.h>

#include <cstdint>

#include "psgd.h"

namespace {

constexpr long NOT_MINE = 1;   // the library's own statuses are zero and negative

struct Library {
    decltype(&psgd_mix_step_deg) mix_step_deg = nullptr;
    decltype(&psgd_mix_step_d1d) mix_step_d1d = nullptr;
    decltype(&psgd_mix_full) mix_full = nullptr;
    decltype(&psgd_build_mixing_device) build_mixing_device = nullptr;
    decltype(&psgd_consensus_dist_ex) consensus_dist_ex = nullptr;
    decltype(&psgd_synth_grad_ex) synth_grad_ex = nullptr;
    decltype(&psgd_consensus_dist) consensus_dist = nullptr;
} lib;

// A plain strided tensor on device `dev` whose pointer means what it says: no subclass, no tensor of a transform or a trace.
const at::Tensor* plain(PyObject* o, int dev) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || t.get_device() != dev || !t.has_storage()) return nullptr;
    const at::TensorImpl* impl = t.unsafeGetTensorImpl();
    if (impl->is_python_dispatch()) return nullptr;
    const c10::DispatchKeySet ks = t.key_set();
    using K = c10::DispatchKey;
    for (K k : {K::FuncTorchBatched, K::FuncTorchGradWrapper, K::Functionalize, K::Conjugate, K::Negative, K::ZeroTensor, K::Python})
        if (ks.has(k)) return nullptr;
    return &t;
}

struct Rows {
    void* p;
    int64_t ld;
};
// [n, d] with unit stride along d; the first tensor says what n and d are (n < 0 on entry).
bool rows(PyObject* o, int dev, c10::ScalarType type, int64_t& n, int64_t& d, Rows& r) {
    const at::Tensor* t = plain(o, dev);
    if (!t || t->scalar_type() != type || t->dim() != 2) return false;
    const int64_t tn = t->size(0), td = t->size(1);
    if (n < 0) {
        n = tn;
        d = td;
    }
    if (tn != n || td != d || n < 1 || n > PSGD_MAX_N || (d > 1 && t->stride(1) != 1)) return false;
    r.p = t->data_ptr();
    r.ld = n > 1 ? t->stride(0) : d;
    return true;
}
// A contiguous table of `type` with a whole number of slots per row.
bool table(PyObject* o, int dev, c10::ScalarType type, int64_t n, int64_t& deg, void*& p) {
    const at::Tensor* t = plain(o, dev);
    if (!t || t->scalar_type() != type || !t->is_contiguous() || t->numel() < n || t->numel() % n || t->numel() / n > PSGD_MAX_DEG)
        return false;
    if (deg < 0) deg = t->numel() / n;
    p = t->data_ptr();
    return deg == t->numel() / n;
}
bool scalar_out(PyObject* o, int dev, double*& p) {
    p = nullptr;
    if (o == Py_None) return true;
    const at::Tensor* t = plain(o, dev);
    if (!t || t->scalar_type() != at::kDouble || t->numel() < 1) return false;
    p = static_cast<double*>(t->data_ptr());
    return true;
}
// The stream's handle: the current one for None, else the object's own.
bool stream_of(PyObject* o, int dev, void*& s) {
    if (o == Py_None) {
        s = c10::hip::getCurrentHIPStream(static_cast<c10::DeviceIndex>(dev)).stream();
        return true;
    }
    PyObject* h = PyObject_GetAttrString(o, "cuda_stream");
    if (!h) {
        PyErr_Clear();
        return false;
    }
    s = PyLong_AsVoidPtr(h);
    Py_DECREF(h);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}
bool number(PyObject* o, float& v) {
    if (!PyFloat_CheckExact(o)) return false;
    v = static_cast<float>(PyFloat_AS_DOUBLE(o));
    return true;
}
bool integer(PyObject* o, int64_t& v) {
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    v = PyLong_AsLongLongAndOverflow(o, &over);
    return !over;
}
int device() { return lib.mix_full ? static_cast<int>(c10::hip::current_device()) : -1; }
PyObject* answer(long rc) { return PyLong_FromLong(rc); }

// Errors of torch's own accessors (C++ exceptions) are not for Python's C API to meet: such a call goes the long way.
template <typename F> PyObject* guarded(const F& f) {
    try {
        return answer(f());
    } catch (...) {
        return answer(NOT_MINE);
    }
}

// The library's calls run without the interpreter's lock, as through ctypes.
struct Unlocked {
    PyThreadState* state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};

bool gradient_type(PyObject* o, c10::ScalarType& type, int& bf16) {
    if (!THPVariable_CheckExact(o)) return false;
    type = THPVariable_Unpack(o).scalar_type();
    bf16 = type != at::kFloat;
    return type == at::kFloat || type == at::kBFloat16;
}

// mix_step(X, X_out, G, nbr, w, lr, delay_mode, stream, cdist_out)
PyObject* mix_step(PyObject*, PyObject* const* a, Py_ssize_t count) {
    return guarded([&]() -> long {
        const int dev = device();
        int64_t n = -1, d = 0, deg = -1, mode = 0;
        Rows x, o, g;
        void *nbr, *w, *s;
        double* cd;
        float lr;
        c10::ScalarType type;
        int bf16 = 0;
        if (count != 9 || dev < 0 || !gradient_type(a[2], type, bf16) || !rows(a[0], dev, at::kFloat, n, d, x) ||
            !rows(a[1], dev, at::kFloat, n, d, o) || !rows(a[2], dev, type, n, d, g) || !table(a[3], dev, at::kInt, n, deg, nbr) ||
            !table(a[4], dev, at::kFloat, n, deg, w) || !number(a[5], lr) || !integer(a[6], mode) || mode < 0 || mode > 1 ||
            !stream_of(a[7], dev, s) || !scalar_out(a[8], dev, cd))
            return NOT_MINE;
        Unlocked run;
        return lib.mix_step_deg(static_cast<float*>(x.p), x.ld, static_cast<float*>(o.p), o.ld, g.p, g.ld, bf16,
                                static_cast<int32_t*>(nbr), static_cast<float*>(w), static_cast<int>(deg), static_cast<int>(n), d, lr,
                                static_cast<int>(mode), cd, s);
    });
}

// mix_full(X, X_out, G, lr, delay_mode, stream, cdist_out)
PyObject* mix_full(PyObject*, PyObject* const* a, Py_ssize_t count) {
    return guarded([&]() -> long {
        const int dev = device();
        int64_t n = -1, d = 0, mode = 0;
        Rows x, o, g;
        void* s;
        double* cd;
        float lr;
        c10::ScalarType type;
        int bf16 = 0;
        if (count != 7 || dev < 0 || !gradient_type(a[2], type, bf16) || !rows(a[0], dev, at::kFloat, n, d, x) ||
            !rows(a[1], dev, at::kFloat, n, d, o) || !rows(a[2], dev, type, n, d, g) || !number(a[3], lr) || !integer(a[4], mode) ||
            mode < 0 || mode > 1 || !stream_of(a[5], dev, s) || !scalar_out(a[6], dev, cd))
            return NOT_MINE;
        Unlocked run;
        return lib.mix_full(static_cast<float*>(x.p), x.ld, static_cast<float*>(o.p), o.ld, g.p, g.ld, bf16, static_cast<int>(n), d, lr,
                            static_cast<int>(mode), cd, s);
    });
}

// mix_step_d1d(X, X_out, G, nbr, w, lr, noise, G_next, c, stream, cdist_out)
PyObject* mix_step_d1d(PyObject*, PyObject* const* a, Py_ssize_t count) {
    return guarded([&]() -> long {
        const int dev = device();
        int64_t n = -1, d = 0, deg = -1;
        Rows x, o, g, z, h;
        void *nbr, *w, *s;
        double* cd;
        float lr, c;
        if (count != 11 || dev < 0 || !rows(a[0], dev, at::kFloat, n, d, x) || !rows(a[1], dev, at::kFloat, n, d, o) ||
            !rows(a[2], dev, at::kFloat, n, d, g) || !table(a[3], dev, at::kInt, n, deg, nbr) || !table(a[4], dev, at::kFloat, n, deg, w) ||
            !number(a[5], lr) || !rows(a[6], dev, at::kFloat, n, d, z) || !rows(a[7], dev, at::kFloat, n, d, h) || !number(a[8], c) ||
            !stream_of(a[9], dev, s) || !scalar_out(a[10], dev, cd))
            return NOT_MINE;
        Unlocked run;
        return lib.mix_step_d1d(static_cast<float*>(x.p), x.ld, static_cast<float*>(o.p), o.ld, static_cast<float*>(g.p), g.ld,
                                static_cast<int32_t*>(nbr), static_cast<float*>(w), static_cast<int>(deg), static_cast<int>(n), d, lr,
                                static_cast<float*>(z.p), z.ld, static_cast<float*>(h.p), h.ld, c, cd, s);
    });
}

// build_mixing_device(topology, n, seed, nbr, w, step_dev, step_offset, advance, stream)
PyObject* build_mixing_device(PyObject*, PyObject* const* a, Py_ssize_t count) {
    return guarded([&]() -> long {
        const int dev = device();
        int64_t topology, n, seed, offset, advance, deg = PSGD_DEG;
        void *nbr, *w, *s;
        uint64_t* step = nullptr;
        if (count != 9 || dev < 0 || !integer(a[0], topology) || !integer(a[1], n) || !integer(a[2], seed) || topology < 0 ||
            topology > 2 || n < 1 || n > PSGD_MAX_N || !table(a[3], dev, at::kInt, n, deg, nbr) || !table(a[4], dev, at::kFloat, n, deg, w) ||
            !integer(a[6], offset) || !integer(a[7], advance) || advance < 0 || advance > INT32_MAX || !stream_of(a[8], dev, s))
            return NOT_MINE;
        if (a[5] != Py_None) {
            const at::Tensor* t = plain(a[5], dev);
            if (!t || (t->scalar_type() != at::kLong && t->scalar_type() != at::kUInt64) || t->numel() < 1) return NOT_MINE;
            step = static_cast<uint64_t*>(t->data_ptr());
        }
        Unlocked run;
        return lib.build_mixing_device(static_cast<int>(topology), static_cast<int>(n), static_cast<uint64_t>(seed), step,
                                       static_cast<uint64_t>(offset), static_cast<int>(advance), static_cast<int32_t*>(nbr),
                                       static_cast<float*>(w), s);
    });
}

// consensus_dist_async(X, out, stream)
PyObject* consensus_dist_async(PyObject*, PyObject* const* a, Py_ssize_t count) {
    return guarded([&]() -> long {
        const int dev = device();
        int64_t n = -1, d = 0;
        Rows x;
        double* out;
        void* s;
        if (count != 3 || dev < 0 || a[1] == Py_None || !rows(a[0], dev, at::kFloat, n, d, x) || !scalar_out(a[1], dev, out) ||
            !stream_of(a[2], dev, s))
            return NOT_MINE;
        Unlocked run;
        return lib.consensus_dist_ex(static_cast<float*>(x.p), x.ld, static_cast<int>(n), d, out, s);
    });
}

// consensus_dist(X): the value, or None where the call is not answered here
PyObject* consensus_dist(PyObject*, PyObject* const* a, Py_ssize_t count) {
    double v = 0.0;
    bool mine = false;
    try {
        const int dev = device();
        int64_t n = -1, d = 0;
        Rows x;
        if (count == 1 && dev >= 0 && rows(a[0], dev, at::kFloat, n, d, x) && THPVariable_Unpack(a[0]).is_contiguous()) {
            Unlocked run;
            v = lib.consensus_dist(static_cast<float*>(x.p), static_cast<int>(n), d);
            mine = true;
        }
    } catch (...) {
    }
    if (!mine) Py_RETURN_NONE;
    return PyFloat_FromDouble(v);
}

// synth_grad(X_prev, noise, G, c, stream)
PyObject* synth_grad(PyObject*, PyObject* const* a, Py_ssize_t count) {
    return guarded([&]() -> long {
        const int dev = device();
        int64_t n = -1, d = 0;
        Rows x, z, g;
        float c;
        void* s;
        if (count != 5 || dev < 0 || !rows(a[0], dev, at::kFloat, n, d, x) || !rows(a[1], dev, at::kFloat, n, d, z) ||
            !rows(a[2], dev, at::kFloat, n, d, g) || !number(a[3], c) || !stream_of(a[4], dev, s))
            return NOT_MINE;
        Unlocked run;
        return lib.synth_grad_ex(static_cast<float*>(x.p), x.ld, static_cast<float*>(z.p), z.ld, static_cast<float*>(g.p), g.ld,
                                 static_cast<int>(n), d, c, s);
    });
}

// bind(addresses of the functions, in the order of struct Library)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t count) {
    void* p[7];
    if (count != 7) return answer(NOT_MINE);
    for (int i = 0; i < 7; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (PyErr_Occurred()) return nullptr;
    }
    lib.mix_step_deg = reinterpret_cast<decltype(lib.mix_step_deg)>(p[0]);
    lib.mix_step_d1d = reinterpret_cast<decltype(lib.mix_step_d1d)>(p[1]);
    lib.mix_full = reinterpret_cast<decltype(lib.mix_full)>(p[2]);
    lib.build_mixing_device = reinterpret_cast<decltype(lib.build_mixing_device)>(p[3]);
    lib.consensus_dist_ex = reinterpret_cast<decltype(lib.consensus_dist_ex)>(p[4]);
    lib.synth_grad_ex = reinterpret_cast<decltype(lib.synth_grad_ex)>(p[5]);
    lib.consensus_dist = reinterpret_cast<decltype(lib.consensus_dist)>(p[6]);
    return answer(0);
}

#define PSGD_METHOD(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {PSGD_METHOD(mix_step),  PSGD_METHOD(mix_full), PSGD_METHOD(mix_step_d1d), PSGD_METHOD(build_mixing_device),
                         PSGD_METHOD(consensus_dist_async), PSGD_METHOD(consensus_dist), PSGD_METHOD(synth_grad), PSGD_METHOD(bind), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call(void) { return PyModule_Create(&module); }
