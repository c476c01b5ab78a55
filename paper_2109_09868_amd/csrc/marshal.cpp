// Argument marshalling of the binding's calls in their ordinary form: exact torch tensors in device memory of the right type,
// shape and contiguity, float64 node arrays, Python ints, outputs given, torch's current stream.  Anything else returns None and
// the binding's own checks take over (they raise, convert or allocate), so what is accepted and refused is decided there.
// Bound by host time: a decode of 64 groups took 6.8 us to enqueue, 3.4 of it in Python around the 3.4 of call and launch.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

#include "approxifer.h"

namespace {

struct Library {
    decltype(&approxifer_encode) encode;
    decltype(&approxifer_decode) decode;
    decltype(&approxifer_decode_top1) decode_top1;
    decltype(&approxifer_decode_byzantine) byzantine;
    decltype(&approxifer_decode_byzantine_homogeneous) homogeneous;
    decltype(&approxifer_pad_last_group) pad_last_group;
    decltype(&approxifer_top1) top1;
    decltype(&approxifer_wait_mask) wait_mask;
};

// The handle of a loaded library: its entry points, by address, in the order above.
constexpr const char *kCapsule = "approxifer.library";
const Library *library(PyObject *o) { return static_cast<const Library *>(PyCapsule_GetPointer(o, kCapsule)); }

PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != 8) {
        PyErr_SetString(PyExc_TypeError, "expected eight addresses");
        return nullptr;
    }
    void *p[8];
    for (int i = 0; i < 8; ++i) {
        p[i] = PyLong_AsVoidPtr(args[i]);
        if (PyErr_Occurred()) return nullptr;
    }
    Library *lib = new Library{
        reinterpret_cast<decltype(Library::encode)>(p[0]),         reinterpret_cast<decltype(Library::decode)>(p[1]),
        reinterpret_cast<decltype(Library::decode_top1)>(p[2]),    reinterpret_cast<decltype(Library::byzantine)>(p[3]),
        reinterpret_cast<decltype(Library::homogeneous)>(p[4]),    reinterpret_cast<decltype(Library::pad_last_group)>(p[5]),
        reinterpret_cast<decltype(Library::top1)>(p[6]),           reinterpret_cast<decltype(Library::wait_mask)>(p[7])};
    PyObject *c = PyCapsule_New(lib, kCapsule, [](PyObject *o) { delete static_cast<Library *>(PyCapsule_GetPointer(o, kCapsule)); });
    if (c == nullptr) delete lib;
    return c;
}

// A plain device tensor: no subclass, no wrapper of a transform or mode, dense and contiguous.
const at::Tensor *plain(PyObject *o, at::ScalarType type) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || t.scalar_type() != type) return nullptr;
    const c10::TensorImpl *impl = t.unsafeGetTensorImpl();
    const c10::DispatchKeySet keys = impl->key_set();
    if (!impl->has_storage() || impl->is_python_dispatch() || keys.has(c10::DispatchKey::FuncTorchBatched) ||
        keys.has(c10::DispatchKey::FuncTorchGradWrapper) || keys.has(c10::DispatchKey::Functionalize) ||
        keys.has(c10::DispatchKey::ZeroTensor) || impl->has_symbolic_sizes_strides() || !t.is_contiguous())
        return nullptr;
    return &t;
}
template <class... Size>
void *shaped(PyObject *o, at::ScalarType type, Size... sizes) {
    const at::Tensor *t = plain(o, type);
    const int64_t want[] = {static_cast<int64_t>(sizes)...};
    if (t == nullptr || t->dim() != static_cast<int64_t>(sizeof...(sizes))) return nullptr;
    for (size_t d = 0; d < sizeof...(sizes); ++d)
        if (t->size(d) != want[d]) return nullptr;
    return t->data_ptr();
}

bool integer(PyObject *o, int &v) {
    if (!PyLong_Check(o)) return false;
    int over = 0;
    const long x = PyLong_AsLongAndOverflow(o, &over);
    if (over != 0 || x != static_cast<int>(x)) return false;
    v = static_cast<int>(x);
    return true;
}

// A float64 array in host memory, held for the call.
struct Nodes {
    Py_buffer b{};
    bool held = false;
    explicit Nodes(PyObject *o) {
        if (PyObject_GetBuffer(o, &b, PyBUF_FORMAT | PyBUF_C_CONTIGUOUS) != 0) {
            PyErr_Clear();
            return;
        }
        held = true;
    }
    ~Nodes() {
        if (held) PyBuffer_Release(&b);
    }
    bool ok() const { return held && b.itemsize == 8 && b.format != nullptr && b.format[0] == 'd' && b.format[1] == '\0'; }
    int64_t size() const { return b.len / 8; }
    const double *data() const { return static_cast<const double *>(b.buf); }
};

void *current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// The call itself without the interpreter lock, as ctypes makes it; its status as a Python int.
template <class F>
PyObject *status_of(F call) {
    int rc;
    void *stream = current_stream();                          // may throw: not without the lock
    Py_BEGIN_ALLOW_THREADS
    rc = call(stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

constexpr at::ScalarType kF32 = at::kFloat, kI32 = at::kInt, kU8 = at::kByte;

// (library, queries, alpha, beta, coded)
PyObject *encode(PyObject *const *a, Py_ssize_t n) {
    const Library *lib = n == 5 ? library(a[0]) : nullptr;
    if (lib == nullptr) return nullptr;
    const Nodes al(a[2]), be(a[3]);
    const at::Tensor *q = plain(a[1], kF32);
    if (q == nullptr || !al.ok() || !be.ok() || q->dim() != 3 || q->size(1) != al.size()) Py_RETURN_NONE;
    const int64_t G = q->size(0), K = q->size(1), D = q->size(2), N = be.size();
    void *coded = shaped(a[4], kF32, G, N, D);
    void *queries = q->data_ptr();
    if (coded == nullptr || queries == nullptr) Py_RETURN_NONE;
    return status_of([&](void *s) {
        return lib->encode(static_cast<const float *>(queries), static_cast<float *>(coded), G, static_cast<int>(K),
                           static_cast<int>(N), D, al.data(), be.data(), s);
    });
}

struct Decode {
    int64_t G, N, C, K;
    void *preds, *mask, *status;
    int S, sign;
    bool ok;
    Decode(PyObject *p, PyObject *m, const Nodes &al, const Nodes &be, PyObject *s, PyObject *g, PyObject *st) : ok(false) {
        const at::Tensor *t = plain(p, kF32);
        if (t == nullptr || !al.ok() || !be.ok() || t->dim() != 3 || t->size(1) != be.size()) return;
        G = t->size(0);
        N = t->size(1);
        C = t->size(2);
        K = al.size();
        preds = t->data_ptr();
        mask = shaped(m, kU8, G, N);
        status = shaped(st, kI32, G);
        ok = preds != nullptr && mask != nullptr && status != nullptr && integer(s, S) && integer(g, sign);
    }
};

// (library, preds, mask, alpha, beta, S, sign_mode, out, status)
PyObject *decode(PyObject *const *a, Py_ssize_t n) {
    const Library *lib = n == 9 ? library(a[0]) : nullptr;
    if (lib == nullptr) return nullptr;
    const Nodes al(a[3]), be(a[4]);
    const Decode d(a[1], a[2], al, be, a[5], a[6], a[8]);
    void *out = d.ok ? shaped(a[7], kF32, d.G, d.K, d.C) : nullptr;
    if (out == nullptr) Py_RETURN_NONE;
    return status_of([&](void *s) {
        return lib->decode(static_cast<const float *>(d.preds), static_cast<const uint8_t *>(d.mask), static_cast<float *>(out),
                           static_cast<int32_t *>(d.status), d.G, static_cast<int>(d.K), static_cast<int>(d.N), d.S, d.C,
                           al.data(), be.data(), d.sign, s);
    });
}

// (library, preds, mask, alpha, beta, S, sign_mode, top1, score or None, status)
PyObject *decode_top1(PyObject *const *a, Py_ssize_t n) {
    const Library *lib = n == 10 ? library(a[0]) : nullptr;
    if (lib == nullptr) return nullptr;
    const Nodes al(a[3]), be(a[4]);
    const Decode d(a[1], a[2], al, be, a[5], a[6], a[9]);
    void *top1 = d.ok ? shaped(a[7], kI32, d.G, d.K) : nullptr;
    if (top1 == nullptr) Py_RETURN_NONE;
    void *score = nullptr;
    if (a[8] != Py_None && (score = shaped(a[8], kF32, d.G, d.K)) == nullptr) Py_RETURN_NONE;
    return status_of([&](void *s) {
        return lib->decode_top1(static_cast<const float *>(d.preds), static_cast<const uint8_t *>(d.mask),
                                static_cast<int32_t *>(top1), static_cast<float *>(score), static_cast<int32_t *>(d.status), d.G,
                                static_cast<int>(d.K), static_cast<int>(d.N), d.S, d.C, al.data(), be.data(), d.sign, s);
    });
}

// (library, homogeneous, preds, mask, alpha, beta, S, A, sign_mode, out, adv, status, workspace or None)
PyObject *byzantine(PyObject *const *a, Py_ssize_t n) {
    const Library *lib = n == 13 ? library(a[0]) : nullptr;
    if (lib == nullptr) return nullptr;
    const Nodes al(a[4]), be(a[5]);
    const Decode d(a[2], a[3], al, be, a[6], a[8], a[11]);
    int A = 0;
    if (!d.ok || !integer(a[7], A) || A < 1) Py_RETURN_NONE;
    void *out = shaped(a[9], kF32, d.G, d.K, d.C);
    void *adv = shaped(a[10], kI32, d.G, A);
    if (out == nullptr || adv == nullptr) Py_RETURN_NONE;
    void *ws = nullptr;
    size_t ws_bytes = 0;
    if (a[12] != Py_None) {
        const at::Tensor *w = plain(a[12], kU8);
        if (w == nullptr) Py_RETURN_NONE;
        ws = w->data_ptr();
        ws_bytes = static_cast<size_t>(w->numel());
    }
    const auto entry = a[1] == Py_True ? lib->homogeneous : lib->byzantine;
    return status_of([&](void *s) {
        return entry(static_cast<const float *>(d.preds), static_cast<const uint8_t *>(d.mask), static_cast<float *>(out),
                     static_cast<int32_t *>(adv), static_cast<int32_t *>(d.status), d.G, static_cast<int>(d.K),
                     static_cast<int>(d.N), d.S, A, d.C, al.data(), be.data(), d.sign, ws, ws_bytes, s);
    });
}

// (library, buffer, Q, K): buffer [rows, D] with rows >= ceil(Q / K) K
PyObject *pad_last_group(PyObject *const *a, Py_ssize_t n) {
    const Library *lib = n == 4 ? library(a[0]) : nullptr;
    if (lib == nullptr) return nullptr;
    const at::Tensor *b = plain(a[1], kF32);
    int Q = 0, K = 0;
    if (b == nullptr || b->dim() != 2 || !integer(a[2], Q) || !integer(a[3], K) || Q < 1 || K < 1) Py_RETURN_NONE;
    const int64_t G = (static_cast<int64_t>(Q) + K - 1) / K;
    void *p = b->data_ptr();
    if (b->size(0) < G * K || p == nullptr) Py_RETURN_NONE;
    const int64_t D = b->size(1);
    return status_of([&](void *s) { return lib->pad_last_group(static_cast<float *>(p), Q, K, D, s); });
}

// (library, values [rows.., C], top1 [rows..], score or None)
PyObject *top1(PyObject *const *a, Py_ssize_t n) {
    const Library *lib = n == 4 ? library(a[0]) : nullptr;
    if (lib == nullptr) return nullptr;
    const at::Tensor *v = plain(a[1], kF32), *t = plain(a[2], kI32);
    if (v == nullptr || t == nullptr || v->dim() < 1 || v->sizes().slice(0, v->dim() - 1) != t->sizes()) Py_RETURN_NONE;
    const at::Tensor *sc = a[3] == Py_None ? nullptr : plain(a[3], kF32);
    if (a[3] != Py_None && (sc == nullptr || sc->sizes() != t->sizes())) Py_RETURN_NONE;
    const int64_t C = v->size(v->dim() - 1), rows = t->numel();
    void *vp = v->data_ptr(), *tp = t->data_ptr(), *sp = sc != nullptr ? sc->data_ptr() : nullptr;
    if (vp == nullptr || tp == nullptr || (sc != nullptr && sp == nullptr)) Py_RETURN_NONE;
    return status_of([&](void *s) {
        return lib->top1(static_cast<const float *>(vp), static_cast<int32_t *>(tp), static_cast<float *>(sp), rows, C, s);
    });
}

// (library, arrival, wait_for, mask, count)
PyObject *wait_mask(PyObject *const *a, Py_ssize_t n) {
    const Library *lib = n == 5 ? library(a[0]) : nullptr;
    if (lib == nullptr) return nullptr;
    const at::Tensor *t = plain(a[1], kF32);
    int wait_for = 0;
    if (t == nullptr || t->dim() != 2 || !integer(a[2], wait_for)) Py_RETURN_NONE;
    const int64_t G = t->size(0), N = t->size(1);
    void *arrival = t->data_ptr(), *mask = shaped(a[3], kU8, G, N), *count = shaped(a[4], kI32, G);
    if (arrival == nullptr || mask == nullptr || count == nullptr) Py_RETURN_NONE;
    return status_of([&](void *s) {
        return lib->wait_mask(static_cast<const float *>(arrival), static_cast<uint8_t *>(mask), static_cast<int32_t *>(count), G,
                              static_cast<int>(N), wait_for, s);
    });
}

// No C++ exception leaves the module: what torch throws makes the call one for the binding's own checks.
template <PyObject *(*F)(PyObject *const *, Py_ssize_t)>
PyObject *guarded(PyObject *, PyObject *const *args, Py_ssize_t n) {
    try {
        PyObject *r = F(args, n);
        if (r == nullptr && !PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return r;
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

#define APPROXIFER_METHOD(name) \
    {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&guarded<name>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&bind)), METH_FASTCALL, nullptr},
    APPROXIFER_METHOD(encode),    APPROXIFER_METHOD(decode),         APPROXIFER_METHOD(decode_top1),
    APPROXIFER_METHOD(byzantine), APPROXIFER_METHOD(pad_last_group), APPROXIFER_METHOD(top1),
    APPROXIFER_METHOD(wait_mask), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: the interpreter and the torch whose layouts are compiled in; the binding uses the module with no other.
PyMODINIT_FUNC PyInit__marshal(void) {
    PyObject *m = PyModule_Create(&module);
    if (m != nullptr && PyModule_AddStringConstant(m, "built_for", APPROXIFER_BUILT_FOR) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
