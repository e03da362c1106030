// lsb_bind.cpp -- CPython module `_bind`: the argument marshalling of the
// Python API in native code.
//
// A call through ctypes spends about 6 us on the host before the library sees
// it (tensor attributes, range-checked arguments, the current stream object);
// the library's own part, a launch included, is about 3.5 us.  Each function
// here takes the ordinary case of its entry point -- plain contiguous tensors
// of the right type on the current device, plain integers in range -- reads
// what the library needs from the tensors and calls it.  For anything else it
// returns None without calling, and the Python layer goes on with its checked
// path, which serves the call or raises the error that names the argument.
//
// The library's functions are looked up in the handle that the Python layer
// has loaded (install); the GIL is released around each call, as ctypes does.
//
// Reading a tensor can throw (storage that refuses to hand out its address, a
// lazy copy that finds no memory): no C++ exception may reach CPython, so each
// function declines then, and the checked path meets the same refusal as a
// Python error.
#include <Python.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <dlfcn.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>

#include "../../../include/lsb.h"

namespace {

struct Library {
    decltype(&lsb_capacity) capacity;
    decltype(&lsb_slice_stream_bytes) slice_stream_bytes;
    decltype(&lsb_embed) embed;
    decltype(&lsb_extract) extract;
    decltype(&lsb_extract_sync) extract_sync;
    decltype(&lsb_embed_raw) embed_raw;
    decltype(&lsb_extract_raw) extract_raw;
    decltype(&lsb_paper_embed) paper_embed;
    decltype(&lsb_paper_extract) paper_extract;
    decltype(&lsb_embed_plane) embed_plane;
    decltype(&lsb_extract_plane) extract_plane;
    decltype(&lsb_sse) sse;
    decltype(&lsb_verify) verify;
    decltype(&lsb_embed_verify) embed_verify;
    decltype(&lsb_plan_run) plan_run;
    decltype(&lsb_embed_batch) embed_batch;
    decltype(&lsb_extract_batch) extract_batch;
} L;

struct Bytes {
    uint8_t *p;
    uint64_t n;
};

// Arguments of one call.  `ok` turns false at the first argument that is not
// the ordinary case; what the readers return is then not used.
class Args {
   public:
    Args(PyObject *const *args, Py_ssize_t given, Py_ssize_t want) : a_(args), ok_(given == want) {
        if (ok_) ok_ = c10::hip::GetDevice(&dev_) == hipSuccess;
    }
    bool ok() const { return ok_; }
    void require(bool cond) { ok_ = ok_ && cond; }

    // A contiguous uint8 tensor on the current device (a null pointer if empty).
    Bytes bytes(int i) {
        const at::Tensor *t = tensor(i);
        if (!t || t->scalar_type() != at::kByte) return fail(), Bytes{};
        return Bytes{t->numel() ? (uint8_t *)t->data_ptr() : nullptr, (uint64_t)t->numel()};
    }
    // Address of at least `count` words of `bits` bits that a kernel writes.
    void *words(int i, int bits, int64_t count) {
        const at::Tensor *t = tensor(i);
        if (!t || t->numel() < count) return fail(), nullptr;
        const auto type = t->scalar_type();
        if (bits == 64 ? type != at::kLong && type != at::kUInt64 : type != at::kInt) return fail(), nullptr;
        return t->data_ptr();
    }
    uint64_t u64(int i) {
        if (!ok_ || !PyLong_CheckExact(a_[i])) return fail(), 0;
        const unsigned long long v = PyLong_AsUnsignedLongLong(a_[i]);
        if (v == (unsigned long long)-1 && PyErr_Occurred()) return PyErr_Clear(), fail(), 0;
        return v;
    }
    uint32_t u32(int i) {
        const uint64_t v = u64(i);
        require(v <= 0xFFFFFFFFull);
        return (uint32_t)v;
    }
    int k(int i) {
        const uint64_t v = u64(i);
        require(v <= 0x7FFFFFFF);
        return (int)v;
    }
    void *pointer(int i) { return (void *)(uintptr_t)u64(i); }
    // The raw handle of a given stream, or the current stream for None.
    void *stream(int i) {
        if (!ok_) return nullptr;
        if (a_[i] == Py_None) return (void *)c10::hip::getCurrentHIPStream(dev_).stream();
        return pointer(i);
    }
    bool none(int i) const { return ok_ && a_[i] == Py_None; }

   private:
    void fail() { ok_ = false; }
    // A plain torch.Tensor on the current device; wrappers (functorch levels,
    // Python dispatch, lazy conjugate or negative views) are not.
    const at::Tensor *tensor(int i) {
        if (!ok_ || !THPVariable_CheckExact(a_[i])) return nullptr;
        const at::Tensor &t = THPVariable_Unpack(a_[i]);
        const c10::DispatchKeySet ks = t.key_set();
        using K = c10::DispatchKey;
        if (!t.is_cuda() || t.layout() != at::kStrided || !t.has_storage() || t.device().index() != dev_ ||
            ks.has(K::FuncTorchBatched) || ks.has(K::FuncTorchGradWrapper) || ks.has(K::Functionalize) ||
            ks.has(K::Python) || ks.has(K::Conjugate) || ks.has(K::Negative) || ks.has(K::ZeroTensor) ||
            !t.is_contiguous())
            return nullptr;
        return &t;
    }
    PyObject *const *a_;
    bool ok_;
    c10::DeviceIndex dev_ = -1;
};

// The library's return code of a call made without the GIL, or None.
template <typename F>
PyObject *call(const Args &a, F f) {
    if (!a.ok()) Py_RETURN_NONE;
    int64_t rc;
    Py_BEGIN_ALLOW_THREADS rc = f();
    Py_END_ALLOW_THREADS return PyLong_FromLongLong(rc);
}

typedef PyObject *(*BindFn)(PyObject *, PyObject *const *, Py_ssize_t);

template <BindFn f>
PyObject *guarded(PyObject *self, PyObject *const *args, Py_ssize_t given) {
    try {
        return f(self, args, given);
    } catch (const std::exception &) {
        Py_RETURN_NONE;
    }
}

#define LSB_BIND(name) PyObject *name(PyObject *, PyObject *const *args, Py_ssize_t given)

LSB_BIND(capacity) {  // n, k
    if (given != 2 || !PyLong_CheckExact(args[0]) || !PyLong_CheckExact(args[1])) Py_RETURN_NONE;
    const unsigned long long n = PyLong_AsUnsignedLongLong(args[0]);
    const long k = PyLong_AsLong(args[1]);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    if (k < 1 || k > 8) Py_RETURN_NONE;
    return PyLong_FromLongLong(L.capacity(n, (int)k));
}

LSB_BIND(embed) {  // cover, stego, msg, k, stream
    Args a(args, given, 5);
    const Bytes c = a.bytes(0), s = a.bytes(1), m = a.bytes(2);
    const int k = a.k(3);
    void *st = a.stream(4);
    a.require(c.n == s.n && m.n <= 0xFFFFFFFFull);
    return call(a, [&] { return L.embed(c.p, s.p, c.n, m.p, (uint32_t)m.n, k, st); });
}

LSB_BIND(extract) {  // stego, out, len_status, k, stream
    Args a(args, given, 5);
    const Bytes s = a.bytes(0), o = a.bytes(1);
    uint32_t *ls = (uint32_t *)a.words(2, 32, 2);
    const int k = a.k(3);
    void *st = a.stream(4);
    return call(a, [&] { return L.extract(s.p, s.n, k, o.p, o.n, ls, (int32_t *)(ls + 1), st); });
}

LSB_BIND(extract_sync) {  // stego, out, k, stream -> (code, length)
    Args a(args, given, 4);
    const Bytes s = a.bytes(0), o = a.bytes(1);
    const int k = a.k(2);
    void *st = a.stream(3);
    if (!a.ok()) Py_RETURN_NONE;
    uint32_t len = 0;
    int rc;
    Py_BEGIN_ALLOW_THREADS rc = L.extract_sync(s.p, s.n, k, o.p, o.n, &len, st);
    Py_END_ALLOW_THREADS return Py_BuildValue("(iI)", rc, len);
}

// Bytes of the stream that a slice touches fit `have`; a k or size that the
// library refuses goes to the checked path.
bool slice_fits(int k, uint64_t t0, uint64_t n, uint64_t bits, uint64_t have) {
    const int64_t need = L.slice_stream_bytes(k, t0, n, bits);
    return need >= 0 && (uint64_t)need <= have;
}

LSB_BIND(embed_raw) {  // cover, stego, t0, stream_bytes, stream_bits, k, stream
    Args a(args, given, 7);
    const Bytes c = a.bytes(0), s = a.bytes(1), b = a.bytes(3);
    const uint64_t t0 = a.u64(2), bits = a.u64(4);
    const int k = a.k(5);
    void *st = a.stream(6);
    a.require(c.n == s.n);
    if (a.ok()) a.require(slice_fits(k, t0, c.n, bits, b.n));
    return call(a, [&] { return L.embed_raw(c.p, s.p, c.n, t0, b.p, bits, k, st); });
}

LSB_BIND(extract_raw) {  // stego, t0, stream_out, stream_bits, k, stream
    Args a(args, given, 6);
    const Bytes s = a.bytes(0), o = a.bytes(2);
    const uint64_t t0 = a.u64(1), bits = a.u64(3);
    const int k = a.k(4);
    void *st = a.stream(5);
    if (a.ok()) a.require(slice_fits(k, t0, s.n, bits, o.n));
    return call(a, [&] { return L.extract_raw(s.p, s.n, t0, o.p, bits, k, st); });
}

// h * w * c == n, without overflow.
bool image_fits(uint32_t h, uint32_t w, uint32_t c, uint64_t n) {
    return (unsigned __int128)h * w * c == (unsigned __int128)n;
}

LSB_BIND(paper_embed) {  // cover, stego, h, w, c, plane, data, stream
    Args a(args, given, 8);
    const Bytes cv = a.bytes(0), s = a.bytes(1), d = a.bytes(6);
    const uint32_t h = a.u32(2), w = a.u32(3), c = a.u32(4), plane = a.u32(5);
    void *st = a.stream(7);
    a.require(cv.n == s.n && image_fits(h, w, c, cv.n));
    return call(a, [&] { return L.paper_embed(cv.p, s.p, h, w, c, plane, d.p, d.n, st); });
}

LSB_BIND(paper_extract) {  // stego, out, h, w, c, plane, length, stream
    Args a(args, given, 8);
    const Bytes s = a.bytes(0), o = a.bytes(1);
    const uint32_t h = a.u32(2), w = a.u32(3), c = a.u32(4), plane = a.u32(5);
    const uint64_t len = a.u64(6);
    void *st = a.stream(7);
    a.require(image_fits(h, w, c, s.n) && len <= o.n);
    return call(a, [&] { return L.paper_extract(s.p, h, w, c, plane, len ? o.p : nullptr, len, st); });
}

LSB_BIND(embed_plane) {  // cover, stego, c, plane, msg, k, stream
    Args a(args, given, 7);
    const Bytes cv = a.bytes(0), s = a.bytes(1), m = a.bytes(4);
    const uint32_t c = a.u32(2), plane = a.u32(3);
    const int k = a.k(5);
    void *st = a.stream(6);
    a.require(c > 0 && cv.n % (c ? c : 1) == 0 && cv.n == s.n && m.n <= 0xFFFFFFFFull);
    return call(a, [&] { return L.embed_plane(cv.p, s.p, cv.n / c, c, plane, m.p, (uint32_t)m.n, k, st); });
}

LSB_BIND(extract_plane) {  // stego, out, len_status, c, plane, k, stream
    Args a(args, given, 7);
    const Bytes s = a.bytes(0), o = a.bytes(1);
    uint32_t *ls = (uint32_t *)a.words(2, 32, 2);
    const uint32_t c = a.u32(3), plane = a.u32(4);
    const int k = a.k(5);
    void *st = a.stream(6);
    a.require(c > 0);
    return call(a, [&] {
        return L.extract_plane(s.p, s.n / c, c, plane, k, o.p, o.n, ls, (int32_t *)(ls + 1), st);
    });
}

LSB_BIND(sse) {  // a, b, out, stream
    Args a(args, given, 4);
    const Bytes x = a.bytes(0), y = a.bytes(1);
    uint64_t *o = (uint64_t *)a.words(2, 64, 1);
    void *st = a.stream(3);
    a.require(x.n == y.n);
    return call(a, [&] { return L.sse(x.p, y.p, x.n, o, st); });
}

LSB_BIND(verify) {  // cover, stego, msg, k, out, stream
    Args a(args, given, 6);
    const Bytes c = a.bytes(0), s = a.bytes(1), m = a.bytes(2);
    const int k = a.k(3);
    uint64_t *o = (uint64_t *)a.words(4, 64, 1);
    void *st = a.stream(5);
    a.require(c.n == s.n && m.n <= 0xFFFFFFFFull);
    return call(a, [&] { return L.verify(c.p, s.p, c.n, m.p, (uint32_t)m.n, k, o, st); });
}

LSB_BIND(embed_verify) {  // cover, stego, msg, k, mismatches, stream
    Args a(args, given, 6);
    const Bytes c = a.bytes(0), s = a.bytes(1), m = a.bytes(2);
    const int k = a.k(3);
    uint64_t *o = (uint64_t *)a.words(4, 64, 1);
    void *st = a.stream(5);
    a.require(c.n == s.n && m.n <= 0xFFFFFFFFull);
    return call(a, [&] { return L.embed_verify(c.p, s.p, c.n, m.p, (uint32_t)m.n, k, o, st); });
}

// Arena of a plan run with at least `need` bytes.
uint8_t *arena(Args &a, int i, uint64_t need) {
    const Bytes b = a.bytes(i);
    a.require(b.n >= need);
    return b.p;
}

LSB_BIND(embed_batch) {  // plan, jobs, need (cover, stego, msg), cover, stego, msg, status, stream
    Args a(args, given, 10);
    lsb_plan *p = (lsb_plan *)a.pointer(0);
    const uint64_t jobs = a.u64(1), nc = a.u64(2), ns = a.u64(3), nm = a.u64(4);
    uint8_t *c = arena(a, 5, nc), *s = arena(a, 6, ns), *m = arena(a, 7, nm);
    int32_t *status = (int32_t *)a.words(8, 32, (int64_t)jobs);
    void *st = a.stream(9);
    return call(a, [&] { return L.embed_batch(p, c, s, m, status, st); });
}

LSB_BIND(extract_batch) {  // plan, jobs, need (stego, msg), stego, msg, len, status, stream
    Args a(args, given, 9);
    lsb_plan *p = (lsb_plan *)a.pointer(0);
    const uint64_t jobs = a.u64(1), ns = a.u64(2), nm = a.u64(3);
    uint8_t *s = arena(a, 4, ns), *m = arena(a, 5, nm);
    uint32_t *len = (uint32_t *)a.words(6, 32, (int64_t)jobs);
    int32_t *status = (int32_t *)a.words(7, 32, (int64_t)jobs);
    void *st = a.stream(8);
    return call(a, [&] { return L.extract_batch(p, s, m, len, status, st); });
}

LSB_BIND(plan_run) {  // plan, jobs, need (cover, stego, msg), cover, stego, msg, len, status, stream
    Args a(args, given, 11);
    lsb_plan *p = (lsb_plan *)a.pointer(0);
    const uint64_t jobs = a.u64(1), nc = a.u64(2), ns = a.u64(3), nm = a.u64(4);
    uint8_t *c = nc == 0 && a.none(5) ? nullptr : arena(a, 5, nc);
    uint8_t *s = arena(a, 6, ns), *m = arena(a, 7, nm);
    uint32_t *len = a.none(8) ? nullptr : (uint32_t *)a.words(8, 32, (int64_t)jobs);
    int32_t *status = (int32_t *)a.words(9, 32, (int64_t)jobs);
    void *st = a.stream(10);
    return call(a, [&] { return L.plan_run(p, c, s, m, len, status, st); });
}

template <typename F>
bool look_up(void *handle, const char *name, F *fn) {
    *fn = (F)dlsym(handle, name);
    if (!*fn) PyErr_Format(PyExc_RuntimeError, "liblsb.so does not export %s", name);
    return *fn != nullptr;
}

// install(handle): the dlopen handle of liblsb.so that the calls go to.
PyObject *install(PyObject *, PyObject *arg) {
    void *h = (void *)PyLong_AsVoidPtr(arg);
    if (!h) return PyErr_Occurred() ? nullptr : PyErr_Format(PyExc_ValueError, "null library handle");
#define LSB_FN(name) look_up(h, "lsb_" #name, &L.name)
    if (LSB_FN(capacity) && LSB_FN(slice_stream_bytes) && LSB_FN(embed) && LSB_FN(extract) && LSB_FN(extract_sync) &&
        LSB_FN(embed_raw) && LSB_FN(extract_raw) && LSB_FN(paper_embed) && LSB_FN(paper_extract) &&
        LSB_FN(embed_plane) && LSB_FN(extract_plane) && LSB_FN(sse) && LSB_FN(verify) && LSB_FN(embed_verify) &&
        LSB_FN(plan_run) && LSB_FN(embed_batch) && LSB_FN(extract_batch))
        Py_RETURN_NONE;
    return nullptr;
}

#define LSB_METHOD(name) {#name, (PyCFunction)(void (*)(void))guarded<name>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {LSB_METHOD(capacity), LSB_METHOD(embed), LSB_METHOD(extract), LSB_METHOD(extract_sync),
                         LSB_METHOD(embed_raw), LSB_METHOD(extract_raw), LSB_METHOD(paper_embed),
                         LSB_METHOD(paper_extract), LSB_METHOD(embed_plane), LSB_METHOD(extract_plane),
                         LSB_METHOD(sse), LSB_METHOD(verify), LSB_METHOD(embed_verify), LSB_METHOD(embed_batch),
                         LSB_METHOD(extract_batch), LSB_METHOD(plan_run),
                         {"install", install, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_bind", "Native argument marshalling over liblsb.so.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__bind(void) { return PyModule_Create(&module); }
