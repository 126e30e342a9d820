// The hot half of the Python binding: the device calls of a plan with lists of tensors or marshalled pointer
// arrays, straight to the C ABI.  Tensors and buffers are taken as lists and tuples of plain tensors or as c_void_p arrays;
// weights, scalars and streams in every form that the ctypes half takes.  For anything else a call returns None and
// that half, which raises every error of marshalling, makes the call.
//
// On small sets the host decides: a pack, reduce and unpack of 158 tensors handed over as lists asked 323 tensors
// for their addresses through Python and copied them twice, 34.5 us a step where the kernels take 18 (18.5 now, the kernels
// alone); three calls on 6 tensors with marshalled arrays took 14.5 us (11.7 to 12.4), where three launches of an empty kernel with as many
// arguments take 10.9 to 11.5 and the three C calls 11.4 to 12.0 in the same process.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <cstring>
#include <string>
#include <vector>

#include "kt.h"

namespace {

PyObject *ctypes_array = nullptr;       // ctypes.Array
PyObject *cuda_stream = nullptr;        // "cuda_stream"
PyObject *get_device = nullptr, *get_stream = nullptr;      // torch._C._cuda_getDevice, _cuda_getCurrentRawStream

// The entry points of one loaded library, as addresses: two libraries may be loaded in one process.
struct Entries {
    kt_status (*pack)(kt_plan *, int, const void *const *, void *const *, void *);
    kt_status (*reduce)(kt_plan *, int, const void *const *, int, const float *, void *const *, void *);
    kt_status (*unpack)(kt_plan *, int, const void *const *, float, void *const *, void *);
    kt_status (*fused)(kt_plan *, int, const void *const *, const void *const *, int, const float *, float, void *const *, void *);
    kt_status (*sgd)(kt_plan *, int, const void *const *, float, void *const *, void *const *, float, float, float, int, void *);
    kt_status (*master)(kt_plan *, int, const void *const *, float, void *const *, void *const *, void *const *, float, float, float,
                        int, void *);
    kt_status (*fused_sgd)(kt_plan *, int, const void *const *, const void *const *, int, const float *, float, void *const *,
                           void *const *, void *const *, float, float, float, int, void *);
};

struct Calls {
    PyObject_HEAD
    Entries f;
};

constexpr int MAX_ARRAYS = 5;

// What one call has converted.  `ok` turns false at the first form that is not taken here; a Python error is never left set.
// Scalars, weights and the stream may run Python (__float__, __index__, the collector with what it finalizes), and with it other
// calls of this thread: they are asked for before the pointers, whose tables the thread has once.
struct Args {
    PyObject *const *a;
    bool ok = true;
    Py_buffer held[MAX_ARRAYS + 1];
    int nheld = 0;
    int arrays = 0;
    float w[KT_MAX_PEERS];

    explicit Args(PyObject *const *args) : a(args) {}
    ~Args()
    {
        for (int i = 0; i < nheld; ++i) PyBuffer_Release(&held[i]);
    }
    Args(const Args &) = delete;
    bool fail()
    {
        PyErr_Clear();
        return ok = false;
    }

    // an int, or what stands for one, that fits a C int
    int integer(int i)
    {
        if (!ok) return 0;
        PyObject *x = a[i], *own = PyLong_CheckExact(x) ? nullptr : PyNumber_Index(x);
        if (!PyLong_CheckExact(x) && !own) return fail(), 0;
        int over = 0;
        const long v = PyLong_AsLongAndOverflow(own ? own : x, &over);
        Py_XDECREF(own);
        if (over || v != (int)v) return fail(), 0;
        return (int)v;
    }
    void *address(PyObject *x)
    {
        if (!PyLong_Check(x)) return fail(), nullptr;
        void *p = PyLong_AsVoidPtr(x);
        if (!p && PyErr_Occurred()) fail();
        return p;
    }
    // float(x)
    float real(PyObject *x)
    {
        if (PyFloat_CheckExact(x)) return (float)PyFloat_AS_DOUBLE(x);
        PyObject *f = PyNumber_Float(x);
        if (!f) return fail(), 0.0f;
        const double v = PyFloat_AS_DOUBLE(f);
        Py_DECREF(f);
        return (float)v;
    }
    float real(int i) { return ok ? real(a[i]) : 0.0f; }
    // bool(x)
    int flag(int i)
    {
        const int v = ok ? PyObject_IsTrue(a[i]) : 0;
        if (v < 0) fail();
        return v > 0;
    }

    // `want` elements of a ctypes array whose items are of struct code `code`; marshal() pads an empty list to one entry
    void *array(PyObject *x, Py_ssize_t want, char code, Py_ssize_t size)
    {
        if (!PyObject_TypeCheck(x, reinterpret_cast<PyTypeObject *>(ctypes_array))) return fail(), nullptr;
        Py_buffer &b = held[nheld];
        if (PyObject_GetBuffer(x, &b, PyBUF_FORMAT | PyBUF_ND) != 0) return fail(), nullptr;
        ++nheld;
        const char *f = b.format ? b.format : "";
        if (*f == '<' || *f == '=' || *f == '@') ++f;
        if (b.ndim != 1 || b.itemsize != size || f[0] != code || f[1] || b.shape[0] != (want > 0 ? want : 1)) return fail(), nullptr;
        return b.buf;
    }
    // `want` device addresses
    void *const *pointers(int i, Py_ssize_t want)
    {
        if (!ok) return nullptr;
        PyObject *x = a[i];
        if (!PyList_CheckExact(x) && !PyTuple_CheckExact(x)) return static_cast<void *const *>(array(x, want, 'P', sizeof(void *)));
        const Py_ssize_t n = PySequence_Fast_GET_SIZE(x);
        if (n != want || at::impl::torch_function_mode_enabled()) return fail(), nullptr;
        static thread_local std::vector<void *> tables[MAX_ARRAYS];      // kept: no allocation per call
        try {
            std::vector<void *> &t = tables[arrays++];
            t.resize(n > 0 ? n : 1);
            for (Py_ssize_t j = 0; j < n; ++j) {
                PyObject *item = PySequence_Fast_GET_ITEM(x, j);
                if (!THPVariable_CheckExact(item)) return fail(), nullptr;
                t[j] = THPVariable_Unpack(item).data_ptr();
            }
            return t.data();
        } catch (...) {         // a tensor without memory of its own, say: asked again through Python, it raises its own error
            return fail(), nullptr;
        }
    }
    const float *weights(int i, int K)
    {
        if (!ok || a[i] == Py_None) return nullptr;      // None: the plan's device-resident ones
        if (PyObject_TypeCheck(a[i], reinterpret_cast<PyTypeObject *>(ctypes_array)))
            return static_cast<const float *>(array(a[i], K, 'f', sizeof(float)));
        if (PyObject_Size(a[i]) != K) return fail(), nullptr;
        PyObject *t = PySequence_Tuple(a[i]);           // its own: __float__ of an item may change the list
        if (!t || PyTuple_GET_SIZE(t) != K) fail();
        for (int k = 0; ok && k < K; ++k) w[k] = real(PyTuple_GET_ITEM(t, k));
        Py_XDECREF(t);
        return w;
    }
    void *stream(PyObject *x)
    {
        if (x == Py_None) {             // torch's current stream on the current device
            PyObject *dev = PyObject_CallNoArgs(get_device);
            PyObject *raw = dev ? PyObject_CallOneArg(get_stream, dev) : nullptr;
            Py_XDECREF(dev);
            void *s = raw ? PyLong_AsVoidPtr(raw) : nullptr;
            Py_XDECREF(raw);
            if (PyErr_Occurred()) fail();
            return s;
        }
        if (PyLong_Check(x)) return address(x);
        PyObject *raw = PyObject_GetAttr(x, cuda_stream);
        void *s = raw ? address(raw) : (fail(), nullptr);
        Py_XDECREF(raw);
        return s;
    }
    int copies(int i)
    {
        const int K = integer(i);
        if (ok && (K < 1 || K > KT_MAX_PEERS)) fail();
        return ok ? K : 1;
    }
};

// Every call starts with: plan handle, number of tensors, number of buckets, bucket.
struct Plan {
    kt_plan *p;
    int T, nb, bucket;
    explicit Plan(Args &x)
    {
        p = static_cast<kt_plan *>(x.address(x.a[0]));
        T = x.integer(1);
        nb = x.integer(2);
        bucket = x.integer(3);
    }
};

// The call itself without the interpreter lock, as ctypes makes it.
template <typename F> PyObject *finish(const Args &x, F call)
{
    if (!x.ok) Py_RETURN_NONE;
    kt_status st;
    Py_BEGIN_ALLOW_THREADS
    st = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong((long)st);
}

const Entries &entries(PyObject *self) { return reinterpret_cast<Calls *>(self)->f; }

#define KT_CALL(name, count)                                                                             \
    PyObject *name(PyObject *self, PyObject *const *args, Py_ssize_t nargs)                              \
    {                                                                                                    \
        if (nargs != count) { PyErr_SetString(PyExc_TypeError, #name ": needs " #count " arguments"); return nullptr; } \
        const Entries &f = entries(self);                                                                \
        Args x(args);                                                                                    \
        void *const s = x.stream(args[nargs - 1]);                                                       \
        const Plan p(x);

KT_CALL(pack, 7)
    void *const *t = x.pointers(4, p.T), *const *b = x.pointers(5, p.nb);
    return finish(x, [&] { return f.pack(p.p, p.bucket, t, b, s); });
}

KT_CALL(reduce, 9)
    const int K = x.copies(4);
    const float *w = x.weights(6, K);
    void *const *in = x.pointers(5, (Py_ssize_t)p.nb * K), *const *out = x.pointers(7, p.nb);
    return finish(x, [&] { return f.reduce(p.p, p.bucket, in, K, w, out, s); });
}

KT_CALL(unpack, 8)
    const float scale = x.real(5);
    void *const *b = x.pointers(4, p.nb), *const *t = x.pointers(6, p.T);
    return finish(x, [&] { return f.unpack(p.p, p.bucket, b, scale, t, s); });
}

KT_CALL(fused, 11)
    const int K = x.copies(4);
    const float *w = x.weights(7, K);
    const float scale = x.real(8);
    void *const *in = x.pointers(5, p.T), *const *peers = x.pointers(6, (Py_ssize_t)p.nb * (K - 1)), *const *out = x.pointers(9, p.T);
    return finish(x, [&] { return f.fused(p.p, p.bucket, in, peers, K, w, scale, out, s); });
}

KT_CALL(sgd, 13)
    const float scale = x.real(5), lr = x.real(8), mu = x.real(9), wd = x.real(10);
    const int first = x.flag(11);
    void *const *b = x.pointers(4, p.nb), *const *params = x.pointers(6, p.T), *const *momenta = x.pointers(7, p.T);
    return finish(x, [&] { return f.sgd(p.p, p.bucket, b, scale, params, momenta, lr, mu, wd, first, s); });
}

KT_CALL(master, 14)
    const float scale = x.real(5), lr = x.real(9), mu = x.real(10), wd = x.real(11);
    const int first = x.flag(12);
    void *const *b = x.pointers(4, p.nb), *const *params = x.pointers(6, p.T), *const *momenta = x.pointers(7, p.T);
    void *const *models = x.pointers(8, p.T);
    return finish(x, [&] { return f.master(p.p, p.bucket, b, scale, params, momenta, models, lr, mu, wd, first, s); });
}

KT_CALL(fused_sgd, 17)
    const int K = x.copies(4);
    const float *w = x.weights(7, K);
    const float scale = x.real(8), lr = x.real(12), mu = x.real(13), wd = x.real(14);
    const int first = x.flag(15);
    void *const *in = x.pointers(5, p.T), *const *peers = x.pointers(6, (Py_ssize_t)p.nb * (K - 1));
    void *const *params = x.pointers(9, p.T), *const *momenta = x.pointers(10, p.T);
    void *const *models = x.a[11] == Py_None ? nullptr : x.pointers(11, p.T);
    return finish(x, [&] { return f.fused_sgd(p.p, p.bucket, in, peers, K, w, scale, params, momenta, models, lr, mu, wd, first, s); });
}

#define KT_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {KT_METHOD(pack), KT_METHOD(reduce), KT_METHOD(unpack), KT_METHOD(fused), KT_METHOD(sgd), KT_METHOD(master),
                         KT_METHOD(fused_sgd), {nullptr, nullptr, 0, nullptr}};

// Calls(addresses of kt_bucket_pack, kt_weighted_reduce, kt_bucket_unpack_scale, kt_fused_step, kt_bucket_unpack_sgd,
// kt_bucket_unpack_sgd_master, kt_fused_step_sgd)
PyObject *calls_new(PyTypeObject *type, PyObject *args, PyObject *)
{
    unsigned long long v[7];
    if (!PyArg_ParseTuple(args, "KKKKKKK", v, v + 1, v + 2, v + 3, v + 4, v + 5, v + 6)) return nullptr;
    Calls *c = reinterpret_cast<Calls *>(type->tp_alloc(type, 0));
    if (!c) return nullptr;
    c->f.pack = reinterpret_cast<decltype(c->f.pack)>(v[0]);
    c->f.reduce = reinterpret_cast<decltype(c->f.reduce)>(v[1]);
    c->f.unpack = reinterpret_cast<decltype(c->f.unpack)>(v[2]);
    c->f.fused = reinterpret_cast<decltype(c->f.fused)>(v[3]);
    c->f.sgd = reinterpret_cast<decltype(c->f.sgd)>(v[4]);
    c->f.master = reinterpret_cast<decltype(c->f.master)>(v[5]);
    c->f.fused_sgd = reinterpret_cast<decltype(c->f.fused_sgd)>(v[6]);
    return reinterpret_cast<PyObject *>(c);
}

PyTypeObject calls_type = {PyVarObject_HEAD_INIT(nullptr, 0)};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_kt_marshal", nullptr, -1, nullptr, nullptr, nullptr, nullptr, nullptr};

PyObject *attribute(const char *mod, const char *name)
{
    PyObject *m = PyImport_ImportModule(mod);
    PyObject *v = m ? PyObject_GetAttrString(m, name) : nullptr;
    Py_XDECREF(m);
    return v;
}

// What looks into a tensor here is inline code of torch's and Python's headers: the objects have to be those that it was
// compiled for.
bool built_for_these()
{
    const std::string python = std::to_string(PY_MAJOR_VERSION) + "." + std::to_string(PY_MINOR_VERSION) + ".";
    const std::string now = std::string(Py_GetVersion()).substr(0, std::strcspn(Py_GetVersion(), " "));
    PyObject *version = attribute("torch", "__version__");
    const char *torch_now = version ? PyUnicode_AsUTF8(version) : nullptr;
    if (!torch_now) return false;
    const bool same = !std::strcmp(torch_now, KT_TORCH_VERSION) && now.compare(0, python.size(), python) == 0;
    if (!same)
        PyErr_Format(PyExc_ImportError, "_kt_marshal.so was built for torch %s and Python %s* and not for torch %s and Python %s",
                     KT_TORCH_VERSION, python.c_str(), torch_now, now.c_str());
    Py_DECREF(version);
    return same;
}

}  // namespace

PyMODINIT_FUNC PyInit__kt_marshal(void)
{
    if (!built_for_these()) return nullptr;
    ctypes_array = attribute("ctypes", "Array");
    get_device = ctypes_array ? attribute("torch._C", "_cuda_getDevice") : nullptr;
    get_stream = get_device ? attribute("torch._C", "_cuda_getCurrentRawStream") : nullptr;
    cuda_stream = get_stream ? PyUnicode_InternFromString("cuda_stream") : nullptr;
    if (!cuda_stream) return nullptr;
    calls_type.tp_name = "_kt_marshal.Calls";
    calls_type.tp_basicsize = sizeof(Calls);
    calls_type.tp_flags = Py_TPFLAGS_DEFAULT;
    calls_type.tp_new = calls_new;
    calls_type.tp_methods = methods;
    if (PyType_Ready(&calls_type) < 0) return nullptr;
    PyObject *m = PyModule_Create(&module);
    if (!m) return nullptr;
    Py_INCREF(&calls_type);
    if (PyModule_AddObject(m, "Calls", reinterpret_cast<PyObject *>(&calls_type)) < 0) { Py_DECREF(m); return nullptr; }
    return m;
}
