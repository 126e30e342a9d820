// The hot half of the Python binding: the device calls of a plan with lists of tensors or marshalled pointer
// arrays, straight to the C ABI.  Only the plainest forms are taken here (lists and tuples of plain tensors, c_void_p and c_float
// arrays, lists of floats, streams that are None or an int); for every other form a call returns None and
// the ctypes half of the binding, which raises every error of marshalling, makes the call.
//
// On small sets the host decides: a pack, reduce and unpack of 158 tensors handed over as lists asked 323 tensors
// for their addresses through Python and copied them twice, 34.5 us a step where the kernels take 18 (18.5 now, the kernels
// alone); three calls on 6 tensors with marshalled arrays took 14.8 us (12.5), where three bare launches take 8.
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
struct Args {
    PyObject *const *a;
    int at = 0;
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

    // an int that fits a C int
    int integer()
    {
        if (!ok || !PyLong_Check(a[at])) return fail(), 0;
        int over = 0;
        const long v = PyLong_AsLongAndOverflow(a[at++], &over);
        if (over || v != (int)v) return fail(), 0;
        return (int)v;
    }
    void *address(PyObject *x)
    {
        if (!PyLong_CheckExact(x)) return fail(), nullptr;
        void *p = PyLong_AsVoidPtr(x);
        if (!p && PyErr_Occurred()) fail();
        return p;
    }
    float real()
    {
        if (!ok) return 0.0f;
        if (PyFloat_CheckExact(a[at])) return (float)PyFloat_AS_DOUBLE(a[at++]);
        if (!PyLong_CheckExact(a[at])) return fail(), 0.0f;
        const double v = PyLong_AsDouble(a[at++]);
        if (v == -1.0 && PyErr_Occurred()) fail();
        return (float)v;
    }
    int flag()
    {
        if (!ok || !PyBool_Check(a[at])) return fail(), 0;
        return a[at++] == Py_True;
    }

    // `want` elements of a ctypes array whose items are of struct code `code`; marshal() pads an empty list to one entry
    void *array(Py_ssize_t want, char code, Py_ssize_t size)
    {
        PyObject *x = a[at];
        if (!PyObject_TypeCheck(x, reinterpret_cast<PyTypeObject *>(ctypes_array))) return fail(), nullptr;
        Py_buffer &b = held[nheld];
        if (PyObject_GetBuffer(x, &b, PyBUF_FORMAT | PyBUF_ND) != 0) return fail(), nullptr;
        ++nheld;
        const char *f = b.format ? b.format : "";
        if (*f == '<' || *f == '=' || *f == '@') ++f;
        if (b.ndim != 1 || b.itemsize != size || f[0] != code || f[1] || b.shape[0] != (want > 0 ? want : 1)) return fail(), nullptr;
        ++at;
        return b.buf;
    }
    // `want` device addresses
    void *const *pointers(Py_ssize_t want)
    {
        if (!ok) return nullptr;
        PyObject *x = a[at];
        if (!PyList_CheckExact(x) && !PyTuple_CheckExact(x)) return static_cast<void *const *>(array(want, 'P', sizeof(void *)));
        const Py_ssize_t n = PySequence_Fast_GET_SIZE(x);
        if (n != want || at::impl::torch_function_mode_enabled()) return fail(), nullptr;
        static thread_local std::vector<void *> tables[MAX_ARRAYS];      // kept: no allocation per call
        try {
            std::vector<void *> &t = tables[arrays++];
            t.resize(n > 0 ? n : 1);
            for (Py_ssize_t i = 0; i < n; ++i) {
                PyObject *item = PySequence_Fast_GET_ITEM(x, i);
                if (!THPVariable_CheckExact(item)) return fail(), nullptr;
                t[i] = THPVariable_Unpack(item).data_ptr();
            }
            ++at;
            return t.data();
        } catch (...) {         // a tensor without memory of its own, say: asked again through Python, it raises its own error
            return fail(), nullptr;
        }
    }
    const float *weights(int K)
    {
        if (!ok) return nullptr;
        PyObject *x = a[at];
        if (x == Py_None) {             // the plan's device-resident ones
            ++at;
            return nullptr;
        }
        if (!PyList_CheckExact(x) && !PyTuple_CheckExact(x)) return static_cast<const float *>(array(K, 'f', sizeof(float)));
        if (PySequence_Fast_GET_SIZE(x) != K) return fail(), nullptr;
        for (int k = 0; k < K; ++k) {
            PyObject *item = PySequence_Fast_GET_ITEM(x, k);
            if (!PyFloat_CheckExact(item)) return fail(), nullptr;
            w[k] = (float)PyFloat_AS_DOUBLE(item);
        }
        ++at;
        return w;
    }
    // Asked for first: it runs Python, and with it whatever the collector finds to finalize.
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
        return address(x);
    }
    int copies()
    {
        const int K = integer();
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
        p = static_cast<kt_plan *>(x.address(x.a[x.at++]));
        T = x.integer();
        nb = x.integer();
        bucket = x.integer();
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
    void *const *t = x.pointers(p.T), *const *b = x.pointers(p.nb);
    return finish(x, [&] { return f.pack(p.p, p.bucket, t, b, s); });
}

KT_CALL(reduce, 9)
    const int K = x.copies();
    void *const *in = x.pointers((Py_ssize_t)p.nb * K);
    const float *w = x.weights(K);
    void *const *out = x.pointers(p.nb);
    return finish(x, [&] { return f.reduce(p.p, p.bucket, in, K, w, out, s); });
}

KT_CALL(unpack, 8)
    void *const *b = x.pointers(p.nb);
    const float scale = x.real();
    void *const *t = x.pointers(p.T);
    return finish(x, [&] { return f.unpack(p.p, p.bucket, b, scale, t, s); });
}

KT_CALL(fused, 11)
    const int K = x.copies();
    void *const *in = x.pointers(p.T), *const *peers = x.pointers((Py_ssize_t)p.nb * (K - 1));
    const float *w = x.weights(K);
    const float scale = x.real();
    void *const *out = x.pointers(p.T);
    return finish(x, [&] { return f.fused(p.p, p.bucket, in, peers, K, w, scale, out, s); });
}

KT_CALL(sgd, 13)
    void *const *b = x.pointers(p.nb);
    const float scale = x.real();
    void *const *params = x.pointers(p.T), *const *momenta = x.pointers(p.T);
    const float lr = x.real(), mu = x.real(), wd = x.real();
    const int first = x.flag();
    return finish(x, [&] { return f.sgd(p.p, p.bucket, b, scale, params, momenta, lr, mu, wd, first, s); });
}

KT_CALL(master, 14)
    void *const *b = x.pointers(p.nb);
    const float scale = x.real();
    void *const *params = x.pointers(p.T), *const *momenta = x.pointers(p.T), *const *models = x.pointers(p.T);
    const float lr = x.real(), mu = x.real(), wd = x.real();
    const int first = x.flag();
    return finish(x, [&] { return f.master(p.p, p.bucket, b, scale, params, momenta, models, lr, mu, wd, first, s); });
}

KT_CALL(fused_sgd, 17)
    const int K = x.copies();
    void *const *in = x.pointers(p.T), *const *peers = x.pointers((Py_ssize_t)p.nb * (K - 1));
    const float *w = x.weights(K);
    const float scale = x.real();
    void *const *params = x.pointers(p.T), *const *momenta = x.pointers(p.T), *const *models = nullptr;
    if (x.ok && x.a[x.at] == Py_None) ++x.at; else models = x.pointers(p.T);
    const float lr = x.real(), mu = x.real(), wd = x.real();
    const int first = x.flag();
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
    if (!get_stream) return nullptr;
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
