// The product calls of the Python binding as native functions: cer_matmul, cser_matmul, cer_matmul_noalloc, csr_matmul.
//
// A batch-1 product of a small layer lasts 3.3 us on the GPU, and enqueueing it through ctypes took 7 us: the interpreter
// spent 4.5 us on attribute look-ups, ctypes' argument conversion and torch.cuda.current_stream() (which builds a Stream
// object), the library and the HIP launch 2.5 us.  The same checks and conversions through the C API take 0.5 us.  The
// module links to neither torch nor the library: the entry points' addresses are handed over by binding.py when it has
// loaded the library (`bind`), tensors are read through their Python attributes.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>

namespace {

using MatmulFn = int (*)(const void*, const float*, float*, int64_t, void*);

enum { kCer, kCser, kNoalloc, kCsr, kFunctions };
const char* const kNames[kFunctions] = {"cer_matmul", "cser_matmul", "cer_matmul_noalloc", "csr_matmul"};
MatmulFn g_fn[kFunctions] = {};
PyObject* g_load = nullptr;    // binding.lib: loads the library and calls bind()
PyObject* g_check = nullptr;   // binding._check(rc, name): raises for an error code
PyObject* g_stream = nullptr;  // binding._stream_ptr(None): the current torch stream, by torch's own path

PyObject *s_ptr, *s_is_cuda, *s_dtype, *s_itemsize, *s_is_contiguous, *s_data_ptr, *s_cuda_stream;
PyObject* g_word_dtype = nullptr;  // a dtype seen to be 4 bytes wide (torch.float32)
PyObject* g_get_device = nullptr;  // torch._C._cuda_getDevice, ._cuda_getCurrentRawStream once torch has initialised the device
PyObject* g_raw_stream = nullptr;

bool address_of(PyObject* o, void** out) {  // an int (or None) as ctypes' c_void_p takes it
    if (o == Py_None) {
        *out = nullptr;
        return true;
    }
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);
    if (v == (unsigned long long)-1 && PyErr_Occurred()) return false;
    *out = reinterpret_cast<void*>((uintptr_t)v);
    return true;
}

bool attribute_address(PyObject* o, PyObject* name, void** out) {
    PyObject* v = PyObject_GetAttr(o, name);
    if (!v) return false;
    const bool ok = address_of(v, out);
    Py_DECREF(v);
    return ok;
}

int is_true(PyObject* v) {  // steals v; -1: error
    if (!v) return -1;
    const int t = v == Py_True ? 1 : (v == Py_False ? 0 : PyObject_IsTrue(v));
    Py_DECREF(v);
    return t;
}

// A raw address, or a contiguous tensor of 4-byte elements in device memory.
bool device_pointer(PyObject* t, void** out) {
    if (PyLong_Check(t)) return address_of(t, out);
    int good = is_true(PyObject_GetAttr(t, s_is_cuda));
    if (good < 0) return false;
    if (good) {
        PyObject* dt = PyObject_GetAttr(t, s_dtype);
        if (!dt) return false;
        if (dt != g_word_dtype) {
            PyObject* size = PyObject_GetAttr(dt, s_itemsize);
            if (!size) {
                Py_DECREF(dt);
                return false;
            }
            good = PyLong_Check(size) && PyLong_AsLong(size) == 4;
            Py_DECREF(size);
            if (good && !g_word_dtype) {
                g_word_dtype = dt;
                Py_INCREF(dt);
            }
        }
        Py_DECREF(dt);
    }
    if (good) {
        good = is_true(PyObject_CallMethodNoArgs(t, s_is_contiguous));
        if (good < 0) return false;
    }
    if (!good) {
        PyErr_SetString(PyExc_ValueError, "expected a contiguous fp32 tensor in device memory");
        return false;
    }
    PyObject* p = PyObject_CallMethodNoArgs(t, s_data_ptr);
    if (!p) return false;
    const bool ok = address_of(p, out);
    Py_DECREF(p);
    return ok;
}

// None: the current torch stream of the current device; an int; or an object with .cuda_stream.
bool stream_pointer(PyObject* s, void** out) {
    if (s && s != Py_None) return PyLong_Check(s) ? address_of(s, out) : attribute_address(s, s_cuda_stream, out);
    PyObject* v;
    if (g_raw_stream) {
        PyObject* dev = PyObject_CallNoArgs(g_get_device);
        if (!dev) return false;
        v = PyObject_CallOneArg(g_raw_stream, dev);
        Py_DECREF(dev);
    } else {
        v = PyObject_CallOneArg(g_stream, Py_None);  // initialises torch's side of the device on first use
        if (v) {
            PyObject* c = PyImport_ImportModule("torch._C");
            PyObject* get = c ? PyObject_GetAttrString(c, "_cuda_getDevice") : nullptr;
            PyObject* raw = get ? PyObject_GetAttrString(c, "_cuda_getCurrentRawStream") : nullptr;
            Py_XDECREF(c);
            if (raw) {
                g_get_device = get;
                g_raw_stream = raw;
            } else {
                PyErr_Clear();
                Py_XDECREF(get);
            }
        }
    }
    if (!v) return false;
    const bool ok = address_of(v, out);
    Py_DECREF(v);
    return ok;
}

const char* const kArgNames[5] = {"h", "X", "Y", "batch", "stream"};

PyObject* product(int which, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    PyObject* a[5] = {};
    const Py_ssize_t nkw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    if (nargs > 5) return PyErr_Format(PyExc_TypeError, "%s() takes from 4 to 5 positional arguments but %zd were given", kNames[which], nargs);
    for (Py_ssize_t i = 0; i < nargs; ++i) a[i] = args[i];
    for (Py_ssize_t k = 0; k < nkw; ++k) {
        PyObject* name = PyTuple_GET_ITEM(kwnames, k);
        int i = 0;
        while (i < 5 && PyUnicode_CompareWithASCIIString(name, kArgNames[i]) != 0) ++i;
        if (i == 5) return PyErr_Format(PyExc_TypeError, "%s() got an unexpected keyword argument '%U'", kNames[which], name);
        if (a[i]) return PyErr_Format(PyExc_TypeError, "%s() got multiple values for argument '%s'", kNames[which], kArgNames[i]);
        a[i] = args[nargs + k];
    }
    for (int i = 0; i < 4; ++i)
        if (!a[i]) return PyErr_Format(PyExc_TypeError, "%s() missing required argument '%s'", kNames[which], kArgNames[i]);
    if (!g_fn[which]) {  // the library is not loaded yet
        PyObject* l = g_load ? PyObject_CallNoArgs(g_load) : PyErr_Format(PyExc_RuntimeError, "binding.py has not set up its native part");
        if (!l) return nullptr;
        Py_DECREF(l);
        if (!g_fn[which]) return PyErr_Format(PyExc_RuntimeError, "%s is not bound", kNames[which]);
    }
    void *h, *X, *Y, *s;
    if (!attribute_address(a[0], s_ptr, &h) || !device_pointer(a[1], &X) || !device_pointer(a[2], &Y)) return nullptr;
    if (PyFloat_Check(a[3])) return PyErr_Format(PyExc_TypeError, "batch must be an integer");
    const int64_t batch = (int64_t)PyLong_AsUnsignedLongLongMask(a[3]);
    if (batch == -1 && PyErr_Occurred()) return nullptr;
    if (!stream_pointer(a[4], &s)) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_fn[which](h, static_cast<const float*>(X), static_cast<float*>(Y), batch, s);
    Py_END_ALLOW_THREADS
    if (rc != 0) {
        PyObject* r = PyObject_CallFunction(g_check, "is", rc, kNames[which]);
        if (!r) return nullptr;
        Py_DECREF(r);
    }
    Py_RETURN_NONE;
}

template <int kWhich>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    return product(kWhich, args, nargs, kwnames);
}

// setup(load, check, stream): binding.py's functions of these roles
PyObject* setup(PyObject*, PyObject* args) {
    PyObject *load, *check, *stream;
    if (!PyArg_ParseTuple(args, "OOO", &load, &check, &stream)) return nullptr;
    Py_INCREF(load);
    Py_INCREF(check);
    Py_INCREF(stream);
    Py_XSETREF(g_load, load);
    Py_XSETREF(g_check, check);
    Py_XSETREF(g_stream, stream);
    Py_RETURN_NONE;
}

// bind(addresses): where the loaded library has the functions of kNames
PyObject* bind(PyObject*, PyObject* args) {
    unsigned long long at[kFunctions];
    if (!PyArg_ParseTuple(args, "KKKK", &at[0], &at[1], &at[2], &at[3])) return nullptr;
    for (int i = 0; i < kFunctions; ++i) g_fn[i] = reinterpret_cast<MatmulFn>((uintptr_t)at[i]);
    Py_RETURN_NONE;
}

#define CER_ENTRY(name, which)                                                                                        \
    {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(entry<which>)), METH_FASTCALL | METH_KEYWORDS, \
     name "(h, X, Y, batch, stream=None)\n--\n\n"}

PyMethodDef g_methods[] = {
    CER_ENTRY("cer_matmul", kCer),
    CER_ENTRY("cser_matmul", kCser),
    CER_ENTRY("cer_matmul_noalloc", kNoalloc),
    CER_ENTRY("csr_matmul", kCsr),
    {"setup", setup, METH_VARARGS, nullptr},
    {"bind", bind, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_cerpy", "Native product calls of the binding.", -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__cerpy(void) {
    s_ptr = PyUnicode_InternFromString("ptr");
    s_is_cuda = PyUnicode_InternFromString("is_cuda");
    s_dtype = PyUnicode_InternFromString("dtype");
    s_itemsize = PyUnicode_InternFromString("itemsize");
    s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    return PyModule_Create(&g_module);
}
