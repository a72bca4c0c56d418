// The calls a program makes once per layer or per map, as Python functions over the C ABI of include/ts.h.
// What bounds small layers and the coarse levels of a network is the host: marshalled by ctypes such a call cost
// 11 us, of which 2 were the library's own (the stream of the calling thread 3.2, tensor descriptors 3, the output
// tensor 1.8).  Here the tensors' own fields are read.  The library is entered without the interpreter lock.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/Functions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/ts.h"

namespace {

PyObject *g_error = nullptr;   // binding.TsError

PyObject *raise_ts(int rc) {
    PyObject *e = PyObject_CallFunction(g_error, "is", rc, ts_last_error());
    if (e) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    return nullptr;
}

// A tensor as the library sees it; false with a Python error set.
bool describe(PyObject *obj, ts_tensor *d) {
    if (!THPVariable_Check(obj)) {
        PyErr_SetString(PyExc_TypeError, "expected a tensor");
        return false;
    }
    const at::Tensor &t = THPVariable_Unpack(obj);
    if (!t.is_cuda() || !t.is_contiguous() || t.dim() < 1) {
        PyErr_SetString(PyExc_ValueError, "tensors must be contiguous device tensors");
        return false;
    }
    if (t.scalar_type() == at::kHalf) d->dtype = TS_F16;
    else if (t.scalar_type() == at::kFloat) d->dtype = TS_F32;
    else {
        PyObject *dt = PyObject_GetAttrString(obj, "dtype");
        if (dt) PyErr_Format(PyExc_TypeError, "unsupported dtype %S", dt);
        Py_XDECREF(dt);
        return false;
    }
    d->data = t.numel() ? t.data_ptr() : nullptr;
    d->rows = t.size(0);
    d->cols = (int32_t)t.size(-1);
    return true;
}

template <class T>
bool pointer(PyObject *obj, T **p) {
    *p = static_cast<T *>(PyLong_AsVoidPtr(obj));
    return !PyErr_Occurred();
}

bool integer(PyObject *obj, long long *v) {   // what int() takes
    PyObject *as_int = PyNumber_Long(obj);
    if (!as_int) return false;
    *v = PyLong_AsLongLong(as_int);
    Py_DECREF(as_int);
    return !(*v == -1 && PyErr_Occurred());
}

bool device_vector(PyObject *obj, const void **p) {
    if (!THPVariable_Check(obj)) {
        PyErr_SetString(PyExc_TypeError, "bias must be a tensor");
        return false;
    }
    *p = THPVariable_Unpack(obj).data_ptr();
    return true;
}

inline void *current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

bool nargs_are(Py_ssize_t got, Py_ssize_t want) {
    if (got == want) return true;
    PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", want, got);
    return false;
}

// What the layer calls share: the output tensor, made here unless the caller brought one.
struct Output {
    at::Tensor made;
    PyObject *given;
    ts_tensor d;
    bool open(PyObject *out, PyObject *feats, const ts_kmap *kmap, int64_t cols) {
        given = out;
        if (out != Py_None) return describe(out, &d);
        const at::Tensor &f = THPVariable_Unpack(feats);
        int64_t rows;
        void *const st = current_stream();
        Py_BEGIN_ALLOW_THREADS
        ts_set_stream(st);              // counting may build the map
        rows = ts_kmap_num_out(kmap);   // may wait for the build to say
        Py_END_ALLOW_THREADS
        if (rows < 0) {
            raise_ts((int)rows);
            return false;
        }
        made = at::empty({rows, cols}, f.options());
        d.data = rows ? made.data_ptr() : nullptr;
        d.rows = rows;
        d.cols = (int32_t)cols;
        d.dtype = f.scalar_type() == at::kHalf ? TS_F16 : TS_F32;
        return true;
    }
    PyObject *close() {
        if (given == Py_None) return THPVariable_Wrap(std::move(made));
        Py_INCREF(given);
        return given;
    }
};

// conv_prepared(feats, feats2 or None, weights handle, c_out, map handle, bias or None, residual or None, relu, out or None)
PyObject *conv_prepared(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (!nargs_are(n, 9)) return nullptr;
    ts_tensor f, f2, r;
    const void *bias = nullptr;
    ts_weights *w;
    ts_kmap *m;
    long long c_out;
    const int relu = PyObject_IsTrue(a[7]);
    if (!integer(a[3], &c_out) || relu < 0 || !pointer(a[2], &w) || !pointer(a[4], &m)) return nullptr;
    const bool two = a[1] != Py_None, res = a[6] != Py_None;
    if (!describe(a[0], &f) || (two && !describe(a[1], &f2)) || (res && !describe(a[6], &r))) return nullptr;
    if (a[5] != Py_None && !device_vector(a[5], &bias)) return nullptr;
    Output o;
    if (!o.open(a[8], a[0], m, c_out)) return nullptr;
    int rc;
    void *const st = current_stream();
    Py_BEGIN_ALLOW_THREADS
    ts_set_stream(st);
    rc = two ? ts_sparse_conv_prepared2(&f, &f2, w, m, bias, res ? &r : nullptr, relu, &o.d)
             : ts_sparse_conv_prepared(&f, w, m, bias, res ? &r : nullptr, relu, &o.d);
    Py_END_ALLOW_THREADS
    if (rc != TS_OK) return raise_ts(rc);
    return o.close();
    END_HANDLE_TH_ERRORS
}

// conv(feats, weights, map handle, out or None, dataflow)
PyObject *conv(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (!nargs_are(n, 5)) return nullptr;
    ts_tensor f, w;
    ts_kmap *m;
    long long dataflow;
    if (!integer(a[4], &dataflow) || !pointer(a[2], &m)) return nullptr;
    if (!describe(a[0], &f)) return nullptr;
    if (!THPVariable_Check(a[1]) || THPVariable_Unpack(a[1]).dim() != 3) {
        PyErr_SetString(PyExc_ValueError, "weights must be [K^3, C_in, C_out]");
        return nullptr;
    }
    if (!describe(a[1], &w)) return nullptr;
    w.rows *= THPVariable_Unpack(a[1]).size(1);
    Output o;
    if (!o.open(a[3], a[0], m, w.cols)) return nullptr;
    int rc;
    void *const st = current_stream();
    Py_BEGIN_ALLOW_THREADS
    ts_set_stream(st);
    rc = ts_sparse_conv_ex(&f, &w, m, &o.d, (int)dataflow);
    Py_END_ALLOW_THREADS
    if (rc != TS_OK) return raise_ts(rc);
    return o.close();
    END_HANDLE_TH_ERRORS
}

PyObject *handle_or_error(int rc, const ts_kmap *m) { return rc == TS_OK ? PyLong_FromVoidPtr(const_cast<ts_kmap *>(m)) : raise_ts(rc); }

// build(coords, kernel size, stride, transposed, wait) -> map handle
PyObject *build(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (!nargs_are(n, 5)) return nullptr;
    long long K, s;
    const int tr = PyObject_IsTrue(a[3]), wait = PyObject_IsTrue(a[4]);
    if (!integer(a[1], &K) || !integer(a[2], &s) || tr < 0 || wait < 0) return nullptr;
    if (!THPVariable_Check(a[0])) {
        PyErr_SetString(PyExc_TypeError, "coords must be a tensor");
        return nullptr;
    }
    const at::Tensor &c = THPVariable_Unpack(a[0]);
    if (c.scalar_type() != at::kInt || c.dim() != 2 || c.size(1) != 4) {
        PyErr_SetString(PyExc_ValueError, "coords must be int32 [N,4]");
        return nullptr;
    }
    if (!c.is_cuda() || !c.is_contiguous()) {
        PyErr_SetString(PyExc_ValueError, "coords must be a contiguous device tensor");
        return nullptr;
    }
    const int32_t *data = c.numel() ? static_cast<const int32_t *>(c.data_ptr()) : nullptr;
    const int64_t rows = c.size(0);
    ts_kmap *m = nullptr;
    int rc;
    void *const st = current_stream();
    Py_BEGIN_ALLOW_THREADS
    ts_set_stream(st);
    rc = wait ? ts_build_kmap(data, rows, (int)K, (int)s, tr, &m) : ts_build_kmap_async(data, rows, (int)K, (int)s, tr, &m);
    Py_END_ALLOW_THREADS
    return handle_or_error(rc, m);
    END_HANDLE_TH_ERRORS
}

PyObject *identity(PyObject *, PyObject *arg) {
    HANDLE_TH_ERRORS
    long long n;
    if (!integer(arg, &n)) return nullptr;
    ts_kmap *m = nullptr;
    int rc;
    void *const st = current_stream();
    Py_BEGIN_ALLOW_THREADS
    ts_set_stream(st);
    rc = ts_identity_kmap(n, &m);
    Py_END_ALLOW_THREADS
    return handle_or_error(rc, m);
    END_HANDLE_TH_ERRORS
}

PyObject *transpose(PyObject *, PyObject *arg) {
    HANDLE_TH_ERRORS
    ts_kmap *f, *m = nullptr;
    if (!pointer(arg, &f)) return nullptr;
    int rc;
    void *const st = current_stream();
    Py_BEGIN_ALLOW_THREADS
    ts_set_stream(st);
    rc = ts_kmap_transpose(f, &m);
    Py_END_ALLOW_THREADS
    return handle_or_error(rc, m);
    END_HANDLE_TH_ERRORS
}

PyObject *prepare(PyObject *, PyObject *arg) {
    HANDLE_TH_ERRORS
    ts_kmap *m;
    if (!pointer(arg, &m)) return nullptr;
    int rc;
    void *const st = current_stream();
    Py_BEGIN_ALLOW_THREADS
    ts_set_stream(st);
    rc = ts_kmap_prepare(m);
    Py_END_ALLOW_THREADS
    if (rc != TS_OK) return raise_ts(rc);
    Py_RETURN_NONE;
    END_HANDLE_TH_ERRORS
}

PyObject *out_coords(PyObject *, PyObject *arg) {
    HANDLE_TH_ERRORS
    ts_kmap *m;
    if (!pointer(arg, &m)) return nullptr;
    int64_t rows;
    void *const st = current_stream();
    Py_BEGIN_ALLOW_THREADS
    ts_set_stream(st);
    rows = ts_kmap_num_out(m);
    Py_END_ALLOW_THREADS
    if (rows < 0) return raise_ts((int)rows);
    at::Tensor dst = at::empty({rows, 4}, at::TensorOptions().dtype(at::kInt).device(at::kCUDA));
    int rc;
    int32_t *const p = rows ? static_cast<int32_t *>(dst.data_ptr()) : nullptr;
    Py_BEGIN_ALLOW_THREADS
    ts_set_stream(st);
    rc = ts_kmap_out_coords(m, p);
    Py_END_ALLOW_THREADS
    if (rc != TS_OK) return raise_ts(rc);
    return THPVariable_Wrap(std::move(dst));
    END_HANDLE_TH_ERRORS
}

PyObject *use_current_stream(PyObject *, PyObject *) {
    HANDLE_TH_ERRORS
    ts_set_stream(current_stream());
    Py_RETURN_NONE;
    END_HANDLE_TH_ERRORS
}

PyObject *set_error(PyObject *, PyObject *cls) {
    Py_INCREF(cls);
    Py_XDECREF(g_error);
    g_error = cls;
    Py_RETURN_NONE;
}

PyMethodDef g_methods[] = {
    {"conv_prepared", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(conv_prepared)), METH_FASTCALL, nullptr},
    {"conv", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(conv)), METH_FASTCALL, nullptr},
    {"build", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(build)), METH_FASTCALL, nullptr},
    {"identity", identity, METH_O, nullptr},
    {"transpose", transpose, METH_O, nullptr},
    {"prepare", prepare, METH_O, nullptr},
    {"out_coords", out_coords, METH_O, nullptr},
    {"use_current_stream", use_current_stream, METH_NOARGS, nullptr},
    {"set_error", set_error, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_native", "Per-layer and per-map calls into libts.so.", -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&g_module); }
