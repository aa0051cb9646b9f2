// CPython module `_call`: the entry points of a decode loop without the interpreter's share of a call.
//
// A step issues two launches of about 2.3 us of host time each; the Python binding in front of them (a check, a pointer object and a
// conversion per argument) took 3 to 5 us more, so that the smallest steps waited for it.  Here the checks read the tensors
// themselves.  A call whose arguments are not all of the plain form (device tensors, or DeviceArg, of the right type) returns None and the
// general binding takes it, with its errors; the GIL is released while the library works, as ctypes does.
#include <torch/csrc/autograd/python_variable.h>

#include <structmember.h>
#include <torch/version.h>

#include <cstdint>
#include <cstring>

#include "../../include/louver.h"

namespace {

// Base of binding.DeviceArg: a device tensor checked and marshalled once.  Python fields as they were (tensor, ptr, dtype, shape), and
// what the calls here read.
struct Arg {
    PyObject_HEAD
    PyObject *tensor, *ptr, *dtype, *shape;
    void *address;
    int scalar_type;
    int64_t dims[4];
    int n_dims;
};

struct Held {   // an argument's pointer and the sizes the calls ask for
    void *p;
    const int64_t *dims;
    int n_dims;
};

bool is_plain(PyObject *o, const at::Tensor *&t) {
    if (!THPVariable_CheckExact(o)) return false;   // subclasses keep their own ways
    t = &THPVariable_Unpack(o);
    return t->is_cuda() && t->layout() == at::kStrided && t->has_storage() && t->is_contiguous();
}

extern PyTypeObject ArgType;

// `want`: a scalar type, or -1 for any.
bool held(PyObject *o, int want, Held &h) {
    if (PyObject_TypeCheck(o, &ArgType)) {
        const Arg *a = reinterpret_cast<const Arg *>(o);
        if (!a->tensor || (want >= 0 && a->scalar_type != want)) return false;
        h = {a->address, a->dims, a->n_dims};
        return true;
    }
    const at::Tensor *t = nullptr;
    if (!is_plain(o, t) || (want >= 0 && (int)t->scalar_type() != want)) return false;
    h = {t->data_ptr(), t->sizes().data(), (int)t->dim()};
    return true;
}

PyObject *s_value;   // "value"

// The address in a ctypes pointer object (None and 0 are NULL).
bool address(PyObject *o, void *&p) {
    PyObject *v = PyObject_GetAttr(o, s_value);
    if (!v) {
        PyErr_Clear();
        return false;
    }
    if (v == Py_None) p = nullptr;
    else p = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

constexpr int F32 = (int)at::kFloat, I32 = (int)at::kInt;

// The library's functions, handed over by the binding once it has loaded the library.
struct {
    decltype(&lvr_decode_step) decode_step;
    decltype(&lvr_append_decode_step) append_decode_step;
    decltype(&lvr_query) query;
    decltype(&lvr_sparse_attention) sparse_attention;
    decltype(&lvr_sparse_attention_static) sparse_attention_static;
    decltype(&lvr_dense_attention) dense_attention;
} lib;

// Runs `call` (which returns an error code) without the GIL.
template <typename F>
PyObject *result_of(F call) {
    int code;
    Py_BEGIN_ALLOW_THREADS
    code = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(code);
}

#define LVR_NOT_PLAIN(COND) do { if (!(COND)) Py_RETURN_NONE; } while (0)
#define LVR_PLAIN(BODY)                             \
    try {                                           \
        BODY                                        \
    } catch (...) {   /* a tensor without memory */ \
        PyErr_Clear();                              \
        Py_RETURN_NONE;                             \
    }

// (h, q, tau, out, out_idx, out_count, stream)
PyObject *decode_step(PyObject *, PyObject *const *a, Py_ssize_t n) {
    void *h, *st;
    Held q, tau, out, idx, count;
    LVR_PLAIN(LVR_NOT_PLAIN(n == 7 && lib.decode_step && address(a[0], h) && held(a[1], F32, q) && held(a[2], F32, tau) && held(a[3], F32, out) &&
                            held(a[4], I32, idx) && idx.n_dims > 0 && held(a[5], I32, count) && address(a[6], st));)
    const int64_t cap = idx.dims[idx.n_dims - 1];
    return result_of([&] {
        return lib.decode_step(static_cast<lvr_index *>(h), (const float *)q.p, (const float *)tau.p, (float *)out.p, (int32_t *)idx.p,
                               (int32_t *)count.p, cap, st);
    });
}

// (h, k_new, v_new, q, tau, out, out_idx, out_count, stream)
PyObject *append_decode_step(PyObject *, PyObject *const *a, Py_ssize_t n) {
    void *h, *st;
    Held k, v, q, tau, out, idx, count;
    LVR_PLAIN(LVR_NOT_PLAIN(n == 9 && lib.append_decode_step && address(a[0], h) && held(a[1], -1, k) && k.n_dims > 2 && held(a[2], -1, v) &&
                            held(a[3], F32, q) && held(a[4], F32, tau) && held(a[5], F32, out) && held(a[6], I32, idx) && idx.n_dims > 0 &&
                            held(a[7], I32, count) && address(a[8], st));)
    const int64_t cap = idx.dims[idx.n_dims - 1], m = k.dims[2];
    return result_of([&] {
        return lib.append_decode_step(static_cast<lvr_index *>(h), k.p, v.p, m, (const float *)q.p, (const float *)tau.p, (float *)out.p,
                                      (int32_t *)idx.p, (int32_t *)count.p, cap, st);
    });
}

// (h, q, tau, out_idx, out_count, stream)
PyObject *query(PyObject *, PyObject *const *a, Py_ssize_t n) {
    void *h, *st;
    Held q, tau, idx, count;
    LVR_PLAIN(LVR_NOT_PLAIN(n == 6 && lib.query && address(a[0], h) && held(a[1], F32, q) && held(a[2], F32, tau) && held(a[3], I32, idx) &&
                            idx.n_dims > 0 && held(a[4], I32, count) && address(a[5], st));)
    const int64_t cap = idx.dims[idx.n_dims - 1];
    return result_of([&] {
        return lib.query(static_cast<lvr_index *>(h), (const float *)q.p, (const float *)tau.p, (int32_t *)idx.p, (int32_t *)count.p, cap, st);
    });
}

// (h, q, idx, count, out, stream)
PyObject *sparse_attention(PyObject *, PyObject *const *a, Py_ssize_t n) {
    void *h, *st;
    Held q, idx, count, out;
    LVR_PLAIN(LVR_NOT_PLAIN(n == 6 && lib.sparse_attention && address(a[0], h) && held(a[1], F32, q) && held(a[2], I32, idx) && idx.n_dims > 0 &&
                            held(a[3], I32, count) && held(a[4], F32, out) && address(a[5], st));)
    const int64_t cap = idx.dims[idx.n_dims - 1];
    return result_of([&] {
        return lib.sparse_attention(static_cast<lvr_index *>(h), (const float *)q.p, (const int32_t *)idx.p, (const int32_t *)count.p, cap,
                                    (float *)out.p, st);
    });
}

// (h, q, out, stream)
PyObject *dense_attention(PyObject *, PyObject *const *a, Py_ssize_t n) {
    void *h, *st;
    Held q, out;
    LVR_PLAIN(LVR_NOT_PLAIN(n == 4 && lib.dense_attention && address(a[0], h) && held(a[1], F32, q) && held(a[2], F32, out) && address(a[3], st));)
    return result_of([&] { return lib.dense_attention(static_cast<lvr_index *>(h), (const float *)q.p, (float *)out.p, st); });
}

// (K, V, q, idx, count, out, scale, stream): K and V tensors of one shape [batch][n_kv_heads][n][128] and one type
PyObject *sparse_attention_static(PyObject *, PyObject *const *a, Py_ssize_t n) {
    void *st;
    Held q, idx, count, out;
    const at::Tensor *K = nullptr, *V = nullptr;
    double scale = 0.0;
    void *kp = nullptr, *vp = nullptr;
    LVR_PLAIN(
        LVR_NOT_PLAIN(n == 8 && lib.sparse_attention_static && is_plain(a[0], K) && is_plain(a[1], V) && K->dim() == 4 && K->sizes() == V->sizes() &&
                      K->scalar_type() == V->scalar_type() && (K->scalar_type() == at::kBFloat16 || K->scalar_type() == at::kFloat) &&
                      held(a[2], F32, q) && q.n_dims > 1 && held(a[3], I32, idx) && idx.n_dims > 0 && held(a[4], I32, count) &&
                      held(a[5], F32, out) && PyFloat_CheckExact(a[6]) && address(a[7], st));
        scale = PyFloat_AS_DOUBLE(a[6]);
        kp = K->data_ptr();
        vp = V->data_ptr();)
    const int64_t cap = idx.dims[idx.n_dims - 1];
    const int32_t type = K->scalar_type() == at::kBFloat16 ? LVR_BF16 : LVR_F32;
    const int64_t batch = K->size(0), heads = K->size(1), rows = K->size(2), hq = q.dims[1];
    LVR_NOT_PLAIN(batch <= INT32_MAX && heads <= INT32_MAX && hq <= INT32_MAX);
    return result_of([&] {
        return lib.sparse_attention_static(kp, vp, rows, type, (int32_t)batch, (int32_t)hq, (int32_t)heads, (float)scale, (const float *)q.p,
                                           (const int32_t *)idx.p, (const int32_t *)count.p, cap, (float *)out.p, st);
    });
}

// bind(name, address): the library's function of that name
PyObject *bind(PyObject *, PyObject *args) {
    const char *name;
    unsigned long long at;
    if (!PyArg_ParseTuple(args, "sK", &name, &at)) return nullptr;
    struct { const char *name; void **slot; } all[] = {
        {"lvr_decode_step", (void **)&lib.decode_step}, {"lvr_append_decode_step", (void **)&lib.append_decode_step},
        {"lvr_query", (void **)&lib.query}, {"lvr_sparse_attention", (void **)&lib.sparse_attention},
        {"lvr_sparse_attention_static", (void **)&lib.sparse_attention_static}, {"lvr_dense_attention", (void **)&lib.dense_attention}};
    for (auto &f : all)
        if (!strcmp(f.name, name)) {
            *f.slot = (void *)(uintptr_t)at;
            Py_RETURN_NONE;
        }
    PyErr_SetString(PyExc_KeyError, name);
    return nullptr;
}

// Arg.__init__(tensor, ptr): a contiguous device tensor (the caller has checked that) and the pointer object of its memory
int arg_init(PyObject *self, PyObject *args, PyObject *) {
    Arg *a = reinterpret_cast<Arg *>(self);
    PyObject *t, *ptr;
    if (!PyArg_ParseTuple(args, "OO", &t, &ptr)) return -1;
    if (a->tensor || !THPVariable_Check(t)) {
        PyErr_SetString(PyExc_TypeError, "a tensor, once");
        return -1;
    }
    void *at = nullptr;
    PyObject *dtype = nullptr, *shape = nullptr, *sizes = nullptr;
    if (!address(ptr, at) || !(dtype = PyObject_GetAttrString(t, "dtype")) || !(sizes = PyObject_GetAttrString(t, "shape")) ||
        !(shape = PySequence_Tuple(sizes))) {
        Py_XDECREF(dtype);
        Py_XDECREF(sizes);
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "no pointer");
        return -1;
    }
    Py_DECREF(sizes);
    const at::Tensor &x = THPVariable_Unpack(t);
    a->address = at;
    a->scalar_type = (int)x.scalar_type();
    // a call that asks for sizes reads the leading three or the last of up to four; others take the general binding
    a->n_dims = x.dim() <= 4 ? (int)x.dim() : 0;
    for (int i = 0; i < a->n_dims; ++i) a->dims[i] = x.size(i);
    Py_INCREF(t);
    Py_INCREF(ptr);
    a->ptr = ptr;
    a->dtype = dtype;
    a->shape = shape;
    a->tensor = t;
    return 0;
}

int arg_traverse(PyObject *self, visitproc visit, void *arg) {
    Arg *a = reinterpret_cast<Arg *>(self);
    Py_VISIT(a->tensor);
    Py_VISIT(a->ptr);
    Py_VISIT(a->dtype);
    Py_VISIT(a->shape);
    return 0;
}

int arg_clear(PyObject *self) {
    Arg *a = reinterpret_cast<Arg *>(self);
    Py_CLEAR(a->tensor);
    Py_CLEAR(a->ptr);
    Py_CLEAR(a->dtype);
    Py_CLEAR(a->shape);
    return 0;
}

void arg_dealloc(PyObject *self) {
    PyObject_GC_UnTrack(self);
    arg_clear(self);
    Py_TYPE(self)->tp_free(self);
}

PyMemberDef arg_members[] = {{"tensor", T_OBJECT_EX, offsetof(Arg, tensor), READONLY, nullptr},
                             {"ptr", T_OBJECT_EX, offsetof(Arg, ptr), READONLY, nullptr},
                             {"dtype", T_OBJECT_EX, offsetof(Arg, dtype), READONLY, nullptr},
                             {"shape", T_OBJECT_EX, offsetof(Arg, shape), READONLY, nullptr},
                             {nullptr, 0, 0, 0, nullptr}};

PyTypeObject ArgType = {PyVarObject_HEAD_INIT(nullptr, 0)};

PyMethodDef methods[] = {{"decode_step", (PyCFunction)(void (*)())decode_step, METH_FASTCALL, nullptr},
                         {"append_decode_step", (PyCFunction)(void (*)())append_decode_step, METH_FASTCALL, nullptr},
                         {"query", (PyCFunction)(void (*)())query, METH_FASTCALL, nullptr},
                         {"sparse_attention", (PyCFunction)(void (*)())sparse_attention, METH_FASTCALL, nullptr},
                         {"sparse_attention_static", (PyCFunction)(void (*)())sparse_attention_static, METH_FASTCALL, nullptr},
                         {"dense_attention", (PyCFunction)(void (*)())dense_attention, METH_FASTCALL, nullptr},
                         {"bind", bind, METH_VARARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__call() {
    ArgType.tp_name = "paper_2605_06763_amd._call.Arg";
    ArgType.tp_basicsize = sizeof(Arg);
    ArgType.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_BASETYPE | Py_TPFLAGS_HAVE_GC;
    ArgType.tp_new = PyType_GenericNew;
    ArgType.tp_init = arg_init;
    ArgType.tp_dealloc = arg_dealloc;
    ArgType.tp_traverse = arg_traverse;
    ArgType.tp_clear = arg_clear;
    ArgType.tp_members = arg_members;
    if (PyType_Ready(&ArgType) < 0) return nullptr;
    if (!(s_value = PyUnicode_InternFromString("value"))) return nullptr;
    PyObject *m = PyModule_Create(&module);
    if (!m) return nullptr;
    Py_INCREF(&ArgType);
    if (PyModule_AddObject(m, "Arg", reinterpret_cast<PyObject *>(&ArgType)) < 0) {
        Py_DECREF(&ArgType);
        Py_DECREF(m);
        return nullptr;
    }
    if (PyModule_AddStringConstant(m, "TORCH_VERSION", TORCH_VERSION) < 0) {   // whose headers this was built with
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
