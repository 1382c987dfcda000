// The per-call part of the Python binding in C: tensors to pointers, descriptors to addresses, the current stream, the call.
// Through ctypes that is 3.6 us of the 6 to 8 us a small layer's call takes (argument objects, one conversion per argument,
// a Python frame per pointer), here 0.6 us; the launch itself is 2.2 us.
//
// Every function returns the entry point's status, or -1 without having called it when an argument is not of the plain
// kind (a tensor, an integer, None, a descriptor of the registered type): binding.py then takes its ctypes path, which
// accepts what it always accepted and raises what it always raised.  Nothing is kept between calls but the types, entry
// points and callables that binding.py hands over once.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "../../include/nq.h"

namespace {

PyObject *t_tensor, *t_weight, *t_epilogue, *t_shape, *t_cfg;      // types
PyObject *f_device, *f_stream;                                     // current device; its current raw stream
PyObject *s_data_ptr, *s_is_contiguous;
int stream_ready;                                                  // set by binding.py once torch has initialised the GPU

typedef nq_status (*gemm_fn)(const int8_t *, int64_t, const nq_weight *, const nq_epilogue *, void *, void *);
typedef nq_status (*conv_fn)(const int8_t *, const nq_conv_shape *, const nq_weight *, const nq_epilogue *, void *, void *);
typedef nq_status (*gconv_fn)(const int8_t *, const nq_conv_shape *, int, const nq_weight *, const nq_epilogue *, void *, void *);
typedef nq_status (*qpack_fn)(const float *, int64_t, int64_t, const nq_cfg *, float *, void *, void *, void *);
gemm_fn gemm_of[2];
conv_fn conv_of[2];
gconv_fn gconv_of[2];
qpack_fn qpack_of;

// A descriptor's memory for the length of a call.
struct Struct {
    Py_buffer view;
    bool held = false;
    bool take(PyObject *o, PyObject *type, size_t bytes)
    {
        if (!PyObject_TypeCheck(o, reinterpret_cast<PyTypeObject *>(type))) return false;
        if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) {
            PyErr_Clear();
            return false;
        }
        held = true;
        return (size_t)view.len >= bytes;
    }
    ~Struct()
    {
        if (held) PyBuffer_Release(&view);
    }
    template <typename T>
    T *as() const { return static_cast<T *>(view.buf); }
};

bool integer(PyObject *o, int64_t *v)
{
    if (!PyLong_Check(o)) return false;
    *v = PyLong_AsLongLong(o);
    if (*v == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

bool number(PyObject *o, float *v)
{
    if (!PyFloat_Check(o) && !PyLong_Check(o)) return false;
    const double d = PyFloat_AsDouble(o);
    if (d == -1.0 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    *v = (float)d;
    return true;
}

// None, an address, or a contiguous tensor.
bool pointer(PyObject *o, void **p)
{
    if (o == Py_None) {
        *p = nullptr;
        return true;
    }
    if (PyLong_Check(o)) {
        *p = PyLong_AsVoidPtr(o);
        if (!*p && PyErr_Occurred()) {
            PyErr_Clear();
            return false;
        }
        return true;
    }
    if (!PyObject_TypeCheck(o, reinterpret_cast<PyTypeObject *>(t_tensor))) return false;
    PyObject *c = PyObject_CallMethodNoArgs(o, s_is_contiguous);
    const bool yes = c == Py_True;
    Py_XDECREF(c);
    PyObject *a = yes ? PyObject_CallMethodNoArgs(o, s_data_ptr) : nullptr;
    if (!a) {
        PyErr_Clear();
        return false;
    }
    *p = PyLong_AsVoidPtr(a);
    Py_DECREF(a);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

bool stream(PyObject *o, void **s)
{
    if (PyLong_Check(o)) return pointer(o, s);
    if (o != Py_None || !stream_ready) return false;        // a Stream object: binding.py asks it
    PyObject *d = PyObject_CallNoArgs(f_device);
    PyObject *r = d ? PyObject_CallOneArg(f_stream, d) : nullptr;
    Py_XDECREF(d);
    if (!r) {
        PyErr_Clear();
        return false;
    }
    *s = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

PyObject *not_plain() { return PyLong_FromLong(-1); }

#define NQ_CALL(status, expr)  \
    nq_status status;          \
    Py_BEGIN_ALLOW_THREADS;    \
    status = expr;             \
    Py_END_ALLOW_THREADS

// (full, x, M, weight, epilogue, y, stream)
PyObject *gemm(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Struct w, e;
    void *x, *y, *s;
    int64_t full, M;
    if (n != 7 || !integer(a[0], &full) || !pointer(a[1], &x) || !integer(a[2], &M) || !w.take(a[3], t_weight, sizeof(nq_weight)) ||
        !e.take(a[4], t_epilogue, sizeof(nq_epilogue)) || !pointer(a[5], &y) || !stream(a[6], &s))
        return not_plain();
    NQ_CALL(st, gemm_of[full != 0]((const int8_t *)x, M, w.as<nq_weight>(), e.as<nq_epilogue>(), y, s));
    return PyLong_FromLong(st);
}

// (full, x, shape, weight, epilogue, y, stream)
PyObject *conv(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Struct sh, w, e;
    void *x, *y, *s;
    int64_t full;
    if (n != 7 || !integer(a[0], &full) || !pointer(a[1], &x) || !sh.take(a[2], t_shape, sizeof(nq_conv_shape)) ||
        !w.take(a[3], t_weight, sizeof(nq_weight)) || !e.take(a[4], t_epilogue, sizeof(nq_epilogue)) || !pointer(a[5], &y) ||
        !stream(a[6], &s))
        return not_plain();
    NQ_CALL(st, conv_of[full != 0]((const int8_t *)x, sh.as<nq_conv_shape>(), w.as<nq_weight>(), e.as<nq_epilogue>(), y, s));
    return PyLong_FromLong(st);
}

// (full, x, shape, groups, weight, epilogue, y, stream)
PyObject *gconv(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Struct sh, w, e;
    void *x, *y, *s;
    int64_t full, groups;
    if (n != 8 || !integer(a[0], &full) || !pointer(a[1], &x) || !sh.take(a[2], t_shape, sizeof(nq_conv_shape)) ||
        !integer(a[3], &groups) || groups != (int)groups || !w.take(a[4], t_weight, sizeof(nq_weight)) ||
        !e.take(a[5], t_epilogue, sizeof(nq_epilogue)) || !pointer(a[6], &y) || !stream(a[7], &s))
        return not_plain();
    NQ_CALL(st, gconv_of[full != 0]((const int8_t *)x, sh.as<nq_conv_shape>(), (int)groups, w.as<nq_weight>(),
                                    e.as<nq_epilogue>(), y, s));
    return PyLong_FromLong(st);
}

// (w, N, K, cfg, scale, high, low, stream)
PyObject *quantize_pack(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Struct c;
    void *w, *scale, *high, *low, *s;
    int64_t N, K;
    if (n != 8 || !pointer(a[0], &w) || !integer(a[1], &N) || !integer(a[2], &K) || !c.take(a[3], t_cfg, sizeof(nq_cfg)) ||
        !pointer(a[4], &scale) || !pointer(a[5], &high) || !pointer(a[6], &low) || !stream(a[7], &s))
        return not_plain();
    NQ_CALL(st, qpack_of((const float *)w, N, K, c.as<nq_cfg>(), (float *)scale, high, low, s));
    return PyLong_FromLong(st);
}

// A convolution (or, with sizes None, a GEMM over M rows) from the values of its descriptors, for a caller that has no
// descriptor objects: (full, x, M, (B, H, W, Cin, Cout, K, stride, pad) or None, weight, act_scale, bias, residual,
// residual_scale, relu, out_int8, inv_out_scale, y, stream)
PyObject *layer(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Struct w;
    nq_conv_shape sh;
    nq_epilogue e;
    void *x, *y, *s, *bias, *resid;
    int64_t full, M, relu, int8;
    if (n != 14 || !integer(a[0], &full) || !pointer(a[1], &x) || !integer(a[2], &M) || !w.take(a[4], t_weight, sizeof(nq_weight)) ||
        !number(a[5], &e.act_scale) || !pointer(a[6], &bias) || !pointer(a[7], &resid) || !number(a[8], &e.residual_scale) ||
        !integer(a[9], &relu) || !integer(a[10], &int8) || !number(a[11], &e.inv_out_scale) || !pointer(a[12], &y) ||
        !stream(a[13], &s))
        return not_plain();
    const bool is_conv = a[3] != Py_None;
    if (is_conv) {
        int64_t v[8];
        if (!PyTuple_CheckExact(a[3]) || PyTuple_GET_SIZE(a[3]) != 8) return not_plain();
        for (int i = 0; i < 8; ++i)
            if (!integer(PyTuple_GET_ITEM(a[3], i), &v[i])) return not_plain();
        for (int i = 5; i < 8; ++i)
            if (v[i] != (int32_t)v[i]) return not_plain();
        sh.B = v[0]; sh.H = v[1]; sh.W = v[2]; sh.Cin = v[3]; sh.Cout = v[4];
        sh.KH = sh.KW = (int32_t)v[5]; sh.stride = (int32_t)v[6]; sh.pad = (int32_t)v[7];
    }
    e.d_bias = (const float *)bias;
    e.d_residual = (const int8_t *)resid;
    e.relu = relu != 0;
    e.out_int8 = int8 != 0;
    e.d_acc_dump = nullptr;
    NQ_CALL(st, is_conv ? conv_of[full != 0]((const int8_t *)x, &sh, w.as<nq_weight>(), &e, y, s)
                        : gemm_of[full != 0]((const int8_t *)x, M, w.as<nq_weight>(), &e, y, s));
    return PyLong_FromLong(st);
}

// (types: tensor, weight, epilogue, shape, cfg; callables: device, raw stream; addresses: gemm part, full, conv part, full,
// gconv part, full, quantise and pack)
PyObject *setup(PyObject *, PyObject *args)
{
    PyObject *o[7], *f[7];
    if (!PyArg_ParseTuple(args, "OOOOOOOOOOOOOO", o, o + 1, o + 2, o + 3, o + 4, o + 5, o + 6, f, f + 1, f + 2, f + 3, f + 4,
                          f + 5, f + 6))
        return nullptr;
    void *at[7];
    for (int i = 0; i < 7; ++i)
        if (!(at[i] = PyLong_AsVoidPtr(f[i]))) return PyErr_Occurred() ? nullptr : PyErr_Format(PyExc_ValueError, "no address");
    for (int i = 0; i < 5; ++i)
        if (!PyType_Check(o[i])) return PyErr_Format(PyExc_TypeError, "not a type");
    for (PyObject *p : o) Py_INCREF(p);                        // held for the life of the process
    t_tensor = o[0]; t_weight = o[1]; t_epilogue = o[2]; t_shape = o[3]; t_cfg = o[4];
    f_device = o[5]; f_stream = o[6];
    gemm_of[0] = (gemm_fn)at[0]; gemm_of[1] = (gemm_fn)at[1];
    conv_of[0] = (conv_fn)at[2]; conv_of[1] = (conv_fn)at[3];
    gconv_of[0] = (gconv_fn)at[4]; gconv_of[1] = (gconv_fn)at[5];
    qpack_of = (qpack_fn)at[6];
    Py_RETURN_NONE;
}

PyObject *set_stream_ready(PyObject *, PyObject *v)
{
    stream_ready = PyObject_IsTrue(v) == 1;
    Py_RETURN_NONE;
}

#define NQ_FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {NQ_FAST(gemm), NQ_FAST(conv), NQ_FAST(gconv), NQ_FAST(quantize_pack), NQ_FAST(layer),
                         {"setup", setup, METH_VARARGS, nullptr},
                         {"set_stream_ready", set_stream_ready, METH_O, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_nqcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__nqcall()
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
    if (!s_data_ptr || !s_is_contiguous) return nullptr;
    return PyModule_Create(&module);
}
