// Argument marshalling of the Python binding's compute calls (CPython extension, host only).
//
// Turning tensors, numpy arrays and pointer tables into the C ABI's pointers and sizes costs about 10 us per call in
// Python (ctypes structures and casts), more than the launches of a decode-sized forward call (7 us) and than the
// kernel of an adapter update (4 us); here it is about 1 us.  Each function takes the arguments of the binding's method of the
// same name, calls the C entry point with the interpreter lock released and returns its status - or returns None,
// without having called anything, where an argument is not of the plain form it expects (contiguous int32 / uint8 arrays,
// pointer tables made beforehand, bfloat16 or float32 tensors): the binding then takes its general path, which
// converts what can be converted and raises for the rest.  Nothing is kept between calls.  The entry points are the
// addresses the binding hands over (bind), not symbols to link: another copy of the library in the process would answer to them.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "collm_lora.h"

namespace {

PyObject *g_bf16 = nullptr, *g_f32 = nullptr, *g_table = nullptr;  // torch.bfloat16, torch.float32, the binding's PointerTable
decltype(&collm_lora_linear_fwd) g_linear_fwd = nullptr;
decltype(&collm_lora_linear_bwd) g_linear_bwd = nullptr;
decltype(&collm_adapter_adamw) g_adamw = nullptr;
decltype(&collm_adapter_fedavg) g_fedavg = nullptr;
PyObject *s_data_ptr, *s_dtype, *s_shape, *s_array, *s_numel, *s_device, *s_index;

// Arguments of one call as they are read; `ok` falls at the first one that is not of the expected form.
struct Reader {
    PyObject *const *args;
    bool ok = true;
    Py_buffer bufs[12];
    int n_bufs = 0;

    explicit Reader(PyObject *const *a) : args(a) {}
    ~Reader()
    {
        for (int i = 0; i < n_bufs; ++i) PyBuffer_Release(&bufs[i]);
        if (PyErr_Occurred()) PyErr_Clear();
    }
    Reader(const Reader &) = delete;
    Reader &operator=(const Reader &) = delete;

    int64_t integer(PyObject *o)
    {
        if (!ok || !PyLong_Check(o)) {
            ok = false;
            return 0;
        }
        const long long v = PyLong_AsLongLong(o);
        if (v == -1 && PyErr_Occurred()) ok = false;
        return v;
    }
    int32_t int32(PyObject *o)
    {
        const int64_t v = integer(o);
        if (v != (int32_t)v) ok = false;
        return (int32_t)v;
    }
    void *pointer(PyObject *o)  // an address; None is NULL
    {
        if (o == Py_None) return nullptr;
        if (!ok || !PyLong_Check(o)) {
            ok = false;
            return nullptr;
        }
        void *p = PyLong_AsVoidPtr(o);
        if (PyErr_Occurred()) ok = false;
        return p;
    }
    double real(PyObject *o)
    {
        const double v = ok ? PyFloat_AsDouble(o) : 0.0;
        if (PyErr_Occurred()) ok = false;
        return v;
    }
    // a tensor's address (None is NULL if `optional`)
    void *tensor(PyObject *o, bool optional = false)
    {
        if (!ok || (o == Py_None && optional)) return nullptr;
        PyObject *v = PyObject_CallMethodNoArgs(o, s_data_ptr);
        if (!v) {
            ok = false;
            return nullptr;
        }
        void *p = pointer(v);
        Py_DECREF(v);
        return p;
    }
    collm_dtype dtype(PyObject *o)
    {
        PyObject *d = ok ? PyObject_GetAttr(o, s_dtype) : nullptr;
        const bool b = d && d == g_bf16, f = d && d == g_f32;
        Py_XDECREF(d);
        if (!b && !f) ok = false;
        return b ? COLLM_BF16 : COLLM_F32;
    }
    void shape2(PyObject *o, int32_t &rows, int32_t &cols)
    {
        PyObject *s = ok ? PyObject_GetAttr(o, s_shape) : nullptr;
        if (s && PyTuple_Check(s) && PyTuple_GET_SIZE(s) == 2) {
            rows = int32(PyTuple_GET_ITEM(s, 0));
            cols = int32(PyTuple_GET_ITEM(s, 1));
        } else {
            ok = false;
        }
        Py_XDECREF(s);
    }
    int64_t numel(PyObject *o)
    {
        PyObject *v = ok ? PyObject_CallMethodNoArgs(o, s_numel) : nullptr;
        const int64_t n = v ? integer(v) : 0;
        if (!v) ok = false;
        Py_XDECREF(v);
        return n;
    }
    int32_t device(PyObject *o)
    {
        PyObject *d = ok ? PyObject_GetAttr(o, s_device) : nullptr;
        PyObject *i = d ? PyObject_GetAttr(d, s_index) : nullptr;
        int32_t v = 0;
        if (!i) ok = false;
        else if (i != Py_None) v = int32(i);
        Py_XDECREF(i);
        Py_XDECREF(d);
        return v;
    }
    // a contiguous one-dimensional array of elements `fmt` ('i': 32-bit, 'B': bytes) and its length
    const void *array(PyObject *o, char fmt, int32_t &n)
    {
        if (!ok || n_bufs == (int)(sizeof bufs / sizeof bufs[0]) ||
            PyObject_GetBuffer(o, &bufs[n_bufs], PyBUF_ND | PyBUF_FORMAT) != 0) {
            ok = false;
            return nullptr;
        }
        const Py_buffer &b = bufs[n_bufs++];
        const Py_ssize_t size = fmt == 'i' ? 4 : 1;
        if (b.ndim != 1 || b.itemsize != size || !b.format || b.format[0] != fmt || b.format[1] != 0 ||
            b.shape[0] > INT32_MAX || ((uintptr_t)b.buf & (uintptr_t)(size - 1))) {
            ok = false;
            return nullptr;
        }
        n = (int32_t)b.shape[0];
        return b.buf;
    }
    // the array of a pointer table (None is NULL if `optional`)
    void *table(PyObject *o, bool optional = false)
    {
        if (!ok || (o == Py_None && optional)) return nullptr;
        PyObject *a = g_table && PyObject_IsInstance(o, g_table) == 1 ? PyObject_GetAttr(o, s_array) : nullptr;
        if (!a || n_bufs == (int)(sizeof bufs / sizeof bufs[0]) || PyObject_GetBuffer(a, &bufs[n_bufs], PyBUF_SIMPLE) != 0) {
            Py_XDECREF(a);
            ok = false;
            return nullptr;
        }
        Py_DECREF(a);  // (the buffer holds it)
        return bufs[n_bufs++].buf;
    }
};

// What every layer call begins with: handle, x, W, A, B, rank, seg_start, seg_adapter, seg_is_train, scale, layout, stream
struct Layer {
    collm_ctx *ctx;
    collm_shape sh;
    void *x, *W;
    const void *const *A, *const *B;
    const int32_t *rank, *seg_start, *seg_adapter;
    const uint8_t *seg_is_train;
    void *stream;

    explicit Layer(Reader &r)
    {
        PyObject *const *a = r.args;
        ctx = (collm_ctx *)r.pointer(a[0]);
        x = r.tensor(a[1]);
        W = r.tensor(a[2]);
        A = (const void *const *)r.table(a[3]);
        B = (const void *const *)r.table(a[4]);
        int32_t n_rank = 0, n_start = 0, n_seg = 0, n_train = 0, tokens = 0, d_in = 0, w0 = 0, w1 = 0;
        rank = (const int32_t *)r.array(a[5], 'i', n_rank);
        seg_start = (const int32_t *)r.array(a[6], 'i', n_start);
        seg_adapter = (const int32_t *)r.array(a[7], 'i', n_seg);
        seg_is_train = (const uint8_t *)r.array(a[8], 'B', n_train);
        if (n_start != n_seg + 1 || n_train != n_seg) r.ok = false;
        r.shape2(a[1], tokens, d_in);
        r.shape2(a[2], w0, w1);
        sh.d_in = d_in;
        sh.n_tokens = tokens;
        sh.n_segments = n_seg;
        sh.n_adapters = n_rank;
        sh.dtype = r.dtype(a[1]);
        sh.scale = (float)r.real(a[9]);
        sh.layout = (decltype(sh.layout))r.int32(a[10]);
        sh.d_out = sh.layout == COLLM_LAYOUT_OUT_IN ? w0 : w1;
        stream = r.pointer(a[11]);
    }
};

PyObject *status(int rc) { return PyLong_FromLong(rc); }

#define COLLM_ARGS(count)                                                   \
    if (n != (count)) {                                                     \
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");      \
        return nullptr;                                                     \
    }                                                                       \
    Reader r(args)

// ..., y, h_save
PyObject *linear_fwd(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    COLLM_ARGS(14);
    Layer l(r);
    void *y = r.tensor(args[12]), *h = r.tensor(args[13], true);
    if (!r.ok || !g_table) Py_RETURN_NONE;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_linear_fwd(l.ctx, &l.sh, l.x, l.W, l.A, l.B, l.rank, l.seg_start, l.seg_adapter, l.seg_is_train, y, (float *)h, l.stream);
    Py_END_ALLOW_THREADS
    return status(rc);
}

// ..., dy, h_save, dx, dA, dB, accumulate
PyObject *linear_bwd(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    COLLM_ARGS(18);
    Layer l(r);
    void *dy = r.tensor(args[12]), *h = r.tensor(args[13], true), *dx = r.tensor(args[14], true);
    float *const *dA = (float *const *)r.table(args[15], true), *const *dB = (float *const *)r.table(args[16], true);
    const int acc = r.int32(args[17]);
    if (!r.ok || !g_table) Py_RETURN_NONE;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_linear_bwd(l.ctx, &l.sh, l.x, l.W, l.A, l.B, l.rank, l.seg_start, l.seg_adapter, l.seg_is_train, dy, (const float *)h, dx, dA,
                               dB, acc, l.stream);
    Py_END_ALLOW_THREADS
    return status(rc);
}

// device is the parameter's; param, grad, m, v, lr, beta1, beta2, eps, weight_decay, step, master, stream
PyObject *adapter_adamw(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    COLLM_ARGS(12);
    const int32_t dev = r.device(args[0]);
    const collm_dtype dt = r.dtype(args[0]);
    void *param = r.tensor(args[0]), *grad = r.tensor(args[1]), *m = r.tensor(args[2]), *v = r.tensor(args[3]);
    const int64_t elems = r.numel(args[0]);
    collm_adamw hp;
    hp.lr = (float)r.real(args[4]);
    hp.beta1 = (float)r.real(args[5]);
    hp.beta2 = (float)r.real(args[6]);
    hp.eps = (float)r.real(args[7]);
    hp.weight_decay = (float)r.real(args[8]);
    hp.step = r.int32(args[9]);
    void *master = r.tensor(args[10], true), *stream = r.pointer(args[11]);
    if (!r.ok || !g_table) Py_RETURN_NONE;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_adamw(dev, dt, param, (float *)master, (const float *)grad, (float *)m, (float *)v, elems, &hp, stream);
    Py_END_ALLOW_THREADS
    return status(rc);
}

// copies (a pointer table), their number, dst, stream
PyObject *adapter_fedavg(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    COLLM_ARGS(4);
    const void *const *src = (const void *const *)r.table(args[0]);
    const int32_t copies = r.int32(args[1]), dev = r.device(args[2]);
    const collm_dtype dt = r.dtype(args[2]);
    void *dst = r.tensor(args[2]);
    const int64_t elems = r.numel(args[2]);
    void *stream = r.pointer(args[3]);
    if (!r.ok || !g_table) Py_RETURN_NONE;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_fedavg(dev, dt, copies, src, dst, elems, stream);
    Py_END_ALLOW_THREADS
    return status(rc);
}

// the two element types as torch has them, the class of pointer tables, and the addresses of the four entry points
PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    COLLM_ARGS(7);
    void *f[4];
    for (int i = 0; i < 4; ++i) f[i] = r.pointer(args[3 + i]);
    if (!r.ok || !f[0] || !f[1] || !f[2] || !f[3]) Py_RETURN_FALSE;
    g_linear_fwd = reinterpret_cast<decltype(g_linear_fwd)>(f[0]);
    g_linear_bwd = reinterpret_cast<decltype(g_linear_bwd)>(f[1]);
    g_adamw = reinterpret_cast<decltype(g_adamw)>(f[2]);
    g_fedavg = reinterpret_cast<decltype(g_fedavg)>(f[3]);
    Py_INCREF(args[0]);
    Py_INCREF(args[1]);
    Py_INCREF(args[2]);
    Py_XSETREF(g_bf16, args[0]);
    Py_XSETREF(g_f32, args[1]);
    Py_XSETREF(g_table, args[2]);
    Py_RETURN_TRUE;
}

#define COLLM_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {COLLM_METHOD(linear_fwd),     COLLM_METHOD(linear_bwd), COLLM_METHOD(adapter_adamw),
                         COLLM_METHOD(adapter_fedavg), COLLM_METHOD(bind), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_dtype = PyUnicode_InternFromString("dtype");
    s_shape = PyUnicode_InternFromString("shape");
    s_array = PyUnicode_InternFromString("array");
    s_numel = PyUnicode_InternFromString("numel");
    s_device = PyUnicode_InternFromString("device");
    s_index = PyUnicode_InternFromString("index");
    return PyModule_Create(&module);
}
