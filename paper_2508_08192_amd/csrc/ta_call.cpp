// The way from Python into libtreeattn for calls that pass plain torch tensors: an extension module that writes the
// descriptors of a call and makes it.  A step of one request keeps the GPU busy for some 15 to 20 us, and the same
// descriptors put together with ctypes, field by field, took the host 22.5 us a call (57 for write-back, attention and
// bookkeeping); here they take 11.5 (24), the launches included.  What is not of the simple form -- a subclass, an object
// that only describes a tensor, an option given in an unusual type -- is left to the caller: the function then returns None
// and has done nothing.
//
// Only attributes that any Python code could read are used (shape, stride(), dtype, data_ptr()), so the module is tied to
// no version of torch.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <string.h>

#include "../../include/treeattn.h"

namespace {

PyObject *g_tensor, *g_parameter;                  // the exact types taken here
PyObject *g_shape, *g_stride, *g_dtype, *g_data_ptr;   // attribute names
constexpr int kMaxDtypes = 8;
PyObject *g_dtypes[kMaxDtypes];
int32_t g_codes[kMaxDtypes];
int g_n_dtypes;

bool is_plain(PyObject *t)
{
    return (PyObject *)Py_TYPE(t) == g_tensor || (PyObject *)Py_TYPE(t) == g_parameter;
}

// The integers of a tuple (a torch.Size is one); their number, or -1.
int read_ints(PyObject *tuple, int64_t out[5])
{
    if (!tuple || !PyTuple_Check(tuple) || PyTuple_GET_SIZE(tuple) > 5)
        return -1;
    const int n = (int)PyTuple_GET_SIZE(tuple);
    for (int i = 0; i < n; ++i) {
        PyObject *x = PyTuple_GET_ITEM(tuple, i);
        if (!PyLong_CheckExact(x))
            return -1;
        out[i] = PyLong_AsLongLong(x);
        if (out[i] == -1 && PyErr_Occurred())
            return -1;
    }
    return n;
}

bool read_ptr(PyObject *t, void **out)
{
    PyObject *x = PyObject_CallMethodNoArgs(t, g_data_ptr);
    if (!x)
        return false;
    *out = PyLong_CheckExact(x) ? (void *)(uintptr_t)PyLong_AsUnsignedLongLong(x) : nullptr;
    const bool ok = PyLong_CheckExact(x) && !PyErr_Occurred();
    Py_DECREF(x);
    return ok;
}

// Descriptor of a plain tensor; false (perhaps with an exception set) if it has to be described elsewhere.
bool describe(PyObject *t, ta_tensor *d)
{
    if (!is_plain(t))
        return false;
    memset(d, 0, sizeof *d);
    PyObject *x = PyObject_GetAttr(t, g_shape);
    const int n = read_ints(x, d->shape);
    Py_XDECREF(x);
    if (n < 0)
        return false;
    x = PyObject_CallMethodNoArgs(t, g_stride);
    const int m = read_ints(x, d->stride);
    Py_XDECREF(x);
    if (m != n)
        return false;
    x = PyObject_GetAttr(t, g_dtype);
    if (!x)
        return false;
    d->ndim = n;
    d->dtype = -1;
    for (int i = 0; i < g_n_dtypes; ++i)
        if (x == g_dtypes[i])
            d->dtype = g_codes[i];
    Py_DECREF(x);
    return read_ptr(t, &d->data);
}

// n tensors, each of which may be None, into descriptors and pointers to them.
bool describe_all(PyObject *const *args, int n, ta_tensor *d, ta_tensor **ptr)
{
    for (int i = 0; i < n; ++i) {
        ptr[i] = args[i] == Py_None ? nullptr : &d[i];
        if (ptr[i] && !describe(args[i], &d[i]))
            return false;
    }
    return true;
}

bool read_int32(PyObject *x, int32_t *out)
{
    if (!PyLong_CheckExact(x))
        return false;
    const long v = PyLong_AsLong(x);
    *out = (int32_t)v;
    return !(v == -1 && PyErr_Occurred()) && *out == v;
}

// The entry point and the stream, as addresses.
bool read_address(PyObject *x, void **out)
{
    if (!PyLong_CheckExact(x))
        return false;
    *out = (void *)(uintptr_t)PyLong_AsUnsignedLongLong(x);
    return !PyErr_Occurred();
}

PyObject *elsewhere()                              // not of the simple form; whatever went wrong will go wrong there
{
    PyErr_Clear();
    Py_RETURN_NONE;
}

// fwd(entry, stream, q, k_cache, v_cache, page_table, seq_lens, tree_parent, out, lse) -> status or None
PyObject *py_fwd(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    typedef int (*fn_t)(const ta_tensor *, const ta_tensor *, const ta_tensor *, const ta_tensor *, const ta_tensor *,
                        const ta_tensor *, ta_tensor *, ta_tensor *, void *);
    ta_tensor d[8], *t[8];
    void *fn, *stream;
    if (nargs != 10 || !read_address(args[0], &fn) || !read_address(args[1], &stream) || !describe_all(args + 2, 8, d, t))
        return elsewhere();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = ((fn_t)fn)(t[0], t[1], t[2], t[3], t[4], t[5], t[6], t[7], stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// fwd_ex(entry, stream, the eight tensors, scale, num_splits, kernel, item_cost, tree_masks, kv_start, q_node_offset, k_new,
// v_new) -> status or None (entry: tree_attn_fwd_ex or tree_attn_fwd_static)
PyObject *py_fwd_ex(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    typedef int (*fn_t)(const ta_tensor *, const ta_tensor *, const ta_tensor *, const ta_tensor *, const ta_tensor *,
                        const ta_tensor *, ta_tensor *, ta_tensor *, void *, const ta_opts *);
    ta_tensor d[8], *t[8], dn[2], *tn[2], dm;
    ta_opts o;
    void *fn, *stream, *at;
    if (nargs != 19 || !read_address(args[0], &fn) || !read_address(args[1], &stream) || !describe_all(args + 2, 8, d, t))
        return elsewhere();
    memset(&o, 0, sizeof o);
    PyObject *scale = args[10], *masks = args[14], *starts = args[15];
    if (scale != Py_None) {
        if (!PyFloat_CheckExact(scale))
            return elsewhere();
        o.scale = (float)PyFloat_AS_DOUBLE(scale);
    }
    if (!read_int32(args[11], &o.num_splits) || !read_int32(args[12], &o.kernel) || !read_int32(args[13], &o.item_cost) ||
        !read_int32(args[16], &o.q_node_offset))
        return elsewhere();
    if (masks != Py_None) {
        if (!describe(masks, &dm))
            return elsewhere();
        o.tree_masks = dm.data;
        o.tree_masks_stride = dm.ndim == 2 ? dm.stride[0] : 0;
    }
    if (starts != Py_None) {
        if (!is_plain(starts) || !read_ptr(starts, &at))
            return elsewhere();
        o.kv_start = at;
    }
    if (!describe_all(args + 17, 2, dn, tn))
        return elsewhere();
    o.k_new = tn[0];
    o.v_new = tn[1];
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = ((fn_t)fn)(t[0], t[1], t[2], t[3], t[4], t[5], t[6], t[7], stream, &o);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// append(entry, stream, k_new, v_new, k_cache, v_cache, page_table, seq_lens) -> status or None
PyObject *py_append(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    typedef int (*fn_t)(const ta_tensor *, const ta_tensor *, ta_tensor *, ta_tensor *, const ta_tensor *, const ta_tensor *,
                        void *);
    ta_tensor d[6], *t[6];
    void *fn, *stream;
    if (nargs != 8 || !read_address(args[0], &fn) || !read_address(args[1], &stream) || !describe_all(args + 2, 6, d, t))
        return elsewhere();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = ((fn_t)fn)(t[0], t[1], t[2], t[3], t[4], t[5], stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// compact(entry, stream, k_cache, v_cache, page_table, seq_lens, accepted, n_accepted, seq_lens_out, tree_size) -> status or
// None
PyObject *py_compact(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    typedef int (*fn_t)(ta_tensor *, ta_tensor *, const ta_tensor *, const ta_tensor *, const ta_tensor *, const ta_tensor *,
                        int32_t, ta_tensor *, void *);
    ta_tensor d[7], *t[7];
    void *fn, *stream;
    int32_t tree_size;
    if (nargs != 10 || !read_address(args[0], &fn) || !read_address(args[1], &stream) ||
        !describe_all(args + 2, 7, d, t) || !read_int32(args[9], &tree_size))
        return elsewhere();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = ((fn_t)fn)(t[0], t[1], t[2], t[3], t[4], t[5], tree_size, t[6], stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// setup(Tensor, Parameter, ((dtype, code), ...)): the types and element types that describe() knows.  Called once.
PyObject *py_setup(PyObject *, PyObject *args)
{
    PyObject *tensor, *parameter, *dtypes;
    if (!PyArg_ParseTuple(args, "OOO!", &tensor, &parameter, &PyTuple_Type, &dtypes))
        return nullptr;
    int n = 0;
    for (; n < PyTuple_GET_SIZE(dtypes) && n < kMaxDtypes; ++n) {
        PyObject *dt;
        int code;
        if (!PyArg_ParseTuple(PyTuple_GET_ITEM(dtypes, n), "Oi", &dt, &code))
            return nullptr;
        Py_INCREF(dt);
        g_dtypes[n] = dt;
        g_codes[n] = code;
    }
    Py_INCREF(tensor);
    Py_INCREF(parameter);
    g_n_dtypes = n;
    g_tensor = tensor;
    g_parameter = parameter;
    Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    {"fwd", (PyCFunction)(void (*)(void))py_fwd, METH_FASTCALL, nullptr},
    {"fwd_ex", (PyCFunction)(void (*)(void))py_fwd_ex, METH_FASTCALL, nullptr},
    {"append", (PyCFunction)(void (*)(void))py_append, METH_FASTCALL, nullptr},
    {"compact", (PyCFunction)(void (*)(void))py_compact, METH_FASTCALL, nullptr},
    {"setup", py_setup, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_call", "Calls into libtreeattn with plain torch tensors.", -1, kMethods,
                       nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call(void)
{
    g_shape = PyUnicode_InternFromString("shape");
    g_stride = PyUnicode_InternFromString("stride");
    g_dtype = PyUnicode_InternFromString("dtype");
    g_data_ptr = PyUnicode_InternFromString("data_ptr");
    if (!g_shape || !g_stride || !g_dtype || !g_data_ptr)
        return nullptr;
    return PyModule_Create(&kModule);
}
