/* The way from a Python call to the library: tensors and integers in, one call of a C entry point, its status out.
 *
 * A call on tensors of some hundred kilobytes is bound by issuing it: through the interpreter and ctypes (a table of addresses built,
 * four arguments converted) that was 1.0 us of 4.4 to 5.3, here 0.3; the launch itself is 3.3 to 3.9.  Only the ordinary call is taken:
 * maps whose sources are known, lists or tuples of things with a data_ptr(), integers that fit.  Whatever else comes is answered
 * with NOT_TAKEN before the library has seen it, and goes the way through ctypes, which raises what there is to raise.  Nothing is kept
 * between calls but the addresses of the entry points and torch's functions. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <pthread.h>
#include <stdint.h>

enum { NOT_TAKEN = -1, MAX_TABLE = 16 };

typedef int (*execute_fn)(void *const *, void *, void *, void *);
typedef int (*multi_fn)(void *const *, void *const *, void *const *, int, void *);
typedef int (*fused_fn)(void *, void *, void *, int64_t, void *, void *);
typedef int (*store_fn)(void *, void *, void *, int64_t, void *, void *, void *);
typedef int (*mapped_fn)(void *, void *, void *, void *, void *, void *, void *);
typedef int (*gather_fn)(void *const *, void *, void *, void *, int64_t, void *, void *, void *);

static execute_fn p_execute;
static multi_fn p_multi;
static fused_fn p_fused;
static store_fn p_store;
static mapped_fn p_mapped;
static gather_fn p_gather;
static PyObject *raw_stream, *get_device, *is_initialized;   /* torch's; NULL: no current stream from here */
static PyObject *s_data_ptr, *s_at, *s_reads;
static int initialized;   /* torch said so in this process (a fork asks again) */

static void forked(void) { initialized = 0; }

/* Each of these is 1, or 0 for a call that is not taken.  An error is the other way's to raise again and is cleared; one that ends the
 * program (an interrupt, an exit: no Exception) stays, and the call returns with it. */

static int not_taken(void)
{
    if (PyErr_Occurred() && PyErr_ExceptionMatches(PyExc_Exception)) PyErr_Clear();
    return 0;
}

static int address(PyObject *o, void **at)
{
    if (o == Py_None) {
        *at = NULL;
        return 1;
    }
    if (!PyLong_CheckExact(o)) return 0;
    *at = PyLong_AsVoidPtr(o);
    return *at || !PyErr_Occurred() || not_taken();
}

static int integer(PyObject *o, void **at) { return o != Py_None && address(o, at); }

static int data_of(PyObject *tensor, void **at)
{
    PyObject *p = PyObject_CallMethodNoArgs(tensor, s_data_ptr);
    if (!p) return not_taken();
    const int ok = integer(p, at);
    Py_DECREF(p);
    return ok;
}

/* a source, which a map may not need; an output is always there */
static int source_of(PyObject *tensor, void **at)
{
    if (tensor != Py_None) return data_of(tensor, at);
    *at = NULL;
    return 1;
}

/* a map: the library's, how long a source table it expects and the last source that it reads (-1: none) */
static int map_of(PyObject *m, void **map, Py_ssize_t *n_src, Py_ssize_t *last)
{
    PyObject *at = PyObject_GetAttr(m, s_at), *reads = at ? PyObject_GetAttr(m, s_reads) : NULL;
    int ok = 0;
    if (reads && integer(at, map) && *map && PyTuple_CheckExact(reads) && PyTuple_GET_SIZE(reads) == 2 && PyTuple_CheckExact(PyTuple_GET_ITEM(reads, 1))) {
        PyObject *ids = PyTuple_GET_ITEM(reads, 1);
        const Py_ssize_t n = PyTuple_GET_SIZE(ids);
        *n_src = PyLong_AsSsize_t(PyTuple_GET_ITEM(reads, 0));
        *last = n ? PyLong_AsSsize_t(PyTuple_GET_ITEM(ids, n - 1)) : -1;
        ok = *n_src >= 0;
    }
    if (PyErr_Occurred()) ok = not_taken();
    Py_XDECREF(at);
    Py_XDECREF(reads);
    return ok;
}

/* a map whose sources are not asked for; None: NULL */
static int handle_of(PyObject *m, void **map)
{
    if (m == Py_None) {
        *map = NULL;
        return 1;
    }
    PyObject *at = PyObject_GetAttr(m, s_at);
    const int ok = (at && integer(at, map) && *map) || not_taken();
    Py_XDECREF(at);
    return ok;
}

static int table(PyObject *list, void **tab, Py_ssize_t *given, int (*of)(PyObject *, void **))
{
    if (!PyList_CheckExact(list) && !PyTuple_CheckExact(list)) return 0;
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(list);
    if (n > MAX_TABLE) return 0;
    for (Py_ssize_t i = 0; i < MAX_TABLE; ++i) tab[i] = NULL;
    for (Py_ssize_t i = 0; i < n; ++i) {
        if (i >= PySequence_Fast_GET_SIZE(list)) return 0;   /* (a data_ptr() may run anything) */
        PyObject *o = PySequence_Fast_GET_ITEM(list, i);
        Py_INCREF(o);
        const int ok = of(o, &tab[i]);
        Py_DECREF(o);
        if (!ok) return 0;
    }
    *given = n;
    return 1;
}

static int stream_of(PyObject *o, void **stream)
{
    if (o != Py_None) return address(o, stream);
    if (!raw_stream) return 0;
    PyObject *r;
    if (!initialized) {
        r = PyObject_CallNoArgs(is_initialized);
        initialized = r ? PyObject_IsTrue(r) == 1 : 0;
        Py_XDECREF(r);
        if (!initialized) return not_taken();
    }
    PyObject *dev = PyObject_CallNoArgs(get_device);
    r = dev ? PyObject_CallOneArg(raw_stream, dev) : NULL;
    const int ok = (r && integer(r, stream)) || not_taken();
    Py_XDECREF(dev);
    Py_XDECREF(r);
    return ok;
}

#define CALLED(expr)                \
    do {                            \
        int status_;                \
        Py_BEGIN_ALLOW_THREADS      \
        status_ = (expr);           \
        Py_END_ALLOW_THREADS        \
        return PyLong_FromLong(status_); \
    } while (0)
#define UNLESS(x) \
    if (!(x)) return PyErr_Occurred() ? NULL : PyLong_FromLong(NOT_TAKEN)

/* execute(map, tensors, tensor, stream or None) */
static PyObject *call_execute(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    void *tab[MAX_TABLE], *dst, *map, *stream;
    Py_ssize_t given, n_src, last;
    (void)self;
    UNLESS(p_execute && n == 4 && map_of(a[0], &map, &n_src, &last) && table(a[1], tab, &given, source_of));
    UNLESS(last < given && n_src <= MAX_TABLE && data_of(a[2], &dst) && stream_of(a[3], &stream));
    CALLED(p_execute(tab, dst, map, stream));
}

/* execute_multi(maps, tensors, tensors, stream or None) */
static PyObject *call_execute_multi(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    void *tab[MAX_TABLE], *dst[MAX_TABLE], *maps[MAX_TABLE], *stream;
    Py_ssize_t given, n_dst, n_maps, n_src, last;
    (void)self;
    UNLESS(p_multi && n == 4 && (PyList_CheckExact(a[0]) || PyTuple_CheckExact(a[0])) && table(a[1], tab, &given, source_of) && table(a[2], dst, &n_dst, data_of));
    n_maps = PySequence_Fast_GET_SIZE(a[0]);
    UNLESS(n_maps >= 1 && n_maps <= n_dst);
    for (Py_ssize_t i = 0; i < n_maps; ++i) {
        UNLESS(i < PySequence_Fast_GET_SIZE(a[0]));
        PyObject *m = PySequence_Fast_GET_ITEM(a[0], i);
        Py_INCREF(m);   /* (asking it for its attributes may take it out of the list) */
        const int ok = map_of(m, &maps[i], &n_src, &last);
        Py_DECREF(m);
        UNLESS(ok && last < given && n_src <= MAX_TABLE);
    }
    UNLESS(stream_of(a[3], &stream));
    CALLED(p_multi(tab, dst, maps, (int)n_maps, stream));
}

static int count_of(PyObject *o, int64_t *n)
{
    if (!PyLong_CheckExact(o)) return 0;
    *n = PyLong_AsLongLong(o);
    return *n != -1 || !PyErr_Occurred() || not_taken();
}

/* gemm(address of A, map, address of W, map or None, n, store map or None, address of the product, stream) */
static PyObject *call_gemm(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    void *src, *a_map, *w, *w_map, *out_map, *out, *stream;
    int64_t cols;
    (void)self;
    UNLESS(p_fused && n == 8 && integer(a[0], &src) && a[1] != Py_None && handle_of(a[1], &a_map) && integer(a[2], &w) && handle_of(a[3], &w_map) &&
           count_of(a[4], &cols) && handle_of(a[5], &out_map) && integer(a[6], &out) && integer(a[7], &stream));
    if (w_map) CALLED(p_mapped(src, a_map, w, w_map, out_map, out, stream));
    if (out_map) CALLED(p_store(src, a_map, w, cols, out_map, out, stream));
    CALLED(p_fused(src, a_map, w, cols, out, stream));
}

/* gather(addresses, map, address of W, map or None, n, store map or None, address of the product, stream) */
static PyObject *call_gather(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    void *tab[MAX_TABLE], *a_map, *w, *w_map, *out_map, *out, *stream;
    Py_ssize_t given, n_src, last;
    int64_t cols;
    (void)self;
    UNLESS(p_gather && n == 8 && table(a[0], tab, &given, address) && map_of(a[1], &a_map, &n_src, &last) && n_src <= MAX_TABLE && integer(a[2], &w) &&
           handle_of(a[3], &w_map) && count_of(a[4], &cols) && handle_of(a[5], &out_map) && integer(a[6], &out) && integer(a[7], &stream));
    CALLED(p_gather(tab, a_map, w, w_map, cols, out_map, out, stream));
}

/* the current stream's handle, or None where torch has to be asked in full */
static PyObject *call_current_stream(PyObject *self, PyObject *none)
{
    void *stream;
    (void)self;
    (void)none;
    if (!stream_of(Py_None, &stream)) {
        if (PyErr_Occurred()) return NULL;
        Py_RETURN_NONE;
    }
    return PyLong_FromVoidPtr(stream);
}

/* library(addresses of amap_execute, _execute_multi, _gemm_fused, _gemm_fused_store, _gemm_mapped, _gemm_gather) */
static PyObject *call_library(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    void *p[6];
    (void)self;
    for (Py_ssize_t i = 0; i < 6; ++i)
        if (n != 6 || !integer(a[i], &p[i])) {
            PyErr_SetString(PyExc_TypeError, "six addresses");
            return NULL;
        }
    p_execute = (execute_fn)(uintptr_t)p[0];
    p_multi = (multi_fn)(uintptr_t)p[1];
    p_fused = (fused_fn)(uintptr_t)p[2];
    p_store = (store_fn)(uintptr_t)p[3];
    p_mapped = (mapped_fn)(uintptr_t)p[4];
    p_gather = (gather_fn)(uintptr_t)p[5];
    Py_RETURN_NONE;
}

/* torch(stream handle of a device, current device, whether CUDA is initialised) */
static PyObject *call_torch(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    (void)self;
    if (n != 3) {
        PyErr_SetString(PyExc_TypeError, "three functions");
        return NULL;
    }
    Py_INCREF(a[0]);
    Py_INCREF(a[1]);
    Py_INCREF(a[2]);
    Py_XSETREF(raw_stream, a[0]);
    Py_XSETREF(get_device, a[1]);
    Py_XSETREF(is_initialized, a[2]);
    initialized = 0;
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
    {"execute", (PyCFunction)(void (*)(void))call_execute, METH_FASTCALL, NULL},
    {"execute_multi", (PyCFunction)(void (*)(void))call_execute_multi, METH_FASTCALL, NULL},
    {"gemm", (PyCFunction)(void (*)(void))call_gemm, METH_FASTCALL, NULL},
    {"gather", (PyCFunction)(void (*)(void))call_gather, METH_FASTCALL, NULL},
    {"current_stream", call_current_stream, METH_NOARGS, NULL},
    {"library", (PyCFunction)(void (*)(void))call_library, METH_FASTCALL, NULL},
    {"torch", (PyCFunction)(void (*)(void))call_torch, METH_FASTCALL, NULL},
    {NULL, NULL, 0, NULL},
};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_amap_call", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__amap_call(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_at = PyUnicode_InternFromString("_at");
    s_reads = PyUnicode_InternFromString("_reads");
    if (!s_data_ptr || !s_at || !s_reads || pthread_atfork(NULL, NULL, forked)) return NULL;
    return PyModule_Create(&module);
}
