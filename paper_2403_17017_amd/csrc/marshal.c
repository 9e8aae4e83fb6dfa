/* Argument marshalling of the asynchronous calls for the Python binding.  These calls only
 * enqueue a few microseconds of GPU work, so what the interpreter spends on describing them is
 * part of their cost: through ctypes (a Structure built per call, seven converted arguments) and
 * a torch.cuda.Stream object about 5 us a call, here about 2 (4096 rows of 16, one
 * seer_spmv_auto 12.3 -> 9.2 us; 19 prepared products of 2.5 M nonzeros 174 -> 93 us).
 * Everything is read from the objects anew on every call; nothing is kept.  The library's
 * functions are handed over as addresses (bind), so the module links against nothing. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "../../include/seer.h"

static int (*f_spmv)(int, const seer_csr *, const float *, float *, void *, size_t, void *);
static int (*f_auto)(const seer_csr *, const seer_tree *, const float *, float *, void *, size_t, void *);
static int (*f_model)(const seer_csr *, const seer_model *, const float *, float *, void *, size_t, void *, int *, int *);
static int (*f_prepared)(const seer_plan *, const seer_csr *, const float *, float *, void *, size_t, void *);

static PyObject *s_rows, *s_cols, *s_nnz, *s_row_ptr, *s_col_idx, *s_values, *s_data_ptr, *s_numel;

/* What ctypes takes: for a size anything that is an integer (None and floats raise TypeError),
 * reduced to the width of the parameter; for an address an int, or None for a null pointer. */
static int as_size(PyObject *o, uint64_t *out)
{
    *out = (uint64_t)PyLong_AsUnsignedLongLongMask(o);
    return PyErr_Occurred() ? -1 : 0;
}

static int as_address(PyObject *o, uint64_t *out)
{
    if (o == Py_None) { *out = 0; return 0; }
    if (!PyLong_Check(o)) {
        PyErr_Format(PyExc_TypeError, "an address must be an int, not %.100s", Py_TYPE(o)->tp_name);
        return -1;
    }
    return as_size(o, out);
}

/* Takes over the reference r (null: an exception is set). */
static int taken(PyObject *r, int (*as)(PyObject *, uint64_t *), uint64_t *out)
{
    if (!r) return -1;
    const int rc = as(r, out);
    Py_DECREF(r);
    return rc;
}

static int size_attr(PyObject *o, PyObject *name, uint64_t *out) { return taken(PyObject_GetAttr(o, name), as_size, out); }

static int address_of(PyObject *tensor, uint64_t *out)
{
    return taken(PyObject_CallMethodNoArgs(tensor, s_data_ptr), as_address, out);
}

static int address_attr(PyObject *o, PyObject *name, uint64_t *out)
{
    PyObject *t = PyObject_GetAttr(o, name);
    if (!t) return -1;
    const int rc = address_of(t, out);
    Py_DECREF(t);
    return rc;
}

/* DeviceCSR.c_struct() */
static int csr_of(PyObject *A, seer_csr *c)
{
    uint64_t rows, cols, nnz, rp, ci = 0, va = 0;
    if (size_attr(A, s_rows, &rows) || size_attr(A, s_cols, &cols) || size_attr(A, s_nnz, &nnz) ||
        address_attr(A, s_row_ptr, &rp))
        return -1;
    if (nnz && (address_attr(A, s_col_idx, &ci) || address_attr(A, s_values, &va))) return -1;
    c->rows = (int32_t)rows;
    c->cols = (int32_t)cols;
    c->nnz = (int32_t)nnz;
    c->row_ptr = (const int32_t *)(uintptr_t)rp;
    c->col_idx = (const int32_t *)(uintptr_t)ci;
    c->values = (const float *)(uintptr_t)va;
    return 0;
}

/* x, y, workspace (may be None) and the stream handle: arguments 2 .. 5 of every call below */
typedef struct {
    seer_csr csr;
    uint64_t handle, x, y, ws, ws_bytes, stream;
} call_args;

static int parse(PyObject *const *a, Py_ssize_t n, call_args *c)
{
    if (n != 6) {
        PyErr_SetString(PyExc_TypeError, "expected (handle, matrix, x, y, workspace, stream)");
        return -1;
    }
    c->ws = c->ws_bytes = 0;
    if (as_size(a[0], &c->handle) || csr_of(a[1], &c->csr) || address_of(a[2], &c->x) || address_of(a[3], &c->y)) return -1;
    if (a[4] != Py_None &&
        (address_of(a[4], &c->ws) || taken(PyObject_CallMethodNoArgs(a[4], s_numel), as_size, &c->ws_bytes)))
        return -1;
    return as_size(a[5], &c->stream);
}

#define P(T, v) ((T)(uintptr_t)(v))

static PyObject *m_spmv(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    call_args c;
    int rc;
    if (parse(a, n, &c)) return NULL;
    Py_BEGIN_ALLOW_THREADS
    rc = f_spmv((int)c.handle, &c.csr, P(const float *, c.x), P(float *, c.y), P(void *, c.ws), (size_t)c.ws_bytes,
                P(void *, c.stream));
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

static PyObject *m_auto(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    call_args c;
    int rc;
    if (parse(a, n, &c)) return NULL;
    Py_BEGIN_ALLOW_THREADS
    rc = f_auto(&c.csr, P(const seer_tree *, c.handle), P(const float *, c.x), P(float *, c.y), P(void *, c.ws),
                (size_t)c.ws_bytes, P(void *, c.stream));
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

static PyObject *m_model(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    call_args c;
    int rc, path = -1, kid = -1;
    if (parse(a, n, &c)) return NULL;
    Py_BEGIN_ALLOW_THREADS
    rc = f_model(&c.csr, P(const seer_model *, c.handle), P(const float *, c.x), P(float *, c.y), P(void *, c.ws),
                 (size_t)c.ws_bytes, P(void *, c.stream), &path, &kid);
    Py_END_ALLOW_THREADS
    return Py_BuildValue("(iii)", rc, path, kid);
}

static PyObject *m_prepared(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    call_args c;
    int rc;
    if (parse(a, n, &c)) return NULL;
    Py_BEGIN_ALLOW_THREADS
    rc = f_prepared(P(const seer_plan *, c.handle), &c.csr, P(const float *, c.x), P(float *, c.y), P(void *, c.ws),
                    (size_t)c.ws_bytes, P(void *, c.stream));
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

static PyObject *m_bind(PyObject *self, PyObject *args)
{
    unsigned long long spmv, autos, model, prepared;
    if (!PyArg_ParseTuple(args, "KKKK", &spmv, &autos, &model, &prepared)) return NULL;
    f_spmv = P(int (*)(int, const seer_csr *, const float *, float *, void *, size_t, void *), spmv);
    f_auto = P(int (*)(const seer_csr *, const seer_tree *, const float *, float *, void *, size_t, void *), autos);
    f_model = P(int (*)(const seer_csr *, const seer_model *, const float *, float *, void *, size_t, void *, int *, int *), model);
    f_prepared = P(int (*)(const seer_plan *, const seer_csr *, const float *, float *, void *, size_t, void *), prepared);
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
    {"bind", m_bind, METH_VARARGS, "bind(spmv, spmv_auto, spmv_model, spmv_prepared): addresses of the library's functions"},
    {"spmv", (PyCFunction)(void (*)(void))m_spmv, METH_FASTCALL, "spmv(kernel_id, A, x, y, workspace, stream) -> status"},
    {"spmv_auto", (PyCFunction)(void (*)(void))m_auto, METH_FASTCALL, "spmv_auto(tree address, A, x, y, workspace, stream) -> status"},
    {"spmv_model", (PyCFunction)(void (*)(void))m_model, METH_FASTCALL,
     "spmv_model(model address, A, x, y, workspace, stream) -> (status, path, kernel id)"},
    {"spmv_prepared", (PyCFunction)(void (*)(void))m_prepared, METH_FASTCALL,
     "spmv_prepared(plan address, A, x, y, workspace, stream) -> status"},
    {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", "argument marshalling of the asynchronous calls", -1,
                                    methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__marshal(void)
{
    s_rows = PyUnicode_InternFromString("rows");
    s_cols = PyUnicode_InternFromString("cols");
    s_nnz = PyUnicode_InternFromString("nnz");
    s_row_ptr = PyUnicode_InternFromString("row_ptr");
    s_col_idx = PyUnicode_InternFromString("col_idx");
    s_values = PyUnicode_InternFromString("values");
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_numel = PyUnicode_InternFromString("numel");
    if (!s_rows || !s_cols || !s_nnz || !s_row_ptr || !s_col_idx || !s_values || !s_data_ptr || !s_numel) return NULL;
    return PyModule_Create(&module);
}
