// binding.cpp -- the marshalling of coda.py in C: tensors to coda_mat / coda_epi_op, and the calls of the entry points that a
// program makes for every layer.  A call on a small problem is host work (its kernels take a few microseconds), and most of
// that was the interpreter and ctypes: a coda_gemm with four ops 10 us before the launch, here 4.2; a 256 x 512 x 256 linear layer of
// four calls 22.2 -> 18.9 us a pass.  Tensors are asked through their Python methods, so whatever answers to them is accepted as
// before; arguments of other types than the usual ones go to the ctypes function of the same name.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "../../include/coda.h"

#include <string.h>

namespace {

PyObject *s_data_ptr, *s_stride, *s_shape, *s_dtype, *s_keep;
static_assert(sizeof(coda_mat) == 40 && sizeof(coda_epi_op) == 96, "the layouts that coda.py mirrors");

// t.data_ptr() as a pointer
bool data_ptr(PyObject *t, void **out)
{
    PyObject *r = PyObject_CallMethodNoArgs(t, s_data_ptr);
    if (!r) return false;
    bool ok = true;
    if (r == Py_None) *out = nullptr;
    else if (PyLong_Check(r)) *out = reinterpret_cast<void *>(PyLong_AsUnsignedLongLongMask(r));
    else {
        PyErr_SetString(PyExc_TypeError, "data_ptr() is no address");
        ok = false;
    }
    Py_DECREF(r);
    return ok && !PyErr_Occurred();
}

// Item i of a sequence as a 64-bit integer
bool item(PyObject *seq, Py_ssize_t i, int64_t *out)
{
    PyObject *o = PySequence_GetItem(seq, i);
    if (!o) return false;
    *out = PyLong_AsLongLong(o);
    Py_DECREF(o);
    return !(*out == -1 && PyErr_Occurred());
}

// op(type, kind, flags, in_, out, out2, in2, in3, in4, out3, i0, i1) -> a coda_epi_op that owns its tensors
PyObject *op(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 12) return PyErr_Format(PyExc_TypeError, "op takes 12 arguments");
    coda_epi_op v;
    memset(&v, 0, sizeof v);
    v.kind = (int32_t)PyLong_AsLong(a[1]);
    v.flags = (uint32_t)PyLong_AsLong(a[2]);
    const int i0 = PyObject_IsTrue(a[10]), i1 = PyObject_IsTrue(a[11]);
    if (i0 < 0 || i1 < 0) return nullptr;
    if (i0 || i1) {
        if (!PyLong_Check(a[10]) || !PyLong_Check(a[11])) return PyErr_Format(PyExc_TypeError, "int expected");
        v.i0 = (int64_t)PyLong_AsUnsignedLongLongMask(a[10]);        // past 64 bits: as a ctypes field takes it
        v.i1 = (int64_t)PyLong_AsUnsignedLongLongMask(a[11]);
    }
    if (PyErr_Occurred()) return nullptr;
    const void **const at[7] = {(const void **)&v.in, (const void **)&v.out, (const void **)&v.out2, (const void **)&v.in2, (const void **)&v.in3,
                                (const void **)&v.in4, (const void **)&v.out3};
    int64_t *const ld[2] = {&v.ld_in, &v.ld_out};
    for (int i = 0; i < 7; ++i) {
        PyObject *t = a[3 + i];
        if (t == Py_None) continue;
        if (!data_ptr(t, (void **)at[i])) return nullptr;
        if (i >= 2) continue;
        PyObject *pitch = PyObject_CallMethodNoArgs(t, s_stride);
        if (!pitch) return nullptr;
        const Py_ssize_t dims = PySequence_Size(pitch);
        const bool ok = dims >= 0 && (dims != 2 || item(pitch, 0, ld[i]));
        Py_DECREF(pitch);
        if (!ok) return nullptr;
    }
    PyObject *self = PyObject_CallNoArgs(a[0]);
    if (!self) return nullptr;
    Py_buffer view;
    PyObject *keep = nullptr;
    if (PyObject_GetBuffer(self, &view, PyBUF_WRITABLE) == 0) {
        const bool fits = view.len == (Py_ssize_t)sizeof v;
        if (fits) memcpy(view.buf, &v, sizeof v);
        else PyErr_SetString(PyExc_TypeError, "not a coda_epi_op");
        PyBuffer_Release(&view);
        if (fits && (keep = PyTuple_Pack(7, a[3], a[4], a[5], a[6], a[7], a[8], a[9])) && PyObject_SetAttr(self, s_keep, keep) == 0) {
            Py_DECREF(keep);
            return self;
        }
    }
    Py_XDECREF(keep);
    Py_DECREF(self);
    return nullptr;
}

bool fill_mat(PyObject *t, bool trans, PyObject *dtypes, coda_mat *m)
{
    memset(m, 0, sizeof *m);
    int64_t step = 1;
    PyObject *shape = PyObject_GetAttr(t, s_shape);
    if (!shape) return false;
    const Py_ssize_t dims = PySequence_Size(shape);
    bool ok = dims >= 0;
    if (ok && dims != 2) {
        PyErr_SetString(PyExc_AssertionError, "row-major 2-D tensor expected");
        ok = false;
    }
    ok = ok && item(shape, 0, &m->rows) && item(shape, 1, &m->cols);
    Py_DECREF(shape);
    if (!ok) return false;
    PyObject *pitch = PyObject_CallMethodNoArgs(t, s_stride);
    if (!pitch) return false;
    ok = item(pitch, 0, &m->ld) && item(pitch, 1, &step);
    Py_DECREF(pitch);
    if (!ok) return false;
    if (m->cols > 1 && step != 1) {
        PyErr_SetString(PyExc_AssertionError, "row-major 2-D tensor expected");
        return false;
    }
    PyObject *dtype = PyObject_GetAttr(t, s_dtype);
    if (!dtype) return false;
    PyObject *code = PyDict_GetItemWithError(dtypes, dtype);      // borrowed
    Py_DECREF(dtype);
    if (!code && PyErr_Occurred()) return false;
    m->dtype = code ? (int32_t)PyLong_AsLong(code) : (int32_t)CODA_F32;
    m->trans = trans ? 1 : 0;
    void *ptr;
    if (!data_ptr(t, &ptr)) return false;
    m->ptr = ptr;
    return true;
}

// mat(t, trans, dtypes) -> the bytes of a coda_mat
PyObject *mat(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 3) return PyErr_Format(PyExc_TypeError, "mat takes 3 arguments");
    const int trans = PyObject_IsTrue(a[1]);
    coda_mat m;
    if (trans < 0 || !fill_mat(a[0], trans, a[2], &m)) return nullptr;
    return PyBytes_FromStringAndSize(reinterpret_cast<const char *>(&m), sizeof m);
}

// gemm_mats(A, B, transA, transB, dtypes) -> (M, N, K, bytes of A, bytes of B)
PyObject *gemm_mats(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 5) return PyErr_Format(PyExc_TypeError, "gemm_mats takes 5 arguments");
    const int ta = PyObject_IsTrue(a[2]), tb = PyObject_IsTrue(a[3]);
    coda_mat A, B;
    if (ta < 0 || tb < 0 || !fill_mat(a[0], ta, a[4], &A) || !fill_mat(a[1], tb, a[4], &B)) return nullptr;
    return Py_BuildValue("LLLy#y#", (long long)(ta ? A.cols : A.rows), (long long)(tb ? B.rows : B.cols), (long long)(ta ? A.rows : A.cols),
                         reinterpret_cast<const char *>(&A), (Py_ssize_t)sizeof A, reinterpret_cast<const char *>(&B), (Py_ssize_t)sizeof B);
}

// prog(ops, type) -> the bytes of the list's coda_epi_op, one after the other; None if there is anything else in it
PyObject *prog(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 2 || !PyList_Check(a[0])) return PyErr_Format(PyExc_TypeError, "prog takes a list and a type");
    const Py_ssize_t ops = PyList_GET_SIZE(a[0]);
    PyObject *out = PyBytes_FromStringAndSize(nullptr, (Py_ssize_t)sizeof(coda_epi_op) * (ops > 0 ? ops : 1));
    if (!out) return nullptr;
    char *to = PyBytes_AS_STRING(out);
    if (ops == 0) memset(to, 0, sizeof(coda_epi_op));
    for (Py_ssize_t i = 0; i < ops; ++i, to += sizeof(coda_epi_op)) {
        PyObject *o = PyList_GetItem(a[0], i);                      // borrowed; checked, should the list change meanwhile
        Py_buffer view;
        if (!o) {
            Py_DECREF(out);
            return nullptr;
        }
        if (Py_TYPE(o) != reinterpret_cast<PyTypeObject *>(a[1])) {
            Py_DECREF(out);
            Py_RETURN_NONE;
        }
        if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) {
            Py_DECREF(out);
            return nullptr;
        }
        memcpy(to, view.buf, sizeof(coda_epi_op));
        PyBuffer_Release(&view);
    }
    return out;
}

// ---- the calls.  Arguments are pointers (an address, None, the bytes of a structure) and numbers; anything else takes the ctypes function.
struct Args {
    PyObject *const *a;
    bool usual = true;
    template <class T>
    T *ptr(int i)
    {
        PyObject *o = a[i];
        if (o == Py_None) return nullptr;
        if (PyLong_CheckExact(o)) return reinterpret_cast<T *>(PyLong_AsUnsignedLongLongMask(o));
        if (PyBytes_CheckExact(o)) return reinterpret_cast<T *>(PyBytes_AS_STRING(o));
        usual = false;
        return nullptr;
    }
    int64_t num(int i)
    {
        if (!PyLong_CheckExact(a[i])) {
            usual = false;
            return 0;
        }
        int over = 0;
        const long long v = PyLong_AsLongLongAndOverflow(a[i], &over);
        if (over) usual = false;
        return v;
    }
    float real(int i)
    {
        if (PyFloat_CheckExact(a[i])) return (float)PyFloat_AS_DOUBLE(a[i]);
        usual = false;
        return 0.0f;
    }
};

enum Call { GEMM, ROW_FINALIZE, ROW_SUMSQ, COL_FINALIZE, LSE_FINALIZE, CALLS };
constexpr int ARITY[CALLS] = {10, 8, 3, 5, 8};
PyObject *g_ctypes[CALLS];           // set once, when coda.py is imported

template <int CALL>
PyObject *call(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Args x{a};
    coda_status st = CODA_OK;
    x.usual = n == ARITY[CALL];
#define CODA_RUN(...)              \
    if (x.usual) {                 \
        Py_BEGIN_ALLOW_THREADS     \
        st = __VA_ARGS__;          \
        Py_END_ALLOW_THREADS       \
    }
    if (x.usual) {
        void *stream = x.ptr<void>(0);
        if constexpr (CALL == GEMM) {
            const int64_t M = x.num(1), N = x.num(2), K = x.num(3), ops = x.num(7), bytes = x.num(9);
            const coda_mat *A = x.ptr<const coda_mat>(4), *B = x.ptr<const coda_mat>(5);
            const coda_epi_op *p = x.ptr<const coda_epi_op>(6);
            void *ws = x.ptr<void>(8);
            if (ops < 0 || ops > INT32_MAX || bytes < 0) x.usual = false;
            CODA_RUN(coda_gemm(stream, M, N, K, A, B, p, (int32_t)ops, ws, (size_t)bytes))
        } else if constexpr (CALL == ROW_FINALIZE) {
            const float *parts = x.ptr<const float>(1);
            const int64_t M = x.num(2), nblk = x.num(3), d = x.num(6);
            float *sum = x.ptr<float>(4), *rstd = x.ptr<float>(5);
            const float eps = x.real(7);
            CODA_RUN(coda_row_finalize(stream, parts, M, nblk, sum, rstd, d, eps))
        } else if constexpr (CALL == ROW_SUMSQ) {
            const coda_mat *X = x.ptr<const coda_mat>(1);
            float *out = x.ptr<float>(2);
            CODA_RUN(coda_row_sumsq(stream, X, out))
        } else if constexpr (CALL == COL_FINALIZE) {
            const float *parts = x.ptr<const float>(1);
            const int64_t N = x.num(2), nblk = x.num(3);
            float *out = x.ptr<float>(4);
            CODA_RUN(coda_col_finalize(stream, parts, N, nblk, out))
        } else {
            const float *pmax = x.ptr<const float>(1), *psum = x.ptr<const float>(2), *ztgt = x.ptr<const float>(5);
            const int64_t M = x.num(3), nblk = x.num(4);
            float *lse = x.ptr<float>(6), *loss = x.ptr<float>(7);
            CODA_RUN(coda_lse_finalize(stream, pmax, psum, M, nblk, ztgt, lse, loss))
        }
    }
#undef CODA_RUN
    if (x.usual) return PyLong_FromLong(st);
    if (!g_ctypes[CALL]) return PyErr_Format(PyExc_TypeError, "unexpected arguments");
    return PyObject_Vectorcall(g_ctypes[CALL], a, (size_t)n, nullptr);
}

// ctypes_calls(gemm, row_finalize, row_sumsq, col_finalize, lse_finalize)
PyObject *ctypes_calls(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != CALLS) return PyErr_Format(PyExc_TypeError, "one function for every call");
    for (int i = 0; i < CALLS; ++i) {
        Py_INCREF(a[i]);
        Py_XSETREF(g_ctypes[i], a[i]);
    }
    Py_RETURN_NONE;
}

#define CODA_FAST(name, fn) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(fn)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {CODA_FAST("op", op),
                         CODA_FAST("mat", mat),
                         CODA_FAST("gemm_mats", gemm_mats),
                         CODA_FAST("prog", prog),
                         CODA_FAST("ctypes_calls", ctypes_calls),
                         CODA_FAST("coda_gemm", call<GEMM>),
                         CODA_FAST("coda_row_finalize", call<ROW_FINALIZE>),
                         CODA_FAST("coda_row_sumsq", call<ROW_SUMSQ>),
                         CODA_FAST("coda_col_finalize", call<COL_FINALIZE>),
                         CODA_FAST("coda_lse_finalize", call<LSE_FINALIZE>),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_stride = PyUnicode_InternFromString("stride");
    s_shape = PyUnicode_InternFromString("shape");
    s_dtype = PyUnicode_InternFromString("dtype");
    s_keep = PyUnicode_InternFromString("_keep");
    if (!s_data_ptr || !s_stride || !s_shape || !s_dtype || !s_keep) return nullptr;
    return PyModule_Create(&module);
}
