// Argument marshalling of the calls a program makes most often, for the Python binding: checks the tensors, reads
// pointers, sizes and pitches and calls libamulet.so, in place of some thirty attribute reads and calls from
// Python.  It takes ordinary arguments only and returns None for anything else, without calling the library: the
// binding then goes through its own checks, which word the errors.  Per call of 64^3, the launch (2.7)
// included, us on the host: 6.3 from Python, 3.3 from here.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include "amulet.h"

namespace {

PyObject *g_get_device, *g_raw_stream;   // torch._C: the current device's index, the raw handle of its current stream

struct Mat {
    void *p;
    int64_t rows, cols, ld;
};

// a dense device tensor of this type
const at::Tensor *device_tensor(PyObject *o, at::ScalarType type)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage() || t.scalar_type() != type) return nullptr;
    return &t;
}

// ... of two dimensions with unit column stride
bool matrix(PyObject *o, at::ScalarType type, Mat &m)
{
    const at::Tensor *t = device_tensor(o, type);
    if (!t || t->dim() != 2) return false;
    m.rows = t->size(0);
    m.cols = t->size(1);
    if (m.cols > 1 && t->stride(1) != 1) return false;
    m.ld = m.rows <= 1 ? m.cols : t->stride(0);
    if (m.ld <= 0) m.ld = 1;
    m.p = t->data_ptr();
    return true;
}

// ... of n contiguous values
bool values(PyObject *o, at::ScalarType type, int64_t n, void *&p)
{
    const at::Tensor *t = device_tensor(o, type);
    if (!t || !t->is_contiguous() || t->numel() != n) return false;
    p = t->data_ptr();
    return true;
}

bool integer(PyObject *o, int &v)
{
    if (!PyLong_Check(o)) return false;
    const long n = PyLong_AsLong(o);
    if (n < -0x7fffffffL || n > 0x7fffffffL) {
        PyErr_Clear();
        return false;
    }
    v = (int)n;
    return true;
}

bool stream_handle(PyObject *o, void *&s)
{
    PyObject *handle;
    if (o == Py_None) {
        PyObject *dev = PyObject_CallNoArgs(g_get_device);
        if (!dev) {
            PyErr_Clear();
            return false;
        }
        handle = PyObject_CallOneArg(g_raw_stream, dev);
        Py_DECREF(dev);
    } else if (PyLong_Check(o)) {
        handle = o;
        Py_INCREF(o);
    } else {
        handle = PyObject_GetAttrString(o, "cuda_stream");
    }
    if (!handle || !PyLong_Check(handle)) {
        PyErr_Clear();
        Py_XDECREF(handle);
        return false;
    }
    s = PyLong_AsVoidPtr(handle);
    Py_DECREF(handle);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

PyObject *not_here() { Py_RETURN_NONE; }

template <class F> PyObject *status(F call)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// (task, A, B, params, R, stream)
PyObject *mmlike_f32(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Mat A, B, R;
    int task;
    void *params = nullptr, *s;
    if (n != 6 || !integer(a[0], task) || !matrix(a[1], at::kFloat, A) || !matrix(a[2], at::kFloat, B) || !matrix(a[4], at::kFloat, R) ||
        A.cols != B.rows || A.rows != R.rows || B.cols != R.cols)
        return not_here();
    const int rows = task == AMULET_DISCOUNT ? 2 : task == AMULET_BOOST || task == AMULET_COUNT_GT ? 1 : 0;
    if (rows > 0 && a[3] != Py_None && !values(a[3], at::kFloat, rows * R.cols, params)) return not_here();
    if (!stream_handle(a[5], s)) return not_here();
    return status([&] {
        return amulet_mmlike_f32(task, R.rows, R.cols, A.cols, (const float *)A.p, A.ld, (const float *)B.p, B.ld, (const float *)params,
                                 (float *)R.p, R.ld, s);
    });
}

// operands, thresholds and discounts of a general-form call
struct General {
    Mat A, B, R;
    int task, form, ta, tb, shape;
    int64_t K, ldt;
    void *thres, *dis, *stream;
};

// (task, A, B, thres, dis, R, thres_form, trans_a, trans_b, shape, stream)
bool general(PyObject *const *a, Py_ssize_t n, at::ScalarType type, General &g)
{
    if (n != 11 || !integer(a[0], g.task) || !integer(a[6], g.form) || !integer(a[7], g.ta) || !integer(a[8], g.tb) || !integer(a[9], g.shape) ||
        !matrix(a[1], type, g.A) || !matrix(a[2], type, g.B) || !matrix(a[5], type, g.R))
        return false;
    g.K = g.ta ? g.A.rows : g.A.cols;
    if ((g.ta ? g.A.cols : g.A.rows) != g.R.rows || (g.tb ? g.B.cols : g.B.rows) != g.K || (g.tb ? g.B.rows : g.B.cols) != g.R.cols)
        return false;
    g.thres = g.dis = nullptr;
    g.ldt = 0;
    if (g.task != AMULET_IDENTITY) {
        if (g.form == AMULET_THRES_ELEM) {
            Mat t;
            if (!matrix(a[3], type, t) || t.rows != g.R.rows || t.cols != g.R.cols) return false;
            g.thres = t.p;
            g.ldt = t.ld;
        } else {
            const int64_t want = g.form == AMULET_THRES_COL ? g.R.cols : g.form == AMULET_THRES_ROW ? g.R.rows : g.form == AMULET_THRES_CONST ? 1 : -1;
            if (!values(a[3], type, want, g.thres)) return false;
        }
    }
    if (g.task == AMULET_DISCOUNT && !values(a[4], type, g.R.cols, g.dis)) return false;
    return stream_handle(a[10], g.stream);
}

PyObject *mmlike_f32_general(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    General g;
    if (!general(a, n, at::kFloat, g)) return not_here();
    return status([&] {
        return amulet_mmlike_f32_general(g.task, g.form, g.ta, g.tb, g.shape, g.R.rows, g.R.cols, g.K, (const float *)g.A.p, g.A.ld,
                                         (const float *)g.B.p, g.B.ld, (const float *)g.thres, g.ldt, (const float *)g.dis, (float *)g.R.p,
                                         g.R.ld, g.stream);
    });
}

PyObject *mmlike_f64(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    General g;
    if (!general(a, n, at::kDouble, g)) return not_here();
    return status([&] {
        return amulet_mmlike_f64_shape(g.task, g.shape, g.form, g.ta, g.tb, g.R.rows, g.R.cols, g.K, (const double *)g.A.p, g.A.ld,
                                       (const double *)g.B.p, g.B.ld, (const double *)g.thres, g.ldt, (const double *)g.dis, (double *)g.R.p,
                                       g.R.ld, g.stream);
    });
}

bool count_operands(PyObject *const *a, bool ta, bool tb, Mat &A, Mat &B, Mat &R)
{
    return matrix(a[0], at::kChar, A) && matrix(a[1], at::kChar, B) && matrix(a[2], at::kInt, R) && (ta ? A.cols : A.rows) == R.rows &&
           (tb ? B.rows : B.cols) == R.cols && (ta ? A.rows : A.cols) == (tb ? B.cols : B.rows);
}

// (A, B, R, stream)
PyObject *count_i8(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Mat A, B, R;
    void *s;
    if (n != 4 || !count_operands(a, false, false, A, B, R) || !stream_handle(a[3], s)) return not_here();
    return status([&] {
        return amulet_count_i8(R.rows, R.cols, A.cols, (const int8_t *)A.p, A.ld, (const int8_t *)B.p, B.ld, (int32_t *)R.p, R.ld, s);
    });
}

// (A, B, R, shape, stream)
PyObject *count_i8_assign(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Mat A, B, R;
    int shape;
    void *s;
    if (n != 5 || !count_operands(a, false, false, A, B, R) || !integer(a[3], shape) || !stream_handle(a[4], s)) return not_here();
    return status([&] {
        return amulet_count_i8_assign(shape, R.rows, R.cols, A.cols, (const int8_t *)A.p, A.ld, (const int8_t *)B.p, B.ld, (int32_t *)R.p, R.ld, s);
    });
}

// (A, B, R, workspace, trans_a, trans_b, stream)
PyObject *count_i8_general(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    Mat A, B, R;
    int ta, tb;
    void *s, *w = nullptr;
    size_t bytes = 0;
    if (n != 7 || !integer(a[4], ta) || !integer(a[5], tb) || !count_operands(a, ta, tb, A, B, R)) return not_here();
    if (a[3] != Py_None) {
        if (!THPVariable_CheckExact(a[3])) return not_here();
        const at::Tensor &t = THPVariable_Unpack(a[3]);
        if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage() || !t.is_contiguous()) return not_here();
        w = t.data_ptr();
        bytes = t.nbytes();
    }
    if (!stream_handle(a[6], s)) return not_here();
    return status([&] {
        return amulet_count_i8_general(ta, tb, R.rows, R.cols, ta ? A.rows : A.cols, (const int8_t *)A.p, A.ld, (const int8_t *)B.p, B.ld,
                                       (int32_t *)R.p, R.ld, w, bytes, s);
    });
}

#define MARSHAL(NAME) {#NAME, (PyCFunction)(void (*)(void))NAME, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {MARSHAL(mmlike_f32),      MARSHAL(mmlike_f32_general), MARSHAL(mmlike_f64), MARSHAL(count_i8),
                         MARSHAL(count_i8_assign), MARSHAL(count_i8_general),   {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal()
{
    PyObject *c = PyImport_ImportModule("torch._C");
    if (!c) return nullptr;
    g_get_device = PyObject_GetAttrString(c, "_cuda_getDevice");
    g_raw_stream = g_get_device ? PyObject_GetAttrString(c, "_cuda_getCurrentRawStream") : nullptr;
    Py_DECREF(c);
    if (!g_raw_stream) {   // a torch without them: the binding does without this module
        PyErr_SetString(PyExc_ImportError, "torch has no raw stream handles");
        return nullptr;
    }
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for_torch", BUILT_FOR_TORCH) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
