// CPython side of the binding: the run calls of include/bspmm.h without ctypes.
//
// A launch of a small batch costs the host about 2.4 us in hipLaunchKernel, and the Python around
// it used to cost twice that (torch.cuda.current_stream() 2.5 us, ctypes argument conversion
// 0.7 us, leading dimensions and pointers 0.7 us: 7.3 us a call in all, so every product of less
// than that on the GPU ran at the rate of the interpreter).  Here a call takes pointers and
// strides from the tensors with interned method names, asks PyTorch for the raw handle of the
// current stream, and calls the C ABI.  Only argument marshalling: no step of the path is here.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>

#include "../../include/bspmm.h"

namespace {

PyObject* s_data_ptr;        // interned method names
PyObject* s_stride;
PyObject* s_cuda_stream;
PyObject* g_check;           // bspmm._check(code, where): raises BspmmError
PyObject* g_ld;              // bspmm._ld(tensor, width): every case the fast path below leaves out
PyObject* g_raw_stream;      // torch._C._cuda_getCurrentRawStream
PyObject* g_device;          // torch._C._cuda_getDevice

// bspmm._native is set up by the module that imports it: setup(check, ld, raw_stream, get_device).
PyObject* setup(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    if (n != 4) {
        PyErr_SetString(PyExc_TypeError, "setup takes four callables");
        return nullptr;
    }
    PyObject** const slot[4] = {&g_check, &g_ld, &g_raw_stream, &g_device};
    for (int i = 0; i < 4; ++i) {
        Py_INCREF(a[i]);
        Py_XSETREF(*slot[i], a[i]);
    }
    Py_RETURN_NONE;
}

PyObject* call_method(PyObject* self, PyObject* name)
{
    PyObject* const args[1] = {self};
    return PyObject_VectorcallMethod(name, args, 1 | PY_VECTORCALL_ARGUMENTS_OFFSET, nullptr);
}

// Address of a tensor, an integer address, or NULL for None.
bool get_ptr(PyObject* o, void** out)
{
    *out = nullptr;
    if (o == Py_None) return true;
    if (PyLong_Check(o)) {
        *out = PyLong_AsVoidPtr(o);
        return !PyErr_Occurred();
    }
    PyObject* r = call_method(o, s_data_ptr);
    if (!r) return false;
    *out = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    return !PyErr_Occurred();
}

// Leading dimension of a row-major matrix: stride(0) of a two-dimensional tensor whose rows are
// at least `width` apart; anything else (fewer than two rows, other ranks, rows too close) is
// decided by the Python function (`own`: told the tensor's own width).
bool get_ld(PyObject* t, int64_t width, int64_t* ld, bool own = false)
{
    PyObject* st = call_method(t, s_stride);
    if (!st) return false;
    if (PyTuple_Check(st) && PyTuple_GET_SIZE(st) == 2) {
        *ld = PyLong_AsLongLong(PyTuple_GET_ITEM(st, 0));
        if (*ld >= width && !PyErr_Occurred()) {
            Py_DECREF(st);
            return true;
        }
        PyErr_Clear();
    }
    Py_DECREF(st);
    PyObject* w = own ? Py_NewRef(Py_None) : PyLong_FromLongLong(width);
    if (!w) return false;
    PyObject* const args[2] = {t, w};
    PyObject* r = PyObject_Vectorcall(g_ld, args, 2, nullptr);
    Py_DECREF(w);
    if (!r) return false;
    *ld = PyLong_AsLongLong(r);
    Py_DECREF(r);
    return !PyErr_Occurred();
}

// None: the current stream of the current device; an integer handle; or an object with one.
bool get_stream(PyObject* o, void** out)
{
    PyObject* r;
    if (o == Py_None) {
        PyObject* dev = PyObject_Vectorcall(g_device, nullptr, 0, nullptr);
        if (!dev) return false;
        PyObject* const args[1] = {dev};
        r = PyObject_Vectorcall(g_raw_stream, args, 1, nullptr);
        Py_DECREF(dev);
    } else if (PyLong_Check(o)) {
        Py_INCREF(o);
        r = o;
    } else {
        r = PyObject_GetAttr(o, s_cuda_stream);
    }
    if (!r) return false;
    *out = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    return !PyErr_Occurred();
}

bool get_i64(PyObject* o, int64_t* out)
{
    *out = PyLong_AsLongLong(o);
    return !(*out == -1 && PyErr_Occurred());
}

bool arity(const char* name, Py_ssize_t n, Py_ssize_t want)
{
    if (n == want) return true;
    PyErr_Format(PyExc_TypeError, "%s takes %zd arguments, got %zd", name, want, n);
    return false;
}

// `value` (a new reference to it) after a successful call, else the error bspmm._check raises.
PyObject* finish(int rc, const char* where, PyObject* value)
{
    if (rc != BSPMM_OK) {
        PyObject* r = PyObject_CallFunction(g_check, "is", rc, where);
        Py_XDECREF(r);
        return nullptr;
    }
    Py_INCREF(value);
    return value;
}

using RunFn = int (*)(bspmm_plan*, const float*, float*, int64_t, int64_t, void*);

// (other Python threads run while the launch is enqueued, as under ctypes)
template <RunFn FN>
int call(void* plan, void* in, void* out, int64_t ld_in, int64_t ld_out, void* stream)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = FN(static_cast<bspmm_plan*>(plan), static_cast<const float*>(in), static_cast<float*>(out), ld_in, ld_out,
            stream);
    Py_END_ALLOW_THREADS
    return rc;
}

// (plan, in, out, F, stream): leading dimensions from the tensors; returns `out`
template <RunFn FN>
PyObject* plan_product(const char* where, PyObject* const* a, Py_ssize_t n)
{
    if (!arity(where, n, 5)) return nullptr;
    void *plan, *in, *out, *stream;
    int64_t F, ld_in, ld_out;
    if (!get_i64(a[3], &F) || !get_ld(a[1], F, &ld_in) || !get_ld(a[2], F, &ld_out) || !get_ptr(a[0], &plan) ||
        !get_ptr(a[1], &in) || !get_ptr(a[2], &out) || !get_stream(a[4], &stream))
        return nullptr;
    return finish(call<FN>(plan, in, out, ld_in, ld_out, stream), where, a[2]);
}

// (plan, in, out, ld_in, ld_out, stream)
template <RunFn FN>
PyObject* product(const char* where, PyObject* const* a, Py_ssize_t n)
{
    if (!arity(where, n, 6)) return nullptr;
    void *plan, *in, *out, *stream;
    int64_t ld_in, ld_out;
    if (!get_ptr(a[0], &plan) || !get_ptr(a[1], &in) || !get_ptr(a[2], &out) || !get_i64(a[3], &ld_in) ||
        !get_i64(a[4], &ld_out) || !get_stream(a[5], &stream))
        return nullptr;
    return finish(call<FN>(plan, in, out, ld_in, ld_out, stream), where, Py_None);
}

PyObject* plan_run(PyObject*, PyObject* const* a, Py_ssize_t n) { return plan_product<bspmm_run>("bspmm_run", a, n); }
PyObject* plan_run_transposed(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return plan_product<bspmm_run_transposed>("bspmm_run_transposed", a, n);
}
PyObject* run(PyObject*, PyObject* const* a, Py_ssize_t n) { return product<bspmm_run>("bspmm_run", a, n); }
PyObject* run_transposed(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    return product<bspmm_run_transposed>("bspmm_run_transposed", a, n);
}

PyObject* gcn(PyObject* const* ptrs, int64_t ldx, int64_t ldw, int64_t ldy, PyObject* accumulate, PyObject* st,
              PyObject* value)
{
    void *plan, *x, *w, *bias, *y, *stream;
    const int acc = PyObject_IsTrue(accumulate);
    if (acc < 0 || !get_ptr(ptrs[0], &plan) || !get_ptr(ptrs[1], &x) || !get_ptr(ptrs[2], &w) ||
        !get_ptr(ptrs[3], &bias) || !get_ptr(ptrs[4], &y) || !get_stream(st, &stream))
        return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = bspmm_run_gcn(static_cast<bspmm_plan*>(plan), static_cast<const float*>(x), ldx, static_cast<const float*>(w),
                       ldw, static_cast<const float*>(bias), static_cast<float*>(y), ldy, acc, stream);
    Py_END_ALLOW_THREADS
    return finish(rc, "bspmm_run_gcn", value);
}

// (plan, X, W, bias, Y, n_X, F, accumulate, stream): leading dimensions from the tensors; returns Y
PyObject* plan_run_gcn(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    int64_t nx, F, ldx, ldw, ldy;
    if (!arity("bspmm_run_gcn", n, 9) || !get_i64(a[5], &nx) || !get_i64(a[6], &F) || !get_ld(a[1], nx, &ldx, true) ||
        !get_ld(a[2], F, &ldw) || !get_ld(a[4], F, &ldy))
        return nullptr;
    return gcn(a, ldx, ldw, ldy, a[7], a[8], a[4]);
}

// (plan, X, W, bias, Y, ldx, ldw, ldy, accumulate, stream)
PyObject* run_gcn(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    int64_t ldx, ldw, ldy;
    if (!arity("bspmm_run_gcn", n, 10) || !get_i64(a[5], &ldx) || !get_i64(a[6], &ldw) || !get_i64(a[7], &ldy))
        return nullptr;
    return gcn(a, ldx, ldw, ldy, a[8], a[9], Py_None);
}

#define FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(setup), FAST(plan_run), FAST(plan_run_transposed), FAST(plan_run_gcn), FAST(run),
                         FAST(run_transposed), FAST(run_gcn), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "Run calls of libbspmm without ctypes.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_stride = PyUnicode_InternFromString("stride");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (!s_data_ptr || !s_stride || !s_cuda_stream) return nullptr;
    return PyModule_Create(&module);
}
