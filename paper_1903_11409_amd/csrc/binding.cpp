// CPython side of the binding: plan creation and the run calls of include/bspmm.h without ctypes.
//
// A launch of a small batch costs the host about 2.4 us in hipLaunchKernel, and the Python around
// it used to cost twice that (torch.cuda.current_stream() 2.5 us, ctypes argument conversion
// 0.7 us, leading dimensions and pointers 0.7 us: 7.3 us a call in all, so every product of less
// than that on the GPU ran at the rate of the interpreter).  Here pointers, strides and the current
// stream come straight from PyTorch's C++ objects.  Making a plan from a data loader's host arrays
// took 110 us for 128 graphs: three blocking copies, ctypes views of ten arrays, and the host
// schedule; now the arrays and the plan's tables go over in one copy (staging.hpp) behind one call.
// The differentiable product (autograd.py) is here for the same reason.
// Only argument marshalling: no step of the path is here.
#define PY_SSIZE_T_CLEAN
#define NPY_NO_DEPRECATED_API NPY_1_7_API_VERSION
#include <Python.h>
#include <numpy/arrayobject.h>

#include <ATen/core/grad_mode.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/zeros.h>
#include <c10/core/impl/PyInterpreter.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/function.h>
#include <torch/csrc/autograd/functions/utils.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>
#include <ATen/PythonTorchFunctionTLS.h>

#include <cstdint>
#include <cstring>
#include <exception>

#include "plan_api.hpp"

namespace {

PyObject* s_data_ptr;        // interned method names
PyObject* s_cuda_stream;
PyObject* s_handle;
PyObject* g_check;           // bspmm._check(code, where): raises BspmmError
PyObject* g_ld;              // bspmm._ld(tensor, width): every case the fast path below leaves out

// bspmm._native is set up by the module that imports it: setup(check, ld).
PyObject* setup(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    if (n != 2) {
        PyErr_SetString(PyExc_TypeError, "setup takes two callables");
        return nullptr;
    }
    PyObject** const slot[2] = {&g_check, &g_ld};
    for (int i = 0; i < 2; ++i) {
        Py_INCREF(a[i]);
        Py_XSETREF(*slot[i], a[i]);
    }
    Py_RETURN_NONE;
}

bool is_tensor(PyObject* o) { return THPVariable_CheckExact(o); }

// Address of a tensor, an integer address, or NULL for None.
bool get_ptr(PyObject* o, void** out)
{
    *out = nullptr;
    if (is_tensor(o)) {
        *out = THPVariable_Unpack(o).data_ptr();
        return true;
    }
    if (o == Py_None) return true;
    if (PyLong_Check(o)) {
        *out = PyLong_AsVoidPtr(o);
        return !PyErr_Occurred();
    }
    PyObject* r = PyObject_CallMethodNoArgs(o, s_data_ptr);
    if (!r) return false;
    *out = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    return !PyErr_Occurred();
}

// Leading dimension of a row-major matrix: stride(0) of a two-dimensional tensor of at least two
// rows; anything else is decided by the Python function (`own`: told the tensor's own width).
bool get_ld(PyObject* o, int64_t width, int64_t* ld, bool own = false)
{
    if (is_tensor(o)) {
        const at::Tensor& t = THPVariable_Unpack(o);
        if (t.dim() == 2 && t.size(0) >= 2) {
            *ld = t.stride(0);
            return true;
        }
    }
    PyObject* w = own ? Py_NewRef(Py_None) : PyLong_FromLongLong(width);
    if (!w) return false;
    PyObject* const args[2] = {o, w};
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
    if (o == Py_None) {
        *out = c10::hip::getCurrentHIPStream().stream();
        return true;
    }
    PyObject* r = PyLong_Check(o) ? Py_NewRef(o) : PyObject_GetAttr(o, s_cuda_stream);
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
    return Py_NewRef(value);
}

// ---- products

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

PyObject* plan_run(PyObject* const* a, Py_ssize_t n) { return plan_product<bspmm_run>("bspmm_run", a, n); }
PyObject* plan_run_transposed(PyObject* const* a, Py_ssize_t n)
{
    return plan_product<bspmm_run_transposed>("bspmm_run_transposed", a, n);
}
PyObject* run(PyObject* const* a, Py_ssize_t n) { return product<bspmm_run>("bspmm_run", a, n); }
PyObject* run_transposed(PyObject* const* a, Py_ssize_t n)
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

// (plan, X, W, bias, Y, n_X, F, accumulate, stream): leading dimensions from the tensors (X's by its own
// width, not by n_X); returns Y
PyObject* plan_run_gcn(PyObject* const* a, Py_ssize_t n)
{
    int64_t nx, F, ldx, ldw, ldy;
    if (!arity("bspmm_run_gcn", n, 9) || !get_i64(a[5], &nx) || !get_i64(a[6], &F) || !get_ld(a[1], nx, &ldx, true) ||
        !get_ld(a[2], F, &ldw) || !get_ld(a[4], F, &ldy))
        return nullptr;
    return gcn(a, ldx, ldw, ldy, a[7], a[8], a[4]);
}

// (plan, X, W, bias, Y, ldx, ldw, ldy, accumulate, stream)
PyObject* run_gcn(PyObject* const* a, Py_ssize_t n)
{
    int64_t ldx, ldw, ldy;
    if (!arity("bspmm_run_gcn", n, 10) || !get_i64(a[5], &ldx) || !get_i64(a[6], &ldw) || !get_i64(a[7], &ldy))
        return nullptr;
    return gcn(a, ldx, ldw, ldy, a[8], a[9], Py_None);
}

// ---- plans

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Data of a one-dimensional C-contiguous array of the given type, or null.
template <typename T>
const T* array_of(PyObject* o, int type, Py_ssize_t* n)
{
    if (!PyArray_Check(o)) return nullptr;
    PyArrayObject* a = reinterpret_cast<PyArrayObject*>(o);
    if (PyArray_NDIM(a) != 1 || PyArray_TYPE(a) != type || !PyArray_ISCARRAY_RO(a)) return nullptr;
    *n = PyArray_SIZE(a);
    return static_cast<const T*>(PyArray_DATA(a));
}

// The per-operation arrays at a[0] ..: `i32` of them int32, the others int64; the first one's length is
// the batch.
bool meta_arrays(PyObject* const* a, int i32, int total, const void** out, int32_t* batch)
{
    Py_ssize_t n0 = -1;
    for (int i = 0; i < total; ++i) {
        Py_ssize_t n = 0;
        if (i < i32)
            out[i] = array_of<int32_t>(a[i], NPY_INT32, &n);
        else
            out[i] = array_of<int64_t>(a[i], NPY_INT64, &n);
        if (n0 < 0) n0 = n;
        if (!out[i] || n0 > INT32_MAX || n < n0) return false;
    }
    *batch = (int32_t)n0;
    return true;
}

// A contiguous device tensor of the given type.
bool device_data(PyObject* o, at::ScalarType type, int64_t device, const void** out)
{
    if (!is_tensor(o)) return false;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.get_device() != device || t.scalar_type() != type || !t.is_contiguous()) return false;
    *out = t.numel() ? t.data_ptr() : nullptr;
    return true;
}

// The memory is the current stream's.  A plan made on another one waits for what the current one holds (the
// block may have been in use there a moment ago), and the call returns when all that creation
// enqueued has run, conversions and builds included: a plan dropped early leaves nothing on its way to
// memory that is somebody else's by then.
at::Tensor device_bytes(size_t n, int64_t device)
{
    return at::empty({(int64_t)n}, at::TensorOptions().dtype(at::kByte).device(at::Device(at::kCUDA, (c10::DeviceIndex)device)));
}

// (plan, memory, bytes in front of the workspace, row pointers, transposed row pointers, entries): the
// caller may reuse the arrays afterwards, so their sums are taken now.
template <typename Batch>
PyObject* made(bspmm_plan* plan, const Batch& b, const at::Tensor& memory, size_t head)
{
    long long rows = b.batch, cols = b.batch, nnz = 0;
    for (int32_t i = 0; i < b.batch; ++i) rows += b.rows[i], cols += b.cols[i], nnz += b.nnz[i];
    PyObject* t = THPVariable_Wrap(memory);
    return t ? Py_BuildValue("(KNnLLL)", (unsigned long long)reinterpret_cast<uintptr_t>(plan), t, (Py_ssize_t)head, rows,
                             cols, nnz)
             : nullptr;
}

// The caller's CSR arrays in host memory, and how they lie in front of the workspace.
struct Csr {
    const void* data[3];
    size_t bytes[3];
    size_t head() const { return align_up(bytes[0]) + align_up(bytes[1]) + align_up(bytes[2]); }
    static void write(const void* from, char* to)
    {
        const Csr& c = *static_cast<const Csr*>(from);
        for (int i = 0; i < 3; ++i) {
            std::memcpy(to, c.data[i], c.bytes[i]);
            to += align_up(c.bytes[i]);
        }
    }
};

// (rows, cols, nnz, rpt_off, nz_off, b_row_off, c_row_off, rpt, colids, values, F, options address or
// None, device index, stream) -> what made() returns, the CSR arrays all host arrays or all device
// tensors; None when an argument is of another kind (the caller converts it) or the arrays cannot be
// staged.
PyObject* create(PyObject* const* a, Py_ssize_t n)
{
    int64_t F, device;
    void *options, *stream;
    if (!arity("bspmm_create", n, 14) || !get_i64(a[10], &F) || !get_ptr(a[11], &options) || !get_i64(a[12], &device))
        return nullptr;
    const void* meta[7];
    bspmm_batch b;
    if (F > INT32_MAX || !meta_arrays(a, 3, 7, meta, &b.batch)) Py_RETURN_NONE;
    b.rows = static_cast<const int32_t*>(meta[0]), b.cols = static_cast<const int32_t*>(meta[1]);
    b.nnz = static_cast<const int32_t*>(meta[2]), b.rpt_off = static_cast<const int64_t*>(meta[3]);
    b.nz_off = static_cast<const int64_t*>(meta[4]), b.b_row_off = static_cast<const int64_t*>(meta[5]);
    b.c_row_off = static_cast<const int64_t*>(meta[6]);
    Csr csr;
    Py_ssize_t len[3];
    csr.data[0] = array_of<int32_t>(a[7], NPY_INT32, &len[0]);
    csr.data[1] = array_of<int32_t>(a[8], NPY_INT32, &len[1]);
    csr.data[2] = array_of<float>(a[9], NPY_FLOAT32, &len[2]);
    const bool host = csr.data[0] && csr.data[1] && csr.data[2];
    const void* dev[3] = {nullptr, nullptr, nullptr};
    if (!host && !(device_data(a[7], at::kInt, device, &dev[0]) && device_data(a[8], at::kInt, device, &dev[1]) &&
                   device_data(a[9], at::kFloat, device, &dev[2]) && dev[0]))
        Py_RETURN_NONE;
    for (int i = 0; i < 3; ++i) csr.bytes[i] = host ? 4 * (size_t)len[i] : 0;
    if (!get_stream(a[13], &stream)) return nullptr;
    // On another stream than the current one the caller copies the arrays first.
    void* const current = c10::hip::getCurrentHIPStream().stream();
    const bool foreign = a[13] != Py_None && stream != current;
    if (host && foreign) Py_RETURN_NONE;
    const bspmm_options* opt = static_cast<const bspmm_options*>(options);
    const size_t head = host ? csr.head() : 0;
    size_t need = 0;
    bspmm_plan* plan = nullptr;
    at::Tensor memory;
    const char* where = "bspmm_workspace_bytes";
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = bspmm_workspace_bytes(&b, (int32_t)F, opt, &need);
    if (rc == BSPMM_OK) {
        where = "bspmm_create";
        need = need < kAlign ? kAlign : need;
        memory = device_bytes(head + need, device);
        char* base = static_cast<char*>(memory.data_ptr());
        if (host) {
            b.rpt = reinterpret_cast<const int32_t*>(base);
            b.colids = reinterpret_cast<const int32_t*>(base + align_up(csr.bytes[0]));
            b.values = reinterpret_cast<const float*>(base + align_up(csr.bytes[0]) + align_up(csr.bytes[1]));
            rc = bspmm::create_from_host(&plan, &b, (int32_t)F, opt, base + head, need, {head, Csr::write, &csr}, stream);
        } else if (!foreign || (rc = bspmm::run_after(stream, current)) == BSPMM_OK) {
            b.rpt = static_cast<const int32_t*>(dev[0]);
            b.colids = static_cast<const int32_t*>(dev[1]);
            b.values = static_cast<const float*>(dev[2]);
            rc = bspmm_create(&plan, &b, (int32_t)F, opt, base, need, stream);
        }
        if (rc == BSPMM_OK && foreign && (rc = bspmm::run_out(stream)) != BSPMM_OK) bspmm_destroy(plan);
    }
    Py_END_ALLOW_THREADS
    if (host && rc == BSPMM_ESTATE) Py_RETURN_NONE;
    return rc == BSPMM_OK ? made(plan, b, memory, head) : finish(rc, where, Py_None);
}

// (rows, cols, nnz, nz_off, b_row_off, c_row_off, ids, values, F, options address or None, device index,
// stream) -> as above; ids and values device tensors; None as above.
PyObject* create_coo(PyObject* const* a, Py_ssize_t n)
{
    int64_t F, device;
    void *options, *stream;
    if (!arity("bspmm_create_coo", n, 12) || !get_i64(a[8], &F) || !get_ptr(a[9], &options) || !get_i64(a[10], &device))
        return nullptr;
    const void *meta[6], *ids, *values;
    bspmm_coo_batch b;
    if (F > INT32_MAX || !meta_arrays(a, 3, 6, meta, &b.batch) || !device_data(a[6], at::kInt, device, &ids) ||
        !device_data(a[7], at::kFloat, device, &values))
        Py_RETURN_NONE;
    b.rows = static_cast<const int32_t*>(meta[0]), b.cols = static_cast<const int32_t*>(meta[1]);
    b.nnz = static_cast<const int32_t*>(meta[2]), b.nz_off = static_cast<const int64_t*>(meta[3]);
    b.b_row_off = static_cast<const int64_t*>(meta[4]), b.c_row_off = static_cast<const int64_t*>(meta[5]);
    b.ids = static_cast<const int32_t*>(ids);
    b.values = static_cast<const float*>(values);
    if (!get_stream(a[11], &stream)) return nullptr;
    void* const current = c10::hip::getCurrentHIPStream().stream();
    const bool foreign = a[11] != Py_None && stream != current;
    const bspmm_options* opt = static_cast<const bspmm_options*>(options);
    size_t need = 0;
    bspmm_plan* plan = nullptr;
    at::Tensor memory;
    const char* where = "bspmm_workspace_bytes_coo";
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = bspmm_workspace_bytes_coo(&b, (int32_t)F, opt, &need);
    if (rc == BSPMM_OK) {
        where = "bspmm_create_coo";
        need = need < kAlign ? kAlign : need;
        memory = device_bytes(need, device);
        if (foreign) rc = bspmm::run_after(stream, current);
        if (rc == BSPMM_OK) rc = bspmm_create_coo(&plan, &b, (int32_t)F, opt, memory.data_ptr(), need, stream);
        if (rc == BSPMM_OK && foreign && (rc = bspmm::run_out(stream)) != BSPMM_OK) bspmm_destroy(plan);
    }
    Py_END_ALLOW_THREADS
    return rc == BSPMM_OK ? made(plan, b, memory, 0) : finish(rc, where, Py_None);
}

// ---- the differentiable product

// Room for a product: the rows that belong to no operation are zero (autograd.py, _output).
at::Tensor room(bspmm_plan* plan, bool transposed, int64_t rows, int64_t F, const at::Device& device)
{
    const auto options = at::TensorOptions().dtype(at::kFloat).device(device);
    return plan && bspmm::covered_rows(plan, transposed) >= rows ? at::empty({rows, F}, options) : at::zeros({rows, F}, options);
}

// The backward pass of autograd.py's BatchedSpMM.  It has the plan object, not its handle: a plan that was closed
// in between is an error there as here.  Compiled autograd traces nodes instead of running them: there it has the
// node that the class would have made (`traced`, a callable that gives a tensor with it).
struct BatchedSpmmBackward : torch::autograd::Node {
    PyObject *plan, *traced;
    int64_t F, n_b_rows, n_c_rows;
    mutable std::shared_ptr<torch::autograd::Node> twin;
    BatchedSpmmBackward(PyObject* p, PyObject* t, int64_t f, int64_t nb, int64_t nc)
        : plan(Py_NewRef(p)), traced(Py_NewRef(t)), F(f), n_b_rows(nb), n_c_rows(nc) {}
    ~BatchedSpmmBackward() override
    {
        if (!Py_IsInitialized()) return;
        const PyGILState_STATE lock = PyGILState_Ensure();
        Py_DECREF(plan);
        Py_DECREF(traced);
        PyGILState_Release(lock);
    }
    torch::autograd::Node& of_class() const
    {
        if (twin) return *twin;
        const PyGILState_STATE lock = PyGILState_Ensure();
        PyObject* t = PyObject_CallFunction(traced, "OLL", plan, (long long)n_b_rows, (long long)n_c_rows);
        if (t && is_tensor(t)) twin = THPVariable_Unpack(t).grad_fn();
        Py_XDECREF(t);
        PyErr_Clear();
        PyGILState_Release(lock);
        TORCH_CHECK(twin, "BatchedSpMM: no node for compiled autograd");
        return *twin;
    }
    void compiled_args(torch::dynamo::autograd::CompiledNodeArgs& args) const override { of_class().compiled_args(args); }
    torch::autograd::variable_list apply_with_saved(const torch::autograd::variable_list& inputs,
                                                    torch::dynamo::autograd::SwapSavedVariables& saved) override
    {
        return of_class().apply_with_saved(inputs, saved);
    }
    std::string name() const override { return "BatchedSpMMBackward"; }
    torch::autograd::variable_list apply(torch::autograd::variable_list&& grads) override
    {
        const at::Device device = input_metadata(0).device();
        at::Tensor dY = grads.at(0).defined() ? grads[0].contiguous()
                                              : at::zeros({n_c_rows, F}, at::TensorOptions().dtype(at::kFloat).device(device));
        struct Lock {
            PyGILState_STATE state = PyGILState_Ensure();
            ~Lock() { PyGILState_Release(state); }
        } lock;
        void* handle = nullptr;
        PyObject* h = PyObject_GetAttr(plan, s_handle);
        const bool ok = h && get_ptr(h, &handle);
        Py_XDECREF(h);
        if (ok) {
            at::Tensor G = room(static_cast<bspmm_plan*>(handle), true, n_b_rows, F, device);
            void* const in = dY.data_ptr();
            void* const out = G.data_ptr();
            PyObject* r = finish(call<bspmm_run_transposed>(handle, in, out, dY.size(0) >= 2 ? dY.stride(0) : F, F,
                                                            c10::hip::getCurrentHIPStream().stream()),
                                 "bspmm_run_transposed", Py_None);
            Py_XDECREF(r);
            if (r) return {G};
        }
        python_error e;
        e.persist();
        throw e;
    }
};

// (plan object, its handle, F, B, rows of C or None, BatchedSpmmBackward::traced) -> C, or None for what BatchedSpMM.apply decides: other
// types and devices, tensor subclasses, active modes, tracing, forward-mode gradients.
PyObject* batched_spmm(PyObject* const* a, Py_ssize_t n)
{
    void *plan, *stream;
    int64_t F, rows;
    if (!arity("batched_spmm", n, 6) || !get_ptr(a[1], &plan) || !get_i64(a[2], &F)) return nullptr;
    if (!is_tensor(a[3]) || (a[4] != Py_None && !PyLong_CheckExact(a[4]))) Py_RETURN_NONE;
    const at::Tensor& given = THPVariable_Unpack(a[3]);
    if (!given.is_cuda() || given.scalar_type() != at::kFloat || given.layout() != at::kStrided || given.dim() != 2 ||
        given.size(0) < 2 || given._fw_grad(0).defined() || c10::impl::dispatch_mode_enabled() ||
        at::impl::torch_function_mode_enabled() || torch::jit::tracer::isTracing() || given.unsafeGetTensorImpl()->is_python_dispatch())
        Py_RETURN_NONE;
    if (a[4] == Py_None)
        rows = given.size(0);
    else if (!get_i64(a[4], &rows))
        return nullptr;
    if (!get_stream(Py_None, &stream)) return nullptr;
    const bool differentiable = at::GradMode::is_enabled() && given.requires_grad();
    at::Tensor B, C;
    {
        at::NoGradGuard none;
        B = given.contiguous();
        C = room(static_cast<bspmm_plan*>(plan), false, rows, F, B.device());
    }
    const int rc = call<bspmm_run>(plan, B.data_ptr(), C.data_ptr(), B.stride(0), F, stream);
    if (rc != BSPMM_OK) return finish(rc, "bspmm_run", Py_None);
    if (differentiable) {
        auto node = std::shared_ptr<BatchedSpmmBackward>(new BatchedSpmmBackward(a[0], a[5], F, given.size(0), rows),
                                                         torch::autograd::deleteNode);
        node->set_next_edges(torch::autograd::collect_next_edges(given));
        torch::autograd::set_history(C, node);
    }
    return THPVariable_Wrap(std::move(C));
}

// (plan, transposed) -> rows from the first on that every product writes
PyObject* covered_rows(PyObject* const* a, Py_ssize_t n)
{
    void* plan;
    if (!arity("covered_rows", n, 2) || !get_ptr(a[0], &plan)) return nullptr;
    const int transposed = PyObject_IsTrue(a[1]);
    if (transposed < 0) return nullptr;
    return PyLong_FromLongLong(plan ? bspmm::covered_rows(static_cast<bspmm_plan*>(plan), transposed) : 0);
}

// (plan, transposed, ld_in, ld_out) -> whether that product runs in the lean kernel
PyObject* takes_lean_kernel(PyObject* const* a, Py_ssize_t n)
{
    void* plan;
    int64_t ld_in, ld_out;
    if (!arity("takes_lean_kernel", n, 4) || !get_ptr(a[0], &plan) || !get_i64(a[2], &ld_in) || !get_i64(a[3], &ld_out))
        return nullptr;
    const int transposed = PyObject_IsTrue(a[1]);
    if (transposed < 0) return nullptr;
    return PyBool_FromLong(plan && bspmm::takes_lean_kernel(static_cast<bspmm_plan*>(plan), transposed, ld_in, ld_out));
}

// C++ exceptions of PyTorch (no device, out of memory) become Python's.
template <PyObject* (*FN)(PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    PyThreadState* const mine = PyThreadState_Get();
    try {
        return FN(a, n);
    } catch (...) {
        const std::exception_ptr e = std::current_exception();
        if (!PyGILState_Check()) PyEval_RestoreThread(mine);     // thrown while the lock was given up
        torch::translate_exception_to_python(e);
        return nullptr;
    }
}

template <PyObject* (*FN)(PyObject* const*, Py_ssize_t)>
PyMethodDef fast(const char* name)
{
    return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(&guarded<FN>)), METH_FASTCALL, nullptr};
}

PyMethodDef methods[] = {
    {"setup", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(&setup)), METH_FASTCALL, nullptr},
    fast<plan_run>("plan_run"), fast<plan_run_transposed>("plan_run_transposed"), fast<plan_run_gcn>("plan_run_gcn"),
    fast<run>("run"), fast<run_transposed>("run_transposed"), fast<run_gcn>("run_gcn"),
    fast<covered_rows>("covered_rows"), fast<takes_lean_kernel>("takes_lean_kernel"), fast<create>("create"), fast<create_coo>("create_coo"),
    fast<batched_spmm>("batched_spmm"),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "Plan creation and run calls of libbspmm.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void)
{
    import_array();
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    s_handle = PyUnicode_InternFromString("handle");
    if (!s_data_ptr || !s_cuda_stream || !s_handle) return nullptr;
    return PyModule_Create(&module);
}
