// One call from Python to a C-ABI entry point with its outputs allocated on the way: what binding.py's tensor-level helpers do
// when the caller brings no buffers.  A small call is bound by the host (16 x 4096 weights: 4.6 us on the GPU), and six
// torch.empty from Python, the descriptor and the foreign-function call made 14.9 us a call of it; this way it is 9.8 (3.4 the
// library's call itself, half a microsecond an allocation).
// Marshalling only: checks on the tensors, allocation through torch's caching allocator, the call with the interpreter lock
// released, torch's exceptions passed on.  The entry points come as addresses from the ctypes view of the library (bind()).
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/full.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <limits>
#include <vector>

#include "soar.h"

namespace {

struct EntryPoints {
    decltype(&soar_workspace_bytes)              workspace_bytes;
    decltype(&soar_quantize_batch)               quantize_batch;
    decltype(&soar_mxfp4_workspace_bytes)        mx_workspace_bytes;
    decltype(&soar_mxfp4_quantize)               mx_quantize;
    decltype(&soar_dequantize_batch)             dequantize_batch;
    decltype(&soar_mxfp4_dequantize_batch)       mx_dequantize_batch;
    decltype(&soar_recon_error_batch)            recon_error_batch;
};
EntryPoints entry;

// The interpreter lock given back for a scope: taken again also where the call ends in a C++ exception, which
// END_HANDLE_TH_ERRORS turns into a Python one.
struct Unlocked {
    PyThreadState *state = PyEval_SaveThread();
    Unlocked() = default;
    ~Unlocked() { PyEval_RestoreThread(state); }
    Unlocked(const Unlocked &) = delete;
    Unlocked &operator=(const Unlocked &) = delete;
};

constexpr int kNoWorkspace = -1;          // the library names no workspace size: its parameter error

at::Tensor empty(at::IntArrayRef sizes, at::ScalarType type, const at::Device &device)
{
    return at::empty(sizes, at::TensorOptions().dtype(type).device(device));
}

bool is_matrix(PyObject *o, const char *what)
{
    if (THPVariable_Check(o)) return true;
    PyErr_Format(PyExc_TypeError, "%s must be a tensor", what);
    return false;
}

// what _check_matrix and _dtype_code of binding.py ask of a matrix, with their errors
bool check_matrix(const at::Tensor &w, int32_t &dtype)
{
    if (!w.is_cuda()) {
        PyErr_SetString(PyExc_RuntimeError, "soar: weights must live on the GPU (no CPU path exists)");
        return false;
    }
    if (w.dim() != 2 || w.stride(1) != 1) {
        PyErr_SetString(PyExc_ValueError, "weights must be 2-D with contiguous rows");
        return false;
    }
    if (w.scalar_type() == at::kBFloat16) dtype = SOAR_BF16;
    else if (w.scalar_type() == at::kFloat) dtype = SOAR_FP32;
    else {
        PyErr_SetString(PyExc_TypeError, "weights must be bfloat16 or float32");
        return false;
    }
    return true;
}

// (codes, scales, global scale or None, sse, status, iters_run or None, trace or None, status of the call)
PyObject *result(const at::Tensor &codes, const at::Tensor &scales, const at::Tensor &gscale, const at::Tensor &sse, const at::Tensor &status,
                 const at::Tensor &iters_run, const at::Tensor &trace, int rc)
{
    PyObject *t = PyTuple_New(8);
    if (!t) return nullptr;
    const at::Tensor *parts[7] = {&codes, &scales, &gscale, &sse, &status, &iters_run, &trace};
    for (int k = 0; k < 7; ++k) {
        PyObject *o = parts[k]->defined() ? THPVariable_Wrap(*parts[k]) : (Py_INCREF(Py_None), Py_None);
        if (!o) {
            Py_DECREF(t);
            return nullptr;
        }
        PyTuple_SET_ITEM(t, k, o);
    }
    PyTuple_SET_ITEM(t, 7, PyLong_FromLong(rc));
    return t;
}

// quantize(w, address of soar_params, trace wanted, maximum or None, stream): soar_quantize_batch with n = 1
PyObject *quantize(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 5 || !is_matrix(args[0], "weights")) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "quantize takes 5 arguments");
        return nullptr;
    }
    const at::Tensor &w = THPVariable_Unpack(args[0]);
    const soar_params *params = static_cast<const soar_params *>(PyLong_AsVoidPtr(args[1]));
    const bool trace_wanted = args[2] == Py_True;
    void *stream = PyLong_AsVoidPtr(args[4]);
    if (PyErr_Occurred()) return nullptr;
    soar_tensor_desc d = {};
    if (!check_matrix(w, d.dtype)) return nullptr;
    if (args[3] != Py_None &&       // an empty tensor has no address, which would mean: measure it
        !(THPVariable_Check(args[3]) && THPVariable_Unpack(args[3]).scalar_type() == at::kFloat && THPVariable_Unpack(args[3]).is_cuda() &&
          THPVariable_Unpack(args[3]).numel() > 0)) {
        PyErr_SetString(PyExc_TypeError, "amax_in must be a float32 tensor on the GPU");
        return nullptr;
    }
    d.rows = w.size(0);
    d.cols = w.size(1);
    d.ld_elems = w.stride(0);
    const at::Device device = w.device();
    at::Tensor iters_run, trace;
    // before the outputs: their sizes come from the parameters that this checks
    const size_t bytes = entry.workspace_bytes(d.rows, d.cols, params);
    if (bytes == 0) return result({}, {}, {}, {}, {}, {}, {}, kNoWorkspace);
    const at::Tensor codes = empty({d.rows, d.cols / 2}, at::kByte, device), scales = empty({d.rows, d.cols / 16}, at::kByte, device);
    const at::Tensor gscale = empty({1}, at::kFloat, device), sse = empty({1}, at::kDouble, device), status = empty({1}, at::kInt, device);
    if (trace_wanted) {
        // NaN where an entry is not written; the number of iterations is written by every call that is carried out
        trace = at::full({(int64_t)params->iters + 1}, std::numeric_limits<double>::quiet_NaN(),
                         at::TensorOptions().dtype(at::kDouble).device(device));
        iters_run = empty({1}, at::kInt, device);
        d.d_iters_run = static_cast<int32_t *>(iters_run.data_ptr());
        d.d_sse_trace = static_cast<double *>(trace.data_ptr());
    }
    if (args[3] != Py_None) d.d_amax_in = static_cast<const float *>(THPVariable_Unpack(args[3]).data_ptr());
    const at::Tensor workspace = empty({(int64_t)bytes}, at::kByte, device);
    d.d_w = w.data_ptr();
    d.d_codes = static_cast<uint8_t *>(codes.data_ptr());
    d.d_scales = static_cast<uint8_t *>(scales.data_ptr());
    d.d_global_scale = static_cast<float *>(gscale.data_ptr());
    d.d_sse = static_cast<double *>(sse.data_ptr());
    d.d_status = static_cast<int32_t *>(status.data_ptr());
    void *ws = workspace.data_ptr();
    int rc;
    {
        const Unlocked scope;
        rc = entry.quantize_batch(1, &d, params, ws, bytes, stream);
    }
    return result(codes, scales, gscale, sse, status, iters_run, trace, rc);
    END_HANDLE_TH_ERRORS
}

// mx_quantize(w, address of soar_mx_params, stream)
PyObject *mx_quantize(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 3 || !is_matrix(args[0], "weights")) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "mx_quantize takes 3 arguments");
        return nullptr;
    }
    const at::Tensor &w = THPVariable_Unpack(args[0]);
    const soar_mx_params *params = static_cast<const soar_mx_params *>(PyLong_AsVoidPtr(args[1]));
    void *stream = PyLong_AsVoidPtr(args[2]);
    if (PyErr_Occurred()) return nullptr;
    int32_t dtype = 0;
    if (!check_matrix(w, dtype)) return nullptr;
    const int64_t rows = w.size(0), cols = w.size(1);
    const at::Device device = w.device();
    const at::Tensor codes = empty({rows, cols / 2}, at::kByte, device), scales = empty({rows, cols / 32}, at::kByte, device);
    const at::Tensor sse = empty({1}, at::kDouble, device), status = empty({1}, at::kInt, device);
    const size_t bytes = entry.mx_workspace_bytes(rows, cols, params);
    if (bytes == 0) return result(codes, scales, at::Tensor(), sse, status, at::Tensor(), at::Tensor(), kNoWorkspace);
    const at::Tensor workspace = empty({(int64_t)bytes}, at::kByte, device);
    const void *p = w.data_ptr();
    const int64_t ld = w.stride(0);
    uint8_t *c = static_cast<uint8_t *>(codes.data_ptr()), *s = static_cast<uint8_t *>(scales.data_ptr());
    double *e = static_cast<double *>(sse.data_ptr());
    int32_t *st = static_cast<int32_t *>(status.data_ptr());
    void *ws = workspace.data_ptr();
    int rc;
    {
        const Unlocked scope;
        rc = entry.mx_quantize(p, (soar_dtype)dtype, rows, cols, ld, params, c, s, e, st, ws, bytes, stream);
    }
    return result(codes, scales, at::Tensor(), sse, status, at::Tensor(), at::Tensor(), rc);
    END_HANDLE_TH_ERRORS
}

// an owned reference, given back at the end of its scope
struct Ref {
    PyObject *o;
    explicit Ref(PyObject *o_) : o(o_) {}
    ~Ref() { Py_XDECREF(o); }
    Ref(const Ref &) = delete;
    Ref &operator=(const Ref &) = delete;
};

PyObject *name_codes, *name_scales, *name_global_scale;

// codes, scales and (unless mx) the global scale of one Quantized
bool stored_fields(PyObject *q, bool mx, soar_stored_desc &d, int64_t &rows, int64_t &cols, at::Device *device)
{
    const Ref codes(PyObject_GetAttr(q, name_codes)), scales(PyObject_GetAttr(q, name_scales));
    if (!codes.o || !scales.o || !is_matrix(codes.o, "codes") || !is_matrix(scales.o, "scales")) return false;
    const at::Tensor &c = THPVariable_Unpack(codes.o), &s = THPVariable_Unpack(scales.o);
    if (s.dim() < 2) {
        PyErr_SetString(PyExc_IndexError, "scales must be 2-D");
        return false;
    }
    d.d_codes = static_cast<const uint8_t *>(c.data_ptr());
    d.d_scales = static_cast<const uint8_t *>(s.data_ptr());
    if (!mx) {
        const Ref g(PyObject_GetAttr(q, name_global_scale));
        if (!g.o || !is_matrix(g.o, "the global scale")) return false;
        d.d_global_scale = static_cast<const float *>(THPVariable_Unpack(g.o).data_ptr());
    }
    rows = s.size(0);
    cols = s.size(1) * (mx ? 32 : 16);
    if (device) *device = c.device();
    return true;
}

// dequantize(list of Quantized, mx, fp32 wanted, stream) -> (list of matrices, status of the call)
PyObject *dequantize(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 4 || !PyList_Check(args[0])) {
        PyErr_SetString(PyExc_TypeError, "dequantize takes a list and 3 arguments");
        return nullptr;
    }
    const bool mx = args[1] == Py_True, fp32 = args[2] == Py_True;
    void *stream = PyLong_AsVoidPtr(args[3]);
    if (PyErr_Occurred()) return nullptr;
    const Py_ssize_t count = PyList_GET_SIZE(args[0]);
    std::vector<soar_stored_desc> descs((size_t)count);
    std::vector<at::Tensor> outs((size_t)count);
    for (Py_ssize_t k = 0; k < count; ++k) {
        soar_stored_desc &d = descs[(size_t)k];
        at::Device device(at::kCPU);
        if (!stored_fields(PyList_GET_ITEM(args[0], k), mx, d, d.rows, d.cols, &device)) return nullptr;
        outs[(size_t)k] = empty({d.rows, d.cols}, fp32 ? at::kFloat : at::kBFloat16, device);
        if (!check_matrix(outs[(size_t)k], d.dtype)) return nullptr;
        d.ld_elems = outs[(size_t)k].stride(0);
        d.d_out = outs[(size_t)k].data_ptr();
    }
    int rc;
    {
        const Unlocked scope;
        rc = (mx ? entry.mx_dequantize_batch : entry.dequantize_batch)((int32_t)count, descs.data(), stream);
    }
    const Ref list(PyList_New(count));
    if (!list.o) return nullptr;
    for (Py_ssize_t k = 0; k < count; ++k) {
        PyObject *o = THPVariable_Wrap(outs[(size_t)k]);
        if (!o) return nullptr;
        PyList_SET_ITEM(list.o, k, o);
    }
    return Py_BuildValue("(Oi)", list.o, rc);
    END_HANDLE_TH_ERRORS
}

// recon_error(list of weights, list of at least as many Quantized, stream) -> (one sum per weight, status of the call)
PyObject *recon_error(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 3 || !PyList_Check(args[0]) || !PyList_Check(args[1])) {
        PyErr_SetString(PyExc_TypeError, "recon_error takes two lists and a stream");
        return nullptr;
    }
    void *stream = PyLong_AsVoidPtr(args[2]);
    if (PyErr_Occurred()) return nullptr;
    const Py_ssize_t weights = PyList_GET_SIZE(args[0]), stored = PyList_GET_SIZE(args[1]);
    if (weights == 0 || !is_matrix(PyList_GET_ITEM(args[0], 0), "weights")) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "no weights");
        return nullptr;
    }
    if (stored < weights) {
        PyErr_Format(PyExc_ValueError, "%zd weights, but only %zd stored tensors", weights, stored);
        return nullptr;
    }
    const at::Tensor sums = empty({weights}, at::kDouble, THPVariable_Unpack(PyList_GET_ITEM(args[0], 0)).device());
    std::vector<soar_stored_desc> descs((size_t)weights);
    for (Py_ssize_t k = 0; k < weights; ++k) {
        soar_stored_desc &d = descs[(size_t)k];
        if (!is_matrix(PyList_GET_ITEM(args[0], k), "weights")) return nullptr;
        const at::Tensor &w = THPVariable_Unpack(PyList_GET_ITEM(args[0], k));
        int64_t rows = 0, cols = 0;
        if (!stored_fields(PyList_GET_ITEM(args[1], k), false, d, rows, cols, nullptr) || !check_matrix(w, d.dtype)) return nullptr;
        d.rows = w.size(0);
        d.cols = w.size(1);
        d.ld_elems = w.stride(0);
        d.d_w = w.data_ptr();
        d.d_sse = static_cast<double *>(sums.data_ptr()) + k;
    }
    int rc;
    {
        const Unlocked scope;
        rc = entry.recon_error_batch((int32_t)weights, descs.data(), stream);
    }
    const Ref o(THPVariable_Wrap(sums));
    return o.o ? Py_BuildValue("(Oi)", o.o, rc) : nullptr;
    END_HANDLE_TH_ERRORS
}

// bind(addresses of the entry points, in the order of EntryPoints)
PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    constexpr Py_ssize_t kCount = sizeof(EntryPoints) / sizeof(void *);
    if (n != kCount) {
        PyErr_Format(PyExc_TypeError, "bind takes %zd addresses", kCount);
        return nullptr;
    }
    void *p[kCount];
    for (Py_ssize_t k = 0; k < kCount; ++k) {
        p[k] = PyLong_AsVoidPtr(args[k]);
        if (!p[k]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "an entry point has no address");
            return nullptr;
        }
    }
    static_assert(sizeof(EntryPoints) == sizeof(p), "addresses only");
    __builtin_memcpy(&entry, p, sizeof(p));
    Py_RETURN_NONE;
}

#define SOAR_ENTRY(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {SOAR_ENTRY(bind), SOAR_ENTRY(quantize), SOAR_ENTRY(mx_quantize), SOAR_ENTRY(dequantize),
                         SOAR_ENTRY(recon_error), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "soar_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_soar_host()
{
    name_codes = PyUnicode_InternFromString("codes");
    name_scales = PyUnicode_InternFromString("scales");
    name_global_scale = PyUnicode_InternFromString("global_scale");
    return PyModule_Create(&module);
}
