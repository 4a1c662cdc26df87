// The calls that a serving loop makes once or more per layer, without Python between the argument checks, the output
// tensor and the launch: one token through one projection (quantise, multiply) took 30 us of which the GPU works for 6.
//
// Every function answers with its result, with the library's error code (an int), or with None: anything but the plain
// case -- other objects than torch.Tensor itself, wrong types, shapes or strides, numbers that do not fit, a workspace
// that has to be made first -- goes back to the caller, whose general path runs it or raises what it always raised.
// The library is reached through the addresses that bind() is handed, so that it is the one that api.py has loaded.
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>
#include <vector>

#include "liquidgemm.h"

namespace {

struct Library {
    decltype(&w4a8_gemm) gemm;
    decltype(&w4a8_gemm_workspace_size) workspace_size;
    decltype(&w4a8_quantize_activations) quantize;
    decltype(&w4a8_grouped_gemm) grouped;
    decltype(&liquidquant_packed_size) packed_size;
} lib{};

// The GIL is given up for the allocation and the launch (both may wait), also where they throw.
struct WithoutGil {
    PyThreadState *const state = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(state); }
};

// What the general path's checks accept: a tensor on the GPU of that type and shape, contiguous
bool plain(PyObject *o, at::ScalarType type, std::initializer_list<int64_t> shape)
{
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    return t.is_cuda() && t.scalar_type() == type && t.layout() == at::kStrided && t.sizes().equals(shape) && t.is_contiguous();
}
const at::Tensor &tensor(PyObject *o) { return THPVariable_Unpack(o); }

bool small_int(PyObject *o, int &v)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long long x = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow || x < INT_MIN || x > INT_MAX) return false;
    v = (int)x;
    return true;
}

// stream: None (torch's current one) or its number
bool stream_of(PyObject *o, void *&stream)
{
    if (o == Py_None) {
        stream = c10::hip::getCurrentHIPStream().stream();
        return true;
    }
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long long x = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow || x < 0) return false;
    stream = reinterpret_cast<void *>((uintptr_t)x);
    return true;
}

// rows of a matrix of `type` on the GPU, or -1
int64_t rows_of(PyObject *o, at::ScalarType type)
{
    if (!THPVariable_CheckExact(o)) return -1;
    const at::Tensor &t = tensor(o);
    if (!t.is_cuda() || t.scalar_type() != type || t.layout() != at::kStrided || t.dim() != 2 || t.size(0) > INT_MAX || t.size(1) > INT_MAX)
        return -1;
    return t.size(0);
}

// quantize(X_f16, smooth, out_q, out_scales, stream) -> (X_i8, act_scales)
PyObject *quantize(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    void *stream;
    const int64_t M = n == 5 ? rows_of(a[0], at::kHalf) : -1;
    if (M < 0) Py_RETURN_NONE;
    const at::Tensor &x = tensor(a[0]);
    const int64_t K = x.size(1);
    if (!x.is_contiguous() || (a[1] != Py_None && !plain(a[1], at::kFloat, {K})) || (a[2] != Py_None && !plain(a[2], at::kChar, {M, K})) ||
        (a[3] != Py_None && !plain(a[3], at::kFloat, {M})) || !stream_of(a[4], stream))
        Py_RETURN_NONE;
    at::Tensor q = a[2] != Py_None ? tensor(a[2]) : at::Tensor(), s = a[3] != Py_None ? tensor(a[3]) : at::Tensor();
    const float *smooth = a[1] != Py_None ? static_cast<const float *>(tensor(a[1]).data_ptr()) : nullptr;
    int rc;
    {
        const WithoutGil released;
        if (!q.defined()) q = at::empty({M, K}, x.options().dtype(at::kChar));
        if (!s.defined()) s = at::empty({M}, x.options().dtype(at::kFloat));
        rc = lib.quantize((int)M, (int)K, static_cast<const uint16_t *>(x.data_ptr()), smooth, static_cast<int8_t *>(q.data_ptr()),
                          static_cast<float *>(s.data_ptr()), stream);
    }
    if (rc != LQ_OK) return PyLong_FromLong(rc);
    PyObject *const pq = a[2] != Py_None ? (Py_INCREF(a[2]), a[2]) : THPVariable_Wrap(std::move(q));
    PyObject *const ps = a[3] != Py_None ? (Py_INCREF(a[3]), a[3]) : THPVariable_Wrap(std::move(s));
    PyObject *const both = pq && ps ? PyTuple_Pack(2, pq, ps) : nullptr;
    Py_XDECREF(pq);
    Py_XDECREF(ps);
    return both;
    END_HANDLE_TH_ERRORS
}

// gemm(X, act_scales, W_packed, gparams, w_scales, N, K, group, out, workspace, stream, workspaces) -> out
PyObject *gemm(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    void *stream;
    int N, K, group;
    size_t codes = 0, gparams = 0;
    const int64_t M = n == 12 ? rows_of(a[0], at::kChar) : -1;
    if (M < 1 || !small_int(a[5], N) || !small_int(a[6], K) || !small_int(a[7], group) ||
        lib.packed_size(N, K, group, &codes, &gparams) != LQ_OK || !plain(a[0], at::kChar, {M, K}) || !plain(a[1], at::kFloat, {M}) ||
        !plain(a[2], at::kByte, {(int64_t)codes}) || !plain(a[3], at::kByte, {(int64_t)gparams}) || !plain(a[4], at::kFloat, {N}) ||
        (a[8] != Py_None && !plain(a[8], at::kHalf, {M, N})) || !stream_of(a[10], stream))
        Py_RETURN_NONE;
    const at::Tensor &x = tensor(a[0]);
    at::Tensor workspace;
    if (a[9] != Py_None) {
        if (!THPVariable_CheckExact(a[9])) Py_RETURN_NONE;
        workspace = tensor(a[9]);
        if (!workspace.is_cuda() || workspace.scalar_type() != at::kByte || workspace.layout() != at::kStrided || !workspace.is_contiguous())
            Py_RETURN_NONE;
    } else if (const size_t need = lib.workspace_size((int)M, N, K, group)) {
        // the buffer of this device and stream, if there is one that is large enough
        PyObject *const key = Py_BuildValue("(iK)", (int)x.device().index(), (unsigned long long)(uintptr_t)stream);
        if (!key) return nullptr;
        PyObject *const found = PyDict_GetItemWithError(a[11], key);
        Py_DECREF(key);
        if (!found) {
            if (PyErr_Occurred()) return nullptr;
            Py_RETURN_NONE;
        }
        if (!THPVariable_CheckExact(found) || (size_t)tensor(found).numel() < need) Py_RETURN_NONE;
        workspace = tensor(found);
    }
    at::Tensor out = a[8] != Py_None ? tensor(a[8]) : at::Tensor();
    int rc;
    {
        const WithoutGil released;
        if (!out.defined()) out = at::empty({M, N}, x.options().dtype(at::kHalf));
        rc = lib.gemm((int)M, N, K, group, static_cast<const int8_t *>(x.data_ptr()), static_cast<const float *>(tensor(a[1]).data_ptr()),
                      tensor(a[2]).data_ptr(), static_cast<const uint8_t *>(tensor(a[3]).data_ptr()),
                      static_cast<const float *>(tensor(a[4]).data_ptr()), static_cast<uint16_t *>(out.data_ptr()),
                      workspace.defined() ? workspace.data_ptr() : nullptr, workspace.defined() ? (size_t)workspace.numel() : 0, stream);
    }
    if (rc != LQ_OK) return PyLong_FromLong(rc);
    return a[8] != Py_None ? (Py_INCREF(a[8]), a[8]) : THPVariable_Wrap(std::move(out));
    END_HANDLE_TH_ERRORS
}

// grouped(row_offsets (a list), X, act_scales, W_packed, gparams, w_scales, N, K, group, out_y, stream) -> out_y
PyObject *grouped(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    void *stream;
    int N, K, group;
    size_t codes = 0, gparams = 0;
    if (n != 11 || !PyList_CheckExact(a[0]) || PyList_GET_SIZE(a[0]) < 2 || PyList_GET_SIZE(a[0]) > 65) Py_RETURN_NONE;
    const int E = (int)PyList_GET_SIZE(a[0]) - 1;
    int offsets[65];
    for (int i = 0; i <= E; ++i)
        if (!small_int(PyList_GET_ITEM(a[0], i), offsets[i])) Py_RETURN_NONE;
    const int64_t M = offsets[E];
    if (M < 1 || !small_int(a[6], N) || !small_int(a[7], K) || !small_int(a[8], group) ||
        lib.packed_size(N, K, group, &codes, &gparams) != LQ_OK || !plain(a[1], at::kChar, {M, K}) || !plain(a[2], at::kFloat, {M}) ||
        !plain(a[3], at::kByte, {(int64_t)codes * E}) || !plain(a[4], at::kByte, {(int64_t)gparams * E}) ||
        !plain(a[5], at::kFloat, {E, N}) || (a[9] != Py_None && !plain(a[9], at::kHalf, {M, N})) || !stream_of(a[10], stream))
        Py_RETURN_NONE;
    const at::Tensor &x = tensor(a[1]);
    at::Tensor out = a[9] != Py_None ? tensor(a[9]) : at::Tensor();
    int rc;
    {
        const WithoutGil released;
        if (!out.defined()) out = at::empty({M, N}, x.options().dtype(at::kHalf));
        rc = lib.grouped(E, offsets, N, K, group, static_cast<const int8_t *>(x.data_ptr()), static_cast<const float *>(tensor(a[2]).data_ptr()),
                         tensor(a[3]).data_ptr(), static_cast<const uint8_t *>(tensor(a[4]).data_ptr()),
                         static_cast<const float *>(tensor(a[5]).data_ptr()), static_cast<uint16_t *>(out.data_ptr()), nullptr, stream);
    }
    if (rc != LQ_OK) return PyLong_FromLong(rc);
    return a[9] != Py_None ? (Py_INCREF(a[9]), a[9]) : THPVariable_Wrap(std::move(out));
    END_HANDLE_TH_ERRORS
}

// bind(w4a8_gemm, w4a8_gemm_workspace_size, w4a8_quantize_activations, w4a8_grouped_gemm, liquidquant_packed_size): their addresses
PyObject *bind(PyObject *, PyObject *args)
{
    unsigned long long g, w, q, m, p;
    if (!PyArg_ParseTuple(args, "KKKKK", &g, &w, &q, &m, &p)) return nullptr;
    lib = Library{reinterpret_cast<decltype(lib.gemm)>(g), reinterpret_cast<decltype(lib.workspace_size)>(w),
                  reinterpret_cast<decltype(lib.quantize)>(q), reinterpret_cast<decltype(lib.grouped)>(m),
                  reinterpret_cast<decltype(lib.packed_size)>(p)};
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"quantize", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(quantize)), METH_FASTCALL, nullptr},
    {"gemm", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(gemm)), METH_FASTCALL, nullptr},
    {"grouped", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(grouped)), METH_FASTCALL, nullptr},
    {"bind", bind, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module{PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__binding()
{
    PyObject *const m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", BUILT_FOR) == 0) return m;  // (api.py looks at it before the first call)
    Py_XDECREF(m);
    return nullptr;
}
