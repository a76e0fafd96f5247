// The calls of the binding that a program makes for every matrix or product, without Python and ctypes between the tensors and the C ABI (include/gcoo.h): the addresses of the C functions
// come from the library that binding.py has loaded.  (us of the host for 256 x 256, 10 %, N = 256, by ctypes, and so: conversion 7.4 5.1, of which the C function takes 4.0; product 6.0 4.1,
// product into a C that is there 4.6 3.45, of which it takes 3.3; mostly launches.)
//
// A call serves tensors and arrays exactly as it expects them, on the current device, and returns None for anything else: binding.py then does what it does for everything, with its
// checks and errors.  A status other than GCOO_OK is returned as a number.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>
#include <c10/core/impl/VirtualGuardImpl.h>

#include <cstdint>
#include <cstring>

#include "gcoo.h"

namespace {

struct {
    decltype(&gcoo_device_bytes) device_bytes;
    decltype(&gcoo_from_csr) from_csr;
    decltype(&gcoo_from_csr_device) from_csr_device;
    decltype(&gcoo_from_csr_device_static) from_csr_device_static;
    decltype(&gcoo_dense_count_bytes) dense_count_bytes;
    decltype(&gcoo_dense_count) dense_count;
    decltype(&gcoo_from_dense_counted) from_dense_counted;
    decltype(&gcoo_spdm_variant) spdm_variant;
    decltype(&gcoo_free) free_matrix;
} gcoo_calls;

// A strided tensor of this type on the current device, itself and not a subclass of torch.Tensor.
const at::Tensor* tensor(PyObject* o, at::ScalarType type, int64_t device)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    return t.scalar_type() == type && t.layout() == at::kStrided && t.is_cuda() && t.get_device() == device ? &t : nullptr;
}
int64_t current_device() { return c10::impl::VirtualGuardImpl(c10::DeviceType::CUDA).getDevice().index(); }

at::Tensor bytes_on(int64_t device, size_t bytes)
{
    return at::empty({(int64_t)(bytes < 256 ? 256 : bytes)}, at::TensorOptions().dtype(at::kByte).device(c10::Device(c10::DeviceType::CUDA, (c10::DeviceIndex)device)));
}
PyObject* matrix_and_buffer(gcoo_matrix* h, const at::Tensor& buf) { return Py_BuildValue("(KN)", (unsigned long long)(uintptr_t)h, THPVariable_Wrap(buf)); }

// The interpreter is left to other threads while a call allocates, launches or waits.
struct NoGil {
    PyThreadState* state = PyEval_SaveThread();
    ~NoGil() { PyEval_RestoreThread(state); }
};

struct Shape { long long m, k, p; bool ok() const { return p >= INT32_MIN && p <= INT32_MAX; } };

PyObject* bind(PyObject*, PyObject* args)
{
    unsigned long long f[9];
    if (!PyArg_ParseTuple(args, "KKKKKKKKK", f, f + 1, f + 2, f + 3, f + 4, f + 5, f + 6, f + 7, f + 8)) return nullptr;
    static_assert(sizeof(gcoo_calls) == sizeof(f), "an address each");
    std::memcpy(&gcoo_calls, f, sizeof(f));
    Py_RETURN_NONE;
}

// (row_ptr, col_idx, vals, m, k, p, stream, known_nnz): device tensors -> (handle, buffer)
PyObject* from_csr_device(PyObject*, PyObject* args)
{
    HANDLE_TH_ERRORS
    PyObject *rp, *ci, *va;
    Shape s;
    unsigned long long stream;
    int known;
    if (!PyArg_ParseTuple(args, "OOOLLLKp", &rp, &ci, &va, &s.m, &s.k, &s.p, &stream, &known)) return nullptr;
    const int64_t device = current_device();
    const at::Tensor *r = tensor(rp, at::kInt, device), *c = tensor(ci, at::kInt, device), *v = tensor(va, at::kFloat, device);
    if (!r || !c || !v || !r->is_contiguous() || !s.ok()) Py_RETURN_NONE;
    const int64_t nnz = c->numel();
    const size_t need = gcoo_calls.device_bytes(s.m, s.k, nnz, (int32_t)s.p);
    if (need == 0) Py_RETURN_NONE;
    const int32_t *rd = (const int32_t*)r->data_ptr(), *cd = (const int32_t*)c->data_ptr();
    const float* vd = (const float*)v->data_ptr();
    at::Tensor buf;
    gcoo_matrix* out = nullptr;
    int status;
    {
        const NoGil released;
        buf = bytes_on(device, need);
        status = known ? gcoo_calls.from_csr_device(s.m, s.k, nnz, rd, cd, vd, (int32_t)s.p, buf.data_ptr(), need, (void*)(uintptr_t)stream, &out)
                       : gcoo_calls.from_csr(s.m, s.k, rd, cd, vd, 1, (int32_t)s.p, buf.data_ptr(), need, (void*)(uintptr_t)stream, &out);
    }
    if (status != GCOO_OK) return PyLong_FromLong(status);
    return matrix_and_buffer(out, buf);
    END_HANDLE_TH_ERRORS
}

// A one-dimensional contiguous array of 4-byte elements of this format.
struct Array {
    Py_buffer b;
    bool held = false;
    bool get(PyObject* o, char format)
    {
        if (PyObject_GetBuffer(o, &b, PyBUF_ND | PyBUF_FORMAT) != 0) { PyErr_Clear(); return false; }
        held = true;
        return b.ndim == 1 && b.itemsize == 4 && b.format && b.format[0] == format && b.format[1] == 0;
    }
    ~Array() { if (held) PyBuffer_Release(&b); }
};
// (row_ptr, col_idx, vals, m, k, p, stream): arrays in host memory, for the current device -> (handle, buffer)
PyObject* from_csr_host(PyObject*, PyObject* args)
{
    HANDLE_TH_ERRORS
    PyObject *rp, *ci, *va;
    Shape s;
    unsigned long long stream;
    if (!PyArg_ParseTuple(args, "OOOLLLK", &rp, &ci, &va, &s.m, &s.k, &s.p, &stream)) return nullptr;
    Array r, c, v;
    if (!r.get(rp, 'i') || !c.get(ci, 'i') || !v.get(va, 'f') || !s.ok()) Py_RETURN_NONE;
    const size_t need = gcoo_calls.device_bytes(s.m, s.k, c.b.shape[0], (int32_t)s.p);
    if (need == 0) Py_RETURN_NONE;
    at::Tensor buf;
    gcoo_matrix* out = nullptr;
    int status;
    {
        const NoGil released;
        buf = bytes_on(current_device(), need);
        status = gcoo_calls.from_csr(s.m, s.k, (const int32_t*)r.b.buf, (const int32_t*)c.b.buf, (const float*)v.b.buf, 0, (int32_t)s.p, buf.data_ptr(), need,
                                     (void*)(uintptr_t)stream, &out);
    }
    if (status != GCOO_OK) return PyLong_FromLong(status);
    return matrix_and_buffer(out, buf);
    END_HANDLE_TH_ERRORS
}

// (row_ptr, col_idx, vals, m, k, p, out_buf, stream) -> handle
PyObject* from_csr_device_static(PyObject*, PyObject* args)
{
    HANDLE_TH_ERRORS
    PyObject *rp, *ci, *va, *ob;
    Shape s;
    unsigned long long stream;
    if (!PyArg_ParseTuple(args, "OOOLLLOK", &rp, &ci, &va, &s.m, &s.k, &s.p, &ob, &stream)) return nullptr;
    const int64_t device = current_device();
    const at::Tensor *r = tensor(rp, at::kInt, device), *c = tensor(ci, at::kInt, device), *v = tensor(va, at::kFloat, device), *o = tensor(ob, at::kByte, device);
    if (!r || !c || !v || !o || !s.ok()) Py_RETURN_NONE;
    const int32_t *rd = (const int32_t*)r->data_ptr(), *cd = (const int32_t*)c->data_ptr();
    const float* vd = (const float*)v->data_ptr();
    const int64_t nnz = c->numel(), room = o->numel();
    void* to = o->data_ptr();
    gcoo_matrix* out = nullptr;
    int status;
    {
        const NoGil released;
        status = gcoo_calls.from_csr_device_static(s.m, s.k, nnz, rd, cd, vd, (int32_t)s.p, to, (size_t)room, (void*)(uintptr_t)stream, &out);
    }
    if (status != GCOO_OK) return Py_BuildValue("(i)", status);
    return PyLong_FromUnsignedLongLong((unsigned long long)(uintptr_t)out);
    END_HANDLE_TH_ERRORS
}

// (A, p, stream): a dense matrix with rows of adjacent elements -> (handle, buffer)
PyObject* from_dense(PyObject*, PyObject* args)
{
    HANDLE_TH_ERRORS
    PyObject* ao;
    Shape s;
    unsigned long long stream;
    if (!PyArg_ParseTuple(args, "OLK", &ao, &s.p, &stream)) return nullptr;
    const int64_t device = current_device();
    const at::Tensor* a = tensor(ao, at::kFloat, device);
    if (!a || a->dim() != 2 || a->stride(1) != 1 || !s.ok()) Py_RETURN_NONE;
    const int64_t m = a->size(0), k = a->size(1), lda = a->stride(0);
    const int32_t p = (int32_t)s.p;
    const size_t count_bytes = gcoo_calls.dense_count_bytes(m, k, p);
    if (count_bytes == 0) Py_RETURN_NONE;
    const float* ad = (const float*)a->data_ptr();
    void* sp = (void*)(uintptr_t)stream;
    at::Tensor buf;
    gcoo_matrix* out = nullptr;
    int status;
    {
        const NoGil released;
        const at::Tensor counts = bytes_on(device, count_bytes);
        int64_t nnz = 0;
        status = gcoo_calls.dense_count(m, k, ad, lda, p, counts.data_ptr(), (size_t)counts.numel(), sp, &nnz);
        if (status == GCOO_OK) {
            buf = bytes_on(device, gcoo_calls.device_bytes(m, k, nnz, p));
            status = gcoo_calls.from_dense_counted(m, k, nnz, ad, lda, p, counts.data_ptr(), buf.data_ptr(), (size_t)buf.numel(), sp, &out);
        }
    }
    if (status != GCOO_OK) return PyLong_FromLong(status);
    return matrix_and_buffer(out, buf);
    END_HANDLE_TH_ERRORS
}

// (handle, m, k, B, C or None, stream, variant) -> C
PyObject* spdm(PyObject*, PyObject* args)
{
    HANDLE_TH_ERRORS
    unsigned long long handle, stream;
    long long m, k;
    PyObject *bo, *co;
    int variant;
    if (!PyArg_ParseTuple(args, "KLLOOKi", &handle, &m, &k, &bo, &co, &stream, &variant)) return nullptr;
    const int64_t device = current_device();
    const at::Tensor* b = tensor(bo, at::kFloat, device);
    if (handle == 0 || !b || b->dim() != 2 || b->size(0) != k) Py_RETURN_NONE;
    const int64_t N = b->size(1), ldb = k <= 1 ? (N > 1 ? N : 1) : b->stride(0);
    if (b->stride(1) != 1 && N > 1) Py_RETURN_NONE;
    const at::Tensor* c = nullptr;
    if (co != Py_None) {
        c = tensor(co, at::kFloat, device);
        if (!c || c->dim() != 2 || c->size(0) != m || c->size(1) != N) Py_RETURN_NONE;
    }
    at::Tensor made;
    int status;
    {
        const NoGil released;
        if (!c) made = at::empty({m, N}, b->options());
        const at::Tensor& to = c ? *c : made;
        status = gcoo_calls.spdm_variant((const gcoo_matrix*)(uintptr_t)handle, (const float*)b->data_ptr(), ldb, N, (float*)to.data_ptr(), m > 1 ? to.stride(0) : (N > 1 ? N : 1),
                                         (void*)(uintptr_t)stream, variant);
    }
    if (status != GCOO_OK) return PyLong_FromLong(status);
    if (!c) return THPVariable_Wrap(made);
    Py_INCREF(co);
    return co;
    END_HANDLE_TH_ERRORS
}

PyObject* free_matrix(PyObject*, PyObject* arg)
{
    const unsigned long long h = PyLong_AsUnsignedLongLong(arg);
    if (PyErr_Occurred()) return nullptr;
    gcoo_calls.free_matrix((gcoo_matrix*)(uintptr_t)h);       // (host memory only)
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"bind", bind, METH_VARARGS, nullptr},
                         {"from_csr_device", from_csr_device, METH_VARARGS, nullptr},
                         {"from_csr_host", from_csr_host, METH_VARARGS, nullptr},
                         {"from_csr_device_static", from_csr_device_static, METH_VARARGS, nullptr},
                         {"from_dense", from_dense, METH_VARARGS, nullptr},
                         {"spdm", spdm, METH_VARARGS, nullptr},
                         {"free", free_matrix, METH_O, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", "Calls of the binding by the C ABI.", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() { return PyModule_Create(&module); }
