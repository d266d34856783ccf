// The per-product call of the Python binding as a CPython extension: smat_spmm on torch tensors.
//
// A product of a small matrix takes the GPU 4 us; the same call marshalled in Python (shape and device checks,
// the handle's dimensions through ctypes, the current stream, six ctypes conversions, the new C) takes the host 11 us,
// so a loop of such products waits for Python.  Here the checks read the tensors' fields, C comes straight from
// the allocator, and what is left is the launch itself.
//
// Only the call that is plainly in order is taken.  Whatever is not -- operands that do not fit, a stream object, a
// tensor subclass -- returns NotImplemented, and smat.py goes through its own checks, which raise with their
// messages or handle the case.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/core/LegacyTypeDispatch.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>

#include "../../include/smat.h"

namespace {

PyObject* not_mine()
{
    Py_RETURN_NOTIMPLEMENTED;
}

// spmm(handle, B, C or None, N or None) -> C, a nonzero status of smat_spmm, or NotImplemented
PyObject* spmm(PyObject*, PyObject* const* args, Py_ssize_t nargs)
{
    if (nargs != 4 || !PyLong_CheckExact(args[0]) || !THPVariable_CheckExact(args[1])) return not_mine();
    const bool make_c = args[2] == Py_None;
    if (!make_c && !THPVariable_CheckExact(args[2])) return not_mine();
    const auto* h = static_cast<const smat_handle_t*>(PyLong_AsVoidPtr(args[0]));
    int64_t M = 0, K = 0, N = -1;
    int dtype = 0;
    if (!h || smat_get_dims(h, &M, &K, &dtype) != SMAT_OK) {
        PyErr_Clear();
        return not_mine();
    }
    if (args[3] != Py_None) {
        if (!PyLong_CheckExact(args[3])) return not_mine();
        int overflow = 0;
        N = PyLong_AsLongLongAndOverflow(args[3], &overflow);
        if (overflow || N < 0) return not_mine();
    }
    const at::Tensor& b = THPVariable_Unpack(args[1]);
    // the same conditions as _check_device_operands in smat.py
    const int64_t elem = dtype == SMAT_F16 || dtype == SMAT_BF16 ? 2 : 1;
    if (!b.is_cuda() || b.dim() != 2 || b.layout() != at::kStrided || static_cast<int64_t>(b.element_size()) != elem ||
        b.stride(1) != 1 || b.size(0) < K)
        return not_mine();
    if (N < 0) N = b.size(1);
    if (N > b.size(1)) return not_mine();
    const int64_t ldb = b.size(0) > 1 ? b.stride(0) : std::max(b.size(1), N);
    if (K > 1 && ldb < N) return not_mine();
    try {
        at::Tensor c;
        if (make_c) {
            at::AutoDispatchBelowADInplaceOrView no_autograd;
            c = at::empty({M, N}, b.options().dtype(dtype == SMAT_I8 ? at::kInt : at::kFloat));
        } else {
            c = THPVariable_Unpack(args[2]);
            if (!c.is_cuda() || c.device() != b.device() || c.dim() != 2 || c.layout() != at::kStrided || c.element_size() != 4 ||
                c.stride(1) != 1 || c.size(0) < M || N > c.size(1))
                return not_mine();
        }
        const int64_t ldc = c.size(0) > 1 ? c.stride(0) : std::max(c.size(1), N);
        if (M > 1 && ldc < N) return not_mine();
        const void* bp = b.data_ptr();
        void* cp = c.data_ptr();
        void* stream = c10::hip::getCurrentHIPStream().stream();
        smat_status_t st;
        Py_BEGIN_ALLOW_THREADS
        st = smat_spmm(h, bp, ldb, cp, ldc, N, stream);
        Py_END_ALLOW_THREADS
        if (st != SMAT_OK) return PyLong_FromLong(st);
        if (make_c) return THPVariable_Wrap(std::move(c));
        Py_INCREF(args[2]);
        return args[2];
    } catch (...) {
        return not_mine();          // out of memory and the like: the Python path raises torch's own exception
    }
}

PyMethodDef methods[] = {
    {"spmm", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(spmm)), METH_FASTCALL,
     "spmm(handle, B, C or None, N or None) -> C, a nonzero status, or NotImplemented"},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_torch_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__torch_call(void) { return PyModule_Create(&module); }
