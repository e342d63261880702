// The compute calls for Python in one step: arguments checked, output allocated, stream looked up, library called.
//
// Small calls are bound by this: through ctypes a call took 13 us of host time (per tensor a handful of attribute reads and
// a pointer object, a device context, a stream object, 17 conversions), more than the GPU needs below some 8 M cells of S.
// Here it takes 4-5 us, the output's allocation and the launches included.
//
// Only what is as expected is done here.  Anything else - a tensor of the wrong kind, a device that is not current, a size
// that is no int, an error from the library - returns None with nothing done, and binding.py goes through the call
// step by step, which says what is wrong.
#include <Python.h>

#include <ATen/core/LegacyTypeDispatch.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/csrk.h"

namespace {

struct Unexpected {};

int to_int(PyObject *o) {
    if (!PyLong_CheckExact(o)) throw Unexpected{};
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow || v < 0 || v > INT32_MAX) throw Unexpected{};
    return (int)v;
}

struct Args {
    c10::Device device{c10::kCUDA, 0};

    const at::Tensor *tensor(PyObject *o) const {
        if (o == Py_None) return nullptr;
        if (!THPVariable_Check(o)) throw Unexpected{};
        return &THPVariable_Unpack(o);
    }
    void *checked(const at::Tensor *t, at::ScalarType type, int64_t rows, int64_t cols) const {     // cols < 0: one dimension
        if (!t) throw Unexpected{};
        if (!t->is_cuda() || t->device() != device || t->scalar_type() != type || !t->is_contiguous()) throw Unexpected{};
        if (t->dim() != (cols < 0 ? 1 : 2) || t->size(0) != rows || (cols >= 0 && t->size(1) != cols)) throw Unexpected{};
        return t->data_ptr();
    }
    void *optional(PyObject *o, at::ScalarType type, int64_t rows, int64_t cols) const {
        return o == Py_None ? nullptr : checked(tensor(o), type, rows, cols);
    }
    // the output: as given, or a new one (`made`)
    void *output(PyObject *o, int64_t rows, int64_t cols, at::Tensor &made) const {
        if (o != Py_None) return checked(tensor(o), at::kFloat, rows, cols);
        at::AutoDispatchBelowADInplaceOrView guard;
        const auto options = at::TensorOptions().dtype(at::kFloat).device(device);
        made = cols < 0 ? at::empty({rows}, options) : at::empty({rows, cols}, options);
        return made.data_ptr();
    }
};

PyObject *result(PyObject *given, at::Tensor &made, csrk_status status) {
    if (status != CSRK_OK) Py_RETURN_NONE;
    if (given == Py_None) return THPVariable_Wrap(std::move(made));
    Py_INCREF(given);
    return given;
}

// the dense operands of an operation; those it has no use for are NULL
struct Operands {
    const void *A = nullptr, *B = nullptr, *C = nullptr;
    Operands(const Args &a, int op, at::ScalarType type, int M, int K, int D, int N, PyObject *pa, PyObject *pb, PyObject *pc) {
        if (op != CSRK_OP_SPMM) {
            A = a.checked(a.tensor(pa), type, M, D);
            B = a.checked(a.tensor(pb), type, K, D);
        }
        if (op != CSRK_OP_SDDMM) C = a.checked(a.tensor(pc), type, K, N);
    }
};

template <typename F>
PyObject *guarded(F &&f) {
    try {
        return f();
    } catch (...) {         // (also what torch throws about tensors without storage and the like)
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

// call(op, bf16, M, K, D, N, rowptr, colidx, vals, A, B, C, out, workspace)
PyObject *call(PyObject *, PyObject *const *v, Py_ssize_t n) {
    return guarded([&]() -> PyObject * {
        if (n != 14) throw Unexpected{};
        const int op = to_int(v[0]), bf16 = to_int(v[1]), M = to_int(v[2]), K = to_int(v[3]), D = to_int(v[4]), N = to_int(v[5]);
        Args a;
        const at::Tensor *rp = a.tensor(v[6]), *ci = a.tensor(v[7]);
        if (!rp || !ci || !rp->is_cuda()) throw Unexpected{};
        a.device = rp->device();
        if (a.device.index() != c10::hip::current_device()) throw Unexpected{};
        const int64_t nnz = ci->numel();
        const void *rowptr = a.checked(rp, at::kInt, (int64_t)M + 1, -1), *colidx = a.checked(ci, at::kInt, nnz, -1);
        const void *vals = a.optional(v[8], at::kFloat, nnz, -1);
        const Operands x(a, op, bf16 ? at::kBFloat16 : at::kFloat, M, K, D, N, v[9], v[10], v[11]);
        void *ws = nullptr;
        size_t ws_bytes = 0;
        if (v[13] != Py_None) {
            const at::Tensor *w = a.tensor(v[13]);
            if (!w->is_cuda() || w->device() != a.device || !w->is_contiguous()) throw Unexpected{};
            ws = w->data_ptr();
            ws_bytes = w->nbytes();
            if (!ws) throw Unexpected{};
        }
        at::Tensor made;
        void *out = op == CSRK_OP_SDDMM ? a.output(v[12], nnz, -1, made) : a.output(v[12], M, N, made);
        const hipStream_t stream = c10::hip::getCurrentHIPStream(a.device.index()).stream();
        csrk_status status;
        Py_BEGIN_ALLOW_THREADS
        status = csrk_call_bounded(op, bf16, nnz, M, K, D, N, (const int32_t *)rowptr, (const int32_t *)colidx, (const float *)vals,
                                   x.A, x.B, x.C, (float *)out, ws, ws_bytes, stream);
        Py_END_ALLOW_THREADS
        return result(v[12], made, status);
    });
}

// call_plan(op, handle, M, K, D, N, colidx, vals, A, B, C, out)
PyObject *call_plan(PyObject *, PyObject *const *v, Py_ssize_t n) {
    return guarded([&]() -> PyObject * {
        if (n != 12 || !PyLong_CheckExact(v[1])) throw Unexpected{};
        const int op = to_int(v[0]), M = to_int(v[2]), K = to_int(v[3]), D = to_int(v[4]), N = to_int(v[5]);
        const csrk_plan *plan = static_cast<const csrk_plan *>(PyLong_AsVoidPtr(v[1]));
        Args a;
        const at::Tensor *ci = a.tensor(v[6]);
        if (!plan || !ci || !ci->is_cuda()) throw Unexpected{};
        a.device = ci->device();
        if (a.device.index() != c10::hip::current_device()) throw Unexpected{};
        const int64_t nnz = ci->numel();
        const float *vals = (const float *)a.optional(v[7], at::kFloat, nnz, -1);
        const Operands x(a, op, at::kFloat, M, K, D, N, v[8], v[9], v[10]);
        at::Tensor made;
        float *out = (float *)(op == CSRK_OP_SDDMM ? a.output(v[11], nnz, -1, made) : a.output(v[11], M, N, made));
        const float *A = (const float *)x.A, *B = (const float *)x.B, *C = (const float *)x.C;
        const hipStream_t stream = c10::hip::getCurrentHIPStream(a.device.index()).stream();
        csrk_status status;
        Py_BEGIN_ALLOW_THREADS
        status = op == CSRK_OP_SPMM    ? spmm_csr_plan(plan, N, vals, C, out, stream)
                 : op == CSRK_OP_SDDMM ? sddmm_csr_plan(plan, D, vals, A, B, out, stream)
                                       : fusedmm_csr_plan(plan, D, N, vals, A, B, C, out, stream);
        Py_END_ALLOW_THREADS
        return result(v[11], made, status);
    });
}

PyMethodDef methods[] = {{"call", (PyCFunction)(void (*)(void))call, METH_FASTCALL, nullptr},
                         {"call_plan", (PyCFunction)(void (*)(void))call_plan, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_torch_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__torch_calls() { return PyModule_Create(&module); }
