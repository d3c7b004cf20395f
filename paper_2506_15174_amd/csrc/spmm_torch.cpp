// Python entry of the product on torch tensors: the checks, the output allocation, the
// stream look-up and the call of spmm_execute in one native function.
//
// A short product is over in 3 to 5 us, less than the interpreter needs for the same steps
// (attribute reads of the tensors and of the stream, torch.empty, a ctypes call: 8.2 us per
// product of a 256 x 256 matrix and 32 columns with the output allocated, 6.3 us with the
// output handed in), so a loop over products waited for Python and not for the GPU.  Here
// a call is bound by the launch itself (about 2.7 us).
//
// PyTorch is used for device memory and streams only, as everywhere in this package.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/Context.h>
#include <ATen/EmptyTensor.h>
#include <ATen/record_function.h>
#include <ATen/hip/impl/HIPCachingAllocatorMasqueradingAsCUDA.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <stdint.h>

#include <exception>

#include "../../include/spmm.h"

namespace {

// Lets other Python threads run: an allocation may have to free and wait, a launch waits while its queue is
// full.  (Handing the interpreter over and back costs 0.05 us where no other thread wants it.)
struct others_run {
    PyThreadState *state = PyEval_SaveThread();
    ~others_run() { PyEval_RestoreThread(state); }
};

// An output beside B.  On its way through the dispatcher at::empty takes 0.3 us of a small product's 4.4 (256 x 256, 32 columns:
// now 4.1).  Where nothing may want to see or change that call (a dispatch mode, a functional transform, inference mode, a profiler,
// the fill of deterministic mode) and the device is set, the tensor is made from the same allocator directly.
at::Tensor output(const at::Tensor &B, int64_t M, int64_t N)
{
    const c10::impl::LocalDispatchKeySet local = c10::impl::tls_local_dispatch_key_set();
    const bool plain = local.included_ == c10::default_included_set && local.excluded_ == c10::default_excluded_set &&
                       !c10::impl::TorchDispatchModeTLS::any_modes_set() && !at::hasCallbacks() && !at::globalContext().deterministicAlgorithms() &&
                       B.key_set().has(c10::DispatchKey::CUDA) && c10::hip::current_device() == B.device().index();
    if (!plain) return at::empty({M, N}, B.options().requires_grad(false));
    const int64_t sizes[2] = {M, N};
    return at::Tensor(at::detail::empty_generic(sizes, c10::hip::HIPCachingAllocatorMasqueradingAsCUDA::get(), c10::DispatchKeySet(c10::DispatchKey::CUDA), at::kFloat, std::nullopt));
}

// execute(plan address, M, K, B, C or None, stream or None) -> C, or the status code as int
PyObject *execute(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    if (nargs != 6) {
        PyErr_SetString(PyExc_TypeError, "execute(plan, M, K, B, C, stream)");
        return nullptr;
    }
    const spmm_plan_t *plan = static_cast<const spmm_plan_t *>(PyLong_AsVoidPtr(args[0]));
    const int64_t M = PyLong_AsLongLong(args[1]), K = PyLong_AsLongLong(args[2]);
    if (PyErr_Occurred()) return nullptr;
    if (!THPVariable_Check(args[3]) || (args[4] != Py_None && !THPVariable_Check(args[4]))) {
        PyErr_SetString(PyExc_TypeError, "B and C must be torch tensors");
        return nullptr;
    }
    try {
        const at::Tensor &B = THPVariable_Unpack(args[3]);  // the caller's references keep B and C while other threads run
        if (!(B.is_cuda() && B.scalar_type() == at::kFloat && B.is_contiguous() && B.dim() == 2)) {
            PyErr_SetString(PyExc_ValueError, "B must be a contiguous 2-D float32 device tensor");
            return nullptr;
        }
        if (B.size(0) != K) {
            PyErr_Format(PyExc_ValueError, "B has %lld rows, A has %lld columns", (long long)B.size(0), (long long)K);
            return nullptr;
        }
        const int64_t N = B.size(1);
        if (N > INT32_MAX) {
            PyErr_SetString(PyExc_ValueError, "B has more columns than the library's 32-bit column count");
            return nullptr;
        }
        const bool given = args[4] != Py_None;
        at::Tensor made;
        const at::Tensor &C = given ? THPVariable_Unpack(args[4]) : made;
        if (given) {
            if (!(C.is_cuda() && C.scalar_type() == at::kFloat && C.is_contiguous() && C.dim() == 2 && C.size(0) == M &&
                  C.size(1) == N)) {
                PyErr_SetString(PyExc_ValueError, "C must be a contiguous float32 device tensor of shape (M, N)");
                return nullptr;
            }
        }
        void *stream;
        if (args[5] == Py_None) {
            stream = c10::hip::getCurrentHIPStream(B.device().index()).stream();
        } else {
            PyObject *s = PyObject_GetAttrString(args[5], "cuda_stream");
            if (!s) return nullptr;
            stream = PyLong_AsVoidPtr(s);
            Py_DECREF(s);
            if (PyErr_Occurred()) return nullptr;
        }
        spmm_status_t st;
        {
            others_run free_to_run;
            if (!given) made = output(B, M, N);
            st = spmm_execute(plan, static_cast<const float *>(B.const_data_ptr()), (int32_t)N, static_cast<float *>(C.data_ptr()), stream);
        }
        if (st != SPMM_OK) return PyLong_FromLong((long)st);
        if (!given) return THPVariable_Wrap(std::move(made));
        Py_INCREF(args[4]);
        return args[4];
    } catch (...) {  // as torch's own functions report it, e.g. torch.OutOfMemoryError for the output
        torch::translate_exception_to_python(std::current_exception());
        return nullptr;
    }
}

PyMethodDef methods[] = {
    {"execute", (PyCFunction)(void (*)(void))execute, METH_FASTCALL,
     "execute(plan, M, K, B, C, stream): spmm_execute on torch tensors; returns C, or a status code"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_spmm_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__spmm_torch(void) { return PyModule_Create(&module_def); }
