// The Python binding's calls that run once per product (binding.ap_gemv, binding.ap_gemm), as native functions: argument checks,
// output and workspace tensors, the current stream and the call of the C-ABI entry point.  They hold no logic of the library.
// A small product takes 3 to 5 us on the GPU; through ctypes and torch.empty its call took the host 6.1 us, of which the launch
// is 2.9.  Here: 4.6 (512 x 512, calls in a row).
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>

#include "../../include/apgemv.h"

namespace {

// `o` as a tensor, or an error set
const at::Tensor *tensor_of(PyObject *o, const char *what)
{
    if (THPVariable_Check(o)) return &THPVariable_Unpack(o);
    PyErr_Format(PyExc_TypeError, "%s must be a torch.Tensor", what);
    return nullptr;
}

// An address given as an int or None (0); false with an error set otherwise
bool address_of(PyObject *o, void **out)
{
    *out = nullptr;
    if (o == Py_None) return true;
    *out = PyLong_AsVoidPtr(o);
    return !PyErr_Occurred();
}

bool stream_of(PyObject *o, void **out)
{
    if (o != Py_None) return address_of(o, out);
    *out = c10::hip::getCurrentHIPStream().stream();
    return true;
}

bool activations_ok(const at::Tensor &x)
{
    if (x.scalar_type() == at::kHalf && x.is_cuda() && x.is_contiguous()) return true;
    PyErr_SetString(PyExc_AssertionError, "x must be a contiguous float16 tensor on the GPU");
    return false;
}

at::Tensor output_like(const at::Tensor &x, int64_t batch, int64_t M)
{
    return at::empty({batch, M}, at::TensorOptions().dtype(at::kHalf).device(x.device()));
}

// gemv(handle, M, b, x, y, stream) -> y, or the status of a failed call
PyObject *gemv(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 6) {
        PyErr_SetString(PyExc_TypeError, "gemv takes 6 arguments");
        return nullptr;
    }
    void *handle, *stream;
    const long M = PyLong_AsLong(args[1]), b = PyLong_AsLong(args[2]);
    if (PyErr_Occurred() || !address_of(args[0], &handle)) return nullptr;
    const at::Tensor *x = tensor_of(args[3], "x");
    if (!x || !activations_ok(*x)) return nullptr;
    const int64_t batch = x->dim() == 1 ? 1 : x->size(0);
    const at::Tensor *given = args[4] == Py_None ? nullptr : tensor_of(args[4], "y");
    if (PyErr_Occurred()) return nullptr;
    const at::Tensor y = given ? *given : output_like(*x, batch, M);
    if (!stream_of(args[5], &stream)) return nullptr;
    const void *xp = x->data_ptr();
    void *yp = y.data_ptr();
    ap_status status;
    Py_BEGIN_ALLOW_THREADS
    status = ap_gemv(static_cast<const ap_matrix *>(handle), (int)b, xp, yp, (int)batch, stream);
    Py_END_ALLOW_THREADS
    if (status != AP_OK) return PyLong_FromLong(status);
    if (given) {
        Py_INCREF(args[4]);
        return args[4];
    }
    return THPVariable_Wrap(y);
    END_HANDLE_TH_ERRORS
}

// gemm(handle, M, b, x, work, y, stream) -> y, or the status of a failed call (negative: of ap_gemm_workspace_size)
PyObject *gemm(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 7) {
        PyErr_SetString(PyExc_TypeError, "gemm takes 7 arguments");
        return nullptr;
    }
    void *handle, *stream;
    const long M = PyLong_AsLong(args[1]), b = PyLong_AsLong(args[2]);
    if (PyErr_Occurred() || !address_of(args[0], &handle)) return nullptr;
    const at::Tensor *x = tensor_of(args[3], "x");
    if (!x || !activations_ok(*x)) return nullptr;
    if (x->dim() != 2) {
        PyErr_SetString(PyExc_AssertionError, "x must have two dimensions");
        return nullptr;
    }
    size_t bytes = 0;
    ap_status status = ap_gemm_workspace_size(static_cast<const ap_matrix *>(handle), &bytes);
    if (status != AP_OK) return PyLong_FromLong(-(long)status);
    const at::Tensor *given_work = args[4] == Py_None ? nullptr : tensor_of(args[4], "work");
    const at::Tensor *given = args[5] == Py_None ? nullptr : tensor_of(args[5], "y");
    if (PyErr_Occurred()) return nullptr;
    const int64_t batch = x->size(0);
    const at::Tensor work = given_work ? *given_work
                                       : at::empty({(int64_t)bytes}, at::TensorOptions().dtype(at::kByte).device(x->device()));
    const at::Tensor y = given ? *given : output_like(*x, batch, M);
    if (!stream_of(args[6], &stream)) return nullptr;
    const void *xp = x->data_ptr();
    void *yp = y.data_ptr(), *wp = work.data_ptr();
    const size_t work_bytes = (size_t)work.numel();
    Py_BEGIN_ALLOW_THREADS
    status = ap_gemm(static_cast<const ap_matrix *>(handle), (int)b, xp, yp, (int)batch, wp, work_bytes, stream);
    Py_END_ALLOW_THREADS
    if (status != AP_OK) return PyLong_FromLong(status);
    if (given) {
        Py_INCREF(args[5]);
        return args[5];
    }
    return THPVariable_Wrap(y);
    END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"gemv", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(gemv)), METH_FASTCALL, nullptr},
    {"gemm", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(gemm)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_torch_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__torch_call() { return PyModule_Create(&module); }
