// The Python binding's calls that run once per product (binding.ap_gemv, binding.ap_gemm), as native functions: argument checks,
// output and workspace tensors, the current stream and the call of the C-ABI entry point.  They hold no logic of the library.
// A small product takes 3 to 5 us on the GPU; through ctypes and torch.empty its call took the host 6.1 us, of which the launch
// is 2.9.  Here: 4.6 (512 x 512, calls in a row).
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <ATen/ops/empty.h>

#include <algorithm>
#include <vector>

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

// The stream of a call: a named one, or (None) the current one
struct CallStream {
    void *address;
    bool named;
};

bool stream_of(PyObject *o, CallStream *out)
{
    out->named = o != Py_None;
    if (out->named) return address_of(o, &out->address);
    out->address = c10::hip::getCurrentHIPStream().stream();
    return true;
}

// x: `batch` rows of K activations or more
bool activations_ok(const at::Tensor &x, int64_t K)
{
    if (x.scalar_type() != at::kHalf || !x.is_cuda() || !x.is_contiguous()) {
        PyErr_SetString(PyExc_AssertionError, "x must be a contiguous float16 tensor on the GPU");
        return false;
    }
    if (x.numel() >= (x.dim() < 2 ? 1 : x.size(0)) * K) return true;
    PyErr_SetString(PyExc_AssertionError, "x holds fewer than K values per row");
    return false;
}

// Bytes of a given tensor's memory from its first element on; 0 for memory that the GPU cannot write
int64_t room(const at::Tensor &t)
{
    if (!t.is_cuda() && !t.is_pinned()) return 0;
    return (int64_t)t.storage().nbytes() - t.storage_offset() * (int64_t)t.element_size();
}

bool output_ok(const at::Tensor &y, int64_t batch, int64_t M)
{
    if (room(y) >= batch * M * 2) return true;
    PyErr_SetString(PyExc_AssertionError, "y must hold batch x M float16 values on the GPU");
    return false;
}

// Memory that work on the call's stream writes.  The caching allocator hands a block out in the order of the stream that is current,
// and again as soon as it is released there.  For a named stream it is therefore asked in that stream's order: from the current
// stream's blocks, work still queued there could use a block that the call overwrites, or be given one that the call still
// uses.  A tensor that is returned is read by the caller on the current stream, so its release waits for that one too.
at::Tensor allocate(at::IntArrayRef sizes, at::ScalarType type, at::Device device, const CallStream &stream, bool returned)
{
    const auto options = at::TensorOptions().dtype(type).device(device);
    if (!stream.named) return at::empty(sizes, options);
    const auto current = c10::hip::getCurrentHIPStreamMasqueradingAsCUDA(device.index());
    if (current.stream() == stream.address) return at::empty(sizes, options);
    struct Restore {
        decltype(current) &stream;
        ~Restore() { c10::hip::setCurrentHIPStreamMasqueradingAsCUDA(stream); }
    } restore{current};
    c10::hip::setCurrentHIPStreamMasqueradingAsCUDA(
        stream.address ? c10::hip::getStreamFromExternalMasqueradingAsCUDA(static_cast<hipStream_t>(stream.address), current.device_index())
                       : c10::hip::getDefaultHIPStreamMasqueradingAsCUDA(current.device_index()));
    at::Tensor t = at::empty(sizes, options);
    if (returned) t.record_stream(current.unwrap());
    return t;
}

// empty(sizes, half, device index, stream) -> a float16 (half != 0) or uint8 tensor that work on the named stream writes
PyObject *empty(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 4 || !PyTuple_Check(args[0])) {
        PyErr_SetString(PyExc_TypeError, "empty takes 4 arguments, a tuple first");
        return nullptr;
    }
    std::vector<int64_t> sizes;
    for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(args[0]); ++i) sizes.push_back(PyLong_AsLongLong(PyTuple_GET_ITEM(args[0], i)));
    const long half = PyLong_AsLong(args[1]), device = PyLong_AsLong(args[2]);
    CallStream stream;
    if (PyErr_Occurred() || !stream_of(args[3], &stream)) return nullptr;
    return THPVariable_Wrap(allocate(sizes, half ? at::kHalf : at::kByte, at::Device(at::kCUDA, (at::DeviceIndex)device), stream, true));
    END_HANDLE_TH_ERRORS
}

// gemv(handle, M, K, b, x, y, stream) -> y, or the status of a failed call
PyObject *gemv(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 7) {
        PyErr_SetString(PyExc_TypeError, "gemv takes 7 arguments");
        return nullptr;
    }
    void *handle;
    CallStream stream;
    const long M = PyLong_AsLong(args[1]), K = PyLong_AsLong(args[2]), b = PyLong_AsLong(args[3]);
    if (PyErr_Occurred() || !address_of(args[0], &handle)) return nullptr;
    const at::Tensor *x = tensor_of(args[4], "x");
    if (!x || !activations_ok(*x, K)) return nullptr;
    const int64_t batch = x->dim() == 1 ? 1 : x->size(0);
    const at::Tensor *given = args[5] == Py_None ? nullptr : tensor_of(args[5], "y");
    if (PyErr_Occurred() || (given && !output_ok(*given, batch, M))) return nullptr;
    if (!stream_of(args[6], &stream)) return nullptr;
    const at::Tensor y = given ? *given : allocate({batch, M}, at::kHalf, x->device(), stream, true);
    const void *xp = x->data_ptr();
    void *yp = y.data_ptr();
    ap_status status;
    Py_BEGIN_ALLOW_THREADS
    status = ap_gemv(static_cast<const ap_matrix *>(handle), (int)b, xp, yp, (int)batch, stream.address);
    Py_END_ALLOW_THREADS
    if (status != AP_OK) return PyLong_FromLong(status);
    if (given) {
        Py_INCREF(args[5]);
        return args[5];
    }
    return THPVariable_Wrap(y);
    END_HANDLE_TH_ERRORS
}

// gemm(handle, M, K, b, x, work, y, stream) -> y, or the status of a failed call (negative: of ap_gemm_workspace_size)
PyObject *gemm(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 8) {
        PyErr_SetString(PyExc_TypeError, "gemm takes 8 arguments");
        return nullptr;
    }
    void *handle;
    CallStream stream;
    const long M = PyLong_AsLong(args[1]), K = PyLong_AsLong(args[2]), b = PyLong_AsLong(args[3]);
    if (PyErr_Occurred() || !address_of(args[0], &handle)) return nullptr;
    const at::Tensor *x = tensor_of(args[4], "x");
    if (!x || !activations_ok(*x, K)) return nullptr;
    if (x->dim() != 2) {
        PyErr_SetString(PyExc_AssertionError, "x must have two dimensions");
        return nullptr;
    }
    size_t bytes = 0;
    ap_status status = ap_gemm_workspace_size(static_cast<const ap_matrix *>(handle), &bytes);
    if (status != AP_OK) return PyLong_FromLong(-(long)status);
    const at::Tensor *given_work = args[5] == Py_None ? nullptr : tensor_of(args[5], "work");
    const at::Tensor *given = args[6] == Py_None ? nullptr : tensor_of(args[6], "y");
    const int64_t batch = x->size(0);
    if (PyErr_Occurred() || (given && !output_ok(*given, batch, M))) return nullptr;
    if (!stream_of(args[7], &stream)) return nullptr;
    const at::Tensor work = given_work ? *given_work : allocate({(int64_t)bytes}, at::kByte, x->device(), stream, false);
    const at::Tensor y = given ? *given : allocate({batch, M}, at::kHalf, x->device(), stream, true);
    const void *xp = x->data_ptr();
    void *yp = y.data_ptr(), *wp = work.data_ptr();
    const size_t work_bytes = (size_t)(given_work ? std::min(work.numel(), room(work)) : work.numel());
    Py_BEGIN_ALLOW_THREADS
    status = ap_gemm(static_cast<const ap_matrix *>(handle), (int)b, xp, yp, (int)batch, wp, work_bytes, stream.address);
    Py_END_ALLOW_THREADS
    if (status != AP_OK) return PyLong_FromLong(status);
    if (given) {
        Py_INCREF(args[6]);
        return args[6];
    }
    return THPVariable_Wrap(y);
    END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"gemv", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(gemv)), METH_FASTCALL, nullptr},
    {"empty", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(empty)), METH_FASTCALL, nullptr},
    {"gemm", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(gemm)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_torch_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__torch_call() { return PyModule_Create(&module); }
