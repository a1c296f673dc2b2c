// The common call of the Python fa2_fwd, from torch tensors to the launch, without a Python frame in between.
//
// What bounds a small problem is the host: B1 H2 N256 d64 runs 5.5 us on the GPU and took 10.0 us a call, of which the launch
// is 2.7; two allocations from Python took 3.0 us, marshalling 16 arguments through ctypes 1.3, and the checks and
// attribute reads the rest.
//
// forward() takes plain strided tensors of the current device and does nothing but what the Python path does with them; for
// everything else (another device, a subclass, a tensor that a transform has wrapped, an active torch function or dispatch
// mode, a capture that needs scratch memory, arguments that are refused) it returns None before it has allocated or launched
// anything, and the Python path goes on, with its own checks and errors.
#include <torch/csrc/python_headers.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/hip/EmptyTensor.h>
#include <ATen/record_function.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/core/impl/VirtualGuardImpl.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>

#include "fa2.h"

namespace {

// A strided tensor of device memory with nothing above it but autograd and autocast.
bool plain(PyObject* obj) {
  if (!THPVariable_CheckExact(obj)) return false;
  const at::Tensor& t = THPVariable_Unpack(obj);
  static const c10::DispatchKeySet allowed =
      c10::DispatchKeySet(c10::DispatchKey::CUDA) | c10::getAutogradRelatedKeySetFromBackend(c10::BackendComponent::CUDABit) |
      c10::getAutocastRelatedKeySetFromBackend(c10::BackendComponent::CUDABit);
  // (the difference keeps the bit of the backend; what is asked for is that no functionality beyond these is left)
  return t.defined() && t.is_cuda() && (t.key_set() - allowed).highestFunctionalityKey() == c10::DispatchKey::Undefined &&
         t.has_storage() && t.is_contiguous();
}

// The interpreter's lock given up for a scope, which an exception may leave.
struct WithoutGil {
  PyThreadState* const state = PyEval_SaveThread();
  WithoutGil() = default;
  WithoutGil(const WithoutGil&) = delete;
  ~WithoutGil() { PyEval_RestoreThread(state); }
};

// Device memory from the allocator that torch's own factory functions use, without their way through the dispatcher: O and LSE
// took 1.1 us of a call's 4.9 so, 0.5 now (B1 H2 N256 d64; the kernel takes 4.4).  Where something has asked to see dispatched calls
// (a transform, a trace, a profiler's record of operators), they are made.
bool calls_are_seen() {
  return !(c10::impl::tls_local_dispatch_key_set().included_ - c10::default_included_set).empty() ||
         at::getStepCallbacksUnlessEmpty(at::RecordScope::FUNCTION).has_value();
}

at::Tensor empty(at::IntArrayRef sizes, at::ScalarType type, c10::Device device, bool seen) {
  if (seen) return at::empty(sizes, at::TensorOptions().dtype(type).device(device));
  return at::Tensor(at::detail::empty_cuda(sizes, type, device, std::nullopt));
}

// ... with the strides of t too: those of sizes of one may be any
at::Tensor empty_as(const at::Tensor& t, bool seen) {
  if (seen) return at::empty_like(t);
  return at::Tensor(at::detail::empty_strided_cuda(t.sizes(), t.strides(), t.scalar_type(), t.device()));
}

// forward(q, k, v, scale, out, lse, return_lse, causal): (O, LSE), or the library's error code, or None
PyObject* forward(PyObject*, PyObject* const* args, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  if (n_args != 8) {
    PyErr_SetString(PyExc_TypeError, "forward() takes 8 arguments");
    return nullptr;
  }
  if (at::impl::PythonTorchFunctionTLS::stack_len() > 0 || c10::impl::TorchDispatchModeTLS::any_modes_set()) Py_RETURN_NONE;
  for (int i = 0; i < 3; ++i)
    if (!plain(args[i])) Py_RETURN_NONE;
  const at::Tensor &q = THPVariable_Unpack(args[0]), &k = THPVariable_Unpack(args[1]), &v = THPVariable_Unpack(args[2]);
  const at::ScalarType type = q.scalar_type();
  if ((type != at::kHalf && type != at::kBFloat16) || k.scalar_type() != type || v.scalar_type() != type) Py_RETURN_NONE;
  if (q.dim() != 4 || k.dim() != 4 || k.sizes() != v.sizes()) Py_RETURN_NONE;
  const c10::Device device = q.device();
  if (k.device() != device || v.device() != device) Py_RETURN_NONE;
  const c10::impl::VirtualGuardImpl guard(c10::DeviceType::CUDA);
  if (guard.getDevice() != device) Py_RETURN_NONE;
  const int64_t B = q.size(0), Nq = q.size(1), H = q.size(2), d = q.size(3), Nk = k.size(1);
  if (k.size(0) != B || k.size(2) != H || k.size(3) != d) Py_RETURN_NONE;
  if (B > INT_MAX || Nq > INT_MAX || H > INT_MAX || d > INT_MAX || Nk > INT_MAX) Py_RETURN_NONE;

  const int return_lse = PyObject_IsTrue(args[6]), causal = PyObject_IsTrue(args[7]);
  if (return_lse < 0 || causal < 0) return nullptr;
  at::Tensor out, lse;
  if (args[4] != Py_None) {
    if (!plain(args[4])) Py_RETURN_NONE;
    out = THPVariable_Unpack(args[4]);
    if (out.sizes() != q.sizes() || out.scalar_type() != type || out.device() != device) Py_RETURN_NONE;
  }
  if (return_lse && args[5] != Py_None) {
    if (!plain(args[5])) Py_RETURN_NONE;
    lse = THPVariable_Unpack(args[5]);
    if (lse.dim() != 3 || lse.size(0) != B || lse.size(1) != H || lse.size(2) != Nq || lse.scalar_type() != at::kFloat ||
        lse.device() != device)
      Py_RETURN_NONE;
  }
  const double scale = PyFloat_AsDouble(args[3]);
  if (scale == -1.0 && PyErr_Occurred()) {   // float() takes more than this, a text for instance
    PyErr_Clear();
    Py_RETURN_NONE;
  }

  const hipStream_t stream = c10::hip::getCurrentHIPStream(device.index()).stream();
  const int mask = causal ? FA2_MASK_CAUSAL : FA2_MASK_NONE;
  const size_t bytes = Nk < FA2_SPLIT_MIN_KEYS ? 0 : fa2_workspace_bytes((int)B, (int)H, (int)Nq, (int)Nk, (int)d, mask);
  if (bytes != 0) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &status) != hipSuccess || status != hipStreamCaptureStatusNone) Py_RETURN_NONE;
  }
  at::Tensor workspace;
  int rc;
  {
    // (an allocation waits for the driver at times, a launch where the queue is full)
    const WithoutGil released;
    const bool seen = calls_are_seen();
    if (!out.defined()) out = empty_as(q, seen);
    if (return_lse && !lse.defined()) lse = empty({B, H, Nq}, at::kFloat, device, seen);
    // Scratch of the launch stream: dropped on return, its memory is handed out again only behind this call's kernels.  Without
    // it the call still runs, its keys unsplit.
    if (bytes != 0) {
      try {
        workspace = empty({(int64_t)bytes}, at::kByte, device, seen);
      } catch (const c10::OutOfMemoryError&) {
      }
    }
    rc = fa2_fwd_ws(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(),
                    lse.defined() ? static_cast<float*>(lse.data_ptr()) : nullptr, (int)B, (int)H, (int)Nq, (int)Nk, (int)d,
                    (float)scale, type == at::kHalf ? FA2_FP16 : FA2_BF16, mask,
                    workspace.defined() ? workspace.data_ptr() : nullptr, bytes, stream);
  }
  if (rc != FA2_OK) return PyLong_FromLong(rc);

  PyObject* const o_obj = args[4] != Py_None ? Py_NewRef(args[4]) : THPVariable_Wrap(out);
  if (o_obj == nullptr) return nullptr;
  PyObject* const l_obj = !return_lse ? Py_NewRef(Py_None) : args[5] != Py_None ? Py_NewRef(args[5]) : THPVariable_Wrap(lse);
  if (l_obj == nullptr) {
    Py_DECREF(o_obj);
    return nullptr;
  }
  PyObject* const result = PyTuple_New(2);
  if (result == nullptr) {
    Py_DECREF(o_obj);
    Py_DECREF(l_obj);
    return nullptr;
  }
  PyTuple_SET_ITEM(result, 0, o_obj);
  PyTuple_SET_ITEM(result, 1, l_obj);
  return result;
  END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"forward", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(forward)), METH_FASTCALL,
     "forward(q, k, v, scale, out, lse, return_lse, causal) -> (O, LSE), an error code, or None: the Python path's"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fa2_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fa2_torch(void) {
  PyObject* const m = PyModule_Create(&module);
  if (m != nullptr && PyModule_AddStringConstant(m, "torch_version", FA2_TORCH_VERSION) != 0) {   // whose headers these are
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
