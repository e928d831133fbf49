// The caller-side sequence of runtime.py for the calls that a program makes most, as one native call each: check the
// operands, read the run-time shapes, allocate the result, take the current stream, run the C entry point.
//
// What bounds a small operator is this sequence, not its kernel: for a 23 x 128 x 128 dense layer (kernel 2.7 us, launch
// 2.2) the steps in Python and their ctypes calls took 8.6 us.  The functions here serve plain operands only (strided
// torch.Tensor or Parameter on the GPU, contiguous, of the right type and extents, no function or dispatch mode, no trace); anything
// else, and every error, is answered with None, and the caller goes through the steps one by one, which also
// raises the errors.  Nothing is kept from call to call but the entry points and the default workspaces that
// runtime.py made.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/InferenceMode.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "nimble.h"
#include "nimble_vm.h"

namespace {

decltype(&nimble_dense_dyn) g_dense;
decltype(&nimble_attention_dyn) g_attention;
decltype(&nimble_attention_chain_dyn) g_attention_chain;
decltype(&nimble_vm_run) g_vm_run;
decltype(&nimble_lstm_seq_preferred) g_seq_preferred;
decltype(&nimble_lstm_seq_workspace_bytes) g_seq_workspace_bytes;
decltype(&nimble_lstm_seq_pre_dyn) g_seq_pre;
decltype(&nimble_lstm_seq_status) g_seq_status;
PyObject* g_current_device;  // torch._C._cuda_getDevice
PyObject* g_raw_stream;      // torch._C._cuda_getCurrentRawStream

constexpr int kMaxDevices = 64;
struct Workspace {
  PyObject* tensor = nullptr;  // (kept alive for as long as its address is used here)
  void* ptr = nullptr;
  size_t bytes = 0;
};
Workspace g_workspace[kMaxDevices];

// Dispatch keys of an ordinary GPU tensor, made outside and inside inference mode.  Wrapped tensors (vmap, grad
// transforms, functionalization, fake tensors) carry other keys.
c10::DispatchKeySet g_plain, g_inference;

bool modes_active() {
  return at::impl::PythonTorchFunctionTLS::stack_len() > 0 || c10::impl::TorchDispatchModeTLS::any_modes_set() ||
         c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::Tracer);
}

const at::Tensor* plain(PyObject* o, at::ScalarType dtype) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || t.scalar_type() != dtype || !t.is_cuda() || !t.is_contiguous()) return nullptr;
  if (!g_raw_stream || (t.key_set() != g_plain && t.key_set() != g_inference)) return nullptr;
  return &t;
}

// The current device's current stream; false with a Python error set.
bool current_stream(void** stream) {
  PyObject* dev = PyObject_CallNoArgs(g_current_device);
  if (!dev) return false;
  PyObject* s = PyObject_CallOneArg(g_raw_stream, dev);
  Py_DECREF(dev);
  if (!s) return false;
  *stream = PyLong_AsVoidPtr(s);
  Py_DECREF(s);
  return !PyErr_Occurred();
}

const Workspace* workspace_of(const at::Tensor& t) {
  const int d = t.get_device();
  return d >= 0 && d < kMaxDevices && g_workspace[d].ptr ? &g_workspace[d] : nullptr;
}

at::Tensor empty_like(const at::Tensor& t, at::IntArrayRef sizes, at::ScalarType dtype) {
  return at::empty(sizes, at::TensorOptions().dtype(dtype).device(t.device()));
}

// dense(x, w, bias or None, epilogue, out_dtype) -> y or None
PyObject* dense(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 5 || modes_active() || !PyLong_CheckExact(args[3]) || !PyLong_CheckExact(args[4])) Py_RETURN_NONE;
  const at::Tensor *x = plain(args[0], at::kBFloat16), *w = plain(args[1], at::kBFloat16), *b = nullptr;
  if (!x || !w || x->dim() != 2 || w->dim() != 2 || x->size(1) != w->size(1)) Py_RETURN_NONE;
  const int64_t M = x->size(0), N = w->size(0), K = x->size(1);
  if (args[2] != Py_None && (!(b = plain(args[2], at::kBFloat16)) || b->numel() != N)) Py_RETURN_NONE;
  const long epilogue = PyLong_AsLong(args[3]), out_dtype = PyLong_AsLong(args[4]);
  if (epilogue < NIMBLE_EPI_NONE || epilogue > NIMBLE_EPI_BIAS_GELU_ERF || (out_dtype != NIMBLE_BF16 && out_dtype != NIMBLE_F32)) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  const Workspace* ws = workspace_of(*x);
  if (!ws) Py_RETURN_NONE;
  at::Tensor y = empty_like(*x, {M, N}, out_dtype == NIMBLE_F32 ? at::kFloat : at::kBFloat16);
  void* stream;
  if (!current_stream(&stream)) return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = g_dense(x->data_ptr(), w->data_ptr(), b ? b->data_ptr() : nullptr, y.data_ptr(), M, N, K, (int)epilogue, (int)out_dtype,
               ws->ptr, ws->bytes, stream);
  Py_END_ALLOW_THREADS
  if (rc != NIMBLE_OK) Py_RETURN_NONE;
  return THPVariable_Wrap(std::move(y));
  END_HANDLE_TH_ERRORS
}

bool qkv_of(PyObject* const* args, const at::Tensor* (&t)[3]) {
  for (int i = 0; i < 3; ++i)
    if (!(t[i] = plain(args[i], at::kBFloat16)) || t[i]->dim() != 3) return false;
  return t[1]->size(0) == t[0]->size(0) && t[2]->size(0) == t[0]->size(0) && t[1]->size(2) == t[0]->size(2) &&
         t[2]->size(1) == t[1]->size(1);
}

// attention(q, k, v, alpha) -> (s, p, o) or None
PyObject* attention(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  const at::Tensor* t[3];
  if (n != 4 || modes_active() || !PyFloat_CheckExact(args[3]) || !qkv_of(args, t)) Py_RETURN_NONE;
  const int64_t T = t[0]->size(0), M = t[0]->size(1), N = t[1]->size(1), D = t[0]->size(2), Dv = t[2]->size(2);
  const Workspace* ws = workspace_of(*t[0]);
  if (!ws) Py_RETURN_NONE;
  at::Tensor s = empty_like(*t[0], {T, M, N}, at::kFloat), p = empty_like(*t[0], {T, M, N}, at::kBFloat16);
  at::Tensor o = empty_like(*t[0], {T, M, Dv}, at::kBFloat16);
  void* stream;
  if (!current_stream(&stream)) return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = g_attention_chain(t[0]->data_ptr(), t[1]->data_ptr(), t[2]->data_ptr(), s.data_ptr(), p.data_ptr(), o.data_ptr(), T, M, N,
                         D, Dv, (float)PyFloat_AS_DOUBLE(args[3]), ws->ptr, ws->bytes, stream);
  Py_END_ALLOW_THREADS
  if (rc != NIMBLE_OK) Py_RETURN_NONE;
  PyObject* out = PyTuple_New(3);
  if (!out) return nullptr;
  at::Tensor* results[3] = {&s, &p, &o};
  for (int i = 0; i < 3; ++i) {
    PyObject* v = THPVariable_Wrap(std::move(*results[i]));
    if (!v) {
      Py_DECREF(out);
      return nullptr;
    }
    PyTuple_SET_ITEM(out, i, v);
  }
  return out;
  END_HANDLE_TH_ERRORS
}

// fused_attention(q, k, v, alpha) -> o or None
PyObject* fused_attention(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  const at::Tensor* t[3];
  if (n != 4 || modes_active() || !PyFloat_CheckExact(args[3]) || !qkv_of(args, t)) Py_RETURN_NONE;
  const int64_t T = t[0]->size(0), L = t[0]->size(1), D = t[0]->size(2);
  if (t[1]->size(1) != L || t[2]->size(2) != D) Py_RETURN_NONE;
  at::Tensor o = empty_like(*t[0], {T, L, D}, at::kBFloat16);
  void* stream;
  if (!current_stream(&stream)) return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = g_attention(t[0]->data_ptr(), t[1]->data_ptr(), t[2]->data_ptr(), o.data_ptr(), T, L, D,
                   (float)PyFloat_AS_DOUBLE(args[3]), stream);
  Py_END_ALLOW_THREADS
  if (rc != NIMBLE_OK) Py_RETURN_NONE;
  return THPVariable_Wrap(std::move(o));
  END_HANDLE_TH_ERRORS
}

// lstm_sequence(xs, w_x, w_h, bias, h0, c0, max_polls) -> (h_seq, c_T, True) from the one-launch token loop; pre, the
// inputs' share of the gates, where the loop gave up; or None.  The loop's launch waits for whatever the host does between it
// and the projection's, and the pass ends with a wait: with these steps in Python / here (means over where the buffers
// lie) one sentence of 128 tokens at H = 512 takes 180 / 168 us, two of 20 at 256 57 / 45, one of 64 at 1024 131 / 121.
PyObject* lstm_sequence(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 7 || modes_active() || !PyLong_CheckExact(args[6])) Py_RETURN_NONE;
  const at::Tensor* t[5];
  for (int i = 0; i < 5; ++i)
    if (!(t[i] = plain(args[i], at::kBFloat16))) Py_RETURN_NONE;
  const at::Tensor &xs = *t[0], &w_x = *t[1], &w_h = *t[2], &bias = *t[3], &h0 = *t[4], *c0 = plain(args[5], at::kFloat);
  if (!c0 || xs.dim() != 3 || w_x.dim() != 2 || w_h.dim() != 2 || h0.dim() != 2 || c0->dim() != 2) Py_RETURN_NONE;
  const int64_t T = xs.size(0), B = xs.size(1), Ix = xs.size(2), H = h0.size(1);
  if (T < 1 || h0.size(0) != B || c0->size(0) != B || c0->size(1) != H || w_x.size(0) != 4 * H || w_x.size(1) != Ix ||
      w_h.size(0) != 4 * H || w_h.size(1) != H || bias.numel() != 4 * H || !g_seq_preferred(B, H))
    Py_RETURN_NONE;
  const long long max_polls = PyLong_AsLongLong(args[6]);
  if (max_polls < 0 || max_polls > UINT32_MAX) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  const Workspace* ws = workspace_of(xs);
  for (int i = 1; i < 5 && ws; ++i)
    if (t[i]->get_device() != xs.get_device()) ws = nullptr;
  if (!ws || c0->get_device() != xs.get_device()) Py_RETURN_NONE;
  at::Tensor pre = empty_like(xs, {T, B, 4 * H}, at::kFloat), h_seq = empty_like(xs, {T, B, H}, at::kBFloat16);
  at::Tensor c_out = empty_like(xs, {B, H}, at::kFloat), words = empty_like(xs, {(int64_t)g_seq_workspace_bytes(B, H)}, at::kByte);
  void* stream;
  if (!current_stream(&stream)) return nullptr;
  int rc, gave_up = 0;
  Py_BEGIN_ALLOW_THREADS
  rc = g_dense(xs.data_ptr(), w_x.data_ptr(), bias.data_ptr(), pre.data_ptr(), T * B, 4 * H, Ix, NIMBLE_EPI_BIAS, NIMBLE_F32, ws->ptr,
               ws->bytes, stream);
  if (rc == NIMBLE_OK)
    rc = g_seq_pre(pre.data_ptr(), w_h.data_ptr(), h0.data_ptr(), c0->data_ptr(), h_seq.data_ptr(), c_out.data_ptr(), T, B, H,
                   words.data_ptr(), words.nbytes(), (uint32_t)max_polls, stream);
  if (rc == NIMBLE_OK) rc = g_seq_status(words.data_ptr(), stream, &gave_up);
  Py_END_ALLOW_THREADS
  if (rc != NIMBLE_OK) Py_RETURN_NONE;
  if (gave_up) return THPVariable_Wrap(std::move(pre));
  PyObject* out = PyTuple_New(3);
  if (!out) return nullptr;
  at::Tensor* results[2] = {&h_seq, &c_out};
  for (int i = 0; i < 2; ++i) {
    PyObject* v = THPVariable_Wrap(std::move(*results[i]));
    if (!v) {
      Py_DECREF(out);
      return nullptr;
    }
    PyTuple_SET_ITEM(out, i, v);
  }
  Py_INCREF(Py_True);
  PyTuple_SET_ITEM(out, 2, Py_True);
  return out;
  END_HANDLE_TH_ERRORS
}

const at::Tensor* plain_vm_tensor(PyObject* o) {
  const at::Tensor* t = plain(o, at::kBFloat16);
  if (!t) t = plain(o, at::kFloat);
  return t && t->dim() <= 4 ? t : nullptr;
}

// A result of the interpreter: an integer, a host shape, or the part of the pool, an input or a constant that it names.
PyObject* vm_result(const nimble_vm_tensor& r, const std::vector<at::Tensor>& owners) {
  if (r.dtype == NIMBLE_I64) {
    if (r.rank == 0) return PyLong_FromLongLong(r.shape[0]);
    const int64_t n = r.shape[0];
    PyObject* list = PyList_New(n);
    for (int64_t i = 0; list && i < n; ++i) PyList_SET_ITEM(list, i, PyLong_FromLongLong(((const int64_t*)r.data)[i]));
    return list;
  }
  const at::ScalarType dtype = r.dtype == NIMBLE_F32 ? at::kFloat : at::kBFloat16;
  int64_t bytes = r.dtype == NIMBLE_F32 ? 4 : 2;
  for (int i = 0; i < r.rank; ++i) bytes *= r.shape[i];
  const char* at_ = (const char*)r.data;
  for (const at::Tensor& owner : owners) {
    const char* lo = (const char*)owner.data_ptr();
    if (lo <= at_ && at_ + bytes <= lo + owner.nbytes()) {
      at::Tensor flat = owner.dim() == 1 ? owner : owner.view(-1);
      if (flat.scalar_type() != at::kByte) flat = flat.view(at::kByte);
      at::Tensor t = flat.narrow(0, at_ - lo, bytes).view(dtype).view(at::IntArrayRef(r.shape, r.rank));
      return THPVariable_Wrap(std::move(t));
    }
  }
  PyErr_SetString(PyExc_RuntimeError, "the VM returned a tensor outside the pool, the inputs and the constants");
  return nullptr;
}

// vm_run(handle, inputs, pool, constants, max_instructions) -> list of results, a status < 0, or None
PyObject* vm_run(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  constexpr int kMaxInputs = 32, kMaxResults = 16;
  if (n != 5 || modes_active() || !PyLong_CheckExact(args[4]) || !PyList_CheckExact(args[3])) Py_RETURN_NONE;
  if (!PyTuple_CheckExact(args[1]) && !PyList_CheckExact(args[1])) Py_RETURN_NONE;
  const at::Tensor* pool = plain(args[2], at::kByte);
  const Py_ssize_t n_in = PySequence_Fast_GET_SIZE(args[1]);
  if (!pool || n_in > kMaxInputs) Py_RETURN_NONE;
  const Workspace* ws = workspace_of(*pool);
  if (!ws) Py_RETURN_NONE;
  nimble_vm_tensor in[kMaxInputs], out[kMaxResults];
  // (tensors of our own: the lists are the caller's, and another thread may change them while the lock is released)
  std::vector<at::Tensor> owners;
  owners.reserve(1 + n_in + PyList_GET_SIZE(args[3]));
  owners.push_back(*pool);
  for (Py_ssize_t i = 0; i < n_in; ++i) {
    const at::Tensor* t = plain_vm_tensor(PySequence_Fast_GET_ITEM(args[1], i));
    if (!t) Py_RETURN_NONE;
    in[i].data = t->data_ptr();
    in[i].dtype = t->scalar_type() == at::kFloat ? NIMBLE_F32 : NIMBLE_BF16;
    in[i].rank = (int32_t)t->dim();
    for (int d = 0; d < 4; ++d) in[i].shape[d] = d < t->dim() ? t->size(d) : 0;
    owners.push_back(*t);
  }
  for (Py_ssize_t i = 0; i < PyList_GET_SIZE(args[3]); ++i) {
    const at::Tensor* t = plain_vm_tensor(PyList_GET_ITEM(args[3], i));
    if (!t) Py_RETURN_NONE;
    owners.push_back(*t);
  }
  nimble_vm* vm = (nimble_vm*)PyLong_AsVoidPtr(args[0]);
  const long long max_instructions = PyLong_AsLongLong(args[4]);
  if (!vm || PyErr_Occurred()) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  void* stream;
  if (!current_stream(&stream)) return nullptr;
  int n_out = 0, rc;
  Py_BEGIN_ALLOW_THREADS
  rc = g_vm_run(vm, in, (int)n_in, pool->data_ptr(), pool->nbytes(), ws->ptr, ws->bytes, stream, max_instructions, out, kMaxResults,
                &n_out);
  Py_END_ALLOW_THREADS
  if (rc != NIMBLE_OK) return PyLong_FromLong(rc);
  PyObject* list = PyList_New(n_out);
  for (int i = 0; list && i < n_out; ++i) {
    PyObject* v = vm_result(out[i], owners);
    if (!v) {
      Py_DECREF(list);
      return nullptr;
    }
    PyList_SET_ITEM(list, i, v);
  }
  return list;
  END_HANDLE_TH_ERRORS
}

// set_workspace(device index, tensor): the default workspace of a device, as runtime.default_workspace made it
PyObject* set_workspace(PyObject*, PyObject* args) {
  HANDLE_TH_ERRORS
  int index;
  PyObject* tensor;
  if (!PyArg_ParseTuple(args, "iO", &index, &tensor)) return nullptr;
  if (index < 0 || index >= kMaxDevices || !THPVariable_Check(tensor)) Py_RETURN_NONE;
  const at::Tensor& t = THPVariable_Unpack(tensor);
  Py_INCREF(tensor);
  Workspace& w = g_workspace[index];
  Py_XDECREF(w.tensor);
  w.tensor = tensor;
  w.ptr = t.data_ptr();
  w.bytes = t.nbytes();
  Py_RETURN_NONE;
  END_HANDLE_TH_ERRORS
}

// bind(dense, attention, attention_chain, vm_run, lstm_seq_preferred, lstm_seq_workspace_bytes, lstm_seq_pre,
// lstm_seq_status, current_device, raw_stream, device index): addresses of the loaded
// library's entry points (the library that binding.py loaded), torch's two functions, and a GPU on which to look at
// what an ordinary tensor is to the dispatcher.  Before this call every other function answers None.
PyObject* bind(PyObject*, PyObject* args) {
  HANDLE_TH_ERRORS
  unsigned long long a[8];
  PyObject *dev, *stream;
  int index;
  if (!PyArg_ParseTuple(args, "KKKKKKKKOOi", &a[0], &a[1], &a[2], &a[3], &a[4], &a[5], &a[6], &a[7], &dev, &stream, &index)) return nullptr;
  const auto options = at::TensorOptions().dtype(at::kByte).device(at::Device(at::kCUDA, (c10::DeviceIndex)index));
  c10::DispatchKeySet keys[2];
  for (int inference = 0; inference < 2; ++inference) {
    c10::InferenceMode mode(inference != 0);
    keys[inference] = at::empty({0}, options).key_set();
  }
  g_dense = (decltype(g_dense))a[0];
  g_attention = (decltype(g_attention))a[1];
  g_attention_chain = (decltype(g_attention_chain))a[2];
  g_vm_run = (decltype(g_vm_run))a[3];
  g_seq_preferred = (decltype(g_seq_preferred))a[4];
  g_seq_workspace_bytes = (decltype(g_seq_workspace_bytes))a[5];
  g_seq_pre = (decltype(g_seq_pre))a[6];
  g_seq_status = (decltype(g_seq_status))a[7];
  Py_INCREF(dev);
  Py_INCREF(stream);
  g_current_device = dev;
  g_raw_stream = stream;
  g_plain = keys[0];
  g_inference = keys[1];
  Py_RETURN_NONE;
  END_HANDLE_TH_ERRORS
}

PyMethodDef kMethods[] = {
    {"dense", (PyCFunction)(void (*)(void))dense, METH_FASTCALL, nullptr},
    {"attention", (PyCFunction)(void (*)(void))attention, METH_FASTCALL, nullptr},
    {"fused_attention", (PyCFunction)(void (*)(void))fused_attention, METH_FASTCALL, nullptr},
    {"lstm_sequence", (PyCFunction)(void (*)(void))lstm_sequence, METH_FASTCALL, nullptr},
    {"vm_run", (PyCFunction)(void (*)(void))vm_run, METH_FASTCALL, nullptr},
    {"set_workspace", set_workspace, METH_VARARGS, nullptr},
    {"bind", bind, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_host_calls", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host_calls(void) { return PyModule_Create(&kModule); }
