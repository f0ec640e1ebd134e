// The calls of binding.py that a program makes at every layer, for the usual arguments, as a CPython extension: tensors of
// torch's own class, contiguous, of the layout's type and shape, on the current device, the result allocated here, the current
// stream.  Anything else returns None before the library is called, and binding.py goes through it step by step and reports what is
// wrong; so this file checks, but explains nothing.  Once the library has been called, the outcome stands: a status other
// than zero becomes binding.py's exception here, because a second call could succeed where the first one's error is consumed, or enqueue work twice.
//
// What it is for: small calls are bound by the host.  A call of binding.py through ctypes takes about 6 us, of which the launch is 2;
// one from here 4 (a step of 256 tokens, four permutations and an attention call, 29.3 / 22.6 us).
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>

namespace {

using Permute = int (*)(const void*, void*, void*, int32_t, void*);
using Attention = int (*)(const void*, const void*, const void*, void*, void*, void*);
using WithWorkspace = int (*)(const void*, const void*, const void*, void*, void*, int32_t, void*, int64_t, void*);
using Mass = int (*)(const void*, const void*, void*, float*, void*);

struct Library {
  Permute permute;
  Attention attention[4];  // forward, natural order, dense, static: the first three numbered as ca_call is
  WithWorkspace with_workspace;
  Mass mass;
  PyObject *device, *stream, *capturing;  // torch._C: current device, handle of its current stream, is that stream being captured
  PyObject* check;                        // of binding.py: raises for a status other than zero
} lib;

struct Calls {
  PyObject_HEAD
  void* layout;
  int64_t batch, heads, tokens[2], head_dim, tiles;  // tokens: natural order, tile order
  at::ScalarType type;
};

// The current device and its current stream; false with a Python error set.
bool current(int64_t& device, void*& stream) {
  PyObject* d = PyObject_CallNoArgs(lib.device);
  if (!d) return false;
  device = PyLong_AsLongLong(d);
  PyObject* s = PyObject_CallOneArg(lib.stream, d);
  Py_DECREF(d);
  if (!s) return false;
  stream = PyLong_AsVoidPtr(s);
  Py_DECREF(s);
  return !PyErr_Occurred();
}

// The tensor behind an argument, or null if it is not an ordinary one of these tokens.
const at::Tensor* usual(const Calls* c, PyObject* arg, bool padded, int64_t device) {
  if (!THPVariable_CheckExact(arg)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(arg);
  if (!t.defined() || !t.has_storage() || t.layout() != at::kStrided || !t.is_cuda() || t.get_device() != device || t.scalar_type() != c->type) return nullptr;
  if (t.dim() != 4 || !t.is_contiguous() || t.is_conj() || t.is_neg()) return nullptr;
  const auto s = t.sizes();
  return s[0] == c->batch && s[1] == c->heads && s[2] == c->tokens[padded] && s[3] == c->head_dim ? &t : nullptr;
}

bool modes() { return at::impl::torch_function_mode_enabled() || c10::impl::dispatch_mode_enabled(); }

// The outcome of a call; None where it has not come to `made`.
template <class Call>
PyObject* guarded(Call&& call) {
  PyObject* result = nullptr;
  bool made = false;
  try {
    result = call(made);
  } catch (const std::exception& e) {
    if (made) PyErr_SetString(PyExc_RuntimeError, e.what());
  } catch (...) {
    if (made) PyErr_SetString(PyExc_RuntimeError, "unknown exception");
  }
  if (result || made) return result;
  PyErr_Clear();
  Py_RETURN_NONE;
}

// Makes the call; false with a Python error set if it fails.
template <class Launch>
bool launched(bool& made, Launch&& launch) {
  int status = -1;
  made = true;
  Py_BEGIN_ALLOW_THREADS  // as ctypes does
  status = launch();
  Py_END_ALLOW_THREADS
  if (status == 0) return true;
  PyObject* raised = PyObject_CallFunction(lib.check, "i", status);
  if (raised) PyErr_Format(PyExc_RuntimeError, "compact_attn status %d", status);
  Py_XDECREF(raised);
  return false;
}

// permute(src, inverse)
PyObject* calls_permute(PyObject* self, PyObject* const* args, Py_ssize_t n) {
  return guarded([&](bool& made) -> PyObject* {
    const Calls* c = reinterpret_cast<Calls*>(self);
    int64_t device;
    void* stream;
    if (n != 2 || modes() || !current(device, stream)) return nullptr;
    const int inverse = PyObject_IsTrue(args[1]);
    const at::Tensor* src = inverse < 0 ? nullptr : usual(c, args[0], inverse != 0, device);
    if (!src) return nullptr;
    at::Tensor out = at::empty({c->batch, c->heads, c->tokens[!inverse], c->head_dim}, src->options());
    const void* from = src->const_data_ptr();
    void* to = out.mutable_data_ptr();
    if (!launched(made, [&] { return lib.permute(from, to, c->layout, inverse, stream); })) return nullptr;
    return THPVariable_Wrap(std::move(out));
  });
}

// attention(call, q, k, v, workspace bytes): call 0 to 3 as in Library; NotImplemented if there is no memory for the workspace
PyObject* calls_attention(PyObject* self, PyObject* const* args, Py_ssize_t n) {
  return guarded([&](bool& made) -> PyObject* {
    const Calls* c = reinterpret_cast<Calls*>(self);
    int64_t device;
    void* stream;
    if (n != 5 || modes() || !current(device, stream)) return nullptr;
    const long call = PyLong_AsLong(args[0]);
    const long long need = PyLong_AsLongLong(args[4]);
    if (call < 0 || call > 3 || need < 0 || (call == 3 && need > 0) || PyErr_Occurred()) return nullptr;
    const at::Tensor *q = usual(c, args[1], call != 1, device), *k = usual(c, args[2], call != 1, device), *v = usual(c, args[3], call != 1, device);
    if (!q || !k || !v) return nullptr;
    if (need > 0) {  // memory of a capture that torch does not run would not be ours: left to binding.py
      PyObject* captured = PyObject_CallNoArgs(lib.capturing);
      const bool plain = captured == Py_False;
      Py_XDECREF(captured);
      if (!plain) return nullptr;
    }
    at::Tensor out = at::empty(q->sizes(), q->options()), workspace;
    if (need > 0) {
      try {
        workspace = at::empty({(int64_t)(need / (long long)q->element_size())}, q->options());
      } catch (const c10::OutOfMemoryError&) {
        Py_RETURN_NOTIMPLEMENTED;
      }
    }
    const void *qp = q->const_data_ptr(), *kp = k->const_data_ptr(), *vp = v->const_data_ptr();
    void *op = out.mutable_data_ptr(), *wp = need > 0 ? workspace.mutable_data_ptr() : nullptr;
    if (!launched(made, [&] {
          return need > 0 ? lib.with_workspace(qp, kp, vp, c->layout, op, (int32_t)call, wp, need, stream) : lib.attention[call](qp, kp, vp, c->layout, op, stream);
        }))
      return nullptr;
    return THPVariable_Wrap(std::move(out));
  });
}

// mass(q, k)
PyObject* calls_mass(PyObject* self, PyObject* const* args, Py_ssize_t n) {
  return guarded([&](bool& made) -> PyObject* {
    const Calls* c = reinterpret_cast<Calls*>(self);
    int64_t device;
    void* stream;
    if (n != 2 || modes() || !current(device, stream)) return nullptr;
    const at::Tensor *q = usual(c, args[0], true, device), *k = usual(c, args[1], true, device);
    if (!q || !k) return nullptr;
    at::Tensor out = at::empty({c->batch, c->heads, c->tiles, c->tiles}, q->options().dtype(at::kFloat));
    const void *qp = q->const_data_ptr(), *kp = k->const_data_ptr();
    float* op = static_cast<float*>(out.mutable_data_ptr());
    if (!launched(made, [&] { return lib.mass(qp, kp, c->layout, op, stream); })) return nullptr;
    return THPVariable_Wrap(std::move(out));
  });
}

PyMethodDef calls_methods[] = {
    {"permute", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(calls_permute)), METH_FASTCALL, nullptr},
    {"attention", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(calls_attention)), METH_FASTCALL, nullptr},
    {"mass", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(calls_mass)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyTypeObject calls_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

// calls(layout handle, batch, heads, tokens, padded tokens, head dim, tiles, is bf16)
PyObject* make_calls(PyObject*, PyObject* args) {
  unsigned long long layout;
  long long v[6];
  int bf16;
  if (!PyArg_ParseTuple(args, "KLLLLLLp", &layout, &v[0], &v[1], &v[2], &v[3], &v[4], &v[5], &bf16)) return nullptr;
  Calls* c = PyObject_New(Calls, &calls_type);
  if (!c) return nullptr;
  c->layout = reinterpret_cast<void*>(layout);
  c->batch = v[0];
  c->heads = v[1];
  c->tokens[0] = v[2];
  c->tokens[1] = v[3];
  c->head_dim = v[4];
  c->tiles = v[5];
  c->type = bf16 ? at::kBFloat16 : at::kFloat;
  return reinterpret_cast<PyObject*>(c);
}

// bind(addresses of permute, forward, natural, dense, static, with_workspace, mass; torch's device, stream and capture functions; check)
PyObject* bind(PyObject*, PyObject* args) {
  unsigned long long f[7];
  PyObject *device, *stream, *capturing, *check;
  if (!PyArg_ParseTuple(args, "KKKKKKKOOOO", &f[0], &f[1], &f[2], &f[3], &f[4], &f[5], &f[6], &device, &stream, &capturing, &check)) return nullptr;
  lib.permute = reinterpret_cast<Permute>(f[0]);
  for (int i = 0; i < 4; ++i) lib.attention[i] = reinterpret_cast<Attention>(f[1 + i]);
  lib.with_workspace = reinterpret_cast<WithWorkspace>(f[5]);
  lib.mass = reinterpret_cast<Mass>(f[6]);
  Py_INCREF(device);
  Py_INCREF(stream);
  Py_INCREF(capturing);
  Py_INCREF(check);
  lib.device = device;
  lib.stream = stream;
  lib.capturing = capturing;
  lib.check = check;
  Py_RETURN_NONE;
}

PyMethodDef module_methods[] = {{"bind", bind, METH_VARARGS, nullptr}, {"calls", make_calls, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, module_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() {
  calls_type.tp_name = "_calls.Calls";
  calls_type.tp_basicsize = sizeof(Calls);
  calls_type.tp_flags = Py_TPFLAGS_DEFAULT;
  calls_type.tp_methods = calls_methods;
  if (PyType_Ready(&calls_type) < 0) return nullptr;
  PyObject* m = PyModule_Create(&module);
  if (m && PyModule_AddStringConstant(m, "torch_version", CALLS_TORCH) < 0) Py_CLEAR(m);
  return m;
}
