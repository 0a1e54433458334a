// Python entry of the layer calls: checks the tensors and forwards bare
// pointers and torch's current stream to the C ABI.
//
// A layer call on a small wave takes the GPU about ten microseconds, so the
// host side of the call must stay below that.  Doing these same checks from
// Python (device, dtype, contiguity and element count of eight tensors, a
// ctypes call with eleven arguments) took 17 us per call; here it takes well
// under one, and what remains is the kernel launches themselves.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <exception>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "prism.h"

namespace {

// Entry points of the libprism.so that the Python side has loaded.
struct Api {
  decltype(&prism_kv_append) append = nullptr;
  decltype(&prism_prefix_attention) attention = nullptr;
  decltype(&prism_prefix_prefill) prefill = nullptr;
  decltype(&prism_prefix_prefill_static) prefill_static = nullptr;
} g_api;

// What a plan's calls need: the handle and the element counts of its tensors.
struct Call {
  prism_plan_t *plan;
  int64_t q, kv, pool, table, workspace;
};
constexpr const char *kCallName = "prism.call";

// Status for "the binding's own checks refused a tensor": the caller then runs
// the same checks in Python, which name the tensor and raise.
constexpr long kRefused = 1;

bool fits(PyObject *o, c10::ScalarType type, int64_t numel, void **ptr) {
  *ptr = nullptr;
  if (o == Py_None) return numel == 0;
  if (!THPVariable_Check(o)) return false;
  const at::Tensor &t = THPVariable_Unpack(o);
  if (!t.is_cuda() || !t.is_contiguous() || t.scalar_type() != type || t.numel() < numel) return false;
  *ptr = t.data_ptr();
  return true;
}

Call *call_of(PyObject *o) { return (Call *)PyCapsule_GetPointer(o, kCallName); }

// Workspace as the library wants it: pointer and bytes.  Returns whether the
// other tensors are to be checked too (a workspace that is missing or too small
// is the library's own error).
bool workspace_of(PyObject *o, const Call *c, void **ptr, size_t *bytes, bool *ok) {
  *ptr = nullptr;
  *bytes = 0;
  *ok = true;
  if (o == Py_None) return false;
  if (!THPVariable_Check(o)) {
    *ok = false;
    return false;
  }
  const at::Tensor &t = THPVariable_Unpack(o);
  *ptr = t.data_ptr();
  *bytes = (size_t)t.numel() * t.element_size();
  if (*bytes < (size_t)c->workspace) return false;   // in bytes, as the library compares them
  *ok = t.is_cuda() && t.is_contiguous() && t.scalar_type() == at::kByte;
  return true;
}

bool raw_pointer(PyObject *o, void **ptr) {       // unchecked, for calls that the library will refuse
  *ptr = nullptr;
  if (o == Py_None) return true;
  if (!THPVariable_Check(o)) return false;
  *ptr = THPVariable_Unpack(o).data_ptr();
  return true;
}

void *stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }

// The entry points run without the interpreter's lock: a launch waits when the
// stream's queue is full, and other Python threads go on meanwhile.
template <class F, class... Args>
PyObject *call_unlocked(F *entry, Args... args) {
  struct Unlocked {
    PyThreadState *state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
  };
  long rc;
  {
    Unlocked unlocked;
    rc = entry(args...);
  }
  return PyLong_FromLong(rc);
}

PyObject *wrong_count(const char *what) {
  PyErr_Format(PyExc_TypeError, "%s: wrong number of arguments", what);
  return nullptr;
}

PyObject *bind_api(PyObject *, PyObject *args) {
  unsigned long long a, b, c, d;
  if (!PyArg_ParseTuple(args, "KKKK", &a, &b, &c, &d)) return nullptr;
  g_api.append = (decltype(g_api.append))(uintptr_t)a;
  g_api.attention = (decltype(g_api.attention))(uintptr_t)b;
  g_api.prefill = (decltype(g_api.prefill))(uintptr_t)c;
  g_api.prefill_static = (decltype(g_api.prefill_static))(uintptr_t)d;
  Py_RETURN_NONE;
}

PyObject *make_call(PyObject *, PyObject *args) {
  unsigned long long plan;
  long long q, kv, pool, table, ws;
  if (!PyArg_ParseTuple(args, "KLLLLL", &plan, &q, &kv, &pool, &table, &ws)) return nullptr;
  Call *c = new Call{(prism_plan_t *)(uintptr_t)plan, q, kv, pool, table, ws};
  return PyCapsule_New(c, kCallName, [](PyObject *o) { delete (Call *)PyCapsule_GetPointer(o, kCallName); });
}

PyObject *close_call(PyObject *, PyObject *o) {   // the plan is being destroyed: later calls see no plan
  Call *c = call_of(o);
  if (!c) return nullptr;
  c->plan = nullptr;
  Py_RETURN_NONE;
}

// kv_append(call, k_suffix, v_suffix, k_pool, v_pool, block_table)
PyObject *kv_append(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 6) return wrong_count("kv_append");
  const Call *c = call_of(a[0]);
  if (!c) return nullptr;
  void *k, *v, *kp, *vp, *bt;
  if (!fits(a[1], at::kBFloat16, c->kv, &k) || !fits(a[2], at::kBFloat16, c->kv, &v) ||
      !fits(a[3], at::kBFloat16, c->pool, &kp) || !fits(a[4], at::kBFloat16, c->pool, &vp) ||
      !fits(a[5], at::kInt, c->table, &bt))
    return PyLong_FromLong(kRefused);
  return call_unlocked(g_api.append, c->plan, k, v, kp, vp, (const int32_t *)bt, stream());
}

// prefix_attention(call, q, k_pool, v_pool, block_table, out, workspace)
PyObject *prefix_attention(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 7) return wrong_count("prefix_attention");
  const Call *c = call_of(a[0]);
  if (!c) return nullptr;
  void *q, *kp, *vp, *bt, *out, *ws;
  size_t bytes;
  bool ok;
  if (workspace_of(a[6], c, &ws, &bytes, &ok)) {
    ok = ok && fits(a[1], at::kBFloat16, c->q, &q) && fits(a[2], at::kBFloat16, c->pool, &kp) &&
         fits(a[3], at::kBFloat16, c->pool, &vp) && fits(a[4], at::kInt, c->table, &bt) &&
         fits(a[5], at::kBFloat16, c->q, &out);
  } else {
    ok = ok && raw_pointer(a[1], &q) && raw_pointer(a[2], &kp) && raw_pointer(a[3], &vp) && raw_pointer(a[4], &bt) &&
         raw_pointer(a[5], &out);
  }
  if (!ok) return PyLong_FromLong(kRefused);
  return call_unlocked(g_api.attention, c->plan, q, kp, vp, (const int32_t *)bt, out, ws, bytes, stream());
}

// prefix_prefill(call, q, k_suffix, v_suffix, k_pool, v_pool, block_table, out, workspace)
PyObject *prefix_prefill(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 9) return wrong_count("prefix_prefill");
  const Call *c = call_of(a[0]);
  if (!c) return nullptr;
  void *q, *k, *v, *kp, *vp, *bt, *out, *ws;
  size_t bytes;
  bool ok;
  if (workspace_of(a[8], c, &ws, &bytes, &ok)) {
    ok = ok && fits(a[1], at::kBFloat16, c->q, &q) && fits(a[2], at::kBFloat16, c->kv, &k) &&
         fits(a[3], at::kBFloat16, c->kv, &v) && fits(a[4], at::kBFloat16, c->pool, &kp) &&
         fits(a[5], at::kBFloat16, c->pool, &vp) && fits(a[6], at::kInt, c->table, &bt) &&
         fits(a[7], at::kBFloat16, c->q, &out);
  } else {
    ok = ok && raw_pointer(a[1], &q) && raw_pointer(a[2], &k) && raw_pointer(a[3], &v) && raw_pointer(a[4], &kp) &&
         raw_pointer(a[5], &vp) && raw_pointer(a[6], &bt) && raw_pointer(a[7], &out);
  }
  if (!ok) return PyLong_FromLong(kRefused);
  return call_unlocked(g_api.prefill, c->plan, q, k, v, kp, vp, (const int32_t *)bt, out, ws, bytes, stream());
}

// prefix_prefill_static(call, q, k_suffix, v_suffix, k_pool, v_pool, block_table, out)
PyObject *prefix_prefill_static(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 8) return wrong_count("prefix_prefill_static");
  const Call *c = call_of(a[0]);
  if (!c) return nullptr;
  void *q, *k, *v, *kp, *vp, *bt, *out;
  if (!fits(a[1], at::kBFloat16, c->q, &q) || !fits(a[2], at::kBFloat16, c->kv, &k) ||
      !fits(a[3], at::kBFloat16, c->kv, &v) || !fits(a[4], at::kBFloat16, c->pool, &kp) ||
      !fits(a[5], at::kBFloat16, c->pool, &vp) || !fits(a[6], at::kInt, c->table, &bt) ||
      !fits(a[7], at::kBFloat16, c->q, &out))
    return PyLong_FromLong(kRefused);
  return call_unlocked(g_api.prefill_static, c->plan, q, k, v, kp, vp, (const int32_t *)bt, out, stream());
}

// A tensor without storage of its own, or a process without a device, makes
// torch's accessors throw; that must not leave through the interpreter's C frames.
template <PyObject *(*F)(PyObject *, PyObject *const *, Py_ssize_t)>
PyObject *guarded(PyObject *self, PyObject *const *a, Py_ssize_t n) {
  try {
    return F(self, a, n);
  } catch (const std::exception &e) {
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, e.what());
  }
  return nullptr;
}

#define LAYER_CALL(f) (PyCFunction)(void (*)(void))guarded<f>, METH_FASTCALL, nullptr
PyMethodDef methods[] = {
    {"bind_api", bind_api, METH_VARARGS, nullptr},
    {"make_call", make_call, METH_VARARGS, nullptr},
    {"close_call", close_call, METH_O, nullptr},
    {"kv_append", LAYER_CALL(kv_append)},
    {"prefix_attention", LAYER_CALL(prefix_attention)},
    {"prefix_prefill", LAYER_CALL(prefix_prefill)},
    {"prefix_prefill_static", LAYER_CALL(prefix_prefill_static)},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_prism_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__prism_torch(void) { return PyModule_Create(&module); }
