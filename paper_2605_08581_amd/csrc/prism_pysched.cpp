// Python entry of the control plane's per-request calls.  A wave makes a dozen
// or more of each; through ctypes the marshalling of token and anchor arrays
// cost several times what the scheduler and the tree do themselves (640 requests
// of a serving trace: 23.6 ms, with this and the flat arrays in prism_sched.cpp
// 9.6 ms).
// Each function takes the handle first and returns the C status (admit: see
// there); arguments that are neither integers nor int32 buffers raise TypeError
// and the Python side then converts them and calls again.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <vector>

#include "prism.h"
#include "prism_sched.h"

namespace {

struct Api {
  decltype(&prism_qas_submit) submit = nullptr;
  decltype(&prism_qas_complete) complete = nullptr;
  decltype(&prism_dart_set_time) set_time = nullptr;
  decltype(&prism_dart_admit) admit = nullptr;
  decltype(&prism_dart_commit) commit = nullptr;
  decltype(&prism_dart_release) release = nullptr;
} g_api;

bool integer(PyObject *o, long long *v) {
  if (!PyIndex_Check(o)) {
    PyErr_SetString(PyExc_TypeError, "an integer is needed");
    return false;
  }
  PyObject *n = PyNumber_Index(o);
  if (!n) return false;
  *v = PyLong_AsLongLong(n);
  Py_DECREF(n);
  return !(*v == -1 && PyErr_Occurred());
}
// A request's id: any integer, of which 64 bits count (ids may be unsigned hashes).
bool request_of(PyObject *o, long long *v) {
  if (!PyIndex_Check(o)) {
    PyErr_SetString(PyExc_TypeError, "an integer is needed");
    return false;
  }
  PyObject *n = PyNumber_Index(o);
  if (!n) return false;
  *v = (long long)PyLong_AsUnsignedLongLongMask(n);
  Py_DECREF(n);
  return true;
}
bool int32_of(PyObject *o, int32_t *v) {
  long long x;
  if (!integer(o, &x)) return false;
  if (x < INT32_MIN || x > INT32_MAX) {
    PyErr_SetString(PyExc_TypeError, "out of the range of int32");
    return false;
  }
  *v = (int32_t)x;
  return true;
}
void *handle(PyObject *o) { return PyLong_AsVoidPtr(o); }

// An int32 array: a contiguous buffer of that type as it lies, or a list or
// tuple of integers, copied.
struct Int32s {
  Py_buffer view{};
  bool has_view = false;
  std::vector<int32_t> copy;
  int32_t *data = nullptr;
  Py_ssize_t n = 0;
  ~Int32s() { if (has_view) PyBuffer_Release(&view); }
  bool take(PyObject *o, bool writable = false) {
    if (PyObject_CheckBuffer(o)) {
      if (PyObject_GetBuffer(o, &view, PyBUF_C_CONTIGUOUS | PyBUF_FORMAT | (writable ? PyBUF_WRITABLE : 0)) != 0) {
        PyErr_Clear();
      } else {
        has_view = true;
        const char *f = view.format;
        if (f && (f[0] == '<' || f[0] == '=' || f[0] == '@')) ++f;
        if (view.itemsize == 4 && f && (f[0] == 'i' || f[0] == 'l') && f[1] == 0) {
          data = (int32_t *)view.buf;
          n = view.len / 4;
          return true;
        }
      }
    } else if (!writable && (PyList_Check(o) || PyTuple_Check(o))) {
      n = PySequence_Fast_GET_SIZE(o);
      copy.resize((size_t)n);
      for (Py_ssize_t i = 0; i < n; ++i)
        if (!int32_of(PySequence_Fast_GET_ITEM(o, i), &copy[(size_t)i])) return false;
      data = copy.data();
      return true;
    }
    PyErr_SetString(PyExc_TypeError, "an int32 array is needed");
    return false;
  }
};

// Admissions, which may evict, and commits run without the interpreter's lock:
// other Python threads go on meanwhile.  The other calls take about as long as
// giving the lock up and taking it back (640 requests of a serving trace: 2 %).
struct Unlocked {
  PyThreadState *state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};
template <class F, class... Args>
int call_unlocked(F *entry, Args... args) {
  Unlocked unlocked;
  return entry(args...);
}

PyObject *wrong_count(const char *what) {
  PyErr_Format(PyExc_TypeError, "%s: wrong number of arguments", what);
  return nullptr;
}

PyObject *bind_api(PyObject *, PyObject *args) {
  unsigned long long a[6];
  if (!PyArg_ParseTuple(args, "KKKKKK", a, a + 1, a + 2, a + 3, a + 4, a + 5)) return nullptr;
  g_api.submit = (decltype(g_api.submit))(uintptr_t)a[0];
  g_api.complete = (decltype(g_api.complete))(uintptr_t)a[1];
  g_api.set_time = (decltype(g_api.set_time))(uintptr_t)a[2];
  g_api.admit = (decltype(g_api.admit))(uintptr_t)a[3];
  g_api.commit = (decltype(g_api.commit))(uintptr_t)a[4];
  g_api.release = (decltype(g_api.release))(uintptr_t)a[5];
  Py_RETURN_NONE;
}

// submit(qas, request, arrival, skeleton, segment_tokens, system_tokens, suffix_tokens): all segments reorderable
PyObject *submit(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 7) return wrong_count("submit");
  long long request;
  int32_t system, suffix;
  Int32s skel, tok;
  const double arrival = PyFloat_AsDouble(a[2]);
  if (arrival == -1.0 && PyErr_Occurred()) return nullptr;
  if (!request_of(a[1], &request) || !skel.take(a[3]) || !tok.take(a[4]) || !int32_of(a[5], &system) ||
      !int32_of(a[6], &suffix))
    return nullptr;
  if (skel.n != tok.n) {
    PyErr_SetString(PyExc_ValueError, "skeleton and segment_tokens must have the same length");
    return nullptr;
  }
  return PyLong_FromLong(g_api.submit((prism_qas_t *)handle(a[0]), request, arrival, skel.data, tok.data, nullptr,
                                      (int32_t)skel.n, system, suffix));
}

// complete(qas, request) / release(dart, request)
PyObject *complete(PyObject *, PyObject *const *a, Py_ssize_t n) {
  long long request;
  if (n != 2) return wrong_count("complete");
  if (!request_of(a[1], &request)) return nullptr;
  return PyLong_FromLong(g_api.complete((prism_qas_t *)handle(a[0]), request));
}
PyObject *release(PyObject *, PyObject *const *a, Py_ssize_t n) {
  long long request;
  if (n != 2) return wrong_count("release");
  if (!request_of(a[1], &request)) return nullptr;
  return PyLong_FromLong(g_api.release((prism_dart_t *)handle(a[0]), request));
}

PyObject *set_time(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 2) return wrong_count("set_time");
  const double now = PyFloat_AsDouble(a[1]);
  if (now == -1.0 && PyErr_Occurred()) return nullptr;
  return PyLong_FromLong(g_api.set_time((prism_dart_t *)handle(a[0]), now));
}

// admit(dart, request, tokens, anchors, reserve_tokens, row): the hit length, or a
// negative status; row is filled (entries beyond the request's pages with -1)
PyObject *admit(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 6) return wrong_count("admit");
  long long request;
  int32_t reserve, hit = 0;
  Int32s tok, row;
  if (!request_of(a[1], &request) || !tok.take(a[2]) || !int32_of(a[4], &reserve) || !row.take(a[5], true)) return nullptr;
  if (!PyList_Check(a[3]) && !PyTuple_Check(a[3])) {
    PyErr_SetString(PyExc_TypeError, "anchors: a list or tuple is needed");
    return nullptr;
  }
  const Py_ssize_t m = PySequence_Fast_GET_SIZE(a[3]);
  std::vector<prism_dart_anchor_t> anchors((size_t)m);
  for (Py_ssize_t i = 0; i < m; ++i) {
    PyObject *t = PySequence_Fast_GET_ITEM(a[3], i);
    if (!PyTuple_Check(t) || PyTuple_GET_SIZE(t) != 3) {
      PyErr_SetString(PyExc_TypeError, "anchors: (end_offset, kind, segment) tuples are needed");
      return nullptr;
    }
    prism_dart_anchor_t &x = anchors[(size_t)i];
    if (!int32_of(PyTuple_GET_ITEM(t, 0), &x.end_offset) || !int32_of(PyTuple_GET_ITEM(t, 1), &x.kind) ||
        !int32_of(PyTuple_GET_ITEM(t, 2), &x.segment))
      return nullptr;
  }
  for (Py_ssize_t i = 0; i < row.n; ++i) row.data[i] = -1;
  const int rc = call_unlocked(g_api.admit, (prism_dart_t *)handle(a[0]), request, tok.data, (int32_t)tok.n,
                               anchors.data(), (int32_t)m, reserve, row.data, (int32_t)row.n, &hit);
  return PyLong_FromLong(rc < 0 ? rc : hit);
}

PyObject *commit(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 3) return wrong_count("commit");
  long long request;
  Int32s row;
  if (!request_of(a[1], &request) || !row.take(a[2], true)) return nullptr;
  return PyLong_FromLong(
      call_unlocked(g_api.commit, (prism_dart_t *)handle(a[0]), request, row.data, (int32_t)row.n));
}

#define FAST(f) (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr
PyMethodDef methods[] = {{"bind_api", bind_api, METH_VARARGS, nullptr},
                         {"submit", FAST(submit)},
                         {"complete", FAST(complete)},
                         {"set_time", FAST(set_time)},
                         {"admit", FAST(admit)},
                         {"commit", FAST(commit)},
                         {"release", FAST(release)},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_prism_sched", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__prism_sched(void) { return PyModule_Create(&module); }
