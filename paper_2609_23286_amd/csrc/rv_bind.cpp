// rv_bind.cpp -- the argument marshalling of rv.py's per-frame calls, as a CPython module.
//
// A frame of 24 layers passes some 150 tensors to one admission call.  Checking shape, type,
// device and layout and taking the address costs about 0.7 us a tensor through Python's
// attributes (112 us for an admission call whose kernels take 40), and about 0.03 us here.
// Checks, their order and their exceptions are those of rv._ptr; tensor subclasses
// and anything that is not a tensor go to that function.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include <cstdint>
#include <exception>

#include "../../include/rv.h"

namespace {

PyObject* g_ptr_fallback = nullptr;  // rv._ptr_python(t, shape, itemsize, what)
// librv's functions, from the handle rv.py loaded it by.
decltype(&rv_mem_view) g_mem_view = nullptr;
decltype(&rv_mem_len) g_mem_len = nullptr;

// A shape as rv.py's calls state it: up to four extents.
struct Shape {
  int n = 0;
  int64_t d[4];
};

bool parse_shape(PyObject* o, Shape* s) {
  if (!PyTuple_CheckExact(o) || PyTuple_GET_SIZE(o) > 4) {
    PyErr_SetString(PyExc_TypeError, "shape: a tuple of up to four integers");
    return false;
  }
  s->n = (int)PyTuple_GET_SIZE(o);
  for (int i = 0; i < s->n; ++i) {
    s->d[i] = PyLong_AsLongLong(PyTuple_GET_ITEM(o, i));
    if (s->d[i] == -1 && PyErr_Occurred()) return false;
  }
  return true;
}

// What the checks accept without a word; anything else is rv._ptr_python's to word or pass.
bool plain_ptr(PyObject* o, const Shape& s, int itemsize, void** out) {
  if (o == Py_None) {
    *out = nullptr;
    return true;
  }
  if (!THPVariable_CheckExact(o)) return false;
  try {
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.unsafeGetTensorImpl()->is_python_dispatch() || !t.is_contiguous() ||
        (int64_t)t.element_size() != itemsize || t.dim() != s.n)
      return false;
    for (int i = 0; i < s.n; ++i)
      if (t.size(i) != s.d[i]) return false;
    *out = t.data_ptr();
    return true;
  } catch (const std::exception&) {
    return false;  // (the same access from Python raises it)
  }
}

// The device address of a tensor argument (NULL for None); false with an exception set.
bool take_ptr(PyObject* o, PyObject* shape_obj, const Shape& s, int itemsize, const char* what, Py_ssize_t index,
              void** out) {
  if (plain_ptr(o, s, itemsize, out)) return true;
  PyObject* name = index < 0 ? PyUnicode_FromString(what) : PyUnicode_FromFormat("%s[%zd]", what, index);
  if (!name) return false;
  PyObject* r = PyObject_CallFunction(g_ptr_fallback, "OOiN", o, shape_obj, itemsize, name);
  if (!r) return false;
  bool ok = true;
  if (r == Py_None) {
    *out = nullptr;
  } else {
    *out = PyLong_AsVoidPtr(r);
    ok = !(*out == nullptr && PyErr_Occurred());
  }
  Py_DECREF(r);
  return ok;
}

// ptr(tensor, shape, itemsize, what) -> address
PyObject* py_ptr(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 4) return PyErr_Format(PyExc_TypeError, "ptr takes 4 arguments (%zd given)", n);
  Shape s;
  const long itemsize = PyLong_AsLong(args[2]);
  if (itemsize == -1 && PyErr_Occurred()) return nullptr;
  const char* what = PyUnicode_AsUTF8(args[3]);
  if (!what || !parse_shape(args[1], &s)) return nullptr;
  void* p;
  if (!take_ptr(args[0], args[1], s, (int)itemsize, what, -1, &p)) return nullptr;
  return PyLong_FromVoidPtr(p);
}

// ptrs(tensors, n_layers, shape, itemsize, what) -> bytes holding n_layers addresses
PyObject* py_ptrs(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 5) return PyErr_Format(PyExc_TypeError, "ptrs takes 5 arguments (%zd given)", n);
  const Py_ssize_t layers = PyLong_AsSsize_t(args[1]);
  if (layers == -1 && PyErr_Occurred()) return nullptr;
  const long itemsize = PyLong_AsLong(args[3]);
  if (itemsize == -1 && PyErr_Occurred()) return nullptr;
  const char* what = PyUnicode_AsUTF8(args[4]);
  Shape s;
  if (!what || !parse_shape(args[2], &s)) return nullptr;
  PyObject* seq = PySequence_Fast(args[0], "expected a sequence of tensors");
  if (!seq) return nullptr;
  PyObject* out = PyBytes_FromStringAndSize(nullptr, layers * (Py_ssize_t)sizeof(void*));
  if (out) {
    void** p = reinterpret_cast<void**>(PyBytes_AS_STRING(out));
    for (Py_ssize_t i = 0; i < layers; ++i) p[i] = nullptr;  // (a shorter list: the library refuses NULLs)
    // (the size is read each time round: a subclass's accessors may run code that changes it)
    for (Py_ssize_t i = 0; i < PySequence_Fast_GET_SIZE(seq); ++i) {
      void* x = nullptr;
      PyObject* o = PySequence_Fast_GET_ITEM(seq, i);
      Py_INCREF(o);
      const bool ok = take_ptr(o, args[2], s, (int)itemsize, what, i, &x);
      Py_DECREF(o);
      if (ok && i >= layers) PyErr_SetString(PyExc_IndexError, "invalid index");
      if (!ok || i >= layers) {
        Py_CLEAR(out);
        break;
      }
      p[i] = x;
    }
  }
  Py_DECREF(seq);
  return out;
}

// mem_state(handle) -> (memK, memV, head stride, length), or the status of a failed view
PyObject* py_mem_state(PyObject*, PyObject* handle) {
  void* h = handle == Py_None ? nullptr : PyLong_AsVoidPtr(handle);
  if (!h && PyErr_Occurred()) return nullptr;
  const void *k = nullptr, *v = nullptr;
  int64_t hs = 0;
  const rv_status st = g_mem_view((rv_mem)h, &k, &v, &hs);
  if (st != RV_OK) return PyLong_FromLong((long)st);
  return Py_BuildValue("(KKLL)", (unsigned long long)(uintptr_t)k, (unsigned long long)(uintptr_t)v, (long long)hs,
                       (long long)g_mem_len((rv_mem)h));
}

// setup(rv._ptr_python, address of rv_mem_view, address of rv_mem_len)
PyObject* py_setup(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 3) return PyErr_Format(PyExc_TypeError, "setup takes 3 arguments (%zd given)", n);
  void *view = PyLong_AsVoidPtr(args[1]), *len = PyLong_AsVoidPtr(args[2]);
  if (!view || !len) return PyErr_Occurred() ? nullptr : PyErr_Format(PyExc_ValueError, "NULL function");
  g_mem_view = reinterpret_cast<decltype(g_mem_view)>(view);
  g_mem_len = reinterpret_cast<decltype(g_mem_len)>(len);
  Py_INCREF(args[0]);
  Py_XDECREF(g_ptr_fallback);
  g_ptr_fallback = args[0];
  Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    {"ptr", (PyCFunction)(void (*)(void))py_ptr, METH_FASTCALL, nullptr},
    {"ptrs", (PyCFunction)(void (*)(void))py_ptrs, METH_FASTCALL, nullptr},
    {"mem_state", py_mem_state, METH_O, nullptr},
    {"setup", (PyCFunction)(void (*)(void))py_setup, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_rv_bind", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: the torch and Python whose headers this was compiled with.  It reads their
// objects directly, so rv.py loads it with the same ones only.
PyMODINIT_FUNC PyInit__rv_bind(void) {
  PyObject* m = PyModule_Create(&kModule);
  if (m && PyModule_AddObject(m, "built_for", Py_BuildValue("(sii)", TORCH_VERSION, PY_MAJOR_VERSION, PY_MINOR_VERSION)))
    Py_CLEAR(m);
  return m;
}
