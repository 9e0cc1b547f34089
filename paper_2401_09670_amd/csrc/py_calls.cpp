// The entry points of include/ds.h as functions of a CPython module: every argument turned into the C type that the
// declaration has at its place, the GIL released during the call, the status returned.
//
// Why not ctypes for these: a small model's step is a handful of launches at 3 us each, and the host was what bounded it.
// The arguments of a decode step, tensors to pointers included, take 1.0 us here and 3.0 with ctypes; together with the
// stream asked for as a number, a request of a small model (2 prompts of 32 tokens) went from 190 to 171 us, and into a
// loop that the GPU bounds (161 us, as much as its graph).  By address, so that the module needs no library at link time
// and serves whichever build of it the process has loaded.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>
#include <cstring>
#include <tuple>
#include <type_traits>
#include <utility>

#include "../../include/ds.h"

namespace {

PyObject *s_data_ptr, *s_nbytes, *s_value;  // interned names

// The arguments beyond a call's plain conversion: the type of the weights struct, and the buffers it has exported.
struct Frame {
  PyObject* weights_type;
  Py_buffer view{};
  ~Frame() {
    if (view.obj) PyBuffer_Release(&view);
  }
};

// A whole number, or a ctypes.c_int; the low 32 bits, as ctypes passes it.
bool convert(Frame&, PyObject* o, int32_t* out) {
  if (PyLong_Check(o)) {
    *out = (int32_t)PyLong_AsUnsignedLongMask(o);
    return true;
  }
  const bool c_int = !strcmp(Py_TYPE(o)->tp_name, "c_int");
  PyObject* v = c_int ? PyObject_GetAttr(o, s_value) : PyNumber_Index(o);
  if (!v) return false;
  *out = (int32_t)PyLong_AsUnsignedLongMask(v);
  Py_DECREF(v);
  return true;
}

// The bytes of a tensor (None: 0).
bool convert(Frame&, PyObject* o, size_t* out) {
  *out = 0;
  if (o == Py_None) return true;
  PyObject* v = PyObject_GetAttr(o, s_nbytes);
  if (!v) return false;
  *out = PyLong_AsSize_t(v);
  Py_DECREF(v);
  return !PyErr_Occurred();
}

bool convert(Frame& f, PyObject* o, const ds_layer_weights** out) {
  const int is = PyObject_IsInstance(o, f.weights_type);
  if (is < 0) return false;
  if (!is) {
    PyErr_Format(PyExc_TypeError, "LayerWeights, not %R", (PyObject*)Py_TYPE(o));
    return false;
  }
  if (PyObject_GetBuffer(o, &f.view, PyBUF_SIMPLE) != 0) return false;
  *out = (const ds_layer_weights*)f.view.buf;
  return true;
}

// An address: the context's and the stream's (None: NULL).
bool address(PyObject* o, void** out) {
  *out = o == Py_None ? nullptr : PyLong_AsVoidPtr(o);
  return !(*out == nullptr && PyErr_Occurred());
}
bool convert(Frame&, PyObject* o, ds_ctx** out) { return address(o, (void**)out); }

// A tensor's memory (None: NULL).
template <class T>
bool convert(Frame&, PyObject* o, T** out) {
  *out = nullptr;
  if (o == Py_None) return true;
  PyObject* v = PyObject_CallMethodNoArgs(o, s_data_ptr);
  if (!v) return false;
  *out = (T*)PyLong_AsVoidPtr(v);
  Py_DECREF(v);
  return !(*out == nullptr && PyErr_Occurred());
}

template <class F>
struct Entry;
template <class... A>
struct Entry<ds_status(A...)> {
  template <size_t... I>
  static PyObject* run(PyObject* self, PyObject* const* args, std::index_sequence<I...>) {
    constexpr size_t last = sizeof...(A) - 1;  // the stream
    Frame f{PyTuple_GET_ITEM(self, 1)};
    auto fn = (ds_status(*)(A...))PyLong_AsVoidPtr(PyTuple_GET_ITEM(self, 0));
    std::tuple<A...> a;
    auto one = [&](auto i) {
      constexpr size_t k = decltype(i)::value;
      if constexpr (k == last) return address(args[k], &std::get<k>(a));
      else return convert(f, args[k], &std::get<k>(a));
    };
    if (!(one(std::integral_constant<size_t, I>{}) && ...)) return nullptr;
    ds_status st;
    Py_BEGIN_ALLOW_THREADS
    st = fn(std::get<I>(a)...);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
  }
  static PyObject* call(PyObject* self, PyObject* const* args, Py_ssize_t n) {
    if (n != (Py_ssize_t)sizeof...(A)) {
      PyErr_Format(PyExc_TypeError, "%zd arguments, not %zd", (Py_ssize_t)sizeof...(A), n);
      return nullptr;
    }
    return run(self, args, std::index_sequence_for<A...>{});
  }
};

#define DS_ENTRY(name) \
  { #name, (PyCFunction)(void (*)(void))Entry<decltype(name)>::call, METH_FASTCALL, nullptr }
PyMethodDef entries[] = {DS_ENTRY(ds_prefill),          DS_ENTRY(ds_kv_migrate),        DS_ENTRY(ds_decode_step),
                         DS_ENTRY(ds_decode_step_static), DS_ENTRY(ds_layernorm),      DS_ENTRY(ds_linear),
                         DS_ENTRY(ds_prefill_attention), DS_ENTRY(ds_decode_attention), DS_ENTRY(ds_embed),
                         DS_ENTRY(ds_next_token)};

// bind(name, address, LayerWeights) -> the entry point of that name whose code lies at `address`
PyObject* bind(PyObject*, PyObject* args) {
  const char* name;
  PyObject *at, *weights_type;
  if (!PyArg_ParseTuple(args, "sO!O", &name, &PyLong_Type, &at, &weights_type)) return nullptr;
  for (PyMethodDef& e : entries)
    if (!strcmp(e.ml_name, name)) {
      PyObject* self = PyTuple_Pack(2, at, weights_type);
      PyObject* fn = self ? PyCFunction_NewEx(&e, self, nullptr) : nullptr;
      Py_XDECREF(self);
      return fn;
    }
  PyErr_Format(PyExc_KeyError, "%s", name);
  return nullptr;
}

PyMethodDef methods[] = {{"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls(void) {
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_nbytes = PyUnicode_InternFromString("nbytes");
  s_value = PyUnicode_InternFromString("value");
  if (!s_data_ptr || !s_nbytes || !s_value) return nullptr;
  return PyModule_Create(&module);
}
