// The calls of libpkv from Python, as a CPython module: takes the tensors' addresses, the current stream and the numbers out of
// the Python objects and calls the C function with the interpreter's lock released, as ctypes does.  A decode step of a small model is bound by
// the host: an append took 4.2 us there, 2.7 of them HIP's launch, and the rest attribute look-ups, one at a time, and ctypes' conversions;
// this way 3.25.  A pass of append and attention of 4 requests of 17..300 tokens 9.8 -> 8.1 us, of two moves of 5 MB 9.9 -> 8.6.
//
// An argument that is not as expected (no tensor, a number of another kind, a shape of another class, no GPU yet) makes a call
// return NotImplemented, having called nothing: the caller goes by ctypes then, which converts it or raises.  An exception that
// is not about an argument's kind (an interrupt, memory, an error of the tensor's or torch's own) goes to the caller as it is.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "../../include/pkv.h"

#include <tuple>
#include <utility>

namespace {

PyObject *s_data_ptr, *s_numel, *s_element_size, *s_cuda_stream;   // names of methods and an attribute
PyObject *g_shape_type, *g_initialized, *g_device, *g_raw_stream;

// An int's value, false if it is no int.
bool take_int(PyObject* o, int64_t* out) {
  if (!PyLong_Check(o)) return false;
  *out = (int64_t)PyLong_AsUnsignedLongLongMask(o);
  return true;
}
bool method_int(PyObject* o, PyObject* name, int64_t* out) {
  PyObject* r = PyObject_VectorcallMethod(name, &o, 1, nullptr);
  if (!r) return false;
  const bool ok = take_int(r, out);
  Py_DECREF(r);
  return ok;
}

// What a parameter of a C function is made of; each takes one Python argument.
struct Address {   // of a tensor, or None
  void* p = nullptr;
  bool take(PyObject* o) {
    int64_t x = 0;
    if (o != Py_None && !method_int(o, s_data_ptr, &x)) return false;
    p = (void*)x;
    return true;
  }
};
struct Workspace : Address {   // and its bytes
  size_t bytes = 0;
  bool take(PyObject* o) {
    int64_t n = 0, size = 0;
    if (!Address::take(o) || (o != Py_None && !(method_int(o, s_numel, &n) && method_int(o, s_element_size, &size)))) return false;
    bytes = (size_t)(n * size);
    return true;
  }
};
struct Number {
  int64_t v = 0;
  bool take(PyObject* o) { return take_int(o, &v); }
};
struct Real {
  float v = 0;
  bool take(PyObject* o) {
    if (!PyFloat_Check(o)) return false;
    v = (float)PyFloat_AS_DOUBLE(o);
    return true;
  }
};
struct Shape {
  Py_buffer view = {};
  bool take(PyObject* o) {
    return Py_IS_TYPE(o, (PyTypeObject*)g_shape_type) && PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) == 0 &&
           view.len == (Py_ssize_t)sizeof(pkv_attn_shape);
  }
  ~Shape() {
    if (view.obj) PyBuffer_Release(&view);
  }
};
struct Stream {   // a handle, an object that has one, or None for the current device's current stream
  void* p = nullptr;
  bool take(PyObject* o) {
    int64_t x = 0;
    if (o != Py_None) {
      if (!take_int(o, &x)) {
        PyObject* handle = PyObject_GetAttr(o, s_cuda_stream);
        const bool ok = handle && take_int(handle, &x);
        Py_XDECREF(handle);
        if (!ok) return false;
      }
    } else {
      if (g_raw_stream == Py_None) return false;
      PyObject* up = PyObject_CallNoArgs(g_initialized);
      const bool ready = up == Py_True;
      Py_XDECREF(up);
      if (!ready) return false;
      PyObject* device = PyObject_CallNoArgs(g_device);
      if (!device) return false;
      PyObject* raw = PyObject_CallOneArg(g_raw_stream, device);
      Py_DECREF(device);
      const bool ok = raw && take_int(raw, &x);
      Py_XDECREF(raw);
      if (!ok) return false;
    }
    p = (void*)x;
    return true;
  }
};

// The C arguments of each.
struct AnyPointer {
  void* p;
  template <typename X> operator X*() const { return (X*)p; }
};
std::tuple<AnyPointer> c_args(const Address& a) { return {AnyPointer{a.p}}; }
std::tuple<AnyPointer, size_t> c_args(const Workspace& a) { return {AnyPointer{a.p}, a.bytes}; }
std::tuple<int64_t> c_args(const Number& a) { return {a.v}; }
std::tuple<float> c_args(const Real& a) { return {a.v}; }
std::tuple<const pkv_attn_shape*> c_args(const Shape& a) { return {(const pkv_attn_shape*)a.view.buf}; }
std::tuple<void*> c_args(const Stream& a) { return {a.p}; }

template <typename... A, typename Fn, size_t... I>
PyObject* call(Fn fn, PyObject* const* args, std::index_sequence<I...>) {
  std::tuple<A...> a;
  if (!(std::get<I>(a).take(args[I]) && ...)) {
    if (PyErr_Occurred()) {
      if (!PyErr_ExceptionMatches(PyExc_TypeError) && !PyErr_ExceptionMatches(PyExc_AttributeError) &&
          !PyErr_ExceptionMatches(PyExc_OverflowError))
        return nullptr;
      PyErr_Clear();
    }
    Py_RETURN_NOTIMPLEMENTED;
  }
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = std::apply(fn, std::tuple_cat(c_args(std::get<I>(a))...));
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

// One entry point: its address, once known, and the kinds of its arguments in order.
template <typename F, typename... A>
struct Entry {
  static inline F* fn = nullptr;
  static PyObject* run(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (!fn || n != (Py_ssize_t)sizeof...(A)) Py_RETURN_NOTIMPLEMENTED;
    return call<A...>(fn, args, std::index_sequence_for<A...>{});
  }
};
using T = Address;
using Append = Entry<decltype(kv_append), T, T, T, T, T, T, Shape, Stream>;
using AppendFp8 = Entry<decltype(kv_append_fp8), T, T, T, T, T, T, Real, Real, Shape, Stream>;
using Attn = Entry<decltype(paged_decode_attn), T, T, T, T, T, Real, T, Shape, Workspace, Stream>;
using AttnFp8 = Entry<decltype(paged_decode_attn_fp8kv), T, T, T, T, T, Real, Real, Real, T, Shape, Workspace, Stream>;
using AttnStatic = Entry<decltype(paged_decode_attn_static), T, T, T, T, T, Real, T, Shape, Stream>;
using Gather = Entry<decltype(kv_blocks_gather), T, T, T, Number, Number, Number, Stream>;
using Scatter = Entry<decltype(kv_blocks_scatter), T, T, T, Number, Number, Number, Stream>;
using Move = Entry<decltype(kv_blocks_move), T, T, T, T, Number, Number, Number, Number, Stream>;
using Offload = Entry<decltype(kv_blocks_offload), T, T, T, T, Number, Number, Number, Stream>;
using Reload = Entry<decltype(kv_blocks_reload), T, T, T, T, Number, Number, Number, Stream>;

template <typename E>
void set_address(PyObject* addresses, const char* name) {
  PyObject* o = PyDict_GetItemString(addresses, name);   // borrowed
  int64_t x = 0;
  E::fn = o && take_int(o, &x) ? (decltype(E::fn))x : nullptr;
}

// setup(addresses of the C functions by name, the class of shapes, and three functions of torch or None: is the GPU initialised, the
// current device, the handle of its current stream)
PyObject* setup(PyObject*, PyObject* args) {
  PyObject *addresses, *shape, *initialized, *device, *raw;
  if (!PyArg_ParseTuple(args, "O!O!OOO", &PyDict_Type, &addresses, &PyType_Type, &shape, &initialized, &device, &raw)) return nullptr;
  set_address<Append>(addresses, "kv_append");
  set_address<AppendFp8>(addresses, "kv_append_fp8");
  set_address<Attn>(addresses, "paged_decode_attn");
  set_address<AttnFp8>(addresses, "paged_decode_attn_fp8kv");
  set_address<AttnStatic>(addresses, "paged_decode_attn_static");
  set_address<Gather>(addresses, "kv_blocks_gather");
  set_address<Scatter>(addresses, "kv_blocks_scatter");
  set_address<Move>(addresses, "kv_blocks_move");
  set_address<Offload>(addresses, "kv_blocks_offload");
  set_address<Reload>(addresses, "kv_blocks_reload");
  const std::pair<PyObject**, PyObject*> keep[] = {
      {&g_shape_type, shape}, {&g_initialized, initialized}, {&g_device, device}, {&g_raw_stream, raw}};
  for (auto& k : keep) {
    Py_INCREF(k.second);
    PyObject* old = *k.first;
    *k.first = k.second;
    Py_XDECREF(old);
  }
  Py_RETURN_NONE;
}

template <typename E>
PyMethodDef method(const char* name) {
  return {name, (PyCFunction)(void (*)(void))E::run, METH_FASTCALL, nullptr};
}
PyMethodDef methods[] = {
    {"setup", setup, METH_VARARGS, nullptr},
    method<Append>("kv_append"),
    method<AppendFp8>("kv_append_fp8"),
    method<Attn>("paged_decode_attn"),
    method<AttnFp8>("paged_decode_attn_fp8kv"),
    method<AttnStatic>("paged_decode_attn_static"),
    method<Gather>("kv_blocks_gather"),
    method<Scatter>("kv_blocks_scatter"),
    method<Move>("kv_blocks_move"),
    method<Offload>("kv_blocks_offload"),
    method<Reload>("kv_blocks_reload"),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pkv_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pkv_call(void) {
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_numel = PyUnicode_InternFromString("numel");
  s_element_size = PyUnicode_InternFromString("element_size");
  s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  if (!s_data_ptr || !s_numel || !s_element_size || !s_cuda_stream) return nullptr;
  return PyModule_Create(&module);
}
