// The calls of include/dp_bk.h for Python: argument conversion in native code, from each function's own type.
//
// Through ctypes a call of eight arguments cost 4.1 to 5.0 us, 2.5 to 3 of them the launch; here 3.0.  Passes from Python, us,
// through ctypes and here: two micro-batches of 32 layers with biases, 18 x 45 tokens 690, 602; of 20 layers, 11 x 32 442, 388;
// a step of ten 64 x 64 layers, one sample of two tokens 19.8, 18.7.
//
// Device pointers take a tensor (its data_ptr()), an address or None; host arrays a ctypes array of the prototype's own element
// type or None (which pointer is which, a C type cannot tell: set_host_arrays); the last argument is the stream, None for
// torch's current one.  Arguments of another kind make the call return None before anything happened, and the caller takes
// the general path, which refuses what ctypes refuses.  The interpreter's lock is released during the call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <string.h>

#include <tuple>
#include <type_traits>
#include <utility>

#include "dp_bk.h"

namespace {

PyObject *data_ptr_name, *type_name;
PyTypeObject* array_type;                     // ctypes.Array
PyObject *torch_c, *device_name, *stream_name;     // torch's module of private functions; null until its GPU side is up

struct Address {
  void* p = nullptr;
  Py_buffer view;
  bool held = false;
  ~Address() {
    if (held) PyBuffer_Release(&view);
  }
};

bool as_address(PyObject* x, Address& out) {
  if (x == Py_None) return true;
  if (PyLong_Check(x)) {
    out.p = (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(x);
    return true;
  }
  PyObject* r = PyObject_CallMethodNoArgs(x, data_ptr_name);
  if (!r) return false;
  const bool ok = PyLong_Check(r);
  if (ok) out.p = (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(r);
  Py_DECREF(r);
  return ok;
}

// A ctypes array whose elements are of type `element`.
bool as_host_array(PyObject* x, PyObject* element, Address& out) {
  if (x == Py_None) return true;
  if (!array_type || !PyObject_TypeCheck(x, array_type)) return false;
  PyObject* type = PyObject_GetAttr(reinterpret_cast<PyObject*>(Py_TYPE(x)), type_name);
  Py_XDECREF(type);                            // (the array's type holds it)
  if (type != element || PyObject_GetBuffer(x, &out.view, PyBUF_SIMPLE) != 0) return false;
  out.held = true;
  out.p = out.view.buf;
  return true;
}

bool as_stream(PyObject* x, Address& out) {
  if (PyLong_Check(x)) return as_address(x, out);
  if (x != Py_None || !torch_c) return false;
  PyObject* device = PyObject_CallMethodNoArgs(torch_c, device_name);
  if (!device) return false;
  PyObject* r = PyObject_CallMethodOneArg(torch_c, stream_name, device);
  Py_DECREF(device);
  if (!r) return false;
  const bool ok = PyLong_Check(r) && as_address(r, out);
  Py_DECREF(r);
  return ok;
}

template <class T>
struct Value {
  T v{};
  bool set(PyObject* x, PyObject*) {
    if constexpr (std::is_floating_point_v<T>) {
      if (!PyFloat_Check(x) && !PyLong_Check(x)) return false;
      const double d = PyFloat_AsDouble(x);
      if (d == -1.0 && PyErr_Occurred()) return false;
      v = (T)d;
    } else {
      if (!PyLong_Check(x)) return false;
      v = (T)PyLong_AsUnsignedLongLongMask(x);
    }
    return true;
  }
  T get() const { return v; }
};
template <class T>
struct Value<T*> {
  Address a;
  bool set(PyObject* x, PyObject* element) { return element ? as_host_array(x, element, a) : as_address(x, a); }
  T* get() const { return static_cast<T*>(a.p); }
};

template <auto F>
struct Call;
template <class... A, dp_status (*F)(A...)>
struct Call<F> {
  static constexpr Py_ssize_t N = sizeof...(A);
  static inline PyObject* element[N];         // of the arguments that are host arrays; null: not one
  static inline bool known = false;
  template <size_t... I>
  static PyObject* run(PyObject* const* args, std::index_sequence<I...>) {
    std::tuple<Value<A>...> v;
    const bool ok = ((I + 1 == N ? as_stream(args[I], address(std::get<I>(v))) : std::get<I>(v).set(args[I], element[I])) && ...);
    if (!ok) {
      PyErr_Clear();
      Py_RETURN_NONE;
    }
    dp_status st;
    Py_BEGIN_ALLOW_THREADS
    st = F(std::get<I>(v).get()...);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong((long)st);
  }
  template <class T>
  static Address& address(Value<T*>& v) { return v.a; }
  template <class T>
  static Address& address(Value<T>&) {        // not reached: the last argument is a pointer
    static Address none;
    return none;
  }
  static PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != N || !known) Py_RETURN_NONE;
    return run(args, std::make_index_sequence<N>{});
  }
  static bool set_elements(PyObject* types) {
    if (!PyTuple_Check(types) || PyTuple_GET_SIZE(types) != N) return false;
    for (Py_ssize_t i = 0; i < N; ++i) {
      PyObject* t = PyTuple_GET_ITEM(types, i);
      Py_XDECREF(element[i]);
      element[i] = t == Py_None ? nullptr : t;
      Py_XINCREF(element[i]);
    }
    return known = true;
  }
};

PyObject* set_array_type(PyObject*, PyObject* type) {
  if (!PyType_Check(type)) Py_RETURN_NONE;
  Py_INCREF(type);
  Py_XDECREF(reinterpret_cast<PyObject*>(array_type));
  array_type = reinterpret_cast<PyTypeObject*>(type);
  Py_RETURN_NONE;
}

PyObject* set_torch(PyObject*, PyObject* module) {
  Py_INCREF(module);
  Py_XDECREF(torch_c);
  torch_c = module;
  Py_RETURN_NONE;
}

#define DP_CALLS(X) \
  X(dp_ghost_norm) \
  X(dp_perex_norm) \
  X(dp_clip_factors) \
  X(dp_clipped_grad) \
  X(dp_add_noise) \
  X(dp_norms_multi) \
  X(dp_clipped_grad_multi) \
  X(dp_clipped_grad_noise_multi) \
  X(dp_clipped_grad_noise_multi_h16) \
  X(dp_bias_norm) \
  X(dp_clipped_bias_grad) \
  X(dp_norms_multi_keep) \
  X(dp_clipped_grad_kept_multi) \
  X(dp_private_step_multi) \
  X(dp_layerwise_clipped_grad)

// set_host_arrays(name, types): for each argument of call `name` the ctypes type of the host array's elements, or None.
PyObject* set_host_arrays(PyObject*, PyObject* args) {
  const char* name;
  PyObject* types;
  if (!PyArg_ParseTuple(args, "sO", &name, &types)) return nullptr;
  bool ok = false;
#define DP_SET(f) \
  if (!strcmp(name, #f)) ok = Call<f>::set_elements(types);
  DP_CALLS(DP_SET)
#undef DP_SET
  return PyBool_FromLong(ok);
}

#define DP_METHOD(f) {#f, (PyCFunction)(void (*)(void))Call<f>::call, METH_FASTCALL, nullptr},
PyMethodDef methods[] = {DP_CALLS(DP_METHOD)
                         {"set_array_type", set_array_type, METH_O, nullptr},
                         {"set_host_arrays", set_host_arrays, METH_VARARGS, nullptr},
                         {"set_torch", set_torch, METH_O, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pycall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pycall(void) {
  data_ptr_name = PyUnicode_InternFromString("data_ptr");
  type_name = PyUnicode_InternFromString("_type_");
  device_name = PyUnicode_InternFromString("_cuda_getDevice");
  stream_name = PyUnicode_InternFromString("_cuda_getCurrentRawStream");
  return data_ptr_name && type_name && device_name && stream_name ? PyModule_Create(&module) : nullptr;
}
