// Argument marshalling for the Python binding: one CPython entry per C ABI function that takes device tensors.  A Python
// call hands over tensors or None for pointers, integers for sizes and modes, for a stream its handle or Ellipsis (the
// current stream of the current device), and for an optimizer step the address of the struct; each is converted to the
// type of the C parameter in that place, and nothing else is taken for it: an integer is no tensor, and a tensor no
// integer.  Doing this through ctypes and attribute look-ups cost 6 to 10 us a call, as much as the launches of a small
// layer.
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <tuple>
#include <type_traits>
#include <utility>

#include "../../include/efqat.h"

namespace {

struct BadArgument {};

[[noreturn]] void refuse(PyObject* type, const char* what, PyObject* got) {
  PyErr_Format(type, "%s expected, got %.100s", what, Py_TYPE(got)->tp_name);
  throw BadArgument();
}

long long integer(PyObject* o, const char* what) {
  // other integer types (numpy's) by their __index__; a tensor's would wait for the GPU
  if (!PyLong_Check(o) && (!PyIndex_Check(o) || THPVariable_Check(o))) refuse(PyExc_TypeError, what, o);
  const long long v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) throw BadArgument();
  return v;
}

void* tensor_address(PyObject* o) {
  if (o == Py_None) return nullptr;
  if (!THPVariable_Check(o)) refuse(PyExc_TypeError, "tensor", o);
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.is_cuda()) {
    PyErr_SetString(PyExc_ValueError, "tensor must live on the GPU");
    throw BadArgument();
  }
  if (!t.is_contiguous()) {
    PyErr_SetString(PyExc_ValueError, "tensor must be contiguous");
    throw BadArgument();
  }
  return t.data_ptr();
}

// STREAM: the parameter is a stream (every entry ends in `void* stream` or `void* stream, void* side_stream`)
template <class T, bool STREAM>
T from_python(PyObject* o) {
  if constexpr (STREAM) {
    if (o == Py_None) return nullptr;
    if (o == Py_Ellipsis) return (T)c10::hip::getCurrentHIPStream().stream();
    return (T)(uintptr_t)integer(o, "stream handle");
  } else if constexpr (std::is_same_v<T, const efqat_opt_step*>) {
    return o == Py_None ? nullptr : (T)(uintptr_t)integer(o, "address of an efqat_opt_step");
  } else if constexpr (std::is_pointer_v<T>) {
    return (T)tensor_address(o);
  } else {
    return (T)integer(o, "integer");
  }
}

template <class... A>
constexpr bool is_stream(size_t i) {
  constexpr bool is_void[] = {std::is_same_v<A, void*>...};
  constexpr size_t n = sizeof...(A);
  static_assert(is_void[n - 1], "an entry ends in a stream");
  return i == n - 1 || (i == n - 2 && is_void[i]);
}

template <class... A, size_t... I>
PyObject* call(int (*fn)(A...), PyObject* const* args, std::index_sequence<I...>) {
  try {
    std::tuple<A...> a{from_python<A, is_stream<A...>(I)>(args[I])...};     // braces: in order, so that the first bad argument is reported
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = std::apply(fn, a);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
  } catch (const BadArgument&) {
    return nullptr;
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}

template <class... A>
PyObject* call_n(int (*fn)(A...), PyObject* const* args, Py_ssize_t n) {
  if (n != (Py_ssize_t)sizeof...(A)) {
    PyErr_Format(PyExc_TypeError, "%zd arguments, %zd expected", n, (Py_ssize_t)sizeof...(A));
    return nullptr;
  }
  return call(fn, args, std::index_sequence_for<A...>{});
}

template <auto FN>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) { return call_n(FN, args, n); }

#define EFQAT_ENTRY(name) {#name, (PyCFunction)(void (*)(void))entry<efqat_##name>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    EFQAT_ENTRY(fakequant_fwd),  EFQAT_ENTRY(channel_select), EFQAT_ENTRY(channel_select_static),
    EFQAT_ENTRY(weight_quant_select), EFQAT_ENTRY(network_select), EFQAT_ENTRY(layer_select),
    EFQAT_ENTRY(bias_grad),      EFQAT_ENTRY(linear_bwd_ex),  EFQAT_ENTRY(linear_bwd_weight_operand),
    EFQAT_ENTRY(conv_bwd_ex),    EFQAT_ENTRY(linear_fwd),     {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_efqat_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__efqat_torch() { return PyModule_Create(&module_def); }
