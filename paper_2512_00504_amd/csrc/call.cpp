// Native half of the ctypes binding: the calls of the decode/evict path from Python with torch tensors.
//
// A decode step of a few units is 5 us of GPU time; through ctypes the call itself took as long: 1.2 us for
// nine is_contiguous() / data_ptr() pairs, 0.5 us of argument conversion, 0.4 us for the stream handle, 0.4 us
// of Python around them, and 2.6 us in the library (the launch).  Here the first four take 0.3 us.
//
// Each function is the C entry point of the same name without its last argument, the stream, which is the
// current device's current one.  Arguments that are not exactly what the path passes (a torch.Tensor, contiguous, or
// None; an int of 32 bits; a float) are not converted here: the function returns None without having called
// anything, and the caller goes through ctypes, which converts or refuses them as it always has.
#include <torch/csrc/autograd/python_variable.h>

#include <c10/hip/HIPStream.h>

#include <cstring>
#include <tuple>
#include <utility>

#include "gkv.h"

namespace {

struct NotForUs {};

void* pointer(PyObject* o) {
  if (o == Py_None) return nullptr;
  if (!THPVariable_CheckExact(o)) throw NotForUs();
  const at::Tensor& t = THPVariable_Unpack(o);
  if (t.layout() != at::kStrided || !t.is_cuda() || !t.is_contiguous() || !t.has_storage()) throw NotForUs();
  return t.data_ptr();
}
void convert(PyObject* o, void*& out) { out = pointer(o); }
void convert(PyObject* o, const void*& out) { out = pointer(o); }
void convert(PyObject* o, int32_t*& out) { out = (int32_t*)pointer(o); }
void convert(PyObject* o, const int32_t*& out) { out = (const int32_t*)pointer(o); }
void convert(PyObject* o, float*& out) { out = (float*)pointer(o); }
void convert(PyObject* o, const float*& out) { out = (const float*)pointer(o); }
void convert(PyObject* o, gkv_ctx*& out) {
  if (!PyLong_CheckExact(o)) throw NotForUs();
  out = (gkv_ctx*)PyLong_AsVoidPtr(o);
  if (!out) { PyErr_Clear(); throw NotForUs(); }
}
void convert(PyObject* o, int32_t& out) {
  if (!PyLong_CheckExact(o)) throw NotForUs();
  int overflow = 0;
  const long v = PyLong_AsLongAndOverflow(o, &overflow);
  if (overflow || v < INT32_MIN || v > INT32_MAX) throw NotForUs();
  out = (int32_t)v;
}
void convert(PyObject* o, float& out) {
  if (!PyFloat_CheckExact(o)) throw NotForUs();
  out = (float)PyFloat_AS_DOUBLE(o);
}

// One type per entry point, with the signature that the header declares and the address that bind() was given
// (the library is loaded through ctypes).
#define GKV_CALLS(X)                                                                                 \
  X(gkv_attend_decode) X(gkv_score_window) X(gkv_global_update) X(gkv_select_topk) X(gkv_compact)    \
  X(gkv_evict) X(gkv_redundancy_combine) X(gkv_evicted_positions)
#define GKV_TYPE(name) struct call_##name { static inline decltype(&::name) address = nullptr; };
GKV_CALLS(GKV_TYPE)

template <typename Call, typename... A, size_t... I>
PyObject* call(gkv_status (*f)(A...), PyObject* const* args, Py_ssize_t n, std::index_sequence<I...>) {
  try {
    if (!f || n != (Py_ssize_t)sizeof...(I)) throw NotForUs();
    std::tuple<A...> v;
    (convert(args[I], std::get<I>(v)), ...);
    std::get<sizeof...(I)>(v) = (void*)c10::hip::getCurrentHIPStream().stream();
    gkv_status st;
    Py_BEGIN_ALLOW_THREADS
    st = std::apply(f, v);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
  } catch (const NotForUs&) {
    Py_RETURN_NONE;
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}
template <typename... A> constexpr size_t arguments(gkv_status (*)(A...)) { return sizeof...(A); }

template <typename Call>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
  constexpr size_t N = arguments(decltype(Call::address){nullptr}) - 1;   // without the stream
  return call<Call>(Call::address, args, n, std::make_index_sequence<N>());
}

PyObject* bind(PyObject*, PyObject* args) {
  const char* name;
  PyObject* address;
  if (!PyArg_ParseTuple(args, "sO!", &name, &PyLong_Type, &address)) return nullptr;
  void* p = PyLong_AsVoidPtr(address);
  if (PyErr_Occurred()) return nullptr;
#define GKV_BIND(call) if (!strcmp(name, #call)) { call_##call::address = (decltype(&::call))p; Py_RETURN_NONE; }
  GKV_CALLS(GKV_BIND)
  PyErr_SetString(PyExc_KeyError, name);
  return nullptr;
}

#define GKV_METHOD(name) {#name, (PyCFunction)(void (*)(void))entry<call_##name>, METH_FASTCALL, nullptr},
PyMethodDef methods[] = {GKV_CALLS(GKV_METHOD){"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_gkv_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__gkv_call() { return PyModule_Create(&module); }
