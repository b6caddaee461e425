// Python entry points of the C ABI: one function per call of include/moe.h, its arguments converted from Python objects by
// the types of the C declaration, the current stream added as the last one, the status returned as an int.
//
// A step of a small layer is a sequence of some twenty calls whose kernels run for a few microseconds each, so the caller's
// own time per call is what bounds it.  In Python and through ctypes every tensor costs three attribute or method calls
// (device, contiguity, pointer); here the same checks are made on the tensor object.  moe_route + moe_route_bwd of 4096
// tokens 20.4 -> 13.0 us, the twenty launches of a small fp32 training step (T = 256, d = 128, f = 256) 120 -> 87 us.
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <tuple>
#include <type_traits>
#include <utility>

#include "../../../include/moe.h"

namespace {

bool refuse_tensor() {
  PyErr_SetString(PyExc_AssertionError, "tensors must be contiguous and on the GPU");
  return false;
}

// Device pointer of a tensor (None -> NULL).  A plain tensor or parameter is read directly; anything else (subclasses with
// their own behaviour, objects that quack like a tensor) is asked through Python.
bool to_pointer(PyObject* o, void** out) {
  if (o == Py_None) { *out = nullptr; return true; }
  if (THPVariable_CheckExact(o)) {
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous()) return refuse_tensor();
    *out = t.data_ptr();
    return true;
  }
  PyObject* cuda = PyObject_GetAttrString(o, "is_cuda");
  if (!cuda) return false;
  const int is_cuda = PyObject_IsTrue(cuda);
  Py_DECREF(cuda);
  if (is_cuda < 0) return false;
  PyObject* cont = PyObject_CallMethod(o, "is_contiguous", nullptr);
  if (!cont) return false;
  const int is_contiguous = PyObject_IsTrue(cont);
  Py_DECREF(cont);
  if (is_contiguous < 0) return false;
  if (!is_cuda || !is_contiguous) return refuse_tensor();
  PyObject* ptr = PyObject_CallMethod(o, "data_ptr", nullptr);
  if (!ptr) return false;
  *out = PyLong_AsVoidPtr(ptr);
  Py_DECREF(ptr);
  return !PyErr_Occurred();
}

template <typename A> bool convert(PyObject* o, A* out) {
  if constexpr (std::is_pointer_v<A>) {
    void* p = nullptr;
    if (!to_pointer(o, &p)) return false;
    *out = static_cast<A>(p);
    return true;
  } else if constexpr (std::is_floating_point_v<A>) {
    const double v = PyFloat_AsDouble(o);
    *out = static_cast<A>(v);
    return !(v == -1.0 && PyErr_Occurred());
  } else {                                        // integers and the enums, wrapped to the C type as ctypes does
    *out = static_cast<A>(static_cast<long long>(PyLong_AsUnsignedLongLongMask(o)));
    return !PyErr_Occurred();
  }
}

template <auto FN> struct Bound;
template <typename... A, int (*FN)(A...)> struct Bound<FN> {
  static constexpr size_t kArgs = sizeof...(A) - 1;                 // the last parameter is the stream

  template <size_t... I> static bool parse(PyObject* const* args, std::tuple<A...>& v, std::index_sequence<I...>) {
    return (convert(args[I], &std::get<I>(v)) && ...);
  }

  static PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != static_cast<Py_ssize_t>(kArgs)) {
      PyErr_Format(PyExc_TypeError, "takes %zu arguments (%zd given)", kArgs, n);
      return nullptr;
    }
    try {
      std::tuple<A...> v{};
      if (!parse(args, v, std::make_index_sequence<kArgs>())) return nullptr;
      std::get<kArgs>(v) = static_cast<void*>(c10::hip::getCurrentHIPStream().stream());
      int rc;
      Py_BEGIN_ALLOW_THREADS
      rc = std::apply(FN, v);
      Py_END_ALLOW_THREADS
      return PyLong_FromLong(rc);
    } catch (const std::exception& e) {
      PyErr_SetString(PyExc_RuntimeError, e.what());
      return nullptr;
    }
  }
};

#define MOE_BOUND(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(&Bound<&name>::call)), METH_FASTCALL, nullptr}

PyMethodDef methods[] = {
    MOE_BOUND(moe_router_fwd), MOE_BOUND(moe_router_bwd), MOE_BOUND(moe_route), MOE_BOUND(moe_route_noalloc),
    MOE_BOUND(moe_route_range), MOE_BOUND(moe_route_capacity), MOE_BOUND(moe_balance_loss), MOE_BOUND(moe_balance_loss_bwd),
    MOE_BOUND(moe_route_bwd), MOE_BOUND(moe_dispatch), MOE_BOUND(moe_combine), MOE_BOUND(moe_gate_grad),
    MOE_BOUND(moe_expert_ffn_fwd), MOE_BOUND(moe_expert_ffn_bwd), MOE_BOUND(moe_row_map), MOE_BOUND(moe_expert_ffn_fused_fwd),
    MOE_BOUND(moe_expert_ffn_fused_bwd), MOE_BOUND(moe_quant_fp8), MOE_BOUND(moe_dequant_fp8), MOE_BOUND(moe_quant_fp8_tgroup),
    MOE_BOUND(moe_transpose), {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_moe_native", "Calls of the MoE library on torch tensors.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__moe_native(void) { return PyModule_Create(&module); }
