// The ordinary call of the four entry points that launch one kernel, without ctypes: plain CUDA tensors on the current device and its current
// stream, default parameters.  The checks are those of binding.py; whatever is not ordinary (another type, device, layout or argument)
// returns None, and binding.py takes its general path, which says what is wrong.  A call takes 0.5 us here, 2 to 2.6 through ctypes
// (six attribute reads and conversions a tensor), where the launch itself takes 3 and the smallest kernels 3 to 4.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <limits>

#include "../../include/swz.h"

namespace {

using GemmFn = decltype(&swz_gemm);
using TransposeFn = decltype(&swz_transpose);
using SoftmaxFn = decltype(&swz_softmax);
using LayernormFn = decltype(&swz_layernorm);
GemmFn g_gemm;
TransposeFn g_transpose;
SoftmaxFn g_softmax;
LayernormFn g_layernorm;
PyObject* g_parameter;         // torch.nn.Parameter

// A torch.Tensor or Parameter (no other subclass) with memory on `device`, contiguous; nullptr otherwise.
const at::Tensor* plain(PyObject* o, c10::DeviceIndex device) {
  PyObject* type = reinterpret_cast<PyObject*>(Py_TYPE(o));
  if (type != THPVariableClass && type != g_parameter) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.get_device() != device || t.layout() != at::kStrided || !t.has_storage() || !t.is_contiguous()) return nullptr;
  return &t;
}

bool is_bf16(const at::Tensor* t, int dim) { return t != nullptr && t->dim() == dim && t->scalar_type() == at::kBFloat16; }

bool as_int(PyObject* o, int* out) {
  if (!PyLong_CheckExact(o)) return false;
  int overflow = 0;
  const long v = PyLong_AsLongAndOverflow(o, &overflow);
  if (overflow != 0 || v < std::numeric_limits<int>::min() || v > std::numeric_limits<int>::max()) return false;
  *out = static_cast<int>(v);
  return true;
}

// call(stream) without the interpreter lock, as ctypes does it; its status as a Python integer
template <class F>
PyObject* launch(c10::DeviceIndex device, F&& call) {
  const hipStream_t stream = c10::hip::getCurrentHIPStream(device).stream();
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = call(stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

// C++ exceptions of the tensor library (a tensor that refuses its pointer, say) go to the general path too
template <class F>
PyObject* guarded(F&& body) {
  try {
    PyObject* r = body();
    if (r != nullptr) return r;
  } catch (...) {
  }
  Py_RETURN_NONE;
}

PyObject* gemm(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    int mode;
    if (n != 4 || !as_int(args[3], &mode)) return nullptr;
    const c10::DeviceIndex dev = c10::hip::current_device();
    const at::Tensor *a = plain(args[0], dev), *b = plain(args[1], dev), *c = plain(args[2], dev);
    if (!is_bf16(a, 2) || !is_bf16(b, 2) || !is_bf16(c, 2)) return nullptr;
    const int64_t M = a->size(0), K = a->size(1), N = b->size(1);
    if (b->size(0) != K || c->size(0) != M || c->size(1) != N) return nullptr;
    void *pa = a->data_ptr(), *pb = b->data_ptr(), *pc = c->data_ptr();
    return launch(dev, [&](hipStream_t s) { return g_gemm(pa, pb, pc, M, N, K, SWZ_DTYPE_BF16, mode, s); });
  });
}

PyObject* transpose(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    int tile, mode;
    if (n != 4 || !as_int(args[2], &tile) || !as_int(args[3], &mode)) return nullptr;
    const c10::DeviceIndex dev = c10::hip::current_device();
    const at::Tensor *x = plain(args[0], dev), *out = plain(args[1], dev);
    if (x == nullptr || out == nullptr || x->dim() != 2 || out->dim() != 2 || x->scalar_type() != out->scalar_type()) return nullptr;
    const int64_t M = x->size(0), N = x->size(1), bytes = static_cast<int64_t>(x->element_size());
    if (out->size(0) != N || out->size(1) != M || (bytes != 2 && bytes != 4)) return nullptr;
    void *px = x->data_ptr(), *po = out->data_ptr();
    return launch(dev, [&](hipStream_t s) { return g_transpose(px, po, M, N, static_cast<int>(bytes), tile, mode, nullptr, s); });
  });
}

PyObject* softmax(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    int chunks, mode;
    if (n != 4 || !as_int(args[2], &chunks) || !as_int(args[3], &mode)) return nullptr;
    const c10::DeviceIndex dev = c10::hip::current_device();
    const at::Tensor *x = plain(args[0], dev), *out = plain(args[1], dev);
    if (!is_bf16(x, 2) || !is_bf16(out, 2) || x->sizes() != out->sizes()) return nullptr;
    const int64_t M = x->size(0), N = x->size(1);
    void *px = x->data_ptr(), *po = out->data_ptr();
    return launch(dev, [&](hipStream_t s) { return g_softmax(px, po, M, N, chunks, mode, nullptr, s); });
  });
}

PyObject* layernorm(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    int chunks, mode;
    if (n != 7 || !PyFloat_CheckExact(args[4]) || !as_int(args[5], &chunks) || !as_int(args[6], &mode)) return nullptr;
    const float eps = static_cast<float>(PyFloat_AS_DOUBLE(args[4]));
    const c10::DeviceIndex dev = c10::hip::current_device();
    const at::Tensor *x = plain(args[0], dev), *g = plain(args[1], dev), *b = plain(args[2], dev), *out = plain(args[3], dev);
    if (!is_bf16(x, 2) || !is_bf16(out, 2) || !is_bf16(g, 1) || !is_bf16(b, 1) || x->sizes() != out->sizes()) return nullptr;
    const int64_t M = x->size(0), N = x->size(1);
    if (g->size(0) != N || b->size(0) != N) return nullptr;
    void *px = x->data_ptr(), *pg = g->data_ptr(), *pb = b->data_ptr(), *po = out->data_ptr();
    return launch(dev, [&](hipStream_t s) { return g_layernorm(px, pg, pb, po, M, N, eps, chunks, mode, nullptr, s); });
  });
}

// The library's functions, as ctypes found them: this module links to no second copy of it.
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n) {
  void* p[4];
  if (n != 5) {
    PyErr_SetString(PyExc_TypeError, "bind(gemm, transpose, softmax, layernorm, Parameter)");
    return nullptr;
  }
  for (int i = 0; i < 4; ++i) {
    p[i] = PyLong_AsVoidPtr(args[i]);
    if (p[i] == nullptr) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null function");
      return nullptr;
    }
  }
  g_gemm = reinterpret_cast<GemmFn>(p[0]);
  g_transpose = reinterpret_cast<TransposeFn>(p[1]);
  g_softmax = reinterpret_cast<SoftmaxFn>(p[2]);
  g_layernorm = reinterpret_cast<LayernormFn>(p[3]);
  Py_INCREF(args[4]);
  Py_XSETREF(g_parameter, args[4]);
  Py_RETURN_NONE;
}

#define SWZ_FAST(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {SWZ_FAST(gemm), SWZ_FAST(transpose), SWZ_FAST(softmax), SWZ_FAST(layernorm), SWZ_FAST(bind), {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall() {
  PyObject* m = PyModule_Create(&kModule);
  if (m != nullptr && PyModule_AddStringConstant(m, "built_for", SWZ_TORCH_TAG) != 0) Py_CLEAR(m);       // binding.py uses it with that torch only
  return m;
}
