// Argument marshalling of the launch calls in C++: what binding.py does per call in Python (attribute checks of every
// tensor, a ctypes call), for the plain case - descriptors and configuration as the binding's own structures, tensors of
// the exact type torch.Tensor, contiguous, float16, on a GPU.  Each function returns the bolt_status as an int, or None
// if an argument is of any other kind: the caller then takes the general path in Python, which accepts or refuses it.
// A launch of a small problem takes about 3 us on the GPU; the Python path took 5 us of host time per call.
#include <torch/csrc/autograd/python_variable.h>

#include <c10/hip/HIPStream.h>

#include "../../include/bolt.h"

namespace {

PyObject *g_gemm_desc, *g_conv_desc, *g_config;  // the ctypes structure types of binding.py

// A structure's bytes, copied: the call below runs without the interpreter lock.
template <typename T>
bool read_struct(PyObject* o, PyObject* type, T* out) {
  if ((PyObject*)Py_TYPE(o) != type) return false;
  Py_buffer view;
  if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) {
    PyErr_Clear();
    return false;
  }
  const bool ok = view.len == (Py_ssize_t)sizeof(T);
  if (ok) std::memcpy(out, view.buf, sizeof(T));
  PyBuffer_Release(&view);
  return ok;
}
bool read(PyObject* o, bolt_gemm_desc* d) { return read_struct(o, g_gemm_desc, d); }
bool read(PyObject* o, bolt_conv_desc* d) { return read_struct(o, g_conv_desc, d); }

struct Config {
  bolt_config value;
  const bolt_config* ptr = nullptr;
  bool read(PyObject* o) {
    if (o == Py_None) return true;
    ptr = &value;
    return read_struct(o, g_config, &value);
  }
};

// Device pointer of a tensor as the binding accepts it (an address only for this call).
bool half_tensor(PyObject* o, void** p) {
  if (!THPVariable_CheckExact(o)) return false;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.is_cuda() || t.scalar_type() != at::kHalf || !t.is_contiguous()) return false;
  *p = t.data_ptr();
  return true;
}
bool half_tensor_or_none(PyObject* o, void** p) {
  *p = nullptr;
  return o == Py_None || half_tensor(o, p);
}
struct Workspace {
  void* ptr = nullptr;
  size_t bytes = 0;
  bool read(PyObject* o) {
    if (o == Py_None) return true;
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous()) return false;
    ptr = t.data_ptr();
    bytes = (size_t)t.numel() * t.element_size();
    return true;
  }
};
bool read_float(PyObject* o, float* f) {
  if (!PyFloat_CheckExact(o)) return false;
  *f = (float)PyFloat_AS_DOUBLE(o);
  return true;
}

template <typename F>
PyObject* call(F&& f) {
  void* const stream = (void*)c10::hip::getCurrentHIPStream().stream();
  bolt_status s;
  Py_BEGIN_ALLOW_THREADS
  s = f(stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong((long)s);
}

// A torch call may throw (a tensor without storage, for one): the general path then meets the same error and raises it.
template <PyObject* (*BODY)(PyObject* const*)>
PyObject* guarded(PyObject* const* a, Py_ssize_t n, Py_ssize_t want) {
  if (n != want) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  try {
    if (PyObject* r = BODY(a)) return r;
  } catch (...) {
  }
  PyErr_Clear();
  Py_RETURN_NONE;
}

// (desc, x, w, bias, y, config, workspace)
template <typename D, bolt_status (*FN)(const D*, const void*, const void*, const void*, void*, const bolt_config*, void*, size_t, void*)>
PyObject* single(PyObject* const* a) {
  D d;
  void *x, *w, *b, *y;
  Config c;
  Workspace ws;
  if (!read(a[0], &d) || !half_tensor(a[1], &x) || !half_tensor(a[2], &w) || !half_tensor_or_none(a[3], &b) || !half_tensor(a[4], &y) ||
      !c.read(a[5]) || !ws.read(a[6]))
    return nullptr;
  return call([&](void* s) { return FN(&d, x, w, b, y, c.ptr, ws.ptr, ws.bytes, s); });
}

// (desc, x, w, bias, residual, y, gamma, config, workspace)
template <typename D>
PyObject* single_residual(PyObject* const* a) {
  D d;
  void *x, *w, *b, *r, *y;
  float gamma;
  Config c;
  Workspace ws;
  if (!read(a[0], &d) || !half_tensor(a[1], &x) || !half_tensor(a[2], &w) || !half_tensor_or_none(a[3], &b) || !half_tensor(a[4], &r) ||
      !half_tensor(a[5], &y) || !read_float(a[6], &gamma) || !c.read(a[7]) || !ws.read(a[8]))
    return nullptr;
  if constexpr (std::is_same_v<D, bolt_gemm_desc>) {
    const at::Tensor& t = THPVariable_Unpack(a[4]);
    if (t.dim() < 1 || t.size(-1) > INT32_MAX) return nullptr;
    const int32_t ldc = (int32_t)t.size(-1);
    return call([&](void* s) { return bolt_gemm_epilogue_residual(&d, x, w, b, r, ldc, gamma, y, c.ptr, ws.ptr, ws.bytes, s); });
  } else {
    return call([&](void* s) { return bolt_conv2d_fprop_nhwc_residual(&d, x, w, b, r, gamma, y, c.ptr, ws.ptr, ws.bytes, s); });
  }
}

// (desc0, desc1, x, w0, b0, w1, b1, y, config)
template <typename D, bolt_status (*FN)(const D*, const D*, const void*, const void*, const void*, const void*, const void*, void*,
                                        const bolt_config*, void*, size_t, void*)>
PyObject* pair(PyObject* const* a) {
  D d0, d1;
  void *x, *w0, *b0, *w1, *b1, *y;
  Config c;
  if (!read(a[0], &d0) || !read(a[1], &d1) || !half_tensor(a[2], &x) || !half_tensor(a[3], &w0) || !half_tensor_or_none(a[4], &b0) ||
      !half_tensor(a[5], &w1) || !half_tensor_or_none(a[6], &b1) || !half_tensor(a[7], &y) || !c.read(a[8]))
    return nullptr;
  return call([&](void* s) { return FN(&d0, &d1, x, w0, b0, w1, b1, y, c.ptr, nullptr, 0, s); });
}

// (desc list, x, weight list, bias list, y, config): chains of three
template <typename D, bolt_status (*FN)(int32_t, const D* const*, const void*, const void* const*, const void* const*, void*, const bolt_config*, void*)>
PyObject* chain(PyObject* const* a) {
  constexpr int N = 3;
  for (int i : {0, 2, 3})
    if (!PyList_CheckExact(a[i]) || PyList_GET_SIZE(a[i]) != N) return nullptr;
  D d[N];
  const D* dp[N];
  void *x, *y, *w[N], *b[N];
  Config c;
  if (!half_tensor(a[1], &x) || !half_tensor(a[4], &y) || !c.read(a[5])) return nullptr;
  for (int i = 0; i < N; ++i) {
    dp[i] = &d[i];
    if (!read(PyList_GET_ITEM(a[0], i), &d[i]) || !half_tensor(PyList_GET_ITEM(a[2], i), &w[i]) || !half_tensor_or_none(PyList_GET_ITEM(a[3], i), &b[i]))
      return nullptr;
  }
  return call([&](void* s) { return FN(N, dp, x, w, b, y, c.ptr, s); });
}

#define FASTCALL(NAME, WANT, ...) \
  PyObject* NAME(PyObject*, PyObject* const* a, Py_ssize_t n) { return guarded<&__VA_ARGS__>(a, n, WANT); }
FASTCALL(gemm, 7, single<bolt_gemm_desc, &bolt_gemm_epilogue>)
FASTCALL(conv, 7, single<bolt_conv_desc, &bolt_conv2d_fprop_nhwc>)
FASTCALL(gemm_residual, 9, single_residual<bolt_gemm_desc>)
FASTCALL(conv_residual, 9, single_residual<bolt_conv_desc>)
FASTCALL(gemm_pair, 9, pair<bolt_gemm_desc, &bolt_b2b_gemm>)
FASTCALL(conv_pair, 9, pair<bolt_conv_desc, &bolt_b2b_conv>)
FASTCALL(gemm_chain, 6, chain<bolt_gemm_desc, &bolt_b2b_gemm_chain>)
FASTCALL(conv_chain, 6, chain<bolt_conv_desc, &bolt_b2b_conv_chain>)

// The structure types, once: GemmDesc, ConvDesc, BoltConfig.
PyObject* types(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 3) {
    PyErr_SetString(PyExc_TypeError, "types(GemmDesc, ConvDesc, BoltConfig)");
    return nullptr;
  }
  PyObject** const at[3] = {&g_gemm_desc, &g_conv_desc, &g_config};
  for (int i = 0; i < 3; ++i) {
    Py_INCREF(a[i]);
    *at[i] = a[i];
  }
  Py_RETURN_NONE;
}

#define METHOD(NAME) {#NAME, (PyCFunction)(void (*)(void))NAME, METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {METHOD(gemm), METHOD(conv), METHOD(gemm_residual), METHOD(conv_residual), METHOD(gemm_pair), METHOD(conv_pair),
                           METHOD(gemm_chain), METHOD(conv_chain), METHOD(types), {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void) { return PyModule_Create(&g_module); }
