// What the sources of the Python binding's extension module share: the entry points of the loaded library, argument
// conversion and error reporting.
#pragma once
#include <Python.h>
#include <dlfcn.h>

#include <cmath>
#include <vector>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "decoder.h"
#include "seco.h"

namespace seco_ext {

using at::Tensor;

#define SECO_ENTRIES(X)                                                                                             \
  X(seco_chunk_attn_fwd) X(seco_chunk_attn_bwd) X(seco_chunk_attn_bwd_noalloc) X(spaco_chunk_attn_bwd)              \
  X(spaco_chunk_attn_bwd_sparse_dq) X(seco_chunk_attn_bwd_gather) X(spaco_chunk_attn_bwd_gather)                    \
  X(seco_workspace_bytes) X(kvgrad_zero) X(kvgrad_accumulate) X(kv_append) X(kvgrad_readout) X(kv_append_rope)      \
  X(kvgrad_readout_rope) X(rope_rotate) X(dec_add_rmsnorm) X(dec_rmsnorm_bwd) X(dec_silu) X(dec_silu_bwd)             \
  X(dec_cross_entropy) X(dec_cross_entropy_both) X(dec_embedding_bwd) X(dec_gemm_supported) X(dec_gemm) X(dec_gemm_grads) X(dec_gemm_first_grads)      \
  X(dec_rope_qkv) X(dec_gemm_qkv) X(dec_gain_sums) X(dec_split_columns) X(dec_embed_rmsnorm_checked)
struct Lib {
#define X(name) decltype(&::name) name = nullptr;
  SECO_ENTRIES(X)
#undef X
};
inline Lib lib;
inline PyObject* g_error = nullptr;   // SecoError(status, where)

// an error that is already set in the interpreter
struct Raised {};
[[noreturn]] inline void raise(PyObject* type, const char* msg) {
  PyErr_SetString(type, msg);
  throw Raised{};
}
inline void check(int status, const char* where) {
  if (status == SECO_OK) return;
  PyObject* e = PyObject_CallFunction(g_error, "is", status, where);
  if (e) {
    PyErr_SetObject(g_error, e);
    Py_DECREF(e);
  }
  throw Raised{};
}

inline const Tensor& tensor(PyObject* o) {
  if (!THPVariable_Check(o)) raise(PyExc_TypeError, "expected a torch tensor");
  return THPVariable_Unpack(o);
}
inline const Tensor* opt_tensor(PyObject* o) { return o == Py_None ? nullptr : &tensor(o); }
inline int64_t integer(PyObject* o) {
  if (PyLong_Check(o)) {
    const int64_t v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw Raised{};
    return v;
  }
  PyObject* n = PyNumber_Long(o);
  if (!n) throw Raised{};
  const int64_t v = PyLong_AsLongLong(n);
  Py_DECREF(n);
  if (v == -1 && PyErr_Occurred()) throw Raised{};
  return v;
}
inline int32_t int32(PyObject* o) { return (int32_t)integer(o); }
inline double real(PyObject* o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw Raised{};
  return v;
}
inline std::vector<float> floats(PyObject* o) {
  PyObject* s = PySequence_Fast(o, "expected a sequence of floats");
  if (!s) throw Raised{};
  std::vector<float> v((size_t)PySequence_Fast_GET_SIZE(s));
  for (size_t i = 0; i < v.size(); ++i) {
    v[i] = (float)PyFloat_AsDouble(PySequence_Fast_GET_ITEM(s, (Py_ssize_t)i));
    if (PyErr_Occurred()) {
      Py_DECREF(s);
      throw Raised{};
    }
  }
  Py_DECREF(s);
  return v;
}
inline void* stream(PyObject* o) {
  if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
  PyObject* n = PyObject_HasAttrString(o, "cuda_stream") ? PyObject_GetAttrString(o, "cuda_stream") : PyNumber_Long(o);
  if (!n) throw Raised{};
  void* s = PyLong_AsVoidPtr(n);
  Py_DECREF(n);
  if (!s && PyErr_Occurred()) throw Raised{};
  return s;
}

inline int dtype_code(const Tensor& t) {
  if (t.scalar_type() == at::kBFloat16) return SECO_BF16;
  if (t.scalar_type() == at::kFloat) return SECO_F32;
  raise(PyExc_TypeError, "unsupported dtype: expected bfloat16 or float32");
}
inline void strides3(const Tensor& t, int64_t out[3]) {
  if (t.dim() != 4 || t.stride(3) != 1)
    raise(PyExc_ValueError, "expected a [batch, head, row, head_dim] tensor with contiguous head_dim");
  for (int i = 0; i < 3; ++i) out[i] = t.stride(i);
}
inline void* ptr(const Tensor* t) { return t ? t->data_ptr() : nullptr; }
inline void* ptr(const Tensor& t) { return t.data_ptr(); }
inline float* fptr(const Tensor* t) { return static_cast<float*>(ptr(t)); }
inline float* fptr(const Tensor& t) { return static_cast<float*>(t.data_ptr()); }

inline Tensor like(const Tensor& t) { return at::empty_strided(t.sizes(), t.strides(), t.options().requires_grad(false)); }
inline Tensor bytes(int64_t n, const Tensor& t) { return at::empty({n}, t.options().dtype(at::kByte).requires_grad(false)); }
inline size_t nbytes(const Tensor& t) { return (size_t)t.numel() * t.element_size(); }

// Scratch of one call, which works on it in stream s: taken from that stream's memory, whatever stream is current, since it
// is given back as soon as the call is enqueued.
inline Tensor scratch(int64_t n, const Tensor& t, void* s) {
  const auto device = t.device().index();
  if (!t.is_cuda() || s == c10::hip::getCurrentHIPStream(device).stream()) return bytes(n, t);
  struct Back {
    c10::hip::HIPStream to;
    ~Back() { c10::hip::setCurrentHIPStream(to); }
  } back{c10::hip::getCurrentHIPStream(device)};
  c10::hip::setCurrentHIPStream(s ? c10::hip::getStreamFromExternal(static_cast<hipStream_t>(s), device)
                                  : c10::hip::getDefaultHIPStream(device));
  return bytes(n, t);
}

inline size_t workspace(const seco_desc& d, int op) {
  const size_t n = lib.seco_workspace_bytes(&d, op);
  if (n == (size_t)-1) check(SECO_ERR_SHAPE, "seco_workspace_bytes");
  return n;
}

template <PyObject* (*F)(PyObject* const*), int N>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != N) {
    PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", N, n);
    return nullptr;
  }
  try {
    return F(args);
  } catch (const Raised&) {
    return nullptr;
  }
  END_HANDLE_TH_ERRORS
}
#define SECO_METHOD(name, f, n) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(&seco_ext::entry<f, n>)), METH_FASTCALL, nullptr}

extern PyMethodDef step_methods[];   // the training step (chunk_step_ext.cpp)

}  // namespace seco_ext
