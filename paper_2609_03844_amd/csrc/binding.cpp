// The Python entry points' call path in native code: argument checks, output tensors, the
// current stream and the libsbw call in one CPython function each.  Small calls are bound by
// the host; through ctypes a watermark call took 6.3 us of host time and a decoding call
// 13 us, most of it attribute reads and argument marshalling.
//
// These functions take the calls whose arguments are what the documentation asks for: plain
// strided tensors on the current device, Python numbers, the current stream.  For anything
// else they return None and do nothing, and the Python code of the entry point handles the
// call or names what is wrong with it.  Otherwise they return the sbw status, or for the
// functions with outputs the tuple of them (the status where it is not SBW_OK).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <exception>

#include "sbw.h"

namespace {

using at::Tensor;

// Keys of a plain tensor on the GPU; a fake, batched, functional or wrapped one has others.
const c10::DispatchKeySet kPlainKeys({c10::DispatchKey::CUDA, c10::DispatchKey::AutogradCUDA,
                                      c10::DispatchKey::ADInplaceOrView,
                                      c10::DispatchKey::AutocastCUDA});

bool plain(const Tensor& t) {
  return t.defined() && t.has_storage() && t.layout() == at::kStrided &&
         (t.key_set().raw_repr() & ~kPlainKeys.raw_repr()) == 0;
}

// The tensor behind a Python object, or null where it is not a plain one of this device,
// type and (for contiguous operands) layout.
const Tensor* tensor_of(PyObject* o, c10::DeviceIndex device) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const Tensor& t = THPVariable_Unpack(o);
  return plain(t) && t.get_device() == device ? &t : nullptr;
}
const Tensor* packed_of(PyObject* o, at::ScalarType type, c10::DeviceIndex device) {
  const Tensor* t = tensor_of(o, device);
  return t != nullptr && t->scalar_type() == type && t->is_contiguous() ? t : nullptr;
}

struct Call {
  const Tensor* matrix = nullptr;    // logits or texts
  int64_t rows, columns, row_stride;
  sbw_dtype_t dtype = SBW_F32;
  const Tensor* context = nullptr;
  int64_t width = 1;
  uint64_t key;
  double gamma, delta = 0.0;
  sbw_seeding_t seeding;
  c10::DeviceIndex device;
};

bool number(PyObject* o, double* out) {
  if (PyFloat_Check(o)) {
    *out = PyFloat_AS_DOUBLE(o);
    return true;
  }
  if (!PyLong_CheckExact(o)) return false;
  *out = PyLong_AsDouble(o);
  if (*out == -1.0 && PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  return true;
}

bool integer(PyObject* o, int64_t* out) {
  if (!PyLong_CheckExact(o)) return false;
  int overflow = 0;
  *out = PyLong_AsLongLongAndOverflow(o, &overflow);
  return overflow == 0;
}

bool key_of(PyObject* o, uint64_t* out) {   // the low 64 bits of any integer
  if (!PyLong_CheckExact(o)) return false;
  *out = PyLong_AsUnsignedLongLongMask(o);
  return true;
}

bool seeding_of(PyObject* o, sbw_seeding_t* out) {
  if (!PyUnicode_CheckExact(o)) return false;
  if (PyUnicode_CompareWithASCIIString(o, "context") == 0) *out = SBW_SEED_CONTEXT;
  else if (PyUnicode_CompareWithASCIIString(o, "self_salt") == 0) *out = SBW_SEED_SELF_SALT;
  else return false;
  return true;
}

// A non-empty matrix with unit stride along its rows, on the current device.
bool matrix_of(PyObject* o, Call* c) {
  if (!THPVariable_CheckExact(o)) return false;
  const Tensor& t = THPVariable_Unpack(o);
  if (!plain(t) || t.dim() != 2 || t.numel() == 0 || t.stride(1) != 1) return false;
  c->device = c10::hip::current_device();
  if (t.get_device() != c->device) return false;
  c->matrix = &t;
  c->rows = t.size(0);
  c->columns = t.size(1);
  c->row_stride = c->rows > 1 ? t.stride(0) : std::max(c->columns, t.stride(0));
  return true;
}

// logits, context, key, gamma, delta, seeding
bool logits_call(PyObject* logits, PyObject* context, PyObject* key, PyObject* gamma, PyObject* delta,
                 PyObject* seeding, Call* c) {
  if (!matrix_of(logits, c)) return false;
  if (c->matrix->scalar_type() == at::kBFloat16) c->dtype = SBW_BF16;
  else if (c->matrix->scalar_type() != at::kFloat) return false;
  c->context = packed_of(context, at::kInt, c->device);
  if (c->context == nullptr || c->context->dim() < 1 || c->context->dim() > 2 ||
      c->context->size(0) != c->rows)
    return false;
  c->width = c->context->dim() == 2 ? c->context->size(1) : 1;
  return key_of(key, &c->key) && number(gamma, &c->gamma) && number(delta, &c->delta) &&
         seeding_of(seeding, &c->seeding);
}

void* stream_of(const Call& c) { return c10::hip::getCurrentHIPStream(c.device).stream(); }

// The caller's output vector, or a new one for None.
bool output_of(PyObject* o, int64_t n, at::ScalarType type, const Call& c, Tensor* out) {
  if (o == Py_None) {
    *out = at::empty({n}, c.matrix->options().dtype(type));
    return plain(*out);
  }
  const Tensor* t = packed_of(o, type, c.device);
  if (t == nullptr || t->dim() != 1 || t->size(0) != n) return false;
  *out = *t;
  return true;
}

PyObject* object_of(PyObject* given, const Tensor& t) {
  if (given != Py_None) {
    Py_INCREF(given);
    return given;
  }
  return THPVariable_Wrap(t);
}

template <typename F>
PyObject* guarded(F&& f) {
  try {
    return f();
  } catch (const std::exception&) {   // the Python path meets the same error and reports it
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

template <typename F>
sbw_status_t unlocked(F&& f) {
  sbw_status_t s;
  Py_BEGIN_ALLOW_THREADS
  s = f();
  Py_END_ALLOW_THREADS
  return s;
}

// Two or three objects in a tuple, built before the launch so that nothing fails after it.
PyObject* tuple_of(PyObject* a, PyObject* b, PyObject* c) {
  PyObject* t = a != nullptr && b != nullptr ? PyTuple_New(c != nullptr ? 3 : 2) : nullptr;
  if (t == nullptr) {
    Py_XDECREF(a);
    Py_XDECREF(b);
    Py_XDECREF(c);
    return nullptr;
  }
  PyTuple_SET_ITEM(t, 0, a);
  PyTuple_SET_ITEM(t, 1, b);
  if (c != nullptr) PyTuple_SET_ITEM(t, 2, c);
  return t;
}

PyObject* outputs_or_status(PyObject* outputs, sbw_status_t s) {
  if (s == SBW_OK) return outputs;
  Py_DECREF(outputs);
  return PyLong_FromLong(s);
}

// watermark(logits, context, key, gamma, delta, seeding, v_offset)
PyObject* watermark(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    Call c;
    int64_t v_offset;
    if (n != 7 || !logits_call(a[0], a[1], a[2], a[3], a[4], a[5], &c) || !integer(a[6], &v_offset))
      Py_RETURN_NONE;
    void* logits = c.matrix->data_ptr();
    const auto* context = static_cast<const int32_t*>(c.context->data_ptr());
    void* stream = stream_of(c);
    return PyLong_FromLong(unlocked([&] {
      return sbw_watermark_shard(logits, c.dtype, c.rows, c.columns, c.row_stride, context, c.width,
                                 v_offset, c.key, c.gamma, static_cast<float>(c.delta), c.seeding, stream);
    }));
  });
}

// watermark_candidates(logits, context, candidates, key, gamma, delta, seeding)
PyObject* watermark_candidates(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    Call c;
    if (n != 7 || !logits_call(a[0], a[1], a[3], a[4], a[5], a[6], &c)) Py_RETURN_NONE;
    const Tensor* cand = packed_of(a[2], at::kInt, c.device);
    if (cand == nullptr || cand->dim() != 2 || cand->size(0) != c.rows) Py_RETURN_NONE;
    void* logits = c.matrix->data_ptr();
    const auto* context = static_cast<const int32_t*>(c.context->data_ptr());
    const auto* ids = static_cast<const int32_t*>(cand->data_ptr());
    const int64_t k = cand->size(1);
    void* stream = stream_of(c);
    return PyLong_FromLong(unlocked([&] {
      return sbw_watermark_candidates(logits, c.dtype, c.rows, c.columns, c.row_stride, ids, k, context,
                                      c.width, c.key, c.gamma, static_cast<float>(c.delta), c.seeding,
                                      stream);
    }));
  });
}

// decode(logits, context, key, gamma, delta, seeding, seeds or None, inv_temperature,
//        tokens, values, workspace, with_values, v_offset): greedy without seeds
PyObject* decode(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    Call c;
    int64_t v_offset;
    double inv_t = 1.0;
    if (n != 13 || !logits_call(a[0], a[1], a[2], a[3], a[4], a[5], &c) || !number(a[7], &inv_t) ||
        !PyBool_Check(a[11]) || !integer(a[12], &v_offset))
      Py_RETURN_NONE;
    const bool sample = a[6] != Py_None;
    const Tensor* seeds = nullptr;
    if (sample) {
      seeds = packed_of(a[6], at::kLong, c.device);
      if (seeds == nullptr || seeds->dim() != 1 || seeds->size(0) != c.rows) Py_RETURN_NONE;
    }
    const bool with_values = a[9] != Py_None || a[11] == Py_True;
    const int64_t need = sbw_watermark_argmax_workspace(c.rows, c.columns);
    Tensor tokens, values, workspace;
    if (!output_of(a[8], c.rows, at::kInt, c, &tokens)) Py_RETURN_NONE;
    if (with_values && !output_of(a[9], c.rows, at::kFloat, c, &values)) Py_RETURN_NONE;
    if (a[10] == Py_None) {
      if (!output_of(Py_None, need, at::kLong, c, &workspace)) Py_RETURN_NONE;
    } else {
      const Tensor* w = packed_of(a[10], at::kLong, c.device);
      if (w == nullptr || w->numel() < need) Py_RETURN_NONE;
      workspace = *w;
    }
    const void* logits = c.matrix->data_ptr();
    const auto* context = static_cast<const int32_t*>(c.context->data_ptr());
    auto* token = static_cast<int32_t*>(tokens.data_ptr());
    auto* value = with_values ? static_cast<float*>(values.data_ptr()) : nullptr;
    auto* partials = static_cast<uint64_t*>(workspace.data_ptr());
    const auto* seed = sample ? static_cast<const uint64_t*>(seeds->data_ptr()) : nullptr;
    void* stream = stream_of(c);
    PyObject* second;
    if (with_values) {
      second = object_of(a[9], values);
    } else {
      Py_INCREF(Py_None);
      second = Py_None;
    }
    PyObject* outputs = tuple_of(object_of(a[8], tokens), second, nullptr);
    if (outputs == nullptr) return nullptr;
    return outputs_or_status(outputs, unlocked([&] {
      const float delta = static_cast<float>(c.delta);
      if (sample)
        return sbw_watermark_sample_shard(logits, c.dtype, c.rows, c.columns, c.row_stride, context, c.width,
                                          v_offset, c.key, c.gamma, delta, c.seeding, seed,
                                          static_cast<float>(inv_t), token, value, partials, stream);
      return sbw_watermark_argmax_shard(logits, c.dtype, c.rows, c.columns, c.row_stride, context, c.width,
                                        v_offset, c.key, c.gamma, delta, c.seeding, token, value, partials,
                                        stream);
    }));
  });
}

// detect(tokens, key, gamma, seeding, width, lengths, ignore_repeated, counts, z[, scored]):
// without `scored` the scored positions are left out (two outputs)
PyObject* detect(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    Call c;
    if (n < 9 || n > 10 || !matrix_of(a[0], &c) || c.matrix->scalar_type() != at::kInt || !key_of(a[1], &c.key) ||
        !number(a[2], &c.gamma) || !seeding_of(a[3], &c.seeding) || !integer(a[4], &c.width) ||
        !PyBool_Check(a[6]))
      Py_RETURN_NONE;
    const Tensor* lengths = nullptr;
    if (a[5] != Py_None) {
      lengths = packed_of(a[5], at::kInt, c.device);
      if (lengths == nullptr || lengths->dim() != 1 || lengths->size(0) != c.rows) Py_RETURN_NONE;
    }
    const bool with_scored = n == 10;
    Tensor counts, scored, z;
    if (!output_of(a[7], c.rows, at::kInt, c, &counts) ||
        (with_scored && !output_of(a[9], c.rows, at::kInt, c, &scored)) ||
        !output_of(a[8], c.rows, at::kDouble, c, &z))
      Py_RETURN_NONE;
    const auto* tokens = static_cast<const int32_t*>(c.matrix->data_ptr());
    const auto* length = lengths != nullptr ? static_cast<const int32_t*>(lengths->data_ptr()) : nullptr;
    auto* count = static_cast<int32_t*>(counts.data_ptr());
    auto* positions = with_scored ? static_cast<int32_t*>(scored.data_ptr()) : nullptr;
    auto* score = static_cast<double*>(z.data_ptr());
    const uint32_t flags = a[6] == Py_True ? SBW_DETECT_IGNORE_REPEATED : 0u;
    void* stream = stream_of(c);
    PyObject* first = object_of(a[7], counts);
    PyObject* last = object_of(a[8], z);
    PyObject* outputs = with_scored ? tuple_of(first, object_of(a[9], scored), last)
                                    : tuple_of(first, last, nullptr);
    if (outputs == nullptr) return nullptr;
    return outputs_or_status(outputs, unlocked([&] {
      return sbw_detect_ex(tokens, c.rows, c.columns, c.row_stride, length, c.width, c.key, c.gamma,
                           c.seeding, flags, count, positions, score, stream);
    }));
  });
}

PyCFunction fast(PyObject* (*f)(PyObject*, PyObject* const*, Py_ssize_t)) {
  return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f));
}

PyMethodDef methods[] = {
    {"watermark", fast(watermark), METH_FASTCALL, nullptr},
    {"watermark_candidates", fast(watermark_candidates), METH_FASTCALL, nullptr},
    {"decode", fast(decode), METH_FASTCALL, nullptr},
    {"detect", fast(detect), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
