// The step calls of the Python binding for their ordinary arguments: tensors of exactly the layout that the shape describes, in
// GPU memory.  What the binding checks attribute by attribute in Python and marshals through ctypes is read here from the tensors
// themselves: 7 -> 3.4 us of host time a call (a full and two cached steps of 2 x 256 x 64 float32 back to back: 20-21 -> 10-12 us).
// Anything else -- another layout, a subclass, a tensor without storage, a wrong type -- returns None, and the binding goes on in
// Python, which accepts or refuses it with its own message.  No arithmetic and no kernels here.
#include <Python.h>

#include <cstring>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../../include/svdcache.h"

namespace {

PyTypeObject* shape_type;       // binding.Shape

// addresses inside the library that the binding loaded
struct Library {
  decltype(&svdcache_packed_basis_bytes) packed_basis_bytes;
  decltype(&svdcache_packed_state_bytes) packed_state_bytes;
  decltype(&svdcache_full_step) full_step;
  decltype(&svdcache_full_step_residual_ema) full_step_residual_ema;
  decltype(&svdcache_full_step_packed) full_step_packed;
  decltype(&svdcache_forecast) forecast;
  decltype(&svdcache_forecast_packed) forecast_packed;
  decltype(&svdcache_forecast_combine) forecast_combine;
} lib;

// The arguments of one call; `ok` falls when one of them is not ordinary.
struct Args {
  svdc_shape s;
  bool ok = false;

  explicit Args(PyObject* shape) {
    Py_buffer view;
    if (Py_TYPE(shape) != shape_type || PyObject_GetBuffer(shape, &view, PyBUF_SIMPLE) != 0) return;
    if (view.len == (Py_ssize_t)sizeof(s)) {
      std::memcpy(&s, view.buf, sizeof(s));
      ok = s.dtype == SVDC_F32 || s.dtype == SVDC_BF16;
    }
    PyBuffer_Release(&view);
  }
  const at::Tensor* tensor(PyObject* o) {
    if (ok && THPVariable_CheckExact(o)) {
      const at::Tensor& t = THPVariable_Unpack(o);
      if (t.is_cuda()) return &t;
    }
    ok = false;
    return nullptr;
  }
  void* features(PyObject* o) {             // [B, N, D] with the strides of the shape
    const at::Tensor* t = tensor(o);
    if (!t) return nullptr;
    ok = t->scalar_type() == (s.dtype == SVDC_F32 ? at::kFloat : at::kBFloat16) && t->dim() == 3 && t->size(0) == s.B &&
         t->size(1) == s.N && t->size(2) == s.D && t->stride(0) == s.block_stride && t->stride(1) == s.ldf && t->stride(2) == 1;
    return ok ? t->data_ptr() : nullptr;
  }
  void* dense(PyObject* o, int64_t count) { // contiguous float32
    const at::Tensor* t = tensor(o);
    if (!t) return nullptr;
    ok = t->scalar_type() == at::kFloat && t->is_contiguous() && t->numel() == count;
    return ok ? t->data_ptr() : nullptr;
  }
  void* basis(PyObject* o) { return dense(o, (int64_t)s.B * s.D * s.k); }
  void* state(PyObject* o) { return dense(o, (int64_t)s.B * s.N * s.k); }
  void* bytes(PyObject* o, size_t need, size_t* have = nullptr) {
    const at::Tensor* t = tensor(o);
    if (!t) return nullptr;
    const size_t n = (size_t)t->numel() * t->element_size();
    ok = need > 0 && t->is_contiguous() && n >= need;
    if (have) *have = n;
    return ok ? t->data_ptr() : nullptr;
  }
  void* packed_basis(PyObject* o) { return ok ? bytes(o, lib.packed_basis_bytes(&s)) : nullptr; }
  void* optional(PyObject* o, void* (Args::*get)(PyObject*)) { return o == Py_None ? nullptr : (this->*get)(o); }
  // Python's own numbers only: the conversion of any other object runs its code, which may change the list that is being read
  float number(PyObject* o) {
    ok = ok && (PyFloat_CheckExact(o) || PyLong_CheckExact(o));
    const double x = ok ? PyFloat_AsDouble(o) : 0.0;
    if (x == -1.0 && PyErr_Occurred()) ok = false;         // an integer beyond the doubles
    return (float)x;
  }
  int32_t flag(PyObject* o) {
    ok = ok && (PyBool_Check(o) || PyLong_CheckExact(o));
    return ok && PyObject_IsTrue(o) > 0;
  }
};

// Runs `body(args)`, which returns a call to make without the interpreter lock; None where the arguments are not ordinary.
template <typename Body>
PyObject* call(PyObject* const* argv, Py_ssize_t argc, Py_ssize_t want, Body body) {
  int32_t rc = 0;
  bool made = false;
  if (argc == want && lib.full_step) {
    try {
      Args a(argv[0]);
      auto launch = body(a);
      if (a.ok) {
        void* stream = c10::hip::getCurrentHIPStream().stream();
        Py_BEGIN_ALLOW_THREADS
        rc = launch(stream);
        Py_END_ALLOW_THREADS
        made = true;
      }
    } catch (const std::exception&) {       // a tensor without storage or strides
    }
  }
  if (made) return PyLong_FromLong(rc);
  PyErr_Clear();
  Py_RETURN_NONE;
}

PyObject* full_step(PyObject*, PyObject* const* v, Py_ssize_t n) {          // shape F V packed R S C alpha init
  return call(v, n, 9, [&](Args& a) {
    void *F = a.features(v[1]), *V = a.basis(v[2]), *P = a.optional(v[3], &Args::packed_basis), *R = a.features(v[4]),
         *S = a.state(v[5]), *C = a.optional(v[6], &Args::state);
    const float alpha = a.number(v[7]);
    const int32_t init = a.flag(v[8]);
    return [=, &a](void* st) { return lib.full_step(&a.s, F, (float*)V, P, R, (float*)S, (float*)C, alpha, init, st); };
  });
}
PyObject* full_step_residual_ema(PyObject*, PyObject* const* v, Py_ssize_t n) {   // shape F V packed R_prev R S C alpha alpha_r init
  return call(v, n, 11, [&](Args& a) {
    void *F = a.features(v[1]), *V = a.basis(v[2]), *P = a.optional(v[3], &Args::packed_basis),
         *Rp = a.optional(v[4], &Args::features), *R = a.features(v[5]), *S = a.state(v[6]), *C = a.optional(v[7], &Args::state);
    const float alpha = a.number(v[8]), alpha_r = a.number(v[9]);
    const int32_t init = a.flag(v[10]);
    return [=, &a](void* st) {
      return lib.full_step_residual_ema(&a.s, F, (float*)V, P, Rp, R, (float*)S, (float*)C, alpha, alpha_r, init, st);
    };
  });
}
PyObject* full_step_packed(PyObject*, PyObject* const* v, Py_ssize_t n) {   // shape F V packed R S C S_packed alpha init
  return call(v, n, 10, [&](Args& a) {
    size_t have = 0;
    void *F = a.features(v[1]), *V = a.basis(v[2]), *P = a.packed_basis(v[3]), *R = a.features(v[4]), *S = a.state(v[5]),
         *C = a.optional(v[6], &Args::state), *Sp = a.ok ? a.bytes(v[7], lib.packed_state_bytes(&a.s), &have) : nullptr;
    const float alpha = a.number(v[8]);
    const int32_t init = a.flag(v[9]);
    return [=, &a](void* st) {
      return lib.full_step_packed(&a.s, F, (float*)V, P, R, (float*)S, (float*)C, Sp, have, alpha, init, st);
    };
  });
}
PyObject* forecast(PyObject*, PyObject* const* v, Py_ssize_t n) {           // shape S V packed R Fhat
  return call(v, n, 6, [&](Args& a) {
    void *S = a.state(v[1]), *V = a.basis(v[2]), *P = a.optional(v[3], &Args::packed_basis), *R = a.features(v[4]),
         *Fhat = a.features(v[5]);
    return [=, &a](void* st) { return lib.forecast(&a.s, (float*)S, (float*)V, P, R, Fhat, st); };
  });
}
PyObject* forecast_packed(PyObject*, PyObject* const* v, Py_ssize_t n) {    // shape S_packed packed R Fhat
  return call(v, n, 5, [&](Args& a) {
    void *Sp = a.ok ? a.bytes(v[1], lib.packed_state_bytes(&a.s)) : nullptr, *P = a.packed_basis(v[2]), *R = a.features(v[3]),
         *Fhat = a.features(v[4]);
    return [=, &a](void* st) { return lib.forecast_packed(&a.s, Sp, P, R, Fhat, st); };
  });
}
PyObject* forecast_combine(PyObject*, PyObject* const* v, Py_ssize_t n) {   // shape S_list weights V packed R X Out
  const float* S[SVDC_MAX_STATES];
  float w[SVDC_MAX_STATES];
  return call(v, n, 8, [&](Args& a) {
    const bool lists = PyList_CheckExact(v[1]) && PyList_CheckExact(v[2]);
    const Py_ssize_t m = lists ? PyList_GET_SIZE(v[1]) : 0;
    if (m < 1 || m > SVDC_MAX_STATES || PyList_GET_SIZE(v[2]) != m) a.ok = false;
    for (Py_ssize_t i = 0; a.ok && i < m; ++i) {
      S[i] = (const float*)a.state(PyList_GET_ITEM(v[1], i));
      w[i] = a.ok ? a.number(PyList_GET_ITEM(v[2], i)) : 0.f;
    }
    void *V = a.ok ? a.basis(v[3]) : nullptr, *P = a.optional(v[4], &Args::packed_basis), *R = a.features(v[5]),
         *X = a.optional(v[6], &Args::features), *Out = a.features(v[7]);
    return [=, &a, &S, &w](void* st) { return lib.forecast_combine(&a.s, (int32_t)m, S, w, (float*)V, P, R, X, Out, st); };
  });
}

// bind(addresses of the loaded library's functions by name, the class of the shape)
PyObject* bind(PyObject*, PyObject* args) {
  PyObject *addresses, *type;
  if (!PyArg_ParseTuple(args, "O!O!", &PyDict_Type, &addresses, &PyType_Type, &type)) return nullptr;
  auto get = [&](const char* name) -> void* {
    PyObject* o = PyDict_GetItemString(addresses, name);
    return o ? PyLong_AsVoidPtr(o) : nullptr;
  };
  Library l;
#define SVDC_BIND(f) l.f = reinterpret_cast<decltype(l.f)>(get("svdcache_" #f))
  SVDC_BIND(packed_basis_bytes);
  SVDC_BIND(packed_state_bytes);
  SVDC_BIND(full_step);
  SVDC_BIND(full_step_residual_ema);
  SVDC_BIND(full_step_packed);
  SVDC_BIND(forecast);
  SVDC_BIND(forecast_packed);
  SVDC_BIND(forecast_combine);
#undef SVDC_BIND
  if (PyErr_Occurred()) return nullptr;
  if (!l.packed_basis_bytes || !l.packed_state_bytes || !l.full_step || !l.full_step_residual_ema || !l.full_step_packed ||
      !l.forecast || !l.forecast_packed || !l.forecast_combine) {
    PyErr_SetString(PyExc_ValueError, "bind: an address is missing");
    return nullptr;
  }
  lib = l;
  Py_INCREF(type);
  Py_XDECREF(shape_type);
  shape_type = reinterpret_cast<PyTypeObject*>(type);
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"full_step", (PyCFunction)(void (*)())full_step, METH_FASTCALL, nullptr},
                         {"full_step_residual_ema", (PyCFunction)(void (*)())full_step_residual_ema, METH_FASTCALL, nullptr},
                         {"full_step_packed", (PyCFunction)(void (*)())full_step_packed, METH_FASTCALL, nullptr},
                         {"forecast", (PyCFunction)(void (*)())forecast, METH_FASTCALL, nullptr},
                         {"forecast_packed", (PyCFunction)(void (*)())forecast_packed, METH_FASTCALL, nullptr},
                         {"forecast_combine", (PyCFunction)(void (*)())forecast_combine, METH_FASTCALL, nullptr},
                         {"bind", bind, METH_VARARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fast_calls", "Step calls with ordinary arguments.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fast_calls(void) { return PyModule_Create(&module); }
