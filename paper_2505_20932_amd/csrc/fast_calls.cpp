// The binding's most frequent calls without ctypes: a Python extension module that reads the tensors' pointers, sizes
// and strides directly, takes the current stream and calls the C entry point.
//
// Why: a call through ctypes takes 9 to 10 us of host time (a dozen tensor attributes and argument conversions through
// Python objects), the launch itself about 3.5; where kernels are shorter than that - a decoding step, one image -
// the host sets the pace.
//
// Every function returns True when the call was made and returned CWAC_OK, and False otherwise: an argument that is
// not exactly what the call documents, or an error status (nothing was launched then).  The caller goes on with
// the ctypes form, which makes the checks again and raises.  So nothing is refused or accepted here that was not before.
// CWAC_E_LAUNCH alone is raised from here: the runtime's error is taken with the status, and a second call could pass.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/TensorBase.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "cwac.h"

namespace {

// The entry points of the library that the ctypes binding loaded (`bind`), and its structure type for parameters.
struct Entries {
  decltype(&::cwac_quantize_act) quantize_act;
  decltype(&::cwac_quantize_rows_sym) quantize_rows_sym;
  decltype(&::qlinear_cwac_forward) forward;
  decltype(&::qlinear_cwac_forward_table) forward_table;
  decltype(&::qlinear_cwac_forward_fixed_point) forward_fixed_point;
  decltype(&::qconv2d_cwac_forward) conv2d;
  decltype(&::qlinear_w4a16_cwac_forward) w4a16;
} g;
PyObject *g_qparams_type = nullptr, *g_check = nullptr;  // the binding's structure type and its check of a status

// What a call is given, checked one by one; `ok` stays true while everything is what the call documents.
struct Args {
  bool ok = true;

  // a plain tensor on the device
  const at::TensorBase *tensor(PyObject *o) {
    if (!ok || !THPVariable_CheckExact(o)) return fail();
    const at::TensorBase &t = THPVariable_Unpack(o);
    return t.is_cuda() ? &t : fail();
  }
  const at::TensorBase *typed(PyObject *o, at::ScalarType type) {
    const at::TensorBase *t = tensor(o);
    return t && t->scalar_type() == type ? t : fail();
  }
  // ... of two dimensions whose rows are contiguous
  const at::TensorBase *matrix(PyObject *o, at::ScalarType type) {
    const at::TensorBase *t = typed(o, type);
    return t && t->dim() == 2 && t->stride(1) == 1 ? t : fail();
  }
  // pointer of a tensor, NULL for None (elements are not looked at, as in the ctypes form)
  void *pointer(PyObject *o) {
    if (o == Py_None) return nullptr;
    const at::TensorBase *t = tensor(o);
    return t ? t->data_ptr() : nullptr;
  }
  long long integer(PyObject *o) {
    if (!PyLong_CheckExact(o)) return ok = false, 0;
    int overflow = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow || v > INT32_MAX || v < INT32_MIN) ok = false;
    return v;
  }
  float number(PyObject *o) {
    if (!PyFloat_CheckExact(o)) return ok = false, 0.0f;
    return (float)PyFloat_AS_DOUBLE(o);
  }
  // the caller's ctypes structure, read in place (the call copies it)
  const cwac_qparams *qparams(PyObject *o, bool nullable) {
    if (nullable && o == Py_None) return nullptr;
    Py_buffer view;
    if (!ok || (PyObject *)Py_TYPE(o) != g_qparams_type || PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) return fail_qp();
    if (view.len == (Py_ssize_t)sizeof(cwac_qparams))
      memcpy(&qp, view.buf, sizeof qp);
    else
      ok = false;
    PyBuffer_Release(&view);
    return &qp;
  }
  // None: the current stream of the current device
  void *stream(PyObject *o) {
    if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
    PyObject *v = PyObject_GetAttrString(o, "cuda_stream");
    void *s = v && PyLong_Check(v) ? PyLong_AsVoidPtr(v) : (ok = false, nullptr);
    Py_XDECREF(v);
    return s;
  }

 private:
  cwac_qparams qp;
  const at::TensorBase *fail() { return ok = false, nullptr; }
  const cwac_qparams *fail_qp() { return ok = false, nullptr; }
};

// A matrix of one row counts as one with the smallest pitch that holds it.
int64_t pitch(const at::TensorBase &t) {
  return t.size(0) > 1 ? t.stride(0) : (t.stride(0) > t.size(1) ? t.stride(0) : t.size(1));
}
bool same_shape(const at::TensorBase &a, const at::TensorBase &b) { return a.size(0) == b.size(0) && a.size(1) == b.size(1); }

// `f` for the entry point `name`: its result, False for tensors without storage (torch throws), an exception
// for a launch that failed.
struct LaunchFailed {};
template <typename F>
PyObject *guarded(const char *name, F &&f) {
  bool done = false;
  try {
    done = f();
  } catch (const LaunchFailed &) {
    PyErr_Clear();
    return PyObject_CallFunction(g_check, "is", (int)CWAC_E_LAUNCH, name);  // raises
  } catch (...) {
    done = false;
  }
  if (PyErr_Occurred()) PyErr_Clear();
  return PyBool_FromLong(done);
}

// Runs `call` with Python's lock released.
struct Unlock {
  PyThreadState *state = PyEval_SaveThread();
  ~Unlock() { PyEval_RestoreThread(state); }
};
template <typename F>
bool unlocked(F &&call) {
  const cwac_status st = [&] {
    Unlock u;
    return call();
  }();
  if (st == CWAC_E_LAUNCH) throw LaunchFailed();
  return st == CWAC_OK;
}

constexpr auto kI8 = at::kChar;
constexpr auto kF32 = at::kFloat;

// (x, s, z, q, stream)
PyObject *py_quantize_act(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded("cwac_quantize_act", [&] {
    Args v;
    if (n != 5) return false;
    const at::TensorBase *x = v.matrix(a[0], kF32), *q = v.matrix(a[3], kI8);
    const float s = v.number(a[1]);
    const int32_t z = (int32_t)v.integer(a[2]);
    if (!v.ok || !same_shape(*x, *q)) return false;
    void *st = v.stream(a[4]);
    const float *xp = static_cast<const float *>(x->data_ptr());
    int8_t *qp = static_cast<int8_t *>(q->data_ptr());
    const int64_t rows = x->size(0), k = x->size(1), lx = pitch(*x), lq = pitch(*q);
    if (!v.ok || k > INT32_MAX) return false;
    return unlocked([&] { return g.quantize_act(xp, lx, rows, (int32_t)k, s, z, qp, lq, st); });
  });
}

// (x, scale, q, stream)
PyObject *py_quantize_rows_sym(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded("cwac_quantize_rows_sym", [&] {
    Args v;
    if (n != 4) return false;
    const at::TensorBase *x = v.matrix(a[0], kF32), *scale = v.typed(a[1], kF32), *q = v.matrix(a[2], kI8);
    if (!v.ok || !same_shape(*x, *q) || scale->numel() != x->size(0)) return false;
    void *st = v.stream(a[3]);
    const float *xp = static_cast<const float *>(x->data_ptr());
    float *sp = static_cast<float *>(scale->data_ptr());
    int8_t *qp = static_cast<int8_t *>(q->data_ptr());
    const int64_t rows = x->size(0), k = x->size(1), lx = pitch(*x), lq = pitch(*q);
    if (!v.ok || k > INT32_MAX) return false;
    return unlocked([&] { return g.quantize_rows_sym(xp, lx, rows, (int32_t)k, sp, qp, lq, st); });
  });
}

// x_q [m, k] and w_q [n, k] of a linear layer and its output [m, n] of the given type
struct Linear {
  const int8_t *x, *w;
  void *out;
  int64_t m, ldx, ldw, ldo;
  int32_t n, k;
  bool take(Args &v, PyObject *xo, PyObject *wo, PyObject *oo, at::ScalarType type) {
    const at::TensorBase *xt = v.matrix(xo, kI8), *wt = v.matrix(wo, kI8), *ot = v.matrix(oo, type);
    if (!v.ok || xt->size(1) != wt->size(1) || ot->size(0) != xt->size(0) || ot->size(1) != wt->size(0) ||
        wt->size(0) > INT32_MAX || xt->size(1) > INT32_MAX)
      return false;
    x = static_cast<const int8_t *>(xt->data_ptr());
    w = static_cast<const int8_t *>(wt->data_ptr());
    out = ot->data_ptr();
    m = xt->size(0), n = (int32_t)wt->size(0), k = (int32_t)xt->size(1);
    ldx = pitch(*xt), ldw = pitch(*wt), ldo = pitch(*ot);
    return true;
  }
};

at::ScalarType out_type(long long kind) {
  return kind == CWAC_OUT_INT8 ? at::kChar : kind == CWAC_OUT_FP32 ? at::kFloat : kind == CWAC_OUT_INT32 ? at::kInt : at::kDouble;
}

// (x_q, w_q, qp, mult, offset, fbias, s_x_row, out_kind, out, stream)
PyObject *py_forward(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded("qlinear_cwac_forward", [&] {
    Args v;
    if (n != 10) return false;
    const int32_t kind = (int32_t)v.integer(a[7]);
    Linear l;
    if (!v.ok || out_type(kind) == at::kDouble || !l.take(v, a[0], a[1], a[8], out_type(kind))) return false;
    const cwac_qparams *qp = v.qparams(a[2], true);
    const float *mult = static_cast<const float *>(v.pointer(a[3])), *fbias = static_cast<const float *>(v.pointer(a[5])),
                *rows = static_cast<const float *>(v.pointer(a[6]));
    const int32_t *offset = static_cast<const int32_t *>(v.pointer(a[4]));
    void *st = v.stream(a[9]);
    if (!v.ok) return false;
    return unlocked([&] {
      return g.forward(l.x, l.ldx, l.w, l.ldw, l.m, l.n, l.k, qp, mult, offset, fbias, rows, kind, l.out, l.ldo, st);
    });
  });
}

// (x_q, w_q, qp, mult, offset, table, out, stream)
PyObject *py_forward_table(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded("qlinear_cwac_forward_table", [&] {
    Args v;
    Linear l;
    if (n != 8 || !l.take(v, a[0], a[1], a[6], kI8)) return false;
    const cwac_qparams *qp = v.qparams(a[2], false);
    const float *mult = static_cast<const float *>(v.pointer(a[3]));
    const int32_t *offset = static_cast<const int32_t *>(v.pointer(a[4]));
    const at::TensorBase *table = v.typed(a[5], kI8);
    if (!v.ok || table->numel() != 256) return false;
    const int8_t *tp = static_cast<const int8_t *>(table->data_ptr());
    void *st = v.stream(a[7]);
    if (!v.ok) return false;
    return unlocked([&] {
      return g.forward_table(l.x, l.ldx, l.w, l.ldw, l.m, l.n, l.k, qp, mult, offset, tp, static_cast<int8_t *>(l.out), l.ldo, st);
    });
  });
}

// (x_q, w_q, qp, m0, shift, offset, out, stream)
PyObject *py_forward_fixed_point(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded("qlinear_cwac_forward_fixed_point", [&] {
    Args v;
    Linear l;
    if (n != 8 || !l.take(v, a[0], a[1], a[6], kI8)) return false;
    const cwac_qparams *qp = v.qparams(a[2], false);
    const at::TensorBase *m0 = v.typed(a[3], at::kInt), *shift = v.typed(a[4], at::kInt);
    const int32_t *offset = static_cast<const int32_t *>(v.pointer(a[5]));
    void *st = v.stream(a[7]);
    if (!v.ok) return false;
    const int32_t *mp = static_cast<const int32_t *>(m0->data_ptr()), *sp = static_cast<const int32_t *>(shift->data_ptr());
    return unlocked([&] {
      return g.forward_fixed_point(l.x, l.ldx, l.w, l.ldw, l.m, l.n, l.k, qp, mp, sp, offset, static_cast<int8_t *>(l.out), l.ldo,
                                   st);
    });
  });
}

// (x_q, w_q, stride, pad, qp, mult, offset, fbias, out_kind, out, stream)
PyObject *py_conv2d(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded("qconv2d_cwac_forward", [&] {
    Args v;
    if (n != 11) return false;
    const at::TensorBase *x = v.typed(a[0], kI8), *w = v.typed(a[1], kI8);
    const int32_t stride = (int32_t)v.integer(a[2]), pad = (int32_t)v.integer(a[3]), kind = (int32_t)v.integer(a[8]);
    if (!v.ok || out_type(kind) == at::kDouble || x->dim() != 4 || w->dim() != 4 || !x->is_contiguous() || !w->is_contiguous() ||
        x->size(3) != w->size(3))
      return false;
    const at::TensorBase *out = v.matrix(a[9], out_type(kind));
    if (!v.ok || out->size(1) != w->size(0)) return false;
    int32_t d[7];  // batch, h, w, c_in; c_out, kh, kw
    for (int i = 0; i < 7; ++i) {
      const int64_t s = i < 4 ? x->size(i) : w->size(i - 4);
      if (s > INT32_MAX) return false;
      d[i] = (int32_t)s;
    }
    const cwac_qparams *qp = v.qparams(a[4], false);
    const float *mult = static_cast<const float *>(v.pointer(a[5])), *fbias = static_cast<const float *>(v.pointer(a[7]));
    const int32_t *offset = static_cast<const int32_t *>(v.pointer(a[6]));
    void *st = v.stream(a[10]);
    if (!v.ok) return false;
    const int8_t *xp = static_cast<const int8_t *>(x->data_ptr()), *wp = static_cast<const int8_t *>(w->data_ptr());
    void *op = out->data_ptr();
    const int64_t ldo = pitch(*out);
    return unlocked([&] {
      return g.conv2d(xp, wp, d[0], d[1], d[2], d[3], d[4], d[5], d[6], stride, pad, qp, mult, offset, fbias, kind, op, ldo, st);
    });
  });
}

// (x, packed_w, packed_sz, n, mult, fbias, out, stream)
PyObject *py_w4a16(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded("qlinear_w4a16_cwac_forward", [&] {
    Args v;
    if (n != 8) return false;
    const at::TensorBase *x = v.matrix(a[0], at::kHalf), *out = v.tensor(a[6]);
    const long long channels = v.integer(a[3]);
    if (!v.ok || (out->scalar_type() != at::kHalf && out->scalar_type() != kF32)) return false;
    out = v.matrix(a[6], out->scalar_type());
    if (!v.ok || out->size(0) != x->size(0) || out->size(1) != channels || x->size(1) > INT32_MAX) return false;
    const void *pw = v.pointer(a[1]);
    const uint32_t *sz = static_cast<const uint32_t *>(v.pointer(a[2]));
    const float *mult = static_cast<const float *>(v.pointer(a[4])), *fbias = static_cast<const float *>(v.pointer(a[5]));
    void *st = v.stream(a[7]);
    if (!v.ok) return false;
    const int32_t kind = out->scalar_type() == at::kHalf ? CWAC_OUT_FP16 : CWAC_OUT_FP32;
    const uint16_t *xp = static_cast<const uint16_t *>(x->data_ptr());
    void *op = out->data_ptr();
    const int64_t m = x->size(0), k = x->size(1), ldx = pitch(*x), ldo = pitch(*out);
    return unlocked([&] {
      return g.w4a16(xp, ldx, pw, sz, m, (int32_t)channels, (int32_t)k, mult, fbias, kind, op, ldo, st);
    });
  });
}

// (the type of cwac_qparams, {entry point: address}, the check of a status)
PyObject *py_bind(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 3 || !PyDict_Check(a[1])) return PyErr_Format(PyExc_TypeError, "bind(type, addresses, check)");
  const struct {
    const char *name;
    void **slot;
  } slots[] = {{"cwac_quantize_act", (void **)&g.quantize_act},
               {"cwac_quantize_rows_sym", (void **)&g.quantize_rows_sym},
               {"qlinear_cwac_forward", (void **)&g.forward},
               {"qlinear_cwac_forward_table", (void **)&g.forward_table},
               {"qlinear_cwac_forward_fixed_point", (void **)&g.forward_fixed_point},
               {"qconv2d_cwac_forward", (void **)&g.conv2d},
               {"qlinear_w4a16_cwac_forward", (void **)&g.w4a16}};
  for (const auto &s : slots) {
    PyObject *v = PyDict_GetItemString(a[1], s.name);
    if (!v || !PyLong_Check(v)) return PyErr_Format(PyExc_KeyError, "%s", s.name);
    *s.slot = PyLong_AsVoidPtr(v);
  }
  Py_INCREF(a[0]);
  Py_XSETREF(g_qparams_type, a[0]);
  Py_INCREF(a[2]);
  Py_XSETREF(g_check, a[2]);
  Py_RETURN_NONE;
}

#define CWAC_METHOD(name) \
  { #name, (PyCFunction)(void (*)(void))py_##name, METH_FASTCALL, nullptr }
PyMethodDef methods[] = {CWAC_METHOD(bind),    CWAC_METHOD(quantize_act),  CWAC_METHOD(quantize_rows_sym),
                         CWAC_METHOD(forward), CWAC_METHOD(forward_table), CWAC_METHOD(forward_fixed_point),
                         CWAC_METHOD(conv2d),  CWAC_METHOD(w4a16),         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fast_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fast_calls() { return PyModule_Create(&module); }
