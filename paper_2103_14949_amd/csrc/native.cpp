// The binding's marshalling in native code: torch tensors and parameter objects in, one C ABI call
// (include/hago.h) out.  What bounds a small operator is the host: the same work done with ctypes took
// 7 - 8 us of Python per call beside the 2.3 us of the kernel launch itself.
//
// Every function takes the arguments of the binding's function of the same name, positionally, and either
// issues the call on the current stream or (prepare) returns a Prepared object that re-issues it.  The
// library's addresses come from the binding, which loads it: this module links to torch only.
#include <Python.h>

#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <functional>
#include <vector>

#include "../../include/hago.h"

namespace {

// ---- the library's entry points, filled in by bind()
#define HAGO_ENTRIES(X)                                                                                            \
  X(hago_simquant) X(hago_simquant_wrap) X(hago_simquant_batched) X(hago_quantize) X(hago_dequantize)              \
  X(hago_simquant_codes) X(hago_absmax) X(hago_requantize) X(hago_qdense) X(hago_qconv2d) X(hago_qconv2d_ws)       \
  X(hago_qconv2d_static) X(hago_bit_range)
struct Library {
#define X(name) decltype(&::name) name;
  HAGO_ENTRIES(X)
#undef X
} L;
PyObject* g_check = nullptr;  // raises the binding's error for a status

struct Raised {};  // a Python error is set

PyObject* intern(const char* s) { return PyUnicode_InternFromString(s); }

int64_t as_int(PyObject* o) {
  const long long v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) throw Raised{};
  return v;
}
// int(o): floats, numpy scalars and one-element tensors too
int64_t as_converted_int(PyObject* o) {
  PyObject* k = PyNumber_Long(o);
  if (!k) throw Raised{};
  const long long v = PyLong_AsLongLong(k);
  Py_DECREF(k);
  if (v == -1 && PyErr_Occurred()) throw Raised{};
  return v;
}
bool as_bool(PyObject* o) {
  const int v = PyObject_IsTrue(o);
  if (v < 0) throw Raised{};
  return v != 0;
}
int64_t attr_int(PyObject* o, PyObject* name) {
  PyObject* v = PyObject_GetAttr(o, name);
  if (!v) throw Raised{};
  const long long r = PyLong_AsLongLong(v);
  Py_DECREF(v);
  if (r == -1 && PyErr_Occurred()) throw Raised{};
  return r;
}
int64_t attr_converted_int(PyObject* o, PyObject* name) {
  PyObject* v = PyObject_GetAttr(o, name);
  if (!v) throw Raised{};
  try {
    const int64_t r = as_converted_int(v);
    Py_DECREF(v);
    return r;
  } catch (...) {
    Py_DECREF(v);
    throw;
  }
}
void require(bool ok) {
  if (!ok) {
    PyErr_SetNone(PyExc_AssertionError);
    throw Raised{};
  }
}
const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_Check(o)) {
    PyErr_SetString(PyExc_TypeError, "a torch tensor is needed");
    throw Raised{};
  }
  return THPVariable_Unpack(o);
}
void* pointer(PyObject* o) { return o == Py_None ? nullptr : tensor(o).data_ptr(); }
void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

void check(hago_status s) {
  if (s == HAGO_OK) return;
  PyObject* r = PyObject_CallFunction(g_check, "i", (int)s);
  Py_XDECREF(r);
  if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, "libhago call failed");
  throw Raised{};
}

at::ScalarType scalar_type(int64_t code) {
  switch (code) {
    case HAGO_U8: return at::kByte;
    case HAGO_I8: return at::kChar;
    case HAGO_I16: return at::kShort;
    case HAGO_I32: case HAGO_I24: return at::kInt;
    case HAGO_F32: return at::kFloat;
  }
  PyErr_SetObject(PyExc_KeyError, PyLong_FromLongLong(code));
  throw Raised{};
}

// `given`, or a new tensor of the shape and type on `like`'s device (a new reference either way).
PyObject* output(PyObject* given, at::IntArrayRef shape, at::ScalarType type, const at::Tensor& like) {
  if (given != Py_None) {
    tensor(given);
    Py_INCREF(given);
    return given;
  }
  PyObject* r = THPVariable_Wrap(at::Tensor(at::detail::empty_cuda(shape, type, like.device(), std::nullopt)));
  if (!r) throw Raised{};
  return r;
}

hago_qtype qtype(PyObject* q) {
  static PyObject *dtype = intern("dtype"), *bits = intern("bits"), *sgn = intern("is_signed"), *zp = intern("zero_point");
  return hago_qtype{(hago_dtype)attr_int(q, dtype), (int32_t)attr_int(q, bits), (int32_t)attr_converted_int(q, sgn), (int32_t)attr_int(q, zp)};
}

struct Ref {  // a reference of our own
  PyObject* o = nullptr;
  Ref() = default;
  Ref(const Ref&) = delete;
  ~Ref() { Py_XDECREF(o); }
};
struct RequantTensors {  // kept by the Prepared object: the attributes they come from may be set to others
  Ref mult, shift;
};

struct MaybeRequant {  // a copy of the caller's parameters
  bool present = false;
  hago_requant rq{};
  const hago_requant* ptr() const { return present ? &rq : nullptr; }
};

MaybeRequant requant(PyObject* o, RequantTensors& tensors) {
  MaybeRequant r;
  if (o == Py_None) return r;
  static PyObject *mult = intern("multiplier"), *shift = intern("shift"), *pc = intern("per_channel"), *out = intern("out"),
                  *lo = intern("clip_lo"), *hi = intern("clip_hi"), *rounding = intern("rounding");
  auto ptr_of = [&](PyObject* name, Ref& t) {
    t.o = PyObject_GetAttr(o, name);
    if (!t.o) throw Raised{};
    return static_cast<const int32_t*>(pointer(t.o));  // (only None is NULL, the shift-only form)
  };
  r.present = true;
  r.rq.multiplier = ptr_of(mult, tensors.mult);
  r.rq.shift = ptr_of(shift, tensors.shift);
  r.rq.per_channel = (int32_t)attr_int(o, pc);
  PyObject* q = PyObject_GetAttr(o, out);
  if (!q) throw Raised{};
  try {
    r.rq.out = qtype(q);
  } catch (...) {
    Py_DECREF(q);
    throw;
  }
  Py_DECREF(q);
  r.rq.clip_lo = (int32_t)attr_int(o, lo);
  r.rq.clip_hi = (int32_t)attr_int(o, hi);
  r.rq.rounding = (int32_t)attr_int(o, rounding);
  return r;
}

// ---- a call with its arguments already marshalled
struct Prepared {
  PyObject_HEAD
  vectorcallfunc vectorcall;
  std::function<hago_status()>* fn;
  PyObject* keep;  // everything the call's pointers belong to
  PyObject* out;
};

PyObject* prepared_call(PyObject* self, PyObject* const*, size_t nargs, PyObject* names) {
  Prepared* p = reinterpret_cast<Prepared*>(self);
  if (PyVectorcall_NARGS(nargs) != 0 || (names && PyTuple_GET_SIZE(names) != 0)) {
    PyErr_SetString(PyExc_TypeError, "a prepared call takes no arguments");
    return nullptr;
  }
  hago_status s;
  Py_BEGIN_ALLOW_THREADS
  s = (*p->fn)();
  Py_END_ALLOW_THREADS
  if (s != HAGO_OK) {
    try {
      check(s);
    } catch (Raised&) {
    }
    return nullptr;
  }
  Py_INCREF(p->out);
  return p->out;
}

int prepared_traverse(PyObject* self, visitproc visit, void* arg) {
  Prepared* p = reinterpret_cast<Prepared*>(self);
  Py_VISIT(p->keep);
  Py_VISIT(p->out);
  return 0;
}
int prepared_clear(PyObject* self) {
  Prepared* p = reinterpret_cast<Prepared*>(self);
  Py_CLEAR(p->keep);
  Py_CLEAR(p->out);
  return 0;
}
void prepared_dealloc(PyObject* self) {
  PyObject_GC_UnTrack(self);
  delete reinterpret_cast<Prepared*>(self)->fn;
  prepared_clear(self);
  Py_TYPE(self)->tp_free(self);
}
PyObject* prepared_out(PyObject* self, void*) {
  PyObject* o = reinterpret_cast<Prepared*>(self)->out;
  Py_INCREF(o);
  return o;
}
int set_prepared_out(PyObject* self, PyObject* value, void*) {
  if (!value) {
    PyErr_SetString(PyExc_AttributeError, "out");
    return -1;
  }
  Py_INCREF(value);
  Py_XSETREF(reinterpret_cast<Prepared*>(self)->out, value);
  return 0;
}
PyGetSetDef prepared_getset[] = {
    {"out", prepared_out, set_prepared_out, "what a call returns: the output tensor(s) (another value does not change where the launch writes)", nullptr}, {}};

PyTypeObject PreparedType = [] {
  PyTypeObject t = {PyVarObject_HEAD_INIT(nullptr, 0)};
  t.tp_name = "paper_2103_14949_amd._native.Prepared";
  t.tp_doc = "A library call with its arguments already marshalled; calling it re-issues the same launch\n"
             "(same buffers, same stream) and returns the output.";
  t.tp_basicsize = sizeof(Prepared);
  t.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_GC | Py_TPFLAGS_HAVE_VECTORCALL;
  t.tp_vectorcall_offset = offsetof(Prepared, vectorcall);
  t.tp_call = PyVectorcall_Call;
  t.tp_dealloc = prepared_dealloc;
  t.tp_traverse = prepared_traverse;
  t.tp_clear = prepared_clear;
  t.tp_getset = prepared_getset;
  return t;
}();

// Issues f now, or wraps it.  Takes over the reference to `out`; `keep`: the other arguments, borrowed (or NULL).
template <class F>
PyObject* issue(const F& f, PyObject* out, bool prepare, std::initializer_list<PyObject*> keep) {
  if (!prepare) {
    hago_status s;
    Py_BEGIN_ALLOW_THREADS
    s = f();
    Py_END_ALLOW_THREADS
    if (s != HAGO_OK) {
      Py_DECREF(out);
      check(s);
    }
    return out;
  }
  PyObject* k = PyTuple_New((Py_ssize_t)keep.size() + 1);
  Prepared* p = k ? PyObject_GC_New(Prepared, &PreparedType) : nullptr;
  if (!p) {
    Py_XDECREF(k);
    Py_DECREF(out);
    throw Raised{};
  }
  Py_ssize_t i = 0;
  auto hold = [&](PyObject* o) {
    Py_INCREF(o);
    PyTuple_SET_ITEM(k, i++, o);
  };
  for (PyObject* o : keep) hold(o ? o : Py_None);
  hold(out);  // (p->out may be set to something else)
  p->vectorcall = prepared_call;
  p->fn = new std::function<hago_status()>(f);
  p->keep = k;
  p->out = out;
  PyObject_GC_Track(p);
  return reinterpret_cast<PyObject*>(p);
}

// ---- the functions
void need_args(Py_ssize_t n, Py_ssize_t want) {
  if (n == want) return;
  PyErr_Format(PyExc_TypeError, "%zd arguments wanted, got %zd", want, n);
  throw Raised{};
}

struct Tensor3 {  // x[outer, channels, inner]
  const at::Tensor& t;
  int64_t outer, channels, inner;
};
Tensor3 tensor3(PyObject* o) {
  const at::Tensor& t = tensor(o);
  require(t.dim() == 3 && t.is_contiguous());
  return Tensor3{t, t.size(0), t.size(1), t.size(2)};
}

int32_t per_channel_of(PyObject* o, PyObject* scale) {
  return o == Py_None ? (tensor(scale).numel() > 1 ? 1 : 0) : (int32_t)as_converted_int(o);
}

struct Clip {
  int32_t lo, hi;
};
Clip clip_of(PyObject* lo, PyObject* hi, const hago_qtype& q, int32_t most_bits) {
  Clip c;
  check(L.hago_bit_range(q.bits < most_bits ? q.bits : most_bits, q.is_signed ? 1 : 0, &c.lo, &c.hi));
  if (lo != Py_None) c.lo = (int32_t)as_converted_int(lo);
  if (hi != Py_None) c.hi = (int32_t)as_converted_int(hi);
  return c;
}

// simquant, simquant_wrap: (x, scale, zero_point, q, clip_lo, clip_hi, per_channel, out, prepare)
template <class Fn>
PyObject* simquant_with(Fn fn, int32_t most_bits, PyObject* const* a, Py_ssize_t n) {
  need_args(n, 9);
  const Tensor3 x = tensor3(a[0]);
  const hago_qtype q = qtype(a[3]);
  const Clip c = clip_of(a[4], a[5], q, most_bits);
  const int32_t pc = per_channel_of(a[6], a[1]);
  const float* scale = static_cast<const float*>(pointer(a[1]));
  const int32_t* zp = static_cast<const int32_t*>(pointer(a[2]));
  PyObject* out = output(a[7], x.t.sizes(), x.t.scalar_type(), x.t);
  const float* src = static_cast<const float*>(x.t.data_ptr());
  float* dst = static_cast<float*>(pointer(out));
  const int64_t o = x.outer, ch = x.channels, in = x.inner;
  void* st = stream();
  return issue([=] { return fn(src, dst, o, ch, in, scale, zp, pc, q, c.lo, c.hi, st); }, out, as_bool(a[8]), {a[0], a[1], a[2]});
}

PyObject* f_simquant(PyObject* const* a, Py_ssize_t n) { return simquant_with(L.hago_simquant, 64, a, n); }
PyObject* f_simquant_wrap(PyObject* const* a, Py_ssize_t n) { return simquant_with(L.hago_simquant_wrap, 25, a, n); }

// (x, scales, zero_points, q, clip_lo, clip_hi, per_channel, out, prepare)
PyObject* f_simquant_batched(PyObject* const* a, Py_ssize_t n) {
  need_args(n, 9);
  const Tensor3 x = tensor3(a[0]);
  const at::Tensor &scales = tensor(a[1]), &zps = tensor(a[2]);
  require(scales.is_contiguous() && zps.is_contiguous());
  auto ints = [](PyObject* seq) {
    std::vector<int32_t> v;
    PyObject* f = PySequence_Fast(seq, "clip limits are sequences");
    if (!f) throw Raised{};
    for (Py_ssize_t i = 0; i < PySequence_Fast_GET_SIZE(f); ++i) {
      try {
        v.push_back((int32_t)as_converted_int(PySequence_Fast_GET_ITEM(f, i)));
      } catch (...) {
        Py_DECREF(f);
        throw;
      }
    }
    Py_DECREF(f);
    return v;
  };
  const std::vector<int32_t> lo = ints(a[4]), hi = ints(a[5]);
  const int64_t nb = (int64_t)lo.size();
  require((int64_t)hi.size() == nb && scales.size(0) == nb && zps.size(0) == nb);
  const hago_qtype q = qtype(a[3]);
  const int32_t pc = as_bool(a[6]) ? 1 : 0;
  const int64_t shape[4] = {nb, x.outer, x.channels, x.inner};
  PyObject* out = output(a[7], at::IntArrayRef(shape, 4), at::kFloat, x.t);
  const float* src = static_cast<const float*>(x.t.data_ptr());
  float* dst = static_cast<float*>(pointer(out));
  const float* sp = static_cast<const float*>(scales.data_ptr());
  const int32_t* zp = static_cast<const int32_t*>(zps.data_ptr());
  const int64_t o = x.outer, ch = x.channels, in = x.inner;
  void* st = stream();
  auto call = [=](const int32_t* l, const int32_t* h) {
    // (an empty list has no address of its own, and the library wants one only for nb > 0)
    return L.hago_simquant_batched(src, dst, o, ch, in, (int32_t)nb, sp, zp, pc, q, l, h, st);
  };
  if (as_bool(a[8])) return issue([call, lo, hi] { return call(lo.data(), hi.data()); }, out, true, {a[0], a[1], a[2]});
  return issue([&] { return call(lo.data(), hi.data()); }, out, false, {});
}

// (x, scale, zero_point, q, clip_lo, clip_hi, per_channel, out, prepare)
PyObject* f_quantize(PyObject* const* a, Py_ssize_t n) {
  need_args(n, 9);
  const Tensor3 x = tensor3(a[0]);
  const hago_qtype q = qtype(a[3]);
  const Clip c = clip_of(a[4], a[5], q, 64);
  const int32_t pc = per_channel_of(a[6], a[1]);
  const float* scale = static_cast<const float*>(pointer(a[1]));
  const int32_t* zp = static_cast<const int32_t*>(pointer(a[2]));
  PyObject* out = output(a[7], x.t.sizes(), scalar_type(q.dtype), x.t);
  const float* src = static_cast<const float*>(x.t.data_ptr());
  void* dst = pointer(out);
  const int64_t o = x.outer, ch = x.channels, in = x.inner;
  void* st = stream();
  return issue([=] { return L.hago_quantize(src, dst, o, ch, in, scale, zp, pc, q, c.lo, c.hi, st); }, out, as_bool(a[8]),
               {a[0], a[1], a[2]});
}

// (x, scale, zero_point, q, clip_lo, clip_hi, per_channel, out, out_codes, prepare)
PyObject* f_simquant_codes(PyObject* const* a, Py_ssize_t n) {
  need_args(n, 10);
  const Tensor3 x = tensor3(a[0]);
  const hago_qtype q = qtype(a[3]);
  const Clip c = clip_of(a[4], a[5], q, 64);
  const int32_t pc = per_channel_of(a[6], a[1]);
  const float* scale = static_cast<const float*>(pointer(a[1]));
  const int32_t* zp = static_cast<const int32_t*>(pointer(a[2]));
  PyObject* y = output(a[7], x.t.sizes(), x.t.scalar_type(), x.t);
  PyObject* codes;
  try {
    codes = output(a[8], x.t.sizes(), scalar_type(q.dtype), x.t);
  } catch (...) {
    Py_DECREF(y);
    throw;
  }
  const float* src = static_cast<const float*>(x.t.data_ptr());
  float* dst = static_cast<float*>(pointer(y));
  void* dq = pointer(codes);
  PyObject* both = PyTuple_New(2);
  if (!both) throw Raised{};
  PyTuple_SET_ITEM(both, 0, y);
  PyTuple_SET_ITEM(both, 1, codes);
  const int64_t o = x.outer, ch = x.channels, in = x.inner;
  void* st = stream();
  return issue([=] { return L.hago_simquant_codes(src, dst, dq, o, ch, in, scale, zp, pc, q, c.lo, c.hi, st); }, both,
               as_bool(a[9]), {a[0], a[1], a[2]});
}

// (codes, q, scale, zero_point, per_channel, out, prepare)
PyObject* f_dequantize(PyObject* const* a, Py_ssize_t n) {
  need_args(n, 7);
  const Tensor3 x = tensor3(a[0]);
  const hago_qtype q = qtype(a[1]);
  const int32_t pc = per_channel_of(a[4], a[2]);
  const float* scale = static_cast<const float*>(pointer(a[2]));
  const int32_t* zp = static_cast<const int32_t*>(pointer(a[3]));
  PyObject* out = output(a[5], x.t.sizes(), at::kFloat, x.t);
  const void* src = x.t.data_ptr();
  float* dst = static_cast<float*>(pointer(out));
  const int64_t o = x.outer, ch = x.channels, in = x.inner;
  void* st = stream();
  return issue([=] { return L.hago_dequantize(src, q, dst, o, ch, in, scale, zp, pc, st); }, out, as_bool(a[6]),
               {a[0], a[2], a[3]});
}

// (x, per_channel, out, prepare)
PyObject* f_absmax(PyObject* const* a, Py_ssize_t n) {
  need_args(n, 4);
  const Tensor3 x = tensor3(a[0]);
  const int32_t pc = as_bool(a[1]) ? 1 : 0;
  const int64_t nthr = pc ? x.channels : 1;
  PyObject* out = output(a[2], at::IntArrayRef(&nthr, 1), at::kFloat, x.t);
  const float* src = static_cast<const float*>(x.t.data_ptr());
  float* dst = static_cast<float*>(pointer(out));
  const int64_t o = x.outer, ch = x.channels, in = x.inner;
  void* st = stream();
  return issue([=] { return L.hago_absmax(src, o, ch, in, pc, dst, st); }, out, as_bool(a[3]), {a[0]});
}

// (acc, rq, out, prepare)
PyObject* f_requantize(PyObject* const* a, Py_ssize_t n) {
  need_args(n, 4);
  const Tensor3 x = tensor3(a[0]);
  RequantTensors tensors;
  const MaybeRequant rq = requant(a[1], tensors);
  int code;
  switch (x.t.scalar_type()) {
    case at::kByte: code = HAGO_U8; break;
    case at::kChar: code = HAGO_I8; break;
    case at::kShort: code = HAGO_I16; break;
    case at::kInt: code = HAGO_I32; break;
    default: code = HAGO_F32;
  }
  PyObject* out = output(a[2], x.t.sizes(), scalar_type(rq.rq.out.dtype), x.t);
  const void* src = x.t.data_ptr();
  void* dst = pointer(out);
  const int64_t o = x.outer, ch = x.channels, in = x.inner;
  void* st = stream();
  return issue([=] { return L.hago_requantize(src, (hago_dtype)code, o, ch, in, rq.ptr(), dst, st); }, out, as_bool(a[3]),
               {a[0], tensors.mult.o, tensors.shift.o});
}

// (a, a_t, w, w_t, bias, acc_dtype, rq, flags, out, prepare)
PyObject* f_qdense(PyObject* const* a, Py_ssize_t n) {
  need_args(n, 10);
  const at::Tensor &act = tensor(a[0]), &w = tensor(a[2]);
  require(act.dim() == 2 && w.dim() == 2 && act.is_contiguous() && w.is_contiguous());
  const int64_t M = act.size(0), K = act.size(1), N = w.size(0);
  require(w.size(1) == K);
  const hago_qtype at_ = qtype(a[1]), wt = qtype(a[3]);
  const int32_t* bias = static_cast<const int32_t*>(pointer(a[4]));
  const int64_t acc = as_int(a[5]);
  RequantTensors tensors;
  const MaybeRequant rq = requant(a[6], tensors);
  const uint32_t flags = (uint32_t)as_int(a[7]);
  const int64_t shape[2] = {M, N};
  PyObject* out = output(a[8], at::IntArrayRef(shape, 2), scalar_type(rq.present ? rq.rq.out.dtype : acc), act);
  const void *ap = act.data_ptr(), *wp = w.data_ptr();
  void* dst = pointer(out);
  void* st = stream();
  return issue([=] { return L.hago_qdense(ap, at_, wp, wt, bias, M, N, K, (hago_dtype)acc, rq.ptr(), dst, flags, st); }, out,
               as_bool(a[9]), {a[0], a[2], a[4], tensors.mult.o, tensors.shift.o});
}

void pair(PyObject* o, int32_t (&v)[2]) {
  for (Py_ssize_t i = 0; i < 2; ++i) {
    PyObject* e = PySequence_GetItem(o, i);
    if (!e) throw Raised{};
    const long long r = PyLong_AsLongLong(e);
    Py_DECREF(e);
    if (r == -1 && PyErr_Occurred()) throw Raised{};
    v[i] = (int32_t)r;
  }
}

// (a, a_t, w, w_t, bias, layout, stride, pad, groups, acc_dtype, rq, flags, out, prepare, workspace, static_scratch)
PyObject* f_qconv2d(PyObject* const* a, Py_ssize_t n) {
  need_args(n, 16);
  const at::Tensor &act = tensor(a[0]), &w = tensor(a[2]);
  require(act.dim() == 4 && w.dim() == 4 && act.is_contiguous() && w.is_contiguous());
  const hago_qtype at_ = qtype(a[1]), wt = qtype(a[3]);
  const int32_t* bias = static_cast<const int32_t*>(pointer(a[4]));
  const int64_t layout = as_int(a[5]);
  const bool nchw = layout == HAGO_NCHW;
  const int64_t B = act.size(0), C = act.size(nchw ? 1 : 3), H = act.size(nchw ? 2 : 1), W = act.size(nchw ? 3 : 2);
  const int64_t O = w.size(0), KH = w.size(nchw ? 2 : 1), KW = w.size(nchw ? 3 : 2);
  int32_t stride[2], pad[2];
  pair(a[6], stride);
  pair(a[7], pad);
  const int32_t groups = (int32_t)as_int(a[8]);
  const int64_t acc = as_int(a[9]);
  RequantTensors tensors;
  const MaybeRequant rq = requant(a[10], tensors);
  const uint32_t flags = (uint32_t)as_int(a[11]);
  auto extent = [&](int64_t size, int64_t k, int i) -> int64_t {
    if (stride[i] == 0) {
      PyErr_SetString(PyExc_ZeroDivisionError, "stride 0");
      throw Raised{};
    }
    const int64_t num = size + 2 * (int64_t)pad[i] - k, s = stride[i];
    int64_t q = num / s;
    if (num % s != 0 && (num < 0) != (s < 0)) --q;  // floor
    return q + 1 > 0 ? q + 1 : 0;
  };
  const int64_t OH = extent(H, KH, 0), OW = extent(W, KW, 1);
  const int64_t cf[4] = {B, O, OH, OW}, cl[4] = {B, OH, OW, O};
  PyObject* out = output(a[12], at::IntArrayRef(nchw ? cf : cl, 4), scalar_type(rq.present ? rq.rq.out.dtype : acc), act);
  const void *ap = act.data_ptr(), *wp = w.data_ptr();
  void* dst = pointer(out);
  const bool prepare = as_bool(a[13]);
  void* st = stream();
  const int32_t kh = (int32_t)KH, kw = (int32_t)KW, sh = stride[0], sw = stride[1], ph = pad[0], pw = pad[1];
  if (a[14] != Py_None) {
    const at::Tensor& wst = tensor(a[14]);
    const int64_t bytes = wst.numel() * (int64_t)wst.element_size();
    void* ws = wst.numel() ? wst.data_ptr() : nullptr;
    return issue([=] { return L.hago_qconv2d_ws(ap, at_, wp, wt, bias, (hago_layout)layout, B, C, H, W, O, kh, kw, sh, sw, ph, pw,
                                                groups, (hago_dtype)acc, rq.ptr(), dst, ws, bytes, flags, st); },
                 out, prepare, {a[0], a[2], a[4], tensors.mult.o, tensors.shift.o, a[14]});
  }
  auto fn = as_bool(a[15]) ? L.hago_qconv2d_static : L.hago_qconv2d;
  return issue([=] { return fn(ap, at_, wp, wt, bias, (hago_layout)layout, B, C, H, W, O, kh, kw, sh, sw, ph, pw, groups,
                               (hago_dtype)acc, rq.ptr(), dst, flags, st); },
               out, prepare, {a[0], a[2], a[4], tensors.mult.o, tensors.shift.o});
}

template <PyObject* (*F)(PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  try {
    return F(args, n);
  } catch (Raised&) {
    return nullptr;
  }
  END_HANDLE_TH_ERRORS
}

// bind({name: address}, check)
PyObject* f_bind(PyObject* const* a, Py_ssize_t n) {
  need_args(n, 2);
  Library lib;
#define X(name)                                                        \
  {                                                                    \
    PyObject* v = PyMapping_GetItemString(a[0], #name);                \
    if (!v) throw Raised{};                                            \
    void* p = PyLong_AsVoidPtr(v);                                     \
    Py_DECREF(v);                                                      \
    if (!p && PyErr_Occurred()) throw Raised{};                        \
    lib.name = reinterpret_cast<decltype(&::name)>(p);                 \
  }
  HAGO_ENTRIES(X)
#undef X
  L = lib;
  Py_INCREF(a[1]);
  Py_XSETREF(g_check, a[1]);
  Py_RETURN_NONE;
}

// entries(): the names bind() wants
PyObject* f_entries(PyObject* const*, Py_ssize_t n) {
  need_args(n, 0);
  static const char* const names[] = {
#define X(name) #name,
      HAGO_ENTRIES(X)
#undef X
  };
  const Py_ssize_t count = (Py_ssize_t)(sizeof(names) / sizeof(names[0]));
  PyObject* t = PyTuple_New(count);
  if (!t) throw Raised{};
  for (Py_ssize_t i = 0; i < count; ++i) PyTuple_SET_ITEM(t, i, PyUnicode_FromString(names[i]));
  return t;
}

#define HAGO_METHOD(name) \
  {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&guarded<f_##name>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {HAGO_METHOD(bind), HAGO_METHOD(entries), HAGO_METHOD(simquant), HAGO_METHOD(simquant_wrap),
                         HAGO_METHOD(simquant_batched), HAGO_METHOD(quantize), HAGO_METHOD(simquant_codes),
                         HAGO_METHOD(dequantize), HAGO_METHOD(absmax), HAGO_METHOD(requantize), HAGO_METHOD(qdense),
                         HAGO_METHOD(qconv2d), {}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "Native marshalling of the libhago binding.", -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__native() {
  if (PyType_Ready(&PreparedType) < 0) return nullptr;
  PyObject* m = PyModule_Create(&module);
  if (!m) return nullptr;
  Py_INCREF(&PreparedType);
  if (PyModule_AddObject(m, "Prepared", reinterpret_cast<PyObject*>(&PreparedType)) < 0) return nullptr;
  return m;
}
