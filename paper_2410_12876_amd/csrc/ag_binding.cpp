// The binding's per-call work: reads shapes, dtypes and addresses of the tensor arguments and makes the C call.
//
// A decode step on short caches is under ten microseconds of device time, so what the host spends per call is part of
// the step: looking the stream up through torch.cuda (2.9 us), checking and fetching a dozen addresses one Python call at
// a time (4 us) and ctypes' conversion of fifteen arguments (2.7 us) was more than the two kernel launches cost.  The
// same work on the tensors' own structures takes well under a microsecond.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "ag.h"

namespace {

struct bad_arg {};  // a Python exception has been set

[[noreturn]] void fail(PyObject *type, const char *msg) {
  PyErr_SetString(type, msg);
  throw bad_arg();
}

const at::Tensor &tensor(PyObject *o) {
  if (!THPVariable_Check(o)) fail(PyExc_TypeError, "a tensor is expected");
  return THPVariable_Unpack(o);
}

// Device address of an argument: None stays NULL, an integer is taken as the address itself.
void *ptr(PyObject *o) {
  if (o == Py_None) return nullptr;
  if (THPVariable_Check(o)) {
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_contiguous()) fail(PyExc_ValueError, "tensor arguments must be contiguous");
    return t.data_ptr();
  }
  if (!PyLong_Check(o)) fail(PyExc_TypeError, "a tensor, an address or None is expected");
  void *p = PyLong_AsVoidPtr(o);
  if (!p && PyErr_Occurred()) throw bad_arg();
  return p;
}
template <typename T> T *ptr_as(PyObject *o) { return static_cast<T *>(ptr(o)); }

int int_of(PyObject *o) {
  const long long v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) throw bad_arg();
  return (int)v;
}
int64_t int64_of(PyObject *o) {
  const long long v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) throw bad_arg();
  return v;
}
float float_of(PyObject *o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw bad_arg();
  return (float)v;
}

ag_dtype dtype_of(const at::Tensor &t) {
  if (t.scalar_type() == at::kBFloat16) return AG_BF16;
  if (t.scalar_type() == at::kFloat) return AG_F32;
  PyErr_Format(PyExc_ValueError, "unsupported tensor dtype %s", c10::toString(t.scalar_type()));
  throw bad_arg();
}

int64_t dim(const at::Tensor &t, int want, int i) {
  if (t.dim() != want) fail(PyExc_ValueError, "a tensor argument has the wrong number of dimensions");
  return t.size(i);
}

// A size of a tensor of which nothing else is looked at: it may have any number of dimensions beyond that one.
int64_t size_of(const at::Tensor &t, int i) {
  if (t.dim() <= i) fail(PyExc_IndexError, "a tensor argument has too few dimensions");
  return t.size(i);
}

// The struct behind a ctypes structure (None: NULL).  The caller holds a reference to it for the length of the call.
template <typename T> T *struct_of(PyObject *o) {
  if (o == Py_None) return nullptr;
  Py_buffer b;
  if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) throw bad_arg();
  void *p = b.buf;
  const bool fits = b.len == (Py_ssize_t)sizeof(T);
  PyBuffer_Release(&b);
  if (!fits) fail(PyExc_TypeError, "a structure of another type");
  return static_cast<T *>(p);
}

// stream argument: None = torch's current stream, an integer = the handle, else an object with a cuda_stream attribute
void *stream_of(PyObject *o) {
  if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
  if (PyLong_Check(o)) return ptr(o);
  PyObject *a = PyObject_GetAttrString(o, "cuda_stream");
  if (!a) throw bad_arg();
  void *p = PyLong_AsVoidPtr(a);
  Py_DECREF(a);
  if (!p && PyErr_Occurred()) throw bad_arg();
  return p;
}

// Runs the C call without the interpreter lock (a launch can wait for room in the queue) and returns its status.
template <typename F> PyObject *call(F &&f) {
  ag_status st;
  Py_BEGIN_ALLOW_THREADS st = f();
  Py_END_ALLOW_THREADS return PyLong_FromLong((long)st);
}

// Every function takes (context, stream, arguments of the Python entry point...).
#define AG_BINDING(name, count)                                                                          \
  PyObject *name##_(ag_ctx *ctx, void *s, PyObject *const *a);                                            \
  PyObject *name(PyObject *, PyObject *const *a, Py_ssize_t n) {                                          \
    try {                                                                                                \
      if (n != 2 + (count)) fail(PyExc_TypeError, #name ": wrong number of arguments");                    \
      ag_ctx *ctx = ptr_as<ag_ctx>(a[0]);                                                                 \
      return name##_(ctx, stream_of(a[1]), a + 2);                                                        \
    } catch (const bad_arg &) {                                                                          \
      return nullptr;                                                                                    \
    } catch (const std::exception &e) {                                                                  \
      PyErr_SetString(PyExc_RuntimeError, e.what());                                                      \
      return nullptr;                                                                                    \
    }                                                                                                    \
  }                                                                                                      \
  PyObject *name##_(ag_ctx *ctx, void *s, PyObject *const *a)

// feat, w_gate, bias, tau, n_sink, logits_out, flags_out
AG_BINDING(gate, 7) {
  const at::Tensor &x = tensor(a[0]), &w = tensor(a[1]);
  const int B = dim(x, 3, 0), L = dim(x, 3, 1), d = dim(x, 3, 2), H = size_of(w, 1), n_sink = int_of(a[4]);
  const ag_dtype dt = dtype_of(x);
  const void *xp = ptr(a[0]), *wp = ptr(a[1]);
  const float *bias = ptr_as<float>(a[2]), tau = float_of(a[3]);
  float *logits = ptr_as<float>(a[5]);
  uint8_t *flags = ptr_as<uint8_t>(a[6]);
  return call([&] { return ag_gate(ctx, s, xp, dt, B, L, d, wp, bias, H, tau, n_sink, logits, flags); });
}

// h, norm_w, eps, w_gate, bias, tau, n_sink, x_out, logits_out, flags_out
AG_BINDING(rmsnorm_gate, 10) {
  const at::Tensor &h = tensor(a[0]), &w = tensor(a[3]);
  const int B = dim(h, 3, 0), L = dim(h, 3, 1), d = dim(h, 3, 2), H = size_of(w, 1), n_sink = int_of(a[6]);
  const ag_dtype dt = dtype_of(h);
  const void *hp = ptr(a[0]), *g = ptr(a[1]), *wp = ptr(a[3]);
  const float eps = float_of(a[2]), *bias = ptr_as<float>(a[4]), tau = float_of(a[5]);
  void *xo = ptr(a[7]);
  float *logits = ptr_as<float>(a[8]);
  uint8_t *flags = ptr_as<uint8_t>(a[9]);
  return call([&] { return ag_rmsnorm_gate(ctx, s, hp, dt, B, L, d, g, eps, wp, bias, H, tau, n_sink, xo, logits, flags); });
}

// k, v, flags, pos0, cache
AG_BINDING(compact_kv, 5) {
  const int L = size_of(tensor(a[0]), 2), pos0 = int_of(a[3]);
  const void *k = ptr(a[0]), *v = ptr(a[1]);
  const uint8_t *f = ptr_as<uint8_t>(a[2]);
  ag_kv_cache *c = struct_of<ag_kv_cache>(a[4]);
  return call([&] { return ag_compact_kv(ctx, s, k, v, f, L, pos0, c); });
}

// flags, room, total_rows, row_off, rows_needed
AG_BINDING(pack_row_off, 5) {
  const at::Tensor &f = tensor(a[0]);
  const int B = dim(f, 3, 0), H = dim(f, 3, 1), L = dim(f, 3, 2), room = int_of(a[1]);
  const int64_t total = int64_of(a[2]);
  const uint8_t *fp = ptr_as<uint8_t>(a[0]);
  int64_t *ro = ptr_as<int64_t>(a[3]), *need = ptr_as<int64_t>(a[4]);
  return call([&] { return ag_pack_row_off(ctx, s, fp, B, H, L, room, total, ro, need); });
}

// x, w_kv, flags, pos0, kv_out, cache
AG_BINDING(project_compact_kv, 6) {
  const at::Tensor &x = tensor(a[0]);
  const int B = dim(x, 3, 0), L = dim(x, 3, 1), d = dim(x, 3, 2), pos0 = int_of(a[3]);
  const ag_dtype dt = dtype_of(x);
  const void *xp = ptr(a[0]), *w = ptr(a[1]);
  const uint8_t *f = ptr_as<uint8_t>(a[2]);
  void *kv = ptr(a[4]);
  ag_kv_cache *c = struct_of<ag_kv_cache>(a[5]);
  return call([&] { return ag_project_compact_kv(ctx, s, xp, dt, B, L, d, w, f, pos0, kv, c); });
}

// q, k, v, flags, scale, cache, n_recent, out
AG_BINDING(prefill_attn, 8) {
  const at::Tensor &q = tensor(a[0]);
  const int B = dim(q, 4, 0), Hq = dim(q, 4, 1), L = dim(q, 4, 2), D = dim(q, 4, 3), Hkv = size_of(tensor(a[1]), 1), n = int_of(a[6]);
  const ag_dtype dt = dtype_of(q);
  const void *qp = ptr(a[0]), *k = ptr(a[1]), *v = ptr(a[2]);
  const uint8_t *f = ptr_as<uint8_t>(a[3]);
  const float scale = float_of(a[4]);
  const ag_kv_cache *c = struct_of<ag_kv_cache>(a[5]);
  void *out = ptr(a[7]);
  return call([&] { return ag_prefill_attn_recent(ctx, s, qp, k, v, f, B, L, Hq, Hkv, D, dt, scale, c, n, out); });
}

// q, k, v, flags, scale, pos0, cache, n_recent, out
AG_BINDING(compact_prefill_attn, 9) {
  const at::Tensor &q = tensor(a[0]);
  const int B = dim(q, 4, 0), Hq = dim(q, 4, 1), L = dim(q, 4, 2), D = dim(q, 4, 3), Hkv = size_of(tensor(a[1]), 1);
  const int pos0 = int_of(a[5]), n = int_of(a[7]);
  const ag_dtype dt = dtype_of(q);
  const void *qp = ptr(a[0]), *k = ptr(a[1]), *v = ptr(a[2]);
  const uint8_t *f = ptr_as<uint8_t>(a[3]);
  const float scale = float_of(a[4]);
  ag_kv_cache *c = struct_of<ag_kv_cache>(a[6]);
  void *out = ptr(a[8]);
  return call([&] { return ag_compact_prefill_attn(ctx, s, qp, k, v, f, B, L, Hq, Hkv, D, dt, scale, pos0, c, n, out); });
}

// q, k_new, v_new, new_flags, pos, scale, cache, ring, out
AG_BINDING(decode_attn, 9) {
  const at::Tensor &q = tensor(a[0]);
  const int Hq = size_of(q, 1), pos = int_of(a[4]);
  const void *qp = ptr(a[0]), *k = ptr(a[1]), *v = ptr(a[2]);
  const uint8_t *f = ptr_as<uint8_t>(a[3]);
  const float scale = float_of(a[5]);
  ag_kv_cache *c = struct_of<ag_kv_cache>(a[6]);
  ag_recent_ring *r = struct_of<ag_recent_ring>(a[7]);
  void *out = ptr(a[8]);
  return call([&] { return ag_decode_attn_recent(ctx, s, qp, k, v, f, pos, Hq, scale, c, r, out); });
}

// q, k_new, v_new, new_flags, pos, scale, cache, out
AG_BINDING(decode_attn_static, 8) {
  const at::Tensor &q = tensor(a[0]);
  const int Hq = size_of(q, 1), pos = int_of(a[4]);
  const void *qp = ptr(a[0]), *k = ptr(a[1]), *v = ptr(a[2]);
  const uint8_t *f = ptr_as<uint8_t>(a[3]);
  const float scale = float_of(a[5]);
  ag_kv_cache *c = struct_of<ag_kv_cache>(a[6]);
  void *out = ptr(a[7]);
  return call([&] { return ag_decode_attn_static(ctx, s, qp, k, v, f, pos, Hq, scale, c, out); });
}

// k, v, flags, pos0, ring
AG_BINDING(recent_fill, 5) {
  const at::Tensor &k = tensor(a[0]);
  const int B = dim(k, 4, 0), H = dim(k, 4, 1), L = dim(k, 4, 2), D = dim(k, 4, 3), pos0 = int_of(a[3]);
  const ag_dtype dt = dtype_of(k);
  const void *kp = ptr(a[0]), *v = ptr(a[1]);
  const uint8_t *f = ptr_as<uint8_t>(a[2]);
  ag_recent_ring *r = struct_of<ag_recent_ring>(a[4]);
  return call([&] { return ag_recent_fill(ctx, s, kp, v, f, B, L, H, D, dt, pos0, r); });
}

// x, w_qkv, h_prime, d_prime, w_o, bias, tau, n_sink, logits_out, flags_out
AG_BINDING(gate_mha, 10) {
  const at::Tensor &x = tensor(a[0]), &wo = tensor(a[4]);
  const int B = dim(x, 3, 0), L = dim(x, 3, 1), d = dim(x, 3, 2), H = size_of(wo, 1);
  const int hp = int_of(a[2]), dp = int_of(a[3]), n_sink = int_of(a[7]);
  const ag_dtype dt = dtype_of(x);
  const void *xp = ptr(a[0]), *w = ptr(a[1]), *wop = ptr(a[4]);
  const float *bias = ptr_as<float>(a[5]), tau = float_of(a[6]);
  float *logits = ptr_as<float>(a[8]);
  uint8_t *flags = ptr_as<uint8_t>(a[9]);
  return call([&] { return ag_gate_mha(ctx, s, xp, dt, B, L, d, w, hp, dp, wop, bias, H, tau, n_sink, logits, flags); });
}

#define AG_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {AG_METHOD(gate), AG_METHOD(rmsnorm_gate), AG_METHOD(compact_kv), AG_METHOD(pack_row_off),
                         AG_METHOD(project_compact_kv), AG_METHOD(prefill_attn), AG_METHOD(compact_prefill_attn),
                         AG_METHOD(decode_attn), AG_METHOD(decode_attn_static), AG_METHOD(recent_fill), AG_METHOD(gate_mha),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", "Calls into libag on torch tensors.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&module); }
