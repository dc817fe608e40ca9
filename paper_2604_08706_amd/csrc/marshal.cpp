// Argument marshalling of the Python binding (_binding.py), in C++: checks the
// torch tensors an entry point is given (device, dtype, contiguity, size) and
// calls the C ABI with their addresses and the current HIP stream.
//
// Checked from Python and passed through ctypes, an argument cost about 1 us
// and a call 2 to 3 more: 15 us for the loss, 30 for the single pass, more than
// the GPU works on a small batch.  Here the checks cost a fraction of that: a
// call with one launch takes 2.9 us in all (a histogram) to 3.2 (a push, a
// draw), the loss with its two launches 5.6.
//
// The GIL is released around the library call, whose launches may block on a
// full queue.  No C++ exception leaves a function: torch's become Python ones.

#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <exception>

#include "rbpolicy.h"

namespace {

struct Raised {};  // a Python error is set

[[noreturn]] void raise(PyObject* type, const char* fmt, const char* name) {
  PyErr_Format(type, fmt, name);
  throw Raised{};
}

const at::Tensor& tensor(PyObject* o, const char* name) {
  if (!THPVariable_Check(o)) raise(PyExc_TypeError, "%s must be a torch.Tensor", name);
  return THPVariable_Unpack(o);
}

// Address of a contiguous device tensor of at least `numel` elements (any
// dtype when `want` is Undefined).
void* device_ptr(PyObject* o, at::ScalarType want, const char* name, int64_t numel) {
  const at::Tensor& t = tensor(o, name);
  if (!t.is_cuda()) raise(PyExc_ValueError, "%s must be a device tensor", name);
  if (want != at::kFloat && want != at::kInt && want != at::kLong && want != at::kBFloat16 &&
      want != at::ScalarType::Undefined)
    raise(PyExc_TypeError, "%s: unexpected dtype", name);
  if (want != at::ScalarType::Undefined && t.scalar_type() != want) {
    const char* s = want == at::kFloat  ? "torch.float32"
                    : want == at::kInt  ? "torch.int32"
                    : want == at::kLong ? "torch.int64"
                                        : "torch.bfloat16";
    PyObject* got = PyObject_GetAttrString(o, "dtype");
    if (got != nullptr) {
      PyErr_Format(PyExc_TypeError, "%s must be %s, got %S", name, s, got);
      Py_DECREF(got);
    }
    throw Raised{};
  }
  if (!t.is_contiguous()) raise(PyExc_ValueError, "%s must be contiguous", name);
  if (t.numel() < numel) {
    PyErr_Format(PyExc_ValueError, "%s holds %lld elements, needs %lld", name,
                 (long long)t.numel(), (long long)numel);
    throw Raised{};
  }
  return t.data_ptr();
}

float* f32(PyObject* o, const char* name, int64_t numel = 0) {
  return static_cast<float*>(device_ptr(o, at::kFloat, name, numel));
}
int32_t* i32(PyObject* o, const char* name, int64_t numel = 0) {
  return static_cast<int32_t*>(device_ptr(o, at::kInt, name, numel));
}
int64_t* i64(PyObject* o, const char* name, int64_t numel = 0) {
  return static_cast<int64_t*>(device_ptr(o, at::kLong, name, numel));
}
uint16_t* bf16(PyObject* o, const char* name, int64_t numel) {
  return static_cast<uint16_t*>(device_ptr(o, at::kBFloat16, name, numel));
}
int32_t* i32_or_null(PyObject* o, const char* name, int64_t numel) {
  return o == Py_None ? nullptr : i32(o, name, numel);
}
float* f32_or_null(PyObject* o, const char* name, int64_t numel) {
  return o == Py_None ? nullptr : f32(o, name, numel);
}

int64_t numel_of(PyObject* o, const char* name) { return tensor(o, name).numel(); }

int64_t size_of(PyObject* o, const char* name, int64_t dim) {
  const at::Tensor& t = tensor(o, name);
  if (dim >= t.dim()) raise(PyExc_ValueError, "%s has too few dimensions", name);
  return t.size(dim);
}

// The two sizes of a matrix.
void sizes_2d(PyObject* o, const char* name, int64_t& rows, int64_t& cols) {
  const at::Tensor& t = tensor(o, name);
  if (t.dim() != 2) raise(PyExc_ValueError, "%s must have two dimensions", name);
  rows = t.size(0);
  cols = t.size(1);
}

struct Workspace {
  void* p;
  size_t bytes;
};
Workspace workspace(PyObject* o) {
  if (o == Py_None) return {nullptr, 0};
  void* p = device_ptr(o, at::ScalarType::Undefined, "ws", 0);
  return {p, (size_t)THPVariable_Unpack(o).nbytes()};
}

// An integer of any size, cut to its low 64 bits as ctypes cuts it (a policy
// version may be a hash).
int64_t integer(PyObject* o) {
  const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);
  if (v == (unsigned long long)-1 && PyErr_Occurred()) throw Raised{};
  return (int64_t)v;
}
float real(PyObject* o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw Raised{};
  return (float)v;
}

// The current stream, or the given one: an object with `cuda_stream`, which is
// an address or None (the null stream).
void* stream(PyObject* o) {
  if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
  PyObject* s = PyObject_GetAttrString(o, "cuda_stream");
  if (s == nullptr) throw Raised{};
  void* p = s == Py_None ? nullptr : PyLong_AsVoidPtr(s);
  Py_DECREF(s);
  if (p == nullptr && PyErr_Occurred()) throw Raised{};
  return p;
}

// The C struct inside a ctypes.Structure (of the class registered for it).
struct StructView {
  Py_buffer b{};
  StructView(PyObject* o, PyObject* type, size_t bytes, const char* what) {
    const int is = type == nullptr ? 0 : PyObject_IsInstance(o, type);
    if (is < 0) throw Raised{};
    if (is == 0) raise(PyExc_TypeError, "expected %s", what);
    if (PyObject_GetBuffer(o, &b, PyBUF_WRITABLE) != 0) throw Raised{};
    if ((size_t)b.len < bytes) {
      PyBuffer_Release(&b);
      raise(PyExc_TypeError, "%s is too small", what);
    }
  }
  ~StructView() { PyBuffer_Release(&b); }
  StructView(const StructView&) = delete;
  StructView& operator=(const StructView&) = delete;
};

PyObject *g_records, *g_cfg, *g_ring, *g_exec;  // the classes, held for good

struct Args {
  PyObject* const* a;
  Py_ssize_t n;
  PyObject* operator[](Py_ssize_t i) const {
    if (i >= n) raise(PyExc_TypeError, "%s", "too few arguments");
    return a[i];
  }
};

// A library call without the GIL; its status as a Python int.
template <class Call>
PyObject* run(Call&& call) {
  int st;
  Py_BEGIN_ALLOW_THREADS
  st = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

template <PyObject* (*kBody)(const Args&)>
PyObject* entry(PyObject*, PyObject* const* a, Py_ssize_t n) {
  try {
    return kBody(Args{a, n});
  } catch (const Raised&) {
  } catch (const std::exception& e) {
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, e.what());
  } catch (...) {
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, "unknown C++ exception");
  }
  return nullptr;
}

PyObject* set_structs(const Args& a) {
  PyObject** to[4] = {&g_records, &g_cfg, &g_ring, &g_exec};
  for (int i = 0; i < 4; ++i) {
    PyObject* old = *to[i];
    Py_INCREF(a[i]);
    *to[i] = a[i];
    Py_XDECREF(old);
  }
  Py_RETURN_NONE;
}

PyObject* group_advantage(const Args& a) {  // reward group_off adv ddof eps stream
  const int64_t n = numel_of(a[0], "reward"), groups = numel_of(a[1], "group_off") - 1;
  const float* reward = f32(a[0], "reward");
  const int32_t* off = i32(a[1], "group_off");
  float* adv = f32(a[2], "adv", n);
  const int32_t ddof = (int32_t)integer(a[3]);
  const float eps = real(a[4]);
  void* s = stream(a[5]);
  return run([&] { return rb_group_advantage(reward, off, (int32_t)groups, ddof, eps, adv, s); });
}

rb_batch batch(PyObject* out, const rb_sample_cfg& c) {
  const int64_t n = c.n_draw;
  const int64_t width = c.layout == RB_LAYOUT_PACKED ? c.max_tokens : n * c.l_max;
  auto at = [&](const char* key, auto&& get) {
    PyObject* t;
    if (PyDict_CheckExact(out)) {
      t = PyDict_GetItemString(out, key);
      if (t == nullptr) {
        PyErr_SetString(PyExc_KeyError, key);
        throw Raised{};
      }
      Py_INCREF(t);
    } else {
      PyObject* k = PyUnicode_FromString(key);
      if (k == nullptr) throw Raised{};
      t = PyObject_GetItem(out, k);
      Py_DECREF(k);
      if (t == nullptr) throw Raised{};
    }
    try {
      auto* p = get(t, key);
      Py_DECREF(t);  // `out` keeps it
      return p;
    } catch (...) {
      Py_DECREF(t);
      throw;
    }
  };
  auto ints = [](int64_t k) { return [k](PyObject* t, const char* s) { return i32(t, s, k); }; };
  auto floats = [](int64_t k) { return [k](PyObject* t, const char* s) { return f32(t, s, k); }; };
  rb_batch b;
  b.idx = at("idx", ints(n));
  b.adv = at("adv", floats(n));
  b.len = at("len", ints(n));
  b.age = at("age", ints(n));
  b.cu_seqlens = at("cu_seqlens", ints(n + 1));
  b.tokens = at("tokens", ints(width));
  b.old_logp = at("old_logp", floats(width));
  b.seq_of_token = at("seq_of_token", ints(width));
  b.n_tokens = at("n_tokens", [](PyObject* t, const char* s) { return i64(t, s, 1); });
  return b;
}

PyObject* sample_gather(const Args& a) {  // rec cfg out ws stream
  StructView rec(a[0], g_records, sizeof(rb_records), "an RbRecords");
  StructView cfg(a[1], g_cfg, sizeof(rb_sample_cfg), "an RbSampleCfg");
  const auto* r = static_cast<const rb_records*>(rec.b.buf);
  const auto* c = static_cast<const rb_sample_cfg*>(cfg.b.buf);
  const rb_batch b = batch(a[2], *c);
  const Workspace ws = workspace(a[3]);
  void* s = stream(a[4]);
  return run([&] { return rb_sample_gather(r, c, &b, ws.p, ws.bytes, s); });
}

PyObject* sample_gather_noalloc(const Args& a) {  // rec cfg out stream
  StructView rec(a[0], g_records, sizeof(rb_records), "an RbRecords");
  StructView cfg(a[1], g_cfg, sizeof(rb_sample_cfg), "an RbSampleCfg");
  const auto* r = static_cast<const rb_records*>(rec.b.buf);
  const auto* c = static_cast<const rb_sample_cfg*>(cfg.b.buf);
  const rb_batch b = batch(a[2], *c);
  void* s = stream(a[3]);
  return run([&] { return rb_sample_gather_noalloc(r, c, &b, s); });
}

PyObject* logprob_fwd(const Args& a) {  // hidden W tokens seq logp lse ws stream
  int64_t T, d;
  sizes_2d(a[0], "hidden", T, d);
  const int64_t V = size_of(a[1], "W", 0);
  if (size_of(a[1], "W", 1) != d) raise(PyExc_ValueError, "%s disagree on d", "hidden and W");
  const Workspace ws = workspace(a[6]);
  const uint16_t *h = bf16(a[0], "hidden", T * d), *W = bf16(a[1], "W", V * d);
  const int32_t *tok = i32(a[2], "tokens", T), *seq = i32_or_null(a[3], "seq_of_token", T);
  float *logp = f32(a[4], "logp", T), *lse = f32(a[5], "lse", T);
  void* s = stream(a[7]);
  return run([&] {
    return policy_logprob_fwd(h, W, tok, seq, T, (int32_t)d, (int32_t)V, logp, lse, ws.p, ws.bytes,
                              s);
  });
}

// logp old_logp seq adv seq_len n_seq_total loss dlogp stats ws eps_low eps_high stream
PyObject* loss_fwd_bwd(const Args& a) {
  const int64_t T = numel_of(a[0], "logp"), B = numel_of(a[3], "adv");
  const Workspace ws = workspace(a[9]);
  const float *logp = f32(a[0], "logp", T), *old = f32(a[1], "old_logp", T);
  const int32_t* seq = i32(a[2], "seq_of_token", T);
  const float* adv = f32(a[3], "adv", B);
  const int32_t* len = i32(a[4], "seq_len", B);
  const int64_t n_seq = integer(a[5]);
  float *loss = f32(a[6], "loss_accum", 1), *dlogp = f32(a[7], "dlogp", T),
        *stats = f32(a[8], "stats", 4);
  const float lo = real(a[10]), hi = real(a[11]);
  void* s = stream(a[12]);
  return run([&] {
    return policy_loss_fwd_bwd(logp, old, seq, adv, len, T, (int32_t)B, n_seq, lo, hi, loss, dlogp,
                               stats, ws.p, ws.bytes, s);
  });
}

// logp old_logp cu adv n_seq_total loss dlogp stats ws eps_low eps_high stream
PyObject* loss_seq_fwd_bwd(const Args& a) {
  const int64_t T = numel_of(a[0], "logp"), B = numel_of(a[3], "adv");
  const Workspace ws = workspace(a[8]);
  const float *logp = f32(a[0], "logp", T), *old = f32(a[1], "old_logp", T);
  const int32_t* cu = i32(a[2], "cu_seqlens", B + 1);
  const float* adv = f32(a[3], "adv", B);
  const int64_t n_seq = integer(a[4]);
  float *loss = f32(a[5], "loss_accum", 1), *dlogp = f32(a[6], "dlogp", T),
        *stats = f32(a[7], "stats", 4);
  const float lo = real(a[9]), hi = real(a[10]);
  void* s = stream(a[11]);
  return run([&] {
    return policy_loss_seq_fwd_bwd(logp, old, cu, adv, T, (int32_t)B, n_seq, lo, hi, loss, dlogp,
                                   stats, ws.p, ws.bytes, s);
  });
}

PyObject* asymre_coef(const Args& a) {  // reward group_off coef delta_v stream
  const int64_t n = numel_of(a[0], "reward"), groups = numel_of(a[1], "group_off") - 1;
  const float* reward = f32(a[0], "reward");
  const int32_t* off = i32(a[1], "group_off");
  const float dv = real(a[3]);
  float* coef = f32(a[2], "coef", n);
  void* s = stream(a[4]);
  return run([&] { return rb_asymre_coef(reward, off, (int32_t)groups, dv, coef, s); });
}

// logp seq coef n_seq_total loss dlogp stats ws stream
PyObject* asymre_fwd_bwd(const Args& a) {
  const int64_t T = numel_of(a[0], "logp"), B = numel_of(a[2], "coef");
  const Workspace ws = workspace(a[7]);
  const float* logp = f32(a[0], "logp", T);
  const int32_t* seq = i32(a[1], "seq_of_token", T);
  const float* coef = f32(a[2], "coef", B);
  const int64_t n_seq = integer(a[3]);
  float *loss = f32(a[4], "loss_accum", 1), *dlogp = f32(a[5], "dlogp", T),
        *stats = f32(a[6], "stats", 2);
  void* s = stream(a[8]);
  return run([&] {
    return policy_asymre_fwd_bwd(logp, seq, coef, T, (int32_t)B, n_seq, loss, dlogp, stats, ws.p,
                                 ws.bytes, s);
  });
}

// hidden W tokens seq lse dlogp dhidden dW ws accumulate stream
PyObject* logprob_bwd(const Args& a) {
  int64_t T, d;
  sizes_2d(a[0], "hidden", T, d);
  const int64_t V = size_of(a[1], "W", 0);
  const Workspace ws = workspace(a[8]);
  const uint16_t *h = bf16(a[0], "hidden", T * d), *W = bf16(a[1], "W", V * d);
  const int32_t *tok = i32(a[2], "tokens", T), *seq = i32_or_null(a[3], "seq_of_token", T);
  const float *lse = f32(a[4], "lse", T), *dlogp = f32(a[5], "dlogp", T);
  float *dh = f32(a[6], "dhidden", T * d), *dW = f32(a[7], "dW", V * d);
  const int acc = (int)integer(a[9]);
  void* s = stream(a[10]);
  return run([&] {
    return policy_logprob_bwd(h, W, tok, seq, lse, dlogp, T, (int32_t)d, (int32_t)V, dh, dW, acc,
                              ws.p, ws.bytes, s);
  });
}

// hidden W tokens seq old adv seq_len n_seq_total logp lse entropy loss dlogp stats dhidden dW
// ws accumulate eps_low eps_high exec stream
PyObject* fused_fwd_bwd(const Args& a) {
  int64_t T, d;
  sizes_2d(a[0], "hidden", T, d);
  const int64_t V = size_of(a[1], "W", 0), B = numel_of(a[5], "adv");
  const Workspace ws = workspace(a[16]);
  const uint16_t *h = bf16(a[0], "hidden", T * d), *W = bf16(a[1], "W", V * d);
  const int32_t *tok = i32(a[2], "tokens", T), *seq = i32(a[3], "seq_of_token", T);
  const float *old = f32(a[4], "old_logp", T), *adv = f32(a[5], "adv", B);
  const int32_t* len = i32(a[6], "seq_len", B);
  const int64_t n_seq = integer(a[7]);
  float *logp = f32(a[8], "logp", T), *lse = f32(a[9], "lse", T),
        *ent = f32_or_null(a[10], "entropy", T), *loss = f32(a[11], "loss_accum", 1),
        *dlogp = f32(a[12], "dlogp", T), *stats = f32(a[13], "stats", 4),
        *dh = f32(a[14], "dhidden", T * d), *dW = f32(a[15], "dW", V * d);
  const int acc = (int)integer(a[17]);
  const float lo = real(a[18]), hi = real(a[19]);
  void* s = stream(a[21]);
  auto call = [&](const rbp_exec* ex) {
    return run([&] {
      return policy_fused_fwd_bwd(h, W, tok, seq, old, adv, len, T, (int32_t)d, (int32_t)V,
                                  (int32_t)B, n_seq, lo, hi, logp, lse, ent, loss, dlogp, stats,
                                  dh, dW, acc, ws.p, ws.bytes, ex, s);
    });
  };
  if (a[20] == Py_None) return call(nullptr);
  StructView ex(a[20], g_exec, sizeof(rbp_exec), "an RbpExec");
  return call(static_cast<const rbp_exec*>(ex.b.buf));
}

// ring group_off length src_off reward version tokens old_logp ddof eps stream
PyObject* push(const Args& a) {
  const int64_t n = numel_of(a[2], "length"), groups = numel_of(a[1], "group_off") - 1;
  StructView ring(a[0], g_ring, sizeof(rb_ring), "an RbRing");
  auto* r = static_cast<rb_ring*>(ring.b.buf);
  const int32_t *off = i32(a[1], "group_off", groups + 1), *len = i32(a[2], "length", n);
  const int64_t* src = i64(a[3], "src_off", n);
  const float* reward = f32(a[4], "reward", n);
  const int32_t version = (int32_t)integer(a[5]);
  const int32_t* tok = i32(a[6], "tokens");
  const float* old = f32(a[7], "old_logp");
  const int32_t ddof = (int32_t)integer(a[8]);
  const float eps = real(a[9]);
  void* s = stream(a[10]);
  return run([&] {
    return rb_push(r, (int32_t)n, (int32_t)groups, off, len, src, reward, version, tok, old, ddof,
                   eps, s);
  });
}

// idx head capacity step use_count last_step since ws stream
PyObject* note_use(const Args& a) {
  const int64_t n = numel_of(a[0], "idx");
  const Workspace ws = workspace(a[7]);
  const int64_t head = integer(a[1]), cap = integer(a[2]), step = integer(a[3]);
  const int32_t* idx = i32(a[0], "idx", n);
  int32_t* uses = i32(a[4], "use_count", cap);
  int64_t* last = i64(a[5], "last_step", cap);
  int32_t* since = i32_or_null(a[6], "since", n);
  void* s = stream(a[8]);
  return run(
      [&] { return rb_note_use(idx, n, head, cap, step, uses, last, since, ws.p, ws.bytes, s); });
}

PyObject* hist_accumulate(const Args& a) {  // values hist lo stream
  const int64_t n = numel_of(a[0], "values"), bins = numel_of(a[1], "hist");
  const int32_t* v = i32(a[0], "values", n);
  const int32_t lo = (int32_t)integer(a[2]);
  int64_t* hist = i64(a[1], "hist");
  void* s = stream(a[3]);
  return run([&] { return rb_hist_accumulate(v, n, lo, (int32_t)bins, hist, s); });
}

#define RBP_ENTRY(name) \
  {#name, (PyCFunction)(void (*)(void))entry<name>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {RBP_ENTRY(set_structs),
                         RBP_ENTRY(group_advantage),
                         RBP_ENTRY(sample_gather),
                         RBP_ENTRY(sample_gather_noalloc),
                         RBP_ENTRY(logprob_fwd),
                         RBP_ENTRY(loss_fwd_bwd),
                         RBP_ENTRY(loss_seq_fwd_bwd),
                         RBP_ENTRY(asymre_coef),
                         RBP_ENTRY(asymre_fwd_bwd),
                         RBP_ENTRY(logprob_bwd),
                         RBP_ENTRY(fused_fwd_bwd),
                         RBP_ENTRY(push),
                         RBP_ENTRY(note_use),
                         RBP_ENTRY(hist_accumulate),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
