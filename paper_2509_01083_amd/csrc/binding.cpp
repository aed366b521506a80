// Marshalling of the Python binding: each function takes the tensors and
// numbers of one entry point of libdsde, checks the tensors (device, type,
// contiguity, size), fetches their device pointers and the current stream, and
// calls the entry point without the interpreter lock.  The same checks in
// Python (40 tensors for a fused step, about half a microsecond each, and
// ctypes' conversion of 45 arguments) took 21 us of host time, as long as the
// step's kernels take in small batches.
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <dlfcn.h>
#include <torch/csrc/autograd/python_variable.h>

#include <string>

#include "dsde.h"

namespace {

PyObject *g_error = nullptr;  // paper_2509_01083_amd.DsdeError

// The entry points, looked up in the library that the package has loaded
// (set_library), which need not be the one beside this file.
#define DSDE_ENTRIES(X)                                                                                         \
  X(dsde_status_string)                                                                                         \
  X(dsde_verify) X(dsde_step) X(dsde_step_static) X(dsde_kld_signal) X(dsde_next_sl) X(dsde_calibration_update) \
  X(dsde_shard_stats) X(dsde_shard_accept) X(dsde_shard_accept_step) X(dsde_shard_draw_mass) X(dsde_shard_draw_pick)
struct Library {
#define X(name) decltype(&::name) name;
  DSDE_ENTRIES(X)
#undef X
} g_lib;

struct Failed {};  // a Python exception is set

[[noreturn]] void fail(const std::string &text) {
  PyErr_SetString(g_error ? g_error : PyExc_RuntimeError, text.c_str());
  throw Failed{};
}

// The arguments of one call, taken in order.
struct Args {
  PyObject *const *at;
  PyObject *const *end;

  PyObject *next() {
    if (at == end) {
      PyErr_SetString(PyExc_TypeError, "too few arguments");
      throw Failed{};
    }
    return *at++;
  }
  int64_t integer() {
    // any object with __index__; wraps like a C conversion (the library checks the ranges)
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(next());
    if (v == ~0ull && PyErr_Occurred()) throw Failed{};
    return int64_t(v);
  }
  int32_t int32() { return int32_t(integer()); }
  float real() {
    const double v = PyFloat_AsDouble(next());
    if (v == -1.0 && PyErr_Occurred()) throw Failed{};
    return float(v);
  }
  bool flag() { return PyObject_IsTrue(next()) > 0; }
  // The raw stream: an integer handle, or None for torch's current stream.
  void *stream() {
    PyObject *o = next();
    if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
    void *p = PyLong_AsVoidPtr(o);
    if (!p && PyErr_Occurred()) throw Failed{};
    return p;
  }
  void done() {
    if (at != end) {
      PyErr_SetString(PyExc_TypeError, "too many arguments");
      throw Failed{};
    }
  }
};

constexpr int kAny = -1;
constexpr int kI32 = int(at::ScalarType::Int), kI64 = int(at::ScalarType::Long), kU8 = int(at::ScalarType::Byte);
constexpr int kF32 = int(at::ScalarType::Float), kF64 = int(at::ScalarType::Double);

const char *type_name(int type) {
  return type == kI32   ? "torch.int32"
         : type == kI64 ? "torch.int64"
         : type == kU8  ? "torch.uint8"
         : type == kF32 ? "torch.float32"
                        : "torch.float64";
}

// Device pointer of a contiguous GPU tensor of `type` with at least `n`
// elements; NULL for None.
void *ptr(PyObject *o, int type, int64_t n, const char *name) {
  if (o == Py_None) return nullptr;
  if (!THPVariable_Check(o)) fail(std::string(name) + " must be a GPU tensor");
  const at::Tensor &t = THPVariable_Unpack(o);
  if (!t.is_cuda()) fail(std::string(name) + " must be a GPU tensor");
  if (type != kAny && int(t.scalar_type()) != type) {
    std::string got = "another type";
    if (PyObject *d = PyObject_GetAttrString(o, "dtype")) {
      if (PyObject *s = PyObject_Str(d)) {
        if (const char *c = PyUnicode_AsUTF8(s)) got = c;
        Py_DECREF(s);
      }
      Py_DECREF(d);
    }
    PyErr_Clear();
    fail(std::string(name) + " must be " + type_name(type) + ", got " + got);
  }
  if (!t.is_contiguous()) fail(std::string(name) + " must be contiguous");
  if (t.numel() < n)
    fail(std::string(name) + " has " + std::to_string(t.numel()) + " elements, needs " + std::to_string(n));
  return t.data_ptr();
}
template <typename T>
T *take(Args &a, int type, int64_t n, const char *name) {
  return static_cast<T *>(ptr(a.next(), type, n, name));
}
int64_t size_of(PyObject *o, int64_t dim, const char *name) {
  if (!THPVariable_Check(o)) fail(std::string(name) + " must be a GPU tensor");
  const at::Tensor &t = THPVariable_Unpack(o);
  if (t.dim() <= dim) fail(std::string(name) + " has too few dimensions");
  return t.size(dim);
}
// Outputs are taken from the caller's dict, or other mapping, by key.  A
// mapping's item is a new reference, dropped once its pointer is known (as
// with the inputs, the caller keeps the tensor itself alive).
template <typename T>
T *out(PyObject *dict, const char *key, int type, int64_t n) {
  if (PyDict_CheckExact(dict)) {
    PyObject *o = PyDict_GetItemString(dict, key);
    if (!o) {
      PyErr_SetString(PyExc_KeyError, key);
      throw Failed{};
    }
    return static_cast<T *>(ptr(o, type, n, key));
  }
  struct Ref {
    PyObject *o;
    ~Ref() { Py_XDECREF(o); }
  };
  const Ref k{PyUnicode_FromString(key)};
  const Ref o{k.o ? PyObject_GetItem(dict, k.o) : nullptr};
  if (!o.o) throw Failed{};
  return static_cast<T *>(ptr(o.o, type, n, key));
}

int32_t logits_type(const at::Tensor &t) {
  if (t.scalar_type() == at::ScalarType::BFloat16) return DSDE_BF16;
  if (t.scalar_type() == at::ScalarType::Float) return DSDE_FP32;
  fail("logits must be bfloat16 or float32");
}

// The target and draft rows of a call.
struct Rows {
  const void *target, *draft;
  int32_t dtype;
  int64_t V, N;
};
// A draft that does not match the target is refused: the kernels index both with
// the target's element size and width.  `empty` refuses one without rows too,
// which nothing reads.
Rows take_rows(Args &a, int64_t B, const char *what, bool empty = true) {
  PyObject *t = a.next(), *d = a.next();
  const int64_t rows = size_of(t, 0, "target"), V = size_of(t, 1, "target");
  const at::Tensor &tt = THPVariable_Unpack(t);
  Rows r;
  r.dtype = logits_type(tt);
  r.V = V;
  r.N = d == Py_None ? 0 : size_of(d, 0, "draft");
  if (d != Py_None && (empty || r.N > 0)) {
    const at::Tensor &dt = THPVariable_Unpack(d);
    if (dt.scalar_type() != tt.scalar_type() || (r.N > 0 && size_of(d, 1, "draft") != V))
      fail(std::string("draft ") + what + " must match the target's dtype and vocabulary");
  }
  if (rows != r.N + B)
    fail("target has " + std::to_string(rows) + " rows, expected N + B = " + std::to_string(r.N + B));
  r.target = ptr(t, kAny, 0, "target");
  r.draft = r.N > 0 ? ptr(d, kAny, 0, "draft") : nullptr;
  return r;
}

// Per-sequence and per-position inputs in the order of the entry points.
struct Batch {
  const int32_t *sl, *cu_sl, *tokens;
  const float *temperature, *u_acc, *u_res;
};
Batch take_batch(PyObject *const *p, int64_t B, int64_t N) {
  Batch x;
  x.sl = static_cast<const int32_t *>(ptr(p[0], kI32, B, "sl"));
  x.cu_sl = static_cast<const int32_t *>(ptr(p[1], kI32, B + 1, "cu_sl"));
  x.tokens = N > 0 ? static_cast<const int32_t *>(ptr(p[2], kI32, N, "draft_tokens")) : nullptr;
  x.temperature = static_cast<const float *>(ptr(p[3], kF32, B, "temperature"));
  x.u_acc = N > 0 ? static_cast<const float *>(ptr(p[4], kF32, N, "u_acc")) : nullptr;
  x.u_res = static_cast<const float *>(ptr(p[5], kF32, B, "u_res"));
  return x;
}

// The outputs every verification call has.
struct VerifyOut {
  int32_t *accepted, *tokens;
  float *kld, *entropy;
  double *row_lse;
};
VerifyOut take_verify_out(PyObject *dict, PyObject *row_lse, bool entropy, int64_t B, int64_t N, int32_t k_max) {
  VerifyOut o;
  o.accepted = out<int32_t>(dict, "accepted", kI32, B);
  o.tokens = out<int32_t>(dict, "tokens", kI32, B * (k_max + 1));
  o.kld = N > 0 ? out<float>(dict, "kld", kF32, N) : nullptr;
  o.row_lse = static_cast<double *>(ptr(row_lse, kF64, 2 * N, "row_lse"));
  o.entropy = entropy && N > 0 ? out<float>(dict, "draft_entropy", kF32, N) : nullptr;
  return o;
}

// The ring, the signal's and the rule's parameters and outputs of the fused calls.
struct Signal {
  float *hist;
  int32_t *head, *count;
  const float *sl_max;
  int32_t W, n_short, n_long;
  float delta, eps, sl_min;
  int32_t sl_hi;
  const int32_t *budget;
  float *mu_last, *var_short, *var_long, *wvir, *sf, *sl_hat, *sl_cap;
  int32_t *sl_next;
};
Signal take_signal(Args &a, PyObject *dict, int64_t B) {
  Signal s;
  PyObject *hist = a.next();
  const int64_t W = size_of(hist, 1, "hist");
  s.W = int32_t(W);
  s.hist = static_cast<float *>(ptr(hist, kF32, B * W, "hist"));
  s.head = take<int32_t>(a, kI32, B, "head");
  s.count = take<int32_t>(a, kI32, B, "count");
  s.sl_max = take<float>(a, kF32, B, "sl_max");
  s.n_short = a.int32();
  s.n_long = a.int32();
  s.delta = a.real();
  s.eps = a.real();
  s.sl_min = a.real();
  s.sl_hi = a.int32();
  s.budget = take<int32_t>(a, kI32, B, "budget");
  s.mu_last = out<float>(dict, "mu_last", kF32, B);
  s.var_short = out<float>(dict, "var_short", kF32, B);
  s.var_long = out<float>(dict, "var_long", kF32, B);
  s.wvir = out<float>(dict, "wvir", kF32, B);
  s.sf = out<float>(dict, "sf", kF32, B);
  s.sl_hat = out<float>(dict, "sl_hat", kF32, B);
  s.sl_cap = out<float>(dict, "sl_cap", kF32, 1);
  s.sl_next = out<int32_t>(dict, "sl_next", kI32, B);
  return s;
}

void *take_workspace(Args &a, size_t *bytes) {
  PyObject *o = a.next();
  void *p = ptr(o, kU8, 0, "workspace");
  *bytes = o == Py_None ? 0 : size_t(THPVariable_Unpack(o).numel());
  return p;
}

template <typename F>
void call(F f) {
  int32_t rc;
  Py_BEGIN_ALLOW_THREADS rc = f();
  Py_END_ALLOW_THREADS if (rc != DSDE_OK)
      fail(std::string("libdsde: ") + g_lib.dsde_status_string(rc) + " (status " + std::to_string(rc) + ")");
}

// Runs one function body; C++ exceptions become Python ones.
template <typename F>
PyObject *guarded(PyObject *const *args, Py_ssize_t n, F f) {
  try {
    Args a{args, args + n};
    f(a);
    Py_RETURN_NONE;
  } catch (const Failed &) {
  } catch (const std::exception &e) {
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, e.what());
  } catch (...) {
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, "unknown C++ exception");
  }
  return nullptr;
}

// verify(target, draft, sl, cu_sl, draft_tokens, temperature, u_acc, u_res, k_max, pad_id, out, row_lse,
//        draft_entropy, workspace, stream)
PyObject *py_verify(PyObject *, PyObject *const *args, Py_ssize_t n) {
  return guarded(args, n, [&](Args &a) {
    if (n < 8) a.at = a.end;
    PyObject *const *batch = args + 2;
    const int64_t B = n < 8 ? 0 : size_of(batch[0], 0, "sl");
    const Rows r = take_rows(a, B, "logits");
    const Batch x = take_batch(batch, B, r.N);
    a.at += 6;
    const int32_t k_max = a.int32(), pad = a.int32();
    PyObject *dict = a.next(), *lse = a.next();
    const VerifyOut o = take_verify_out(dict, lse, a.flag(), B, r.N, k_max);
    uint32_t *err = out<uint32_t>(dict, "seq_err", kAny, B);
    size_t bytes;
    void *ws = take_workspace(a, &bytes), *stream = a.stream();
    a.done();
    call([&] {
      return g_lib.dsde_verify(r.target, r.draft, r.dtype, r.V, int32_t(B), r.N, k_max, x.sl, x.cu_sl, x.tokens,
                         x.temperature, x.u_acc, x.u_res, pad, o.accepted, o.tokens, o.kld, err, o.row_lse, o.entropy,
                         ws, bytes, stream);
    });
  });
}

// step(target, draft, sl, cu_sl, draft_tokens, temperature, u_acc, u_res, k_max, pad_id, out, row_lse,
//      draft_entropy, hist, head, count, sl_max, n_short, n_long, delta, eps, sl_min, sl_hi, budget, workspace,
//      stream); workspace False: dsde_step_static
PyObject *py_step(PyObject *, PyObject *const *args, Py_ssize_t n) {
  return guarded(args, n, [&](Args &a) {
    if (n < 8) a.at = a.end;
    PyObject *const *batch = args + 2;
    const int64_t B = n < 8 ? 0 : size_of(batch[0], 0, "sl");
    const Rows r = take_rows(a, B, "logits", false);
    const Batch x = take_batch(batch, B, r.N);
    a.at += 6;
    const int32_t k_max = a.int32(), pad = a.int32();
    PyObject *dict = a.next(), *lse = a.next();
    const VerifyOut o = take_verify_out(dict, lse, a.flag(), B, r.N, k_max);
    const Signal s = take_signal(a, dict, B);
    uint32_t *err = out<uint32_t>(dict, "seq_err", kAny, B);
    const bool fixed = a.at < a.end && *a.at == Py_False;
    size_t bytes = 0;
    void *ws = nullptr;
    if (fixed)
      a.next();
    else
      ws = take_workspace(a, &bytes);
    void *stream = a.stream();
    a.done();
    call([&] {
      if (fixed)
        return g_lib.dsde_step_static(r.target, r.draft, r.dtype, r.V, int32_t(B), r.N, k_max, x.sl, x.cu_sl, x.tokens,
                                x.temperature, x.u_acc, x.u_res, pad, o.accepted, o.tokens, o.kld, o.row_lse,
                                o.entropy, s.hist, s.head, s.count, s.W, s.n_short, s.n_long, s.delta, s.eps,
                                s.mu_last, s.var_short, s.var_long, s.wvir, s.sf, s.sl_max, s.sl_min, s.sl_hi,
                                s.budget, s.sl_hat, s.sl_cap, s.sl_next, err, stream);
      return g_lib.dsde_step(r.target, r.draft, r.dtype, r.V, int32_t(B), r.N, k_max, x.sl, x.cu_sl, x.tokens,
                       x.temperature, x.u_acc, x.u_res, pad, o.accepted, o.tokens, o.kld, o.row_lse, o.entropy, s.hist,
                       s.head, s.count, s.W, s.n_short, s.n_long, s.delta, s.eps, s.mu_last, s.var_short, s.var_long,
                       s.wvir, s.sf, s.sl_max, s.sl_min, s.sl_hi, s.budget, s.sl_hat, s.sl_cap, s.sl_next, err, ws,
                       bytes, stream);
    });
  });
}

// kld_signal(sl, cu_sl, kld, hist, head, count, n_short, n_long, delta, eps, out, stream)
PyObject *py_kld_signal(PyObject *, PyObject *const *args, Py_ssize_t n) {
  return guarded(args, n, [&](Args &a) {
    PyObject *sl_o = a.next(), *cu_o = a.next(), *kld_o = a.next(), *hist_o = a.next();
    const int64_t B = size_of(sl_o, 0, "sl"), N = size_of(kld_o, 0, "kld"), W = size_of(hist_o, 1, "hist");
    const auto *sl = static_cast<const int32_t *>(ptr(sl_o, kI32, B, "sl"));
    const auto *cu = static_cast<const int32_t *>(ptr(cu_o, kI32, B + 1, "cu_sl"));
    const auto *kld = N > 0 ? static_cast<const float *>(ptr(kld_o, kF32, N, "kld")) : nullptr;
    auto *hist = static_cast<float *>(ptr(hist_o, kF32, B * W, "hist"));
    int32_t *head = take<int32_t>(a, kI32, B, "head"), *count = take<int32_t>(a, kI32, B, "count");
    const int32_t n_short = a.int32(), n_long = a.int32();
    const float delta = a.real(), eps = a.real();
    PyObject *d = a.next();
    float *mu = out<float>(d, "mu_last", kF32, B), *vs = out<float>(d, "var_short", kF32, B);
    float *vl = out<float>(d, "var_long", kF32, B), *wvir = out<float>(d, "wvir", kF32, B);
    float *sf = out<float>(d, "sf", kF32, B);
    uint32_t *err = out<uint32_t>(d, "seq_err", kAny, B);
    void *stream = a.stream();
    a.done();
    call([&] {
      return g_lib.dsde_kld_signal(int32_t(B), N, sl, cu, kld, hist, head, count, int32_t(W), n_short, n_long, delta, eps, mu,
                             vs, vl, wvir, sf, err, stream);
    });
  });
}

// next_sl(sf, wvir, sl_max, sl_min, sl_hi, budget, out, stream)
PyObject *py_next_sl(PyObject *, PyObject *const *args, Py_ssize_t n) {
  return guarded(args, n, [&](Args &a) {
    PyObject *sf_o = a.next();
    const int64_t B = size_of(sf_o, 0, "sf");
    const auto *sf = static_cast<const float *>(ptr(sf_o, kF32, B, "sf"));
    const float *wvir = take<float>(a, kF32, B, "wvir"), *sl_max = take<float>(a, kF32, B, "sl_max");
    const float sl_min = a.real();
    const int32_t sl_hi = a.int32();
    const int32_t *budget = take<int32_t>(a, kI32, B, "budget");
    PyObject *d = a.next();
    float *hat = out<float>(d, "sl_hat", kF32, B), *cap = out<float>(d, "sl_cap", kF32, 1);
    int32_t *next = out<int32_t>(d, "sl_next", kI32, B);
    uint32_t *err = out<uint32_t>(d, "seq_err", kAny, B);
    void *stream = a.stream();
    a.done();
    call([&] {
      return g_lib.dsde_next_sl(int32_t(B), sf, wvir, sl_max, sl_min, sl_hi, budget, hat, cap, next, err, stream);
    });
  });
}

// calibration_update(sl, cu_sl, accepted, kld, seq_err, state, stream)
PyObject *py_calibration_update(PyObject *, PyObject *const *args, Py_ssize_t n) {
  return guarded(args, n, [&](Args &a) {
    PyObject *sl_o = a.next(), *cu_o = a.next(), *acc_o = a.next(), *kld_o = a.next(), *err_o = a.next();
    PyObject *d = a.next();
    const int64_t B = size_of(sl_o, 0, "sl"), N = size_of(kld_o, 0, "kld");
    const auto *sl = static_cast<const int32_t *>(ptr(sl_o, kI32, B, "sl"));
    const auto *cu = static_cast<const int32_t *>(ptr(cu_o, kI32, B + 1, "cu_sl"));
    const auto *acc = static_cast<const int32_t *>(ptr(acc_o, kI32, B, "accepted"));
    const auto *kld = N > 0 ? static_cast<const float *>(ptr(kld_o, kF32, N, "kld")) : nullptr;
    const auto *err = static_cast<const uint32_t *>(ptr(err_o, kAny, B, "seq_err"));
    int32_t *a_max = out<int32_t>(d, "a_max", kI32, B);
    double *sum = out<double>(d, "kld_sum", kF64, B);
    int64_t *cnt = out<int64_t>(d, "kld_count", kI64, B);
    float *kmax = out<float>(d, "kld_max", kF32, B);
    void *stream = a.stream();
    a.done();
    call([&] { return g_lib.dsde_calibration_update(int32_t(B), N, sl, cu, acc, kld, err, a_max, sum, cnt, kmax, stream); });
  });
}

// shard_stats(target, draft, v_begin, V, sl, cu_sl, draft_tokens, temperature, k_max, workspace, part, seq_err, stream)
PyObject *py_shard_stats(PyObject *, PyObject *const *args, Py_ssize_t n) {
  return guarded(args, n, [&](Args &a) {
    if (n < 8) a.at = a.end;
    const int64_t B = n < 8 ? 0 : size_of(args[4], 0, "sl");
    const Rows r = take_rows(a, B, "slice");
    const int64_t v_begin = a.integer(), V = a.integer();
    const int32_t *sl = take<int32_t>(a, kI32, B, "sl"), *cu = take<int32_t>(a, kI32, B + 1, "cu_sl");
    PyObject *tok_o = a.next();
    const auto *tok = r.N > 0 ? static_cast<const int32_t *>(ptr(tok_o, kI32, r.N, "draft_tokens")) : nullptr;
    const float *temp = take<float>(a, kF32, B, "temperature");
    const int32_t k_max = a.int32();
    size_t bytes;
    void *ws = take_workspace(a, &bytes);
    PyObject *part_o = a.next();
    void *part = r.N > 0 ? ptr(part_o, kU8, r.N * int64_t(sizeof(dsde_shard_partial)), "part") : nullptr;
    uint32_t *err = take<uint32_t>(a, kAny, B, "seq_err");
    void *stream = a.stream();
    a.done();
    call([&] {
      return g_lib.dsde_shard_stats(r.target, r.draft, r.dtype, r.V, v_begin, V, int32_t(B), r.N, k_max, sl, cu, tok, temp,
                              static_cast<dsde_shard_partial *>(part), err, ws, bytes, stream);
    });
  });
}

// shard_accept(fused, parts, V, sl, cu_sl, draft_tokens, temperature, u_acc, u_res, k_max, pad_id, out, row_lse,
//              draft_entropy, seq_err[, hist, head, count, sl_max, n_short, n_long, delta, eps, sl_min, sl_hi, budget],
//              stream); parts packed [G, N, 64]
PyObject *py_shard_accept(PyObject *, PyObject *const *args, Py_ssize_t n) {
  return guarded(args, n, [&](Args &a) {
    const bool fused = a.flag();
    PyObject *parts_o = a.next();
    const int64_t G = size_of(parts_o, 0, "parts"), V = a.integer();
    if (a.end - a.at < 6) a.at = a.end;
    PyObject *const *batch = a.at;
    PyObject *sl_o = a.next();
    const int64_t B = size_of(sl_o, 0, "sl");
    const int64_t N = batch[2] == Py_None ? 0 : size_of(batch[2], 0, "draft_tokens");
    a.at = batch + 6;
    const Batch x = take_batch(batch, B, N);
    const auto *parts = N > 0 ? static_cast<const dsde_shard_partial *>(
                                    ptr(parts_o, kU8, G * N * int64_t(sizeof(dsde_shard_partial)), "parts"))
                              : nullptr;
    const int32_t k_max = a.int32(), pad = a.int32();
    PyObject *dict = a.next(), *lse = a.next();
    const VerifyOut o = take_verify_out(dict, lse, a.flag(), B, N, k_max);
    auto *jobs = out<dsde_draw_job>(dict, "jobs", kU8, B * int64_t(sizeof(dsde_draw_job)));
    uint32_t *err = take<uint32_t>(a, kAny, B, "seq_err");
    Signal s{};
    if (fused) s = take_signal(a, dict, B);
    void *stream = a.stream();
    a.done();
    call([&] {
      if (!fused)
        return g_lib.dsde_shard_accept(int32_t(G), parts, V, int32_t(B), N, k_max, x.sl, x.cu_sl, x.tokens, x.temperature,
                                 x.u_acc, x.u_res, pad, o.accepted, o.tokens, o.kld, o.row_lse, o.entropy, jobs, err,
                                 stream);
      return g_lib.dsde_shard_accept_step(int32_t(G), parts, V, int32_t(B), N, k_max, x.sl, x.cu_sl, x.tokens, x.temperature,
                                    x.u_acc, x.u_res, pad, o.accepted, o.tokens, o.kld, o.row_lse, o.entropy, jobs,
                                    s.hist, s.head, s.count, s.W, s.n_short, s.n_long, s.delta, s.eps, s.mu_last,
                                    s.var_short, s.var_long, s.wvir, s.sf, s.sl_max, s.sl_min, s.sl_hi, s.budget,
                                    s.sl_hat, s.sl_cap, s.sl_next, err, stream);
    });
  });
}

// shard_draw_mass(target, draft, v_begin, part, jobs, k_max, workspace, mass, stream)
PyObject *py_shard_draw_mass(PyObject *, PyObject *const *args, Py_ssize_t n) {
  return guarded(args, n, [&](Args &a) {
    if (n < 5) a.at = a.end;
    const int64_t B = n < 5 ? 0 : size_of(args[4], 0, "jobs");
    const Rows r = take_rows(a, B, "slice");
    const int64_t v_begin = a.integer();
    PyObject *part_o = a.next();
    void *part = r.N > 0 ? ptr(part_o, kU8, r.N * int64_t(sizeof(dsde_shard_partial)), "part") : nullptr;
    auto *jobs = take<dsde_draw_job>(a, kU8, B * int64_t(sizeof(dsde_draw_job)), "jobs");
    const int32_t k_max = a.int32();
    size_t bytes;
    void *ws = take_workspace(a, &bytes);
    auto *mass = take<dsde_shard_mass>(a, kU8, B * int64_t(sizeof(dsde_shard_mass)), "mass");
    void *stream = a.stream();
    a.done();
    call([&] {
      return g_lib.dsde_shard_draw_mass(r.target, r.draft, r.dtype, r.V, v_begin, int32_t(B), r.N, k_max,
                                  static_cast<const dsde_shard_partial *>(part), jobs, mass, ws, bytes, stream);
    });
  });
}

// shard_draw_pick(g, masses, target, draft, v_begin, jobs, k_max, pad_id, accepted, tokens, drawn, seq_err, workspace,
//                 stream)
PyObject *py_shard_draw_pick(PyObject *, PyObject *const *args, Py_ssize_t n) {
  return guarded(args, n, [&](Args &a) {
    const int32_t g = a.int32();
    PyObject *masses_o = a.next();
    if (n < 6) a.at = a.end;
    const int64_t G = size_of(masses_o, 0, "masses"), B = n < 6 ? 0 : size_of(args[5], 0, "jobs");
    const Rows r = take_rows(a, B, "slice");
    const auto *masses = static_cast<const dsde_shard_mass *>(
        ptr(masses_o, kU8, G * B * int64_t(sizeof(dsde_shard_mass)), "masses"));
    const int64_t v_begin = a.integer();
    auto *jobs = take<dsde_draw_job>(a, kU8, B * int64_t(sizeof(dsde_draw_job)), "jobs");
    const int32_t k_max = a.int32(), pad = a.int32();
    int32_t *accepted = take<int32_t>(a, kI32, B, "accepted");
    int32_t *tokens = take<int32_t>(a, kI32, B * (k_max + 1), "tokens"), *drawn = take<int32_t>(a, kI32, B, "drawn");
    uint32_t *err = take<uint32_t>(a, kAny, B, "seq_err");
    size_t bytes;
    void *ws = take_workspace(a, &bytes), *stream = a.stream();
    a.done();
    call([&] {
      return g_lib.dsde_shard_draw_pick(int32_t(G), g, masses, r.target, r.draft, r.dtype, r.V, v_begin, int32_t(B), r.N,
                                  k_max, jobs, pad, accepted, tokens, drawn, err, ws, bytes, stream);
    });
  });
}

// set_error(type): the exception the checks raise
PyObject *py_set_error(PyObject *, PyObject *type) {
  Py_INCREF(type);
  Py_XDECREF(g_error);
  g_error = type;
  Py_RETURN_NONE;
}

// set_library(handle): takes the entry points from a library's dlopen handle
PyObject *py_set_library(PyObject *, PyObject *handle) {
  void *h = PyLong_AsVoidPtr(handle);
  if (!h) {
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "no library handle");
    return nullptr;
  }
  Library lib;
#define X(name)                                                                      \
  if (!(lib.name = reinterpret_cast<decltype(lib.name)>(dlsym(h, #name)))) {         \
    PyErr_SetString(g_error ? g_error : PyExc_RuntimeError, "libdsde lacks " #name); \
    return nullptr;                                                                  \
  }
  DSDE_ENTRIES(X)
#undef X
  g_lib = lib;
  Py_RETURN_NONE;
}

using Fast = PyObject *(*)(PyObject *, PyObject *const *, Py_ssize_t);
PyMethodDef entry(const char *name, Fast f) {
  return PyMethodDef{name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr};
}
PyMethodDef g_methods[] = {entry("verify", py_verify),
                           entry("step", py_step),
                           entry("kld_signal", py_kld_signal),
                           entry("next_sl", py_next_sl),
                           entry("calibration_update", py_calibration_update),
                           entry("shard_stats", py_shard_stats),
                           entry("shard_accept", py_shard_accept),
                           entry("shard_draw_mass", py_shard_draw_mass),
                           entry("shard_draw_pick", py_shard_draw_pick),
                           {"set_error", py_set_error, METH_O, nullptr},
                           {"set_library", py_set_library, METH_O, nullptr},
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, g_methods};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&g_module); }
