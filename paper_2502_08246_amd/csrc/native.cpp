// _native: the calls of include/saap.h as functions on torch tensors, in C++ against the CPython and ATen interfaces.
//
// A decode step is three or four calls whose kernels take 4 to 13 us each; marshalled in Python (ctypes, shapes as
// tuples, a workspace record per call) every call held the host for 10 to 15 us, so that a step called from Python
// took 44 us for 28 us of kernels.  Here a call costs a couple of microseconds on top of its kernel launches.
//
// Marshalling only: shapes are read off the tensors, outputs are allocated unless the caller passes them, the
// workspace is the shared one of the current stream unless the caller passes one, pointers and the current stream go to the
// C call, a status other than SAAP_OK is raised as SaapError.  The interpreter lock is released around the C call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <ATen/ops/zeros.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <initializer_list>
#include <string>
#include <thread>
#include <vector>

#include "saap.h"

namespace {

using at::Tensor;

// ---- errors ------------------------------------------------------------------------------------------
[[noreturn]] void raise_saap(const char* call, int32_t status) {
  PyObject* mod = PyImport_ImportModule("paper_2502_08246_amd.binding");
  PyObject* cls = mod ? PyObject_GetAttrString(mod, "SaapError") : nullptr;
  PyObject* err = cls ? PyObject_CallFunction(cls, "si", call, (int)status) : nullptr;
  if (err) PyErr_SetObject(cls, err);
  Py_XDECREF(err);
  Py_XDECREF(cls);
  Py_XDECREF(mod);
  throw python_error();
}
void check(const char* call, int32_t status) {
  if (status != SAAP_OK) raise_saap(call, status);
}
[[noreturn]] void raise_value(const char* what) {
  PyErr_SetString(PyExc_ValueError, what);
  throw python_error();
}
[[noreturn]] void raise_type(const char* what) {
  PyErr_SetString(PyExc_TypeError, what);
  throw python_error();
}

// ---- arguments ---------------------------------------------------------------------------------------
// The parameters of one function: positional or by name, the first `required` of them mandatory.
constexpr int kMaxParams = 24;
struct Params {
  const char* func;
  int required, n;
  PyObject* names[kMaxParams];
  Params(const char* f, int req, std::initializer_list<const char*> list) : func(f), required(req), n(0) {
    for (const char* s : list) names[n++] = PyUnicode_InternFromString(s);
  }
};

struct Args {
  PyObject* v[kMaxParams];
  Args(const Params& p, PyObject* const* a, Py_ssize_t n_pos, PyObject* kw) {
    if (n_pos > p.n) {
      PyErr_Format(PyExc_TypeError, "%s() takes at most %d arguments (%zd given)", p.func, p.n, n_pos);
      throw python_error();
    }
    for (int i = 0; i < p.n; ++i) v[i] = i < n_pos ? a[i] : nullptr;
    const Py_ssize_t n_kw = kw ? PyTuple_GET_SIZE(kw) : 0;
    for (Py_ssize_t k = 0; k < n_kw; ++k) {
      PyObject* name = PyTuple_GET_ITEM(kw, k);
      int at = -1;
      for (int i = 0; i < p.n && at < 0; ++i)
        if (p.names[i] == name) at = i;
      for (int i = 0; i < p.n && at < 0; ++i)
        if (PyUnicode_Compare(p.names[i], name) == 0) at = i;
      if (at < 0) {
        PyErr_Format(PyExc_TypeError, "%s() got an unexpected keyword argument '%U'", p.func, name);
        throw python_error();
      }
      if (v[at]) {
        PyErr_Format(PyExc_TypeError, "%s() got multiple values for argument '%U'", p.func, name);
        throw python_error();
      }
      v[at] = a[n_pos + k];
    }
    for (int i = 0; i < p.required; ++i)
      if (!v[i]) {
        PyErr_Format(PyExc_TypeError, "%s() missing required argument '%U'", p.func, p.names[i]);
        throw python_error();
      }
  }
  bool has(int i) const { return v[i] && v[i] != Py_None; }
  // A tensor that something is read off here.  One that is only passed on is taken with maybe(): the C call says whether it
  // may be missing.
  const Tensor& tensor(int i) const {
    if (!v[i] || !THPVariable_Check(v[i])) raise_type("a tensor is expected");
    return THPVariable_Unpack(v[i]);
  }
  const Tensor* maybe(int i) const { return has(i) ? &tensor(i) : nullptr; }
  int32_t integer(int i, int32_t dflt = 0) const {
    if (!v[i]) return dflt;
    long r;
    if (PyLong_Check(v[i])) {
      r = PyLong_AsLong(v[i]);
    } else {
      PyObject* o = PyNumber_Long(v[i]);
      if (!o) throw python_error();
      r = PyLong_AsLong(o);
      Py_DECREF(o);
    }
    if (r == -1 && PyErr_Occurred()) throw python_error();
    return (int32_t)r;
  }
  double real(int i, double dflt = 0.0) const {
    if (!v[i]) return dflt;
    const double r = PyFloat_AsDouble(v[i]);
    if (r == -1.0 && PyErr_Occurred()) throw python_error();
    return r;
  }
  bool truth(int i, bool dflt) const {
    if (!v[i]) return dflt;
    const int r = PyObject_IsTrue(v[i]);
    if (r < 0) throw python_error();
    return r != 0;
  }
  at::ScalarType dtype(int i, at::ScalarType dflt) const {
    if (!has(i)) return dflt;
    if (!THPDtype_Check(v[i])) raise_type("a torch dtype is expected");
    return reinterpret_cast<THPDtype*>(v[i])->scalar_type;
  }
};

// ---- tensors -----------------------------------------------------------------------------------------
void want_dims(const Tensor& t, int n) {
  if (t.dim() != n) {
    PyErr_Format(PyExc_ValueError, "a tensor of %d dimensions is expected, got %d", n, (int)t.dim());
    throw python_error();
  }
}
int32_t size(const Tensor& t, int i) { return (int32_t)t.size(i); }

void* ptr(const Tensor& t) {
  if (!t.is_cuda()) raise_value("SAAP tensors must live in GPU memory; there is no CPU path");
  if (!t.is_contiguous()) raise_value("SAAP tensors must be contiguous");
  return t.data_ptr();
}
template <typename T> T* ptr_as(const Tensor& t) { return static_cast<T*>(ptr(t)); }
void* ptr(const Tensor* t) { return t ? ptr(*t) : nullptr; }
template <typename T> T* ptr_as(const Tensor* t) { return static_cast<T*>(ptr(t)); }

int32_t dtype_code(const Tensor& t) {
  if (t.scalar_type() == at::kFloat) return SAAP_F32;
  if (t.scalar_type() == at::kBFloat16) return SAAP_BF16;
  PyErr_Format(PyExc_TypeError, "unsupported dtype %s", c10::toString(t.scalar_type()));
  throw python_error();
}
void want_fp8_cache(const Tensor& q, const Tensor& K8, const Tensor& V8) {
  if (q.scalar_type() != at::kBFloat16 || K8.scalar_type() != at::kByte || V8.scalar_type() != at::kByte)
    raise_type("q must be bf16, K8 and V8 uint8");
}

// An output: the caller's tensor if one was passed (returned as the object it is), else a new one.
struct Out {
  Tensor t;
  PyObject* given;
  Out(const Args& a, int i, at::IntArrayRef shape, at::ScalarType type, const Tensor& like)
      : given(i >= 0 && a.has(i) ? a.v[i] : nullptr) {
    t = given ? a.tensor(i) : at::empty(shape, like.options().dtype(type));
  }
  Out(Tensor made) : t(std::move(made)), given(nullptr) {}
  PyObject* object() const {
    if (given) {
      Py_INCREF(given);
      return given;
    }
    return THPVariable_Wrap(t);
  }
};
PyObject* tuple_of(std::initializer_list<const Out*> outs) {
  PyObject* r = PyTuple_New((Py_ssize_t)outs.size());
  if (!r) throw python_error();
  Py_ssize_t i = 0;
  for (const Out* o : outs) {
    PyObject* x = o->object();
    if (!x) {
      Py_DECREF(r);
      throw python_error();
    }
    PyTuple_SET_ITEM(r, i++, x);
  }
  return r;
}

// ---- workspaces --------------------------------------------------------------------------------------
// The shared buffers: one per device and stream, so that calls on two streams, which may run at the same time, never meet
// in one.  A buffer is made, zero-filled (the arrival counters in its header start at zero) and used in the order of its
// stream; one that has become too small is dropped, and the allocator hands its memory out again in that order (unless
// the program has asked for the buffer itself and may have its address: that one is never freed).
//
// A HIP graph holds the raw address of the buffer that its calls were given, and is replayed on any stream: the first
// captured call takes the buffer of the calls before it away from their stream (which makes a new one when it needs it),
// later captures use it too, and it is never freed.  Making or growing a buffer while the stream captures is refused.
// The tables are guarded by the interpreter lock; the launches of two threads' calls on one stream by the library.
struct StreamBuffer {
  c10::DeviceIndex device;
  hipStream_t stream;
  Tensor buf;
  std::thread::id thread = {};                // that used it last
  uint64_t used = 0;                          // and when, counted in calls
  bool asked_for = false;                     // by the program
};
constexpr size_t kMaxStreamBuffers = 64;      // streams may come and go: the one made first is dropped
struct Workspaces {
  std::vector<StreamBuffer> streams;
  std::vector<StreamBuffer> captured;         // one per device (no stream of its own)
  std::vector<Tensor> retired;                // replaced ones that a graph or the program may hold
  uint64_t calls = 0;
};
Workspaces& workspaces() {
  static Workspaces* w = new Workspaces;      // not destroyed: the device may be gone by then
  return *w;
}
bool capturing(hipStream_t stream) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &status) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return status != hipStreamCaptureStatusNone;
}
bool holds(const Tensor& buf, size_t bytes) { return buf.defined() && (size_t)buf.numel() >= bytes; }

Tensor captured_workspace(Workspaces& w, size_t bytes, c10::DeviceIndex device) {
  StreamBuffer* slot = nullptr;
  for (auto& c : w.captured)
    if (c.device == device) slot = &c;
  if (slot && holds(slot->buf, bytes)) return slot->buf;
  // the one that this thread's calls used last (the warm-up's, on whichever stream), or else another thread's
  const StreamBuffer* from = nullptr;
  const auto me = std::this_thread::get_id();
  for (const auto& b : w.streams)
    if (b.device == device && holds(b.buf, bytes) &&
        (!from || (b.thread == me) > (from->thread == me) || ((b.thread == me) == (from->thread == me) && b.used > from->used)))
      from = &b;
  if (!from) {
    PyErr_SetString(PyExc_RuntimeError,
                    "the shared SAAP workspace would have to grow during stream capture: call the operation once "
                    "eagerly before capturing, or pass ws=");
    throw python_error();
  }
  const Tensor buf = from->buf;
  w.streams.erase(w.streams.begin() + (from - w.streams.data()));
  if (slot) {
    w.retired.push_back(slot->buf);
    slot->buf = buf;
  } else {
    w.captured.push_back({device, nullptr, buf});
  }
  return buf;
}
Tensor shared_workspace(size_t bytes, at::Device device, bool asked_for = false) {
  Workspaces& w = workspaces();
  auto drop = [&](StreamBuffer& b) {
    if (b.asked_for) w.retired.push_back(b.buf);
    b.asked_for = false;
  };
  const c10::DeviceIndex dev = device.index() < 0 ? 0 : device.index();
  const hipStream_t stream = c10::hip::getCurrentHIPStream(dev).stream();
  if (capturing(stream)) return captured_workspace(w, bytes, dev);
  size_t at = 0;
  while (at < w.streams.size() && (w.streams[at].device != dev || w.streams[at].stream != stream)) ++at;
  if (at == w.streams.size() || !holds(w.streams[at].buf, bytes)) {
    const Tensor buf = at::zeros({(int64_t)std::max<size_t>(bytes, SAAP_WS_HEADER_BYTES)},
                                 at::TensorOptions().dtype(at::kByte).device(at::kCUDA, dev));
    if (at == w.streams.size()) {
      if (w.streams.size() >= kMaxStreamBuffers) {
        drop(w.streams.front());
        w.streams.erase(w.streams.begin());
      }
      w.streams.push_back({dev, stream, buf});
      at = w.streams.size() - 1;
    } else {
      drop(w.streams[at]);
      w.streams[at].buf = buf;
    }
  }
  StreamBuffer& b = w.streams[at];
  b.asked_for |= asked_for;
  b.thread = std::this_thread::get_id();
  b.used = ++w.calls;
  return b.buf;
}
struct Ws {
  Tensor keep;          // another thread may replace the shared buffer while this call is being enqueued
  void* p;
  size_t bytes;
  Ws(const Args& a, int i, const Tensor& like, size_t need) {
    if (need == 0) raise_saap("saap_workspace_bytes", SAAP_INVALID_ARG);
    if (!a.has(i) && !like.is_cuda()) raise_value("SAAP tensors must live in GPU memory; there is no CPU path");
    keep = a.has(i) ? a.tensor(i) : shared_workspace(need, like.device());
    p = ptr(keep);
    bytes = (size_t)keep.numel();
  }
  Ws(const Args& a, int i, const Tensor& like, int32_t op, const saap_shape& sh)
      : Ws(a, i, like, saap_workspace_bytes(op, &sh)) {}
};
saap_shape shape_of(int S, int Hq, int Hkv, int mode = 0) {
  saap_shape sh{};
  sh.S = S; sh.Hq = Hq; sh.Hkv = Hkv; sh.mode = mode;
  return sh;
}

void* stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }

// The C call without the interpreter lock (other Python threads may run while a launch waits for queue space).
template <typename F>
void call(const char* name, F f) {
  PyThreadState* s = PyEval_SaveThread();
  const int32_t st = f();
  PyEval_RestoreThread(s);
  check(name, st);
}

#define SAAP_FUNCTION(name) PyObject* name(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames)
#define SAAP_BEGIN(n_required, ...)                                     \
  HANDLE_TH_ERRORS                                                      \
  static const Params params(__func__, n_required, {__VA_ARGS__});      \
  const Args a(params, args, nargs, kwnames);
#define SAAP_END END_HANDLE_TH_ERRORS

// ---- prefill -----------------------------------------------------------------------------------------
SAAP_FUNCTION(assign_keys) {
  SAAP_BEGIN(2, "x", "centroids", "bias", "out", "ws")
  const Tensor &x = a.tensor(0), &cent = a.tensor(1);
  want_dims(x, 4);
  want_dims(cent, 3);
  const int32_t S = size(x, 0), Hkv = size(x, 1), N = size(x, 2), d = size(x, 3), B = size(cent, 1);
  if (size(cent, 0) != Hkv || size(cent, 2) != d || cent.scalar_type() != x.scalar_type())
    raise_value("centroids must be [Hkv,B,d] in the dtype of x");
  Out ids(a, 3, {S, Hkv, N}, at::kInt, x);
  saap_shape sh = shape_of(S, 0, Hkv);
  sh.N = N; sh.B = B; sh.d = d;
  const Ws ws(a, 4, x, SAAP_OP_ASSIGN_KEYS, sh);
  void *px = ptr(x), *pc = ptr(cent), *po = ptr(ids.t), *st = nullptr;
  float* bias = ptr_as<float>(a.maybe(2));
  const int32_t dt = dtype_code(x);
  st = stream();
  call("saap_assign_keys", [&] {
    return saap_assign_keys(px, pc, bias, static_cast<int32_t*>(po), S, Hkv, N, B, d, dt, ws.p, ws.bytes, st);
  });
  return ids.object();
  SAAP_END
}

SAAP_FUNCTION(build_bucket_index) {
  SAAP_BEGIN(4, "bucket_ids", "K", "V", "B", "slack", "ws")
  const Tensor& K = a.tensor(1);
  want_dims(K, 4);
  const int32_t S = size(K, 0), Hkv = size(K, 1), N = size(K, 2), d = size(K, 3);
  const int32_t B = a.integer(3), slack = a.integer(4, 0), Ncap = N + B * slack, dt = dtype_code(K);
  Out off(a, -1, {S, Hkv, B + 1}, at::kInt, K), len(a, -1, {S, Hkv, B}, at::kInt, K), idx(a, -1, {S, Hkv, Ncap}, at::kInt, K);
  Out Ks(a, -1, {S, Hkv, Ncap, d}, K.scalar_type(), K), Vs(a, -1, {S, Hkv, Ncap, d}, K.scalar_type(), K);
  saap_shape sh = shape_of(S, 0, Hkv);
  sh.N = N; sh.B = B;
  const Ws ws(a, 5, K, SAAP_OP_BUILD_BUCKET_INDEX, sh);
  const int32_t* pi = ptr_as<int32_t>(a.maybe(0));
  void *pk = ptr(K), *pv = ptr(a.maybe(2)), *pks = ptr(Ks.t), *pvs = ptr(Vs.t);
  int32_t *po = ptr_as<int32_t>(off.t), *pl = ptr_as<int32_t>(len.t), *px = ptr_as<int32_t>(idx.t);
  void* st = stream();
  call("saap_build_bucket_index", [&] {
    return saap_build_bucket_index_zeroed(pi, pk, pv, po, pl, px, pks, pvs, S, Hkv, N, Ncap, B, d, dt, slack, ws.p, ws.bytes, st);
  });
  return tuple_of({&off, &len, &idx, &Ks, &Vs});
  SAAP_END
}

SAAP_FUNCTION(build_windowed_index) {
  SAAP_BEGIN(7, "bucket_ids", "K", "V", "B", "slack", "n_sink", "n_recent", "ws")
  const Tensor& K = a.tensor(1);
  want_dims(K, 4);
  const int32_t S = size(K, 0), Hkv = size(K, 1), N = size(K, 2), d = size(K, 3);
  const int32_t B = a.integer(3), slack = a.integer(4), n_sink = a.integer(5), n_recent = a.integer(6), dt = dtype_code(K);
  const int32_t W = n_sink + n_recent, Ncap = std::max(N - W, 0) + B * slack + W;
  Out off(a, -1, {S, Hkv, B + 2}, at::kInt, K), len(a, -1, {S, Hkv, B + 1}, at::kInt, K), idx(a, -1, {S, Hkv, Ncap}, at::kInt, K);
  Out Ks(a, -1, {S, Hkv, Ncap, d}, K.scalar_type(), K), Vs(a, -1, {S, Hkv, Ncap, d}, K.scalar_type(), K);
  // W may be 0: an address for the call all the same, and an empty tensor for the caller
  Tensor res = at::empty({S, Hkv, std::max(W, 1)}, K.options().dtype(at::kInt));
  int32_t* pr = ptr_as<int32_t>(res);
  saap_shape sh = shape_of(S, 0, Hkv);
  sh.N = N; sh.B = B;
  const Ws ws(a, 7, K, SAAP_OP_BUILD_BUCKET_INDEX, sh);
  const int32_t* pi = ptr_as<int32_t>(a.maybe(0));
  void *pk = ptr(K), *pv = ptr(a.maybe(2)), *pks = ptr(Ks.t), *pvs = ptr(Vs.t);
  int32_t *po = ptr_as<int32_t>(off.t), *pl = ptr_as<int32_t>(len.t), *px = ptr_as<int32_t>(idx.t);
  void* st = stream();
  call("saap_build_windowed_index", [&] {
    return saap_build_windowed_index_zeroed(pi, pk, pv, po, pl, px, pks, pvs, pr, S, Hkv, N, Ncap, B, d, dt, slack, n_sink,
                                     n_recent, ws.p, ws.bytes, st);
  });
  Out res_out(W > 0 ? res : res.slice(2, 0, 0));
  return tuple_of({&off, &len, &idx, &Ks, &Vs, &res_out});
  SAAP_END
}

SAAP_FUNCTION(quantize_kv) {
  SAAP_BEGIN(2, "Ks", "Vs", "ws")
  const Tensor& Ks = a.tensor(0);
  want_dims(Ks, 4);
  const int32_t S = size(Ks, 0), Hkv = size(Ks, 1), Ncap = size(Ks, 2), d = size(Ks, 3), dt = dtype_code(Ks);
  Out K8(a, -1, {S, Hkv, Ncap, d}, at::kByte, Ks), V8(a, -1, {S, Hkv, Ncap, d}, at::kByte, Ks);
  Out ks(a, -1, {S, Hkv}, at::kFloat, Ks), vs(a, -1, {S, Hkv}, at::kFloat, Ks);
  const Ws ws(a, 2, Ks, SAAP_WS_HEADER_BYTES);
  void *pk = ptr(Ks), *pv = ptr(a.maybe(1));
  uint8_t *p8 = ptr_as<uint8_t>(K8.t), *q8 = ptr_as<uint8_t>(V8.t);
  float *psk = ptr_as<float>(ks.t), *psv = ptr_as<float>(vs.t);
  void* st = stream();
  call("saap_quantize_kv", [&] { return saap_quantize_kv(pk, pv, p8, q8, psk, psv, S, Hkv, Ncap, d, dt, ws.p, ws.bytes, st); });
  return tuple_of({&K8, &V8, &ks, &vs});
  SAAP_END
}

// ---- routing -----------------------------------------------------------------------------------------
SAAP_FUNCTION(classify_queries) {
  SAAP_BEGIN(6, "xq", "W1", "b1", "W2", "b2", "Hkv", "output_kind", "out", "ws")
  const Tensor &xq = a.tensor(0), &W2 = a.tensor(3);
  want_dims(xq, 3);
  want_dims(W2, 3);
  const int32_t S = size(xq, 0), Hq = size(xq, 1), d = size(xq, 2), Hw = size(W2, 0), B = size(W2, 1);
  int32_t hidden = 0;
  const Tensor *W1 = a.maybe(1), *b1 = nullptr;
  if (!W1) {
    if (size(W2, 2) != d || W2.scalar_type() != xq.scalar_type())
      raise_value("one-layer model: W2 must be [Hw,B,d] in xq's dtype");
  } else {
    want_dims(*W1, 3);
    hidden = size(*W1, 1);
    b1 = a.maybe(2);
    if (size(*W1, 0) != Hw || size(W2, 2) != hidden || W1->scalar_type() != xq.scalar_type() ||
        W2.scalar_type() != xq.scalar_type())
      raise_value("W1 [Hw,hidden,d] and W2 [Hw,B,hidden] must match xq's dtype");
  }
  Out scores(a, 7, {S, Hq, B}, at::kFloat, xq);
  saap_shape sh = shape_of(S, Hq, 0);
  sh.hidden = hidden;
  const Ws ws(a, 8, xq, SAAP_OP_CLASSIFY_QUERIES, sh);
  void *px = ptr(xq), *pw1 = ptr(W1), *pw2 = ptr(W2);
  float *pb1 = ptr_as<float>(b1), *pb2 = ptr_as<float>(a.maybe(4)), *po = ptr_as<float>(scores.t);
  const int32_t Hkv = a.integer(5), kind = a.integer(6, SAAP_PROBS), dt = dtype_code(xq);
  void* st = stream();
  call("saap_classify_queries", [&] {
    return saap_classify_queries(px, pw1, pb1, pw2, pb2, Hw, po, S, Hq, Hkv, d, hidden, B, dt, kind, ws.p, ws.bytes, st);
  });
  return scores.object();
  SAAP_END
}

SAAP_FUNCTION(select_buckets) {
  SAAP_BEGIN(3, "scores", "Hkv", "nprobe", "mode", "out", "ws")
  const Tensor& scores = a.tensor(0);
  want_dims(scores, 3);
  const int32_t S = size(scores, 0), Hq = size(scores, 1), B = size(scores, 2);
  const int32_t Hkv = a.integer(1), nprobe = a.integer(2), mode = a.integer(3, SAAP_GROUP_SUM);
  Out sel(a, 4, {S, mode == SAAP_INDEPENDENT ? Hq : Hkv, nprobe}, at::kInt, scores);
  const Ws ws(a, 5, scores, SAAP_OP_SELECT_BUCKETS, saap_shape{});
  const float* ps = ptr_as<float>(scores);
  int32_t* po = ptr_as<int32_t>(sel.t);
  void* st = stream();
  call("saap_select_buckets", [&] { return saap_select_buckets(ps, po, S, Hq, Hkv, B, nprobe, mode, ws.p, ws.bytes, st); });
  return sel.object();
  SAAP_END
}

SAAP_FUNCTION(select_buckets_from_logits) {
  SAAP_BEGIN(3, "logits", "Hkv", "nprobe", "mode", "probs", "out", "ws")
  const Tensor& logits = a.tensor(0);
  want_dims(logits, 3);
  const int32_t S = size(logits, 0), Hq = size(logits, 1), B = size(logits, 2);
  const int32_t Hkv = a.integer(1), nprobe = a.integer(2), mode = a.integer(3, SAAP_GROUP_SUM);
  Out sel(a, 5, {S, mode == SAAP_INDEPENDENT ? Hq : Hkv, nprobe}, at::kInt, logits);
  const Ws ws(a, 6, logits, SAAP_OP_SELECT_BUCKETS, saap_shape{});
  float *pl = ptr_as<float>(logits), *pp = ptr_as<float>(a.maybe(4));
  int32_t* po = ptr_as<int32_t>(sel.t);
  void* st = stream();
  call("saap_select_buckets_from_logits", [&] {
    return saap_select_buckets_from_logits(pl, pp, po, S, Hq, Hkv, B, nprobe, mode, ws.p, ws.bytes, st);
  });
  return sel.object();
  SAAP_END
}

// ---- visit plans -------------------------------------------------------------------------------------
int64_t plan_ints(int32_t S, int32_t Hq, int32_t Hkv, int32_t nruns, int32_t mode) {
  const size_t bytes = saap_visit_plan_bytes(S, Hq, Hkv, nruns, mode);
  if (bytes == 0) raise_saap("saap_visit_plan_bytes", SAAP_INVALID_ARG);
  return (int64_t)(bytes / 4);
}
const Tensor* given_plan(const Args& a, int i, int64_t ints) {
  const Tensor* t = a.maybe(i);
  if (t && (t->scalar_type() != at::kInt || t->numel() < ints)) {
    PyErr_Format(PyExc_ValueError, "plan must be int32 with at least %lld elements", (long long)ints);
    throw python_error();
  }
  return t;
}
Out plan_buffer(const Args& a, int i, int64_t ints, const Tensor& like) {
  given_plan(a, i, ints);
  return Out(a, i, {ints}, at::kInt, like);
}

SAAP_FUNCTION(build_visit_plan) {
  SAAP_BEGIN(4, "selected", "off", "ln", "Hq", "mode", "resident_run", "plan")
  const Tensor &sel = a.tensor(0), &ln = a.tensor(2);
  want_dims(sel, 3);
  want_dims(ln, 3);
  const int32_t S = size(sel, 0), nprobe = size(sel, 2), Hkv = size(ln, 1), runs = size(ln, 2);
  const int32_t Hq = a.integer(3), mode = a.integer(4, SAAP_GROUP_SUM), resident = a.integer(5, -1);
  Out plan = plan_buffer(a, 6, plan_ints(S, Hq, Hkv, nprobe + (resident >= 0 ? 1 : 0), mode), ln);
  const int32_t *ps = nprobe > 0 ? ptr_as<int32_t>(sel) : nullptr, *po = ptr_as<int32_t>(a.maybe(1)), *pl = ptr_as<int32_t>(ln);
  int32_t* pp = ptr_as<int32_t>(plan.t);
  void* st = stream();
  call("saap_build_visit_plan", [&] { return saap_build_visit_plan(ps, po, pl, nprobe, mode, resident, pp, S, Hq, Hkv, runs, st); });
  return plan.object();
  SAAP_END
}

SAAP_FUNCTION(select_buckets_planned) {
  SAAP_BEGIN(5, "scores", "off", "ln", "Hkv", "nprobe", "input_kind", "mode", "resident_run", "probs", "out", "plan", "ws")
  const Tensor& scores = a.tensor(0);
  want_dims(scores, 3);
  const int32_t S = size(scores, 0), Hq = size(scores, 1), B = size(scores, 2);
  const int32_t Hkv = a.integer(3), nprobe = a.integer(4), kind = a.integer(5, SAAP_PROBS), mode = a.integer(6, SAAP_GROUP_SUM);
  const int32_t resident = a.integer(7, -1);
  Out sel(a, 9, {S, mode == SAAP_INDEPENDENT ? Hq : Hkv, nprobe}, at::kInt, scores);
  Out plan = plan_buffer(a, 10, plan_ints(S, Hq, Hkv, nprobe + (resident >= 0 ? 1 : 0), mode), scores);
  const Ws ws(a, 11, scores, SAAP_OP_SELECT_BUCKETS, saap_shape{});
  float *ps = ptr_as<float>(scores), *pp = ptr_as<float>(a.maybe(8));
  const int32_t *po = ptr_as<int32_t>(a.maybe(1)), *pl = ptr_as<int32_t>(a.maybe(2));
  int32_t *psel = ptr_as<int32_t>(sel.t), *pplan = ptr_as<int32_t>(plan.t);
  void* st = stream();
  call("saap_select_buckets_planned", [&] {
    return saap_select_buckets_planned(ps, kind, pp, po, pl, resident, psel, pplan, S, Hq, Hkv, B, nprobe, mode, ws.p, ws.bytes, st);
  });
  return tuple_of({&sel, &plan});
  SAAP_END
}

// ---- attention ---------------------------------------------------------------------------------------
// What every decode attention call takes apart from its lists: q [S,Hq,d], the cache [S,Hkv,rows,d], out and lse.
struct Attend {
  int32_t S, Hq, d, Hkv, rows;
  void *pq, *pk, *pv;
  Out out, lse;
  Attend(const Args& a, const Tensor& q, const Tensor& K, const Tensor* V, int i_dtype, int i_out, int i_lse)
      : out(a, i_out, (want_dims(q, 3), want_dims(K, 4), at::IntArrayRef({q.size(0), q.size(1), q.size(2)})),
            a.dtype(i_dtype, at::kFloat), q),
        lse(a, i_lse, {q.size(0), q.size(1)}, at::kFloat, q) {
    S = size(q, 0); Hq = size(q, 1); d = size(q, 2); Hkv = size(K, 1); rows = size(K, 2);
    pq = ptr(q); pk = ptr(K); pv = ptr(V);
  }
  int32_t out_code() const { return dtype_code(out.t); }
  PyObject* result() const { return tuple_of({&out, &lse}); }
};

SAAP_FUNCTION(sparse_decode_attention) {
  SAAP_BEGIN(7, "q", "Ks", "Vs", "off", "ln", "selected", "scale", "mode", "out_dtype", "out", "lse", "ws")
  const Tensor &q = a.tensor(0), &ln = a.tensor(4), &sel = a.tensor(5);
  Attend t(a, q, a.tensor(1), a.maybe(2), 8, 9, 10);
  want_dims(ln, 3);
  want_dims(sel, 3);
  const int32_t B = size(ln, 2), nprobe = size(sel, 2), mode = a.integer(7, SAAP_GROUP_SUM), dt = dtype_code(q);
  const Ws ws(a, 11, q, SAAP_OP_SPARSE_DECODE_ATTENTION, shape_of(t.S, t.Hq, t.Hkv, mode));
  const int32_t *po = ptr_as<int32_t>(a.maybe(3)), *pl = ptr_as<int32_t>(ln), *ps = nprobe > 0 ? ptr_as<int32_t>(sel) : nullptr;
  const float scale = (float)a.real(6);
  void *out = ptr(t.out.t), *st = nullptr;
  float* lse = ptr_as<float>(t.lse.t);
  const int32_t od = t.out_code();
  st = stream();
  call("saap_sparse_decode_attention", [&] {
    return saap_sparse_decode_attention(t.pq, t.pk, t.pv, po, pl, ps, nprobe, mode, scale, out, od, lse, t.S, t.Hq, t.Hkv,
                                        t.rows, B, t.d, dt, ws.p, ws.bytes, st);
  });
  return t.result();
  SAAP_END
}

SAAP_FUNCTION(sparse_decode_attention_fp8) {
  SAAP_BEGIN(9, "q", "K8", "V8", "kscale", "vscale", "off", "ln", "selected", "scale", "mode", "out_dtype", "out", "lse", "ws")
  const Tensor &q = a.tensor(0), &K8 = a.tensor(1), &V8 = a.tensor(2), &ln = a.tensor(6), &sel = a.tensor(7);
  want_fp8_cache(q, K8, V8);
  Attend t(a, q, K8, &V8, 10, 11, 12);
  want_dims(ln, 3);
  want_dims(sel, 3);
  const int32_t B = size(ln, 2), nprobe = size(sel, 2), mode = a.integer(9, SAAP_GROUP_SUM);
  const Ws ws(a, 13, q, SAAP_OP_SPARSE_DECODE_ATTENTION, shape_of(t.S, t.Hq, t.Hkv, mode));
  const float *ks = ptr_as<float>(a.maybe(3)), *vs = ptr_as<float>(a.maybe(4));
  const int32_t *po = ptr_as<int32_t>(a.maybe(5)), *pl = ptr_as<int32_t>(ln), *ps = nprobe > 0 ? ptr_as<int32_t>(sel) : nullptr;
  const float scale = (float)a.real(8);
  void* out = ptr(t.out.t);
  float* lse = ptr_as<float>(t.lse.t);
  const int32_t od = t.out_code();
  void* st = stream();
  call("saap_sparse_decode_attention_fp8", [&] {
    return saap_sparse_decode_attention_fp8(t.pq, static_cast<uint8_t*>(t.pk), static_cast<uint8_t*>(t.pv), ks, vs, po, pl, ps,
                                            nprobe, mode, scale, out, od, lse, t.S, t.Hq, t.Hkv, t.rows, B, t.d, ws.p,
                                            ws.bytes, st);
  });
  return t.result();
  SAAP_END
}

SAAP_FUNCTION(windowed_decode_attention) {
  SAAP_BEGIN(8, "q", "Ks", "Vs", "off", "ln", "selected", "resident_run", "scale", "mode", "out_dtype", "out", "lse", "ws")
  const Tensor &q = a.tensor(0), &ln = a.tensor(4), &sel = a.tensor(5);
  Attend t(a, q, a.tensor(1), a.maybe(2), 9, 10, 11);
  want_dims(ln, 3);
  want_dims(sel, 3);
  const int32_t runs = size(ln, 2), nprobe = size(sel, 2), resident = a.integer(6), mode = a.integer(8, SAAP_GROUP_SUM);
  const int32_t dt = dtype_code(q);
  const Ws ws(a, 12, q, SAAP_OP_SPARSE_DECODE_ATTENTION, shape_of(t.S, t.Hq, t.Hkv, mode));
  const int32_t *po = ptr_as<int32_t>(a.maybe(3)), *pl = ptr_as<int32_t>(ln), *ps = nprobe > 0 ? ptr_as<int32_t>(sel) : nullptr;
  const float scale = (float)a.real(7);
  void* out = ptr(t.out.t);
  float* lse = ptr_as<float>(t.lse.t);
  const int32_t od = t.out_code();
  void* st = stream();
  call("saap_windowed_decode_attention", [&] {
    return saap_windowed_decode_attention(t.pq, t.pk, t.pv, po, pl, ps, nprobe, mode, resident, scale, out, od, lse, t.S, t.Hq,
                                          t.Hkv, t.rows, runs, t.d, dt, ws.p, ws.bytes, st);
  });
  return t.result();
  SAAP_END
}

SAAP_FUNCTION(windowed_decode_attention_fp8) {
  SAAP_BEGIN(10, "q", "K8", "V8", "kscale", "vscale", "off", "ln", "selected", "resident_run", "scale", "mode", "out_dtype",
             "out", "lse", "ws")
  const Tensor &q = a.tensor(0), &K8 = a.tensor(1), &V8 = a.tensor(2), &ln = a.tensor(6), &sel = a.tensor(7);
  want_fp8_cache(q, K8, V8);
  Attend t(a, q, K8, &V8, 11, 12, 13);
  want_dims(ln, 3);
  want_dims(sel, 3);
  const int32_t runs = size(ln, 2), nprobe = size(sel, 2), resident = a.integer(8), mode = a.integer(10, SAAP_GROUP_SUM);
  const Ws ws(a, 14, q, SAAP_OP_SPARSE_DECODE_ATTENTION, shape_of(t.S, t.Hq, t.Hkv, mode));
  const float *ks = ptr_as<float>(a.maybe(3)), *vs = ptr_as<float>(a.maybe(4));
  const int32_t *po = ptr_as<int32_t>(a.maybe(5)), *pl = ptr_as<int32_t>(ln), *ps = nprobe > 0 ? ptr_as<int32_t>(sel) : nullptr;
  const float scale = (float)a.real(9);
  void* out = ptr(t.out.t);
  float* lse = ptr_as<float>(t.lse.t);
  const int32_t od = t.out_code();
  void* st = stream();
  call("saap_windowed_decode_attention_fp8", [&] {
    return saap_windowed_decode_attention_fp8(t.pq, static_cast<uint8_t*>(t.pk), static_cast<uint8_t*>(t.pv), ks, vs, po, pl, ps,
                                              nprobe, mode, resident, scale, out, od, lse, t.S, t.Hq, t.Hkv, t.rows, runs, t.d,
                                              ws.p, ws.bytes, st);
  });
  return t.result();
  SAAP_END
}

SAAP_FUNCTION(dense_decode_attention) {
  SAAP_BEGIN(4, "q", "K", "V", "scale", "off", "ln", "out_dtype", "out", "lse", "ws")
  const Tensor& q = a.tensor(0);
  Attend t(a, q, a.tensor(1), a.maybe(2), 6, 7, 8);
  const Tensor *off = a.maybe(4), *ln = a.maybe(5);
  if (ln) want_dims(*ln, 3);
  const int32_t B = ln ? size(*ln, 2) : 0, dt = dtype_code(q);
  const Ws ws(a, 9, q, SAAP_OP_DENSE_DECODE_ATTENTION, shape_of(t.S, t.Hq, t.Hkv));
  const int32_t *po = ptr_as<int32_t>(off), *pl = ptr_as<int32_t>(ln);
  const float scale = (float)a.real(3);
  void* out = ptr(t.out.t);
  float* lse = ptr_as<float>(t.lse.t);
  const int32_t od = t.out_code();
  void* st = stream();
  call("saap_dense_decode_attention", [&] {
    return saap_dense_decode_attention(t.pq, t.pk, t.pv, po, pl, B, scale, out, od, lse, t.S, t.Hq, t.Hkv, t.rows, t.d, dt, ws.p,
                                       ws.bytes, st);
  });
  return t.result();
  SAAP_END
}

SAAP_FUNCTION(dense_decode_attention_fp8) {
  SAAP_BEGIN(6, "q", "K8", "V8", "kscale", "vscale", "scale", "off", "ln", "out_dtype", "out", "lse", "ws")
  const Tensor &q = a.tensor(0), &K8 = a.tensor(1), &V8 = a.tensor(2);
  want_fp8_cache(q, K8, V8);
  Attend t(a, q, K8, &V8, 8, 9, 10);
  const Tensor *off = a.maybe(6), *ln = a.maybe(7);
  if (ln) want_dims(*ln, 3);
  const int32_t B = ln ? size(*ln, 2) : 0;
  const Ws ws(a, 11, q, SAAP_OP_DENSE_DECODE_ATTENTION, shape_of(t.S, t.Hq, t.Hkv));
  const float *ks = ptr_as<float>(a.maybe(3)), *vs = ptr_as<float>(a.maybe(4));
  const int32_t *po = ptr_as<int32_t>(off), *pl = ptr_as<int32_t>(ln);
  const float scale = (float)a.real(5);
  void* out = ptr(t.out.t);
  float* lse = ptr_as<float>(t.lse.t);
  const int32_t od = t.out_code();
  void* st = stream();
  call("saap_dense_decode_attention_fp8", [&] {
    return saap_dense_decode_attention_fp8(t.pq, static_cast<uint8_t*>(t.pk), static_cast<uint8_t*>(t.pv), ks, vs, po, pl, B,
                                           scale, out, od, lse, t.S, t.Hq, t.Hkv, t.rows, t.d, ws.p, ws.bytes, st);
  });
  return t.result();
  SAAP_END
}

SAAP_FUNCTION(select_attend) {
  SAAP_BEGIN(8, "logits", "q", "Ks", "Vs", "off", "ln", "nprobe", "scale", "out_dtype", "selected", "out", "lse", "ws",
             "resident_run")
  const Tensor &q = a.tensor(1), &ln = a.tensor(5);
  Attend t(a, q, a.tensor(2), a.maybe(3), 8, 10, 11);
  want_dims(ln, 3);
  const int32_t nprobe = a.integer(6), resident = a.integer(13, -1), dt = dtype_code(q);
  // with a resident run the index has one run more than the logits have buckets
  const int32_t B = size(ln, 2) - (resident >= 0 ? 1 : 0);
  Out sel(a, 9, {t.S, t.Hkv, nprobe}, at::kInt, q);
  const Ws ws(a, 12, q, SAAP_OP_SPARSE_DECODE_ATTENTION, shape_of(t.S, t.Hq, t.Hkv));
  const float* pg = ptr_as<float>(a.maybe(0));
  const int32_t *po = ptr_as<int32_t>(a.maybe(4)), *pl = ptr_as<int32_t>(ln);
  int32_t* ps = nprobe > 0 ? ptr_as<int32_t>(sel.t) : nullptr;
  const float scale = (float)a.real(7);
  void* out = ptr(t.out.t);
  float* lse = ptr_as<float>(t.lse.t);
  const int32_t od = t.out_code();
  void* st = stream();
  if (resident >= 0)
    call("saap_select_attend_windowed", [&] {
      return saap_select_attend_windowed(pg, t.pq, t.pk, t.pv, po, pl, nprobe, resident, scale, ps, out, od, lse, t.S, t.Hq, t.Hkv,
                                         t.rows, B, t.d, dt, ws.p, ws.bytes, st);
    });
  else
    call("saap_select_attend", [&] {
      return saap_select_attend(pg, t.pq, t.pk, t.pv, po, pl, nprobe, scale, ps, out, od, lse, t.S, t.Hq, t.Hkv, t.rows, B, t.d,
                                dt, ws.p, ws.bytes, st);
    });
  return tuple_of({&sel, &t.out, &t.lse});
  SAAP_END
}

SAAP_FUNCTION(select_attend_fp8) {
  SAAP_BEGIN(10, "logits", "q", "K8", "V8", "kscale", "vscale", "off", "ln", "nprobe", "scale", "out_dtype", "selected", "out",
             "lse", "ws")
  const Tensor &q = a.tensor(1), &K8 = a.tensor(2), &V8 = a.tensor(3), &ln = a.tensor(7);
  want_fp8_cache(q, K8, V8);
  Attend t(a, q, K8, &V8, 10, 12, 13);
  want_dims(ln, 3);
  const int32_t nprobe = a.integer(8), B = size(ln, 2);
  Out sel(a, 11, {t.S, t.Hkv, nprobe}, at::kInt, q);
  const Ws ws(a, 14, q, SAAP_OP_SPARSE_DECODE_ATTENTION, shape_of(t.S, t.Hq, t.Hkv));
  const float *pg = ptr_as<float>(a.maybe(0)), *ks = ptr_as<float>(a.maybe(4)), *vs = ptr_as<float>(a.maybe(5));
  const int32_t *po = ptr_as<int32_t>(a.maybe(6)), *pl = ptr_as<int32_t>(ln);
  int32_t* ps = nprobe > 0 ? ptr_as<int32_t>(sel.t) : nullptr;
  const float scale = (float)a.real(9);
  void* out = ptr(t.out.t);
  float* lse = ptr_as<float>(t.lse.t);
  const int32_t od = t.out_code();
  void* st = stream();
  call("saap_select_attend_fp8", [&] {
    return saap_select_attend_fp8(pg, t.pq, static_cast<uint8_t*>(t.pk), static_cast<uint8_t*>(t.pv), ks, vs, po, pl, nprobe,
                                  scale, ps, out, od, lse, t.S, t.Hq, t.Hkv, t.rows, B, t.d, ws.p, ws.bytes, st);
  });
  return tuple_of({&sel, &t.out, &t.lse});
  SAAP_END
}

SAAP_FUNCTION(planned_decode_attention) {
  SAAP_BEGIN(6, "q", "Ks", "Vs", "plan", "nruns", "scale", "mode", "out_dtype", "out", "lse", "ws")
  const Tensor& q = a.tensor(0);
  Attend t(a, q, a.tensor(1), a.maybe(2), 7, 8, 9);
  const int32_t nruns = a.integer(4), mode = a.integer(6, SAAP_GROUP_SUM);
  const Tensor* plan = given_plan(a, 3, plan_ints(t.S, t.Hq, t.Hkv, nruns, mode));
  const Ws ws(a, 10, q, SAAP_OP_PLANNED_DECODE_ATTENTION, shape_of(t.S, t.Hq, t.Hkv, mode));
  const int32_t *pp = ptr_as<int32_t>(plan), dt = dtype_code(q), od = t.out_code();
  const float scale = (float)a.real(5);
  void* out = ptr(t.out.t);
  float* lse = ptr_as<float>(t.lse.t);
  void* st = stream();
  call("saap_planned_decode_attention", [&] {
    return saap_planned_decode_attention(t.pq, t.pk, t.pv, pp, nruns, mode, scale, out, od, lse, t.S, t.Hq, t.Hkv, t.rows, t.d,
                                         dt, ws.p, ws.bytes, st);
  });
  return t.result();
  SAAP_END
}

SAAP_FUNCTION(planned_decode_attention_fp8) {
  SAAP_BEGIN(8, "q", "K8", "V8", "kscale", "vscale", "plan", "nruns", "scale", "mode", "out_dtype", "out", "lse", "ws")
  const Tensor &q = a.tensor(0), &K8 = a.tensor(1), &V8 = a.tensor(2);
  want_fp8_cache(q, K8, V8);
  Attend t(a, q, K8, &V8, 9, 10, 11);
  const int32_t nruns = a.integer(6), mode = a.integer(8, SAAP_GROUP_SUM);
  const Tensor* plan = given_plan(a, 5, plan_ints(t.S, t.Hq, t.Hkv, nruns, mode));
  const Ws ws(a, 12, q, SAAP_OP_PLANNED_DECODE_ATTENTION, shape_of(t.S, t.Hq, t.Hkv, mode));
  const float *ks = ptr_as<float>(a.maybe(3)), *vs = ptr_as<float>(a.maybe(4));
  const int32_t *pp = ptr_as<int32_t>(plan), od = t.out_code();
  const float scale = (float)a.real(7);
  void* out = ptr(t.out.t);
  float* lse = ptr_as<float>(t.lse.t);
  void* st = stream();
  call("saap_planned_decode_attention_fp8", [&] {
    return saap_planned_decode_attention_fp8(t.pq, static_cast<uint8_t*>(t.pk), static_cast<uint8_t*>(t.pv), ks, vs, pp, nruns,
                                             mode, scale, out, od, lse, t.S, t.Hq, t.Hkv, t.rows, t.d, ws.p, ws.bytes, st);
  });
  return t.result();
  SAAP_END
}

SAAP_FUNCTION(prefill_sparse_attention) {
  SAAP_BEGIN(13, "q", "K", "V", "Ks", "Vs", "off", "ln", "idx", "selected", "pos0", "n_sink", "n_recent", "scale", "out_dtype",
             "out", "lse", "ws")
  const Tensor &q = a.tensor(0), &K = a.tensor(1), &Ks = a.tensor(3), &ln = a.tensor(6);
  const Tensor& sel = a.tensor(8);
  want_dims(q, 4);
  want_dims(K, 4);
  want_dims(Ks, 4);
  want_dims(ln, 3);
  want_dims(sel, 4);
  const int32_t S = size(q, 0), Tq = size(q, 1), Hq = size(q, 2), d = size(q, 3), Hkv = size(K, 1), Nt = size(K, 2);
  const int32_t Ncap = size(Ks, 2), B = size(ln, 2), nprobe = size(sel, 3), n_sink = a.integer(10), n_recent = a.integer(11);
  Out out(a, 14, {S, Tq, Hq, d}, a.dtype(13, at::kFloat), q), lse(a, 15, {S, Tq, Hq}, at::kFloat, q);
  saap_shape sh = shape_of(S, Hq, Hkv);
  sh.N = Tq; sh.nprobe = nprobe; sh.dtype = dtype_code(q);
  const Ws ws(a, 16, q, SAAP_OP_PREFILL_SPARSE_ATTENTION, sh);
  void *pq = ptr(q), *pk = ptr(K), *pv = ptr(a.maybe(2)), *pks = ptr(Ks), *pvs = ptr(a.maybe(4)), *po = ptr(out.t);
  const int32_t *poff = ptr_as<int32_t>(a.maybe(5)), *pl = ptr_as<int32_t>(ln), *pi = ptr_as<int32_t>(a.maybe(7));
  const int32_t *ps = nprobe > 0 ? ptr_as<int32_t>(sel) : nullptr, *pp = ptr_as<int32_t>(a.maybe(9));
  float* plse = ptr_as<float>(lse.t);
  const float scale = (float)a.real(12);
  const int32_t od = dtype_code(out.t), dt = dtype_code(q);
  void* st = stream();
  call("saap_prefill_sparse_attention", [&] {
    return saap_prefill_sparse_attention(pq, pk, pv, pks, pvs, poff, pl, pi, ps, pp, nprobe, n_sink, n_recent, scale, po, od, plse,
                                         S, Hq, Hkv, Tq, Nt, Ncap, B, d, dt, ws.p, ws.bytes, st);
  });
  return tuple_of({&out, &lse});
  SAAP_END
}

// ---- keys generated after prefill ----------------------------------------------------------------------
// The arguments append_keys and window_push share, in this order from position 0: x_new, k_new, v_new, pos_new,
// centroids, bias, off, ln, idx, Ks, Vs and, for an 8-bit cache, kscale, vscale.
struct NewKeys {
  int32_t S, Hkv, d, B, Ncap;
  void *x, *k, *v, *cent, *K, *V;
  const int32_t *pos, *off;
  int32_t *len, *idx;
  const float *bias, *kscale = nullptr, *vscale = nullptr;
  NewKeys(const Args& a, bool fp8) {
    const Tensor &xt = a.tensor(0), &ct = a.tensor(4), &it = a.tensor(8);
    if (fp8)
      for (int i : {0, 1, 2, 4})
        if (a.tensor(i).scalar_type() != at::kBFloat16) raise_type("bf16 features and rows expected");
    want_dims(xt, 3);
    want_dims(ct, 3);
    want_dims(it, 3);
    S = size(xt, 0); Hkv = size(xt, 1); d = size(xt, 2); B = size(ct, 1); Ncap = size(it, 2);
    x = ptr(xt); k = ptr(a.maybe(1)); v = ptr(a.maybe(2)); cent = ptr(ct);
    pos = ptr_as<int32_t>(a.maybe(3)); bias = ptr_as<float>(a.maybe(5));
    off = ptr_as<int32_t>(a.maybe(6)); len = ptr_as<int32_t>(a.maybe(7)); idx = ptr_as<int32_t>(it);
    K = ptr(a.maybe(9)); V = ptr(a.maybe(10));
    if (fp8) {
      kscale = ptr_as<float>(a.maybe(11));
      vscale = ptr_as<float>(a.maybe(12));
    }
  }
  saap_shape shape() const {
    saap_shape sh = shape_of(S, 0, Hkv);
    sh.B = B;
    return sh;
  }
};
Out flag_buffer(const Args& a, int i, const Tensor& like) {
  if (a.has(i)) return Out(a, i, {4}, at::kInt, like);
  return Out(at::zeros({4}, like.options().dtype(at::kInt)));
}

SAAP_FUNCTION(append_keys) {
  SAAP_BEGIN(11, "x_new", "k_new", "v_new", "pos_new", "centroids", "bias", "off", "ln", "idx", "Ks", "Vs", "overflow_flag",
             "new_ids", "ws")
  const Tensor& x = a.tensor(0);
  const NewKeys n(a, false);
  Out flag = flag_buffer(a, 11, x), ids(a, 12, {n.S, n.Hkv}, at::kInt, x);
  const Ws ws(a, 13, x, SAAP_OP_APPEND_KEYS, n.shape());
  int32_t *pi = ptr_as<int32_t>(ids.t), *pf = ptr_as<int32_t>(flag.t);
  const int32_t dt = dtype_code(x);
  void* st = stream();
  call("saap_append_keys", [&] {
    return saap_append_keys(n.x, n.k, n.v, n.pos, n.cent, n.bias, n.off, n.len, n.idx, n.K, n.V, pi, pf, n.S, n.Hkv, n.Ncap, n.B,
                            n.d, dt, ws.p, ws.bytes, st);
  });
  return tuple_of({&ids, &flag});
  SAAP_END
}

SAAP_FUNCTION(append_keys_fp8) {
  SAAP_BEGIN(13, "x_new", "k_new", "v_new", "pos_new", "centroids", "bias", "off", "ln", "idx", "K8", "V8", "kscale", "vscale",
             "overflow_flag", "new_ids", "ws")
  const Tensor& x = a.tensor(0);
  const NewKeys n(a, true);
  Out flag = flag_buffer(a, 13, x), ids(a, 14, {n.S, n.Hkv}, at::kInt, x);
  const Ws ws(a, 15, x, SAAP_OP_APPEND_KEYS, n.shape());
  int32_t *pi = ptr_as<int32_t>(ids.t), *pf = ptr_as<int32_t>(flag.t);
  void* st = stream();
  call("saap_append_keys_fp8", [&] {
    return saap_append_keys_fp8(n.x, n.k, n.v, n.pos, n.cent, n.bias, n.off, n.len, n.idx, static_cast<uint8_t*>(n.K),
                                static_cast<uint8_t*>(n.V), n.kscale, n.vscale, pi, pf, n.S, n.Hkv, n.Ncap, n.B, n.d, ws.p,
                                ws.bytes, st);
  });
  return tuple_of({&ids, &flag});
  SAAP_END
}

SAAP_FUNCTION(window_push) {
  SAAP_BEGIN(14, "x_new", "k_new", "v_new", "pos_new", "centroids", "bias", "off", "ln", "idx", "Ks", "Vs", "resident_ids",
             "n_sink", "n_recent", "overflow_flag", "new_ids", "ws")
  const Tensor& x = a.tensor(0);
  const NewKeys n(a, false);
  Out flag = flag_buffer(a, 14, x), ids(a, 15, {n.S, n.Hkv}, at::kInt, x);
  const Ws ws(a, 16, x, SAAP_OP_WINDOW_PUSH, n.shape());
  int32_t *pr = ptr_as<int32_t>(a.maybe(11)), *pi = ptr_as<int32_t>(ids.t), *pf = ptr_as<int32_t>(flag.t);
  const int32_t n_sink = a.integer(12), n_recent = a.integer(13), dt = dtype_code(x);
  void* st = stream();
  call("saap_window_push", [&] {
    return saap_window_push(n.x, n.k, n.v, n.pos, n.cent, n.bias, n.off, n.len, n.idx, n.K, n.V, pr, pi, pf, n.S, n.Hkv, n.Ncap,
                            n.B, n.d, dt, n_sink, n_recent, ws.p, ws.bytes, st);
  });
  return tuple_of({&ids, &flag});
  SAAP_END
}

SAAP_FUNCTION(window_push_fp8) {
  SAAP_BEGIN(16, "x_new", "k_new", "v_new", "pos_new", "centroids", "bias", "off", "ln", "idx", "K8", "V8", "kscale", "vscale",
             "resident_ids", "n_sink", "n_recent", "overflow_flag", "new_ids", "ws")
  const Tensor& x = a.tensor(0);
  const NewKeys n(a, true);
  Out flag = flag_buffer(a, 16, x), ids(a, 17, {n.S, n.Hkv}, at::kInt, x);
  const Ws ws(a, 18, x, SAAP_OP_WINDOW_PUSH, n.shape());
  int32_t *pr = ptr_as<int32_t>(a.maybe(13)), *pi = ptr_as<int32_t>(ids.t), *pf = ptr_as<int32_t>(flag.t);
  const int32_t n_sink = a.integer(14), n_recent = a.integer(15);
  void* st = stream();
  call("saap_window_push_fp8", [&] {
    return saap_window_push_fp8(n.x, n.k, n.v, n.pos, n.cent, n.bias, n.off, n.len, n.idx, static_cast<uint8_t*>(n.K),
                                static_cast<uint8_t*>(n.V), n.kscale, n.vscale, pr, pi, pf, n.S, n.Hkv, n.Ncap, n.B, n.d, n_sink,
                                n_recent, ws.p, ws.bytes, st);
  });
  return tuple_of({&ids, &flag});
  SAAP_END
}

// ---- training ----------------------------------------------------------------------------------------
SAAP_FUNCTION(adam_update) {
  SAAP_BEGIN(6, "param", "grad", "m", "v", "step", "lr", "beta1", "beta2", "eps")
  float* p[4];
  const int64_t n = a.tensor(0).numel();
  for (int i = 0; i < 4; ++i) {
    const Tensor& t = a.tensor(i);
    if (t.scalar_type() != at::kFloat || t.numel() != n) raise_type("adam_update works on fp32 tensors of one size");
    p[i] = ptr_as<float>(t);
  }
  const int32_t step = a.integer(4);
  const float lr = (float)a.real(5), b1 = (float)a.real(6, 0.9), b2 = (float)a.real(7, 0.999), eps = (float)a.real(8, 1e-8);
  void* st = stream();
  call("saap_adam_update", [&] { return saap_adam_update(p[0], p[1], p[2], p[3], (size_t)n, step, lr, b1, b2, eps, st); });
  Py_RETURN_NONE;
  SAAP_END
}

// ---- module ------------------------------------------------------------------------------------------
SAAP_FUNCTION(workspace) {
  SAAP_BEGIN(2, "nbytes", "device_index", "asked_for")
  const int64_t n = a.has(0) ? (int64_t)PyLong_AsLongLong(a.v[0]) : 0;
  if (n == -1 && PyErr_Occurred()) throw python_error();
  return THPVariable_Wrap(
      shared_workspace((size_t)std::max<int64_t>(n, 0), at::Device(at::kCUDA, (int8_t)a.integer(1)), a.truth(2, true)));
  SAAP_END
}

#define SAAP_METHOD(name, doc) {#name, (PyCFunction)(void (*)())name, METH_FASTCALL | METH_KEYWORDS, doc}
PyMethodDef methods[] = {
    SAAP_METHOD(assign_keys,
                "assign_keys(x, centroids, bias=None, out=None, ws=None)\n--\n\n"
                "x [S,Hkv,N,d], centroids [Hkv,B,d], bias [Hkv,B] fp32 or None -> bucket_ids int32 [S,Hkv,N]."),
    SAAP_METHOD(build_bucket_index,
                "build_bucket_index(bucket_ids, K, V, B, slack=0, ws=None)\n--\n\n"
                "-> off [S,Hkv,B+1], len [S,Hkv,B], idx [S,Hkv,Ncap] (int32), Ksorted, Vsorted [S,Hkv,Ncap,d]."),
    SAAP_METHOD(build_windowed_index,
                "build_windowed_index(bucket_ids, K, V, B, slack, n_sink, n_recent, ws=None)\n--\n\n"
                "Index with a resident run of W = n_sink + n_recent slots behind the B buckets.\n"
                "-> off [S,Hkv,B+2], len [S,Hkv,B+1], idx [S,Hkv,Ncap], Ksorted, Vsorted [S,Hkv,Ncap,d], resident_ids [S,Hkv,W]."),
    SAAP_METHOD(quantize_kv,
                "quantize_kv(Ks, Vs, ws=None)\n--\n\n"
                "Ks, Vs [S,Hkv,Ncap,d] (bucket-sorted) -> K8, V8 uint8 [S,Hkv,Ncap,d] (OCP FP8 E4M3 codes),\n"
                "kscale, vscale fp32 [S,Hkv] (one power of two per unit)."),
    SAAP_METHOD(classify_queries,
                "classify_queries(xq, W1, b1, W2, b2, Hkv, output_kind=PROBS, out=None, ws=None)\n--\n\n"
                "xq [S,Hq,d]; W1 [Hw,hidden,d]; W2 [Hw,B,hidden]; b1,b2 fp32 or None -> scores fp32 [S,Hq,B].\n"
                "W1 = None: the one-layer model z = W2 x + b2 with W2 [Hw,B,d]."),
    SAAP_METHOD(select_buckets,
                "select_buckets(scores, Hkv, nprobe, mode=GROUP_SUM, out=None, ws=None)\n--\n\n"
                "scores fp32 [S,Hq,B] -> selected int32 [S,Hkv,nprobe] (GROUP_SUM) or [S,Hq,nprobe] (INDEPENDENT)."),
    SAAP_METHOD(select_buckets_from_logits,
                "select_buckets_from_logits(logits, Hkv, nprobe, mode=GROUP_SUM, probs=None, out=None, ws=None)\n--\n\n"
                "logits fp32 [S,Hq,B] (classify_queries with LOGITS) -> selected; `probs` (optional fp32 [S,Hq,B]) receives\n"
                "the softmax the selection was made from."),
    SAAP_METHOD(build_visit_plan,
                "build_visit_plan(selected, off, ln, Hq, mode=GROUP_SUM, resident_run=-1, plan=None)\n--\n\n"
                "selected int32 [S,lists,nprobe]; off [S,Hkv,runs+1], ln [S,Hkv,runs] -> plan (int32, flat)."),
    SAAP_METHOD(select_buckets_planned,
                "select_buckets_planned(scores, off, ln, Hkv, nprobe, input_kind=PROBS, mode=GROUP_SUM, resident_run=-1, "
                "probs=None, out=None, plan=None, ws=None)\n--\n\n"
                "select_buckets (PROBS) or select_buckets_from_logits (LOGITS) that also writes the lists' visit plan.\n"
                "-> (selected, plan)."),
    SAAP_METHOD(sparse_decode_attention,
                "sparse_decode_attention(q, Ks, Vs, off, ln, selected, scale, mode=GROUP_SUM, out_dtype=None, out=None, "
                "lse=None, ws=None)\n--\n\n"
                "q [S,Hq,d]; Ks,Vs [S,Hkv,Ncap,d]; off,ln from build_bucket_index; selected from select_buckets\n"
                "-> out [S,Hq,d] of out_dtype (None: float32, here and below), lse fp32 [S,Hq]."),
    SAAP_METHOD(sparse_decode_attention_fp8,
                "sparse_decode_attention_fp8(q, K8, V8, kscale, vscale, off, ln, selected, scale, mode=GROUP_SUM, "
                "out_dtype=None, out=None, lse=None, ws=None)\n--\n\n"
                "sparse_decode_attention on a cache written by quantize_kv; q bf16 [S,Hq,d]."),
    SAAP_METHOD(windowed_decode_attention,
                "windowed_decode_attention(q, Ks, Vs, off, ln, selected, resident_run, scale, mode=GROUP_SUM, "
                "out_dtype=None, out=None, lse=None, ws=None)\n--\n\n"
                "sparse_decode_attention over the selected buckets plus the always-visited run `resident_run`\n"
                "(-1 for none); off [S,Hkv,runs+1], ln [S,Hkv,runs]."),
    SAAP_METHOD(windowed_decode_attention_fp8,
                "windowed_decode_attention_fp8(q, K8, V8, kscale, vscale, off, ln, selected, resident_run, scale, mode=GROUP_SUM, "
                "out_dtype=None, out=None, lse=None, ws=None)\n--\n\n"
                "windowed_decode_attention on a cache written by quantize_kv; q bf16 [S,Hq,d]."),
    SAAP_METHOD(dense_decode_attention,
                "dense_decode_attention(q, K, V, scale, off=None, ln=None, out_dtype=None, out=None, lse=None, "
                "ws=None)\n--\n\n"
                "q [S,Hq,d]; K,V [S,Hkv,N,d] (packed, or a bucket-sorted cache with off/ln) -> out, lse."),
    SAAP_METHOD(dense_decode_attention_fp8,
                "dense_decode_attention_fp8(q, K8, V8, kscale, vscale, scale, off=None, ln=None, out_dtype=None, "
                "out=None, lse=None, ws=None)\n--\n\n"
                "dense_decode_attention on 8-bit K/V (packed, or a bucket-sorted cache with off/ln); q bf16."),
    SAAP_METHOD(select_attend,
                "select_attend(logits, q, Ks, Vs, off, ln, nprobe, scale, out_dtype=None, selected=None, out=None, "
                "lse=None, ws=None, resident_run=-1)\n--\n\n"
                "select_buckets_from_logits + sparse_decode_attention in one call (one launch where the library can):\n"
                "logits fp32 [S,Hq,B] -> (selected int32 [S,Hkv,nprobe], out [S,Hq,d], lse fp32 [S,Hq]).  With\n"
                "resident_run = B (an index from build_windowed_index: off [S,Hkv,B+2], ln [S,Hkv,B+1]) the always-visited\n"
                "run is attended too, as by windowed_decode_attention."),
    SAAP_METHOD(select_attend_fp8,
                "select_attend_fp8(logits, q, K8, V8, kscale, vscale, off, ln, nprobe, scale, out_dtype=None, "
                "selected=None, out=None, lse=None, ws=None)\n--\n\n"
                "select_attend on a cache written by quantize_kv; q bf16 [S,Hq,d]."),
    SAAP_METHOD(planned_decode_attention,
                "planned_decode_attention(q, Ks, Vs, plan, nruns, scale, mode=GROUP_SUM, out_dtype=None, out=None, "
                "lse=None, ws=None)\n--\n\n"
                "q [S,Hq,d]; Ks,Vs [S,Hkv,Ncap,d]; plan from select_buckets_planned / build_visit_plan -> out, lse."),
    SAAP_METHOD(planned_decode_attention_fp8,
                "planned_decode_attention_fp8(q, K8, V8, kscale, vscale, plan, nruns, scale, mode=GROUP_SUM, "
                "out_dtype=None, out=None, lse=None, ws=None)\n--\n\n"
                "planned_decode_attention on a cache written by quantize_kv; q bf16 [S,Hq,d]."),
    SAAP_METHOD(prefill_sparse_attention,
                "prefill_sparse_attention(q, K, V, Ks, Vs, off, ln, idx, selected, pos0, n_sink, n_recent, scale, "
                "out_dtype=None, out=None, lse=None, ws=None)\n--\n\n"
                "q [S,Tq,Hq,d]; position-ordered K,V [S,Hkv,Nt,d]; Ks,Vs,off,ln,idx from build_bucket_index over them;\n"
                "selected int32 [S,Hkv,Tq,nprobe]; pos0 int32 [S] -> out [S,Tq,Hq,d], lse fp32 [S,Tq,Hq]."),
    SAAP_METHOD(append_keys,
                "append_keys(x_new, k_new, v_new, pos_new, centroids, bias, off, ln, idx, Ks, Vs, overflow_flag=None, "
                "new_ids=None, ws=None)\n--\n\n"
                "In-place append of one key per (sequence, KV head). -> (new_bucket_ids [S,Hkv], overflow_flag)."),
    SAAP_METHOD(append_keys_fp8,
                "append_keys_fp8(x_new, k_new, v_new, pos_new, centroids, bias, off, ln, idx, K8, V8, kscale, vscale, "
                "overflow_flag=None, new_ids=None, ws=None)\n--\n\n"
                "append_keys on an 8-bit cache (K8, V8 uint8 with the scales of quantize_kv), in place."),
    SAAP_METHOD(window_push,
                "window_push(x_new, k_new, v_new, pos_new, centroids, bias, off, ln, idx, Ks, Vs, resident_ids, n_sink, n_recent, "
                "overflow_flag=None, new_ids=None, ws=None)\n--\n\n"
                "In-place push of one key per (sequence, KV head) into the resident run; the displaced key moves\n"
                "to its bucket. -> (new_bucket_ids [S,Hkv], overflow_flag)."),
    SAAP_METHOD(window_push_fp8,
                "window_push_fp8(x_new, k_new, v_new, pos_new, centroids, bias, off, ln, idx, K8, V8, kscale, vscale, "
                "resident_ids, n_sink, n_recent, overflow_flag=None, new_ids=None, ws=None)\n--\n\n"
                "window_push on an 8-bit cache (K8, V8 uint8 with the scales of quantize_kv), in place."),
    SAAP_METHOD(adam_update,
                "adam_update(param, grad, m, v, step, lr, beta1=0.9, beta2=0.999, eps=1e-8)\n--\n\n"
                "One Adam step on one fp32 tensor, in place (param, m, v)."),
    SAAP_METHOD(workspace,
                "workspace(nbytes, device_index, asked_for=True)\n--\n\n"
                "The shared workspace buffer of the device's current stream, at least nbytes long; asked_for: by the\n"
                "program, which may keep its address."),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "The library's calls on torch tensors.", -1, methods,
                      nullptr,               nullptr,   nullptr,                                  nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() {
  PyObject* m = PyModule_Create(&module);
  // the names the signatures above use
  if (m && (PyModule_AddIntConstant(m, "GROUP_SUM", SAAP_GROUP_SUM) || PyModule_AddIntConstant(m, "PROBS", SAAP_PROBS))) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
