// csd — the per-call part of binding.py in native code: checks the tensors, allocates the outputs
// and calls the C-ABI.  A decode loop calls step() once per token, and in Python that took five
// times as long as the kernel that it launches (4 paths x 256 tokens, us a call: kernel 4.2, step()
// 21 in Python and 6.7 here, draft() 15 and 6.1, accept() 13 and 4.5, reset() 6 and 3.3, most of
// which is the launch).
//
// Every function returns None where an argument is not what the call usually gets (another type,
// a tensor of another kind): binding.py then goes its own way, which raises the error or serves it.
// Otherwise it returns (error code, result).
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/Context.h>
#include <ATen/EmptyTensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/DeviceGuard.h>
#include <c10/core/impl/LocalDispatchKeySet.h>

#include "csd.h"

namespace {

// What a call's arguments are turned into; `usual` falls when one of them is not.
struct Call {
  PyObject* const* args;
  Py_ssize_t n, at = 0;
  bool usual = true;

  PyObject* next() {
    if (at < n) return args[at++];
    usual = false;
    return Py_None;
  }
  int64_t integer() {
    PyObject* o = next();
    int overflow = 1;
    if (PyLong_CheckExact(o)) {
      const long long x = PyLong_AsLongLongAndOverflow(o, &overflow);
      if (overflow == 0) return x;
    }
    usual = false;
    return 0;
  }
  int32_t small() {                                     // an int of the C-ABI
    const int64_t x = integer();
    if (x != (int32_t)x) usual = false;
    return (int32_t)x;
  }
  void* pointer() {
    PyObject* o = next();
    if (PyLong_CheckExact(o)) {
      void* p = PyLong_AsVoidPtr(o);
      if (!PyErr_Occurred()) return p;
      PyErr_Clear();
    }
    usual = false;
    return nullptr;
  }
  bool truth() {
    PyObject* o = next();
    if (o != Py_True && o != Py_False) usual = false;
    return o == Py_True;
  }
  // a contiguous device tensor of `type` with at least `numel` elements, or (`maybe`) None
  void* tensor(at::ScalarType type, int64_t numel, bool maybe) {
    PyObject* o = next();
    if (o == Py_None) {
      usual = usual && maybe;
      return nullptr;
    }
    if (!THPVariable_CheckExact(o)) {
      usual = false;
      return nullptr;
    }
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.scalar_type() != type || !t.is_contiguous() || t.numel() < numel) {
      usual = false;
      return nullptr;
    }
    return t.data_ptr();
  }
  const int32_t* ints(int64_t numel, bool maybe = false) {
    return static_cast<const int32_t*>(tensor(at::kInt, numel, maybe));
  }
  const float* floats(int64_t numel) { return static_cast<const float*>(tensor(at::kFloat, numel, true)); }
};

// The handle and its sizes: the first arguments of every call.
struct Pool {
  csd_index* handle;
  void* stream;
  c10::Device device{c10::DeviceType::CUDA, -1};
  int64_t P, N, rows;
  explicit Pool(Call& c) {
    handle = static_cast<csd_index*>(c.pointer());
    stream = c.pointer();
    const int64_t index = c.integer();
    P = c.integer();
    N = c.integer();
    rows = P * N;
    if (index < -1 || index > 127 || P <= 0 || N <= 0) c.usual = false;
    else device = c10::Device(c10::DeviceType::CUDA, (c10::DeviceIndex)index);
  }
};

// The outputs of a call: int32 or float32 [steps][P][N][L] each, without the leading axis where
// steps < 0, without the trailing one where L < 0.
struct Shape {
  int64_t at[4], n = 0;
  Shape(const Pool& p, int64_t steps, int64_t L) {
    if (steps >= 0) put(steps);
    put(p.P);
    put(p.N);
    if (L >= 0) put(L);
  }
  void put(int64_t x) { at[n++] = x; }
  c10::IntArrayRef sizes() const { return c10::IntArrayRef(at, n); }
};

// Allocates them, each with a storage of its own: a caller may resize one, save it, free it or write to it
// as out=.  The first comes from at::empty; the others straight from the allocator that served it,
// without the dispatcher's part, half of an allocation (step() 8.1 and 6.7 us, draft() 7.2 and 6.1;
// cut from one storage they take 5.3 and 5.1, but then an output that is resized grows into the next
// one).  Whatever may want to see an output made (modes, tracing, function transforms, the filling
// of new memory) gets at::empty for all.
class Maker {
 public:
  explicit Maker(const Pool& p) : device_(p.device) {}
  at::Tensor operator()(at::ScalarType type, const Shape& s) {
    if (allocator_) return at::detail::empty_generic(s.sizes(), allocator_, at::DispatchKeySet(at::DispatchKey::CUDA), type, c10::nullopt);
    at::Tensor t = at::empty(s.sizes(), at::TensorOptions().dtype(type).device(device_));
    if (t.has_storage() && alone()) {
      allocator_ = t.storage().allocator();
      guard_.reset_device(t.device());                   // (an allocator serves the current device)
    }
    return t;
  }

 private:
  static bool alone() {
    const at::DispatchKeySet usual = c10::default_included_set | c10::autocast_dispatch_keyset;
    return (c10::impl::tls_local_dispatch_key_set().included_ - usual).empty() &&
           !(at::globalContext().deterministicAlgorithms() && at::globalContext().deterministicFillUninitializedMemory());
  }
  c10::Device device_;
  c10::Allocator* allocator_ = nullptr;
  c10::OptionalDeviceGuard guard_;
};

int32_t* int_data(const at::Tensor& t) { return t.defined() ? static_cast<int32_t*>(t.data_ptr()) : nullptr; }
float* float_data(const at::Tensor& t) { return t.defined() ? static_cast<float*>(t.data_ptr()) : nullptr; }

bool put(PyObject* dict, const char* name, const at::Tensor& t) {
  PyObject* o = t.defined() ? THPVariable_Wrap(t) : Py_NewRef(Py_None);
  const bool ok = o && PyDict_SetItemString(dict, name, o) == 0;
  Py_XDECREF(o);
  return ok;
}

// a draft's outputs, and the accepted lengths
struct Outputs {
  at::Tensor tokens, length, token_scores, path_scores, accept;
  Outputs(const Pool& p, int64_t steps, int64_t L, bool scores, bool with_accept = false) {
    const Shape per_token(p, steps, L), per_row(p, steps, -1);
    Maker make(p);
    tokens = make(at::kInt, per_token);
    length = make(at::kInt, per_row);
    if (scores) {
      token_scores = make(at::kFloat, per_token);
      path_scores = make(at::kFloat, per_row);
    }
    if (with_accept) accept = make(at::kInt, per_row);
  }
  // (code, dict); with_accept: also the accepted lengths, made here or the caller's (`given`)
  PyObject* result(int code, bool with_accept = false, PyObject* given = nullptr) const {
    PyObject* dict = PyDict_New();
    if (!dict) return nullptr;
    bool ok = put(dict, "tokens", tokens) && put(dict, "length", length) &&
              put(dict, "token_scores", token_scores) && put(dict, "path_scores", path_scores);
    if (ok && with_accept) ok = given ? PyDict_SetItemString(dict, "accept", given) == 0 : put(dict, "accept", accept);
    if (!ok) {
      Py_DECREF(dict);
      return nullptr;
    }
    return Py_BuildValue("(iN)", code, dict);
  }
};

// reset(pool)
PyObject* reset(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Call c{args, n};
  const Pool p(c);
  if (!c.usual) Py_RETURN_NONE;
  int code;
  Py_BEGIN_ALLOW_THREADS
  code = csd_reset(p.handle, p.stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(code);
  END_HANDLE_TH_ERRORS
}

// append(pool, tokens, probs, counts, n)
PyObject* append(PyObject*, PyObject* const* args, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  Call c{args, n_args};
  const Pool p(c);
  const int32_t n = c.small();
  const int32_t* tokens = c.ints(p.rows * n);
  const float* probs = c.floats(p.rows * n);
  const int32_t* counts = c.ints(p.rows, true);
  if (!c.usual) Py_RETURN_NONE;
  int code;
  Py_BEGIN_ALLOW_THREADS
  code = csd_append(p.handle, tokens, probs, counts, n, p.stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(code);
  END_HANDLE_TH_ERRORS
}

// draft(pool, query_len, draft_len, scores)
PyObject* draft(PyObject*, PyObject* const* args, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  Call c{args, n_args};
  const Pool p(c);
  const int32_t k = c.small(), L = c.small();
  const bool scores = c.truth();
  if (!c.usual || L < 0) Py_RETURN_NONE;
  const Outputs o(p, -1, L, scores);
  int code;
  Py_BEGIN_ALLOW_THREADS
  code = csd_draft(p.handle, k, L, int_data(o.tokens), int_data(o.length), float_data(o.token_scores),
                   float_data(o.path_scores), p.stream);
  Py_END_ALLOW_THREADS
  return o.result(code);
  END_HANDLE_TH_ERRORS
}

// accept(pool, draft_tokens, draft_len_t, targets, draft_len)
PyObject* accept(PyObject*, PyObject* const* args, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  Call c{args, n_args};
  const Pool p(c);
  const int32_t L = c.small();
  const int32_t* tokens = c.ints(p.rows * L);
  const int32_t* length = c.ints(p.rows);
  const int32_t* targets = c.ints(p.rows * L);
  if (!c.usual) Py_RETURN_NONE;
  const Shape per_row(p, -1, -1);
  const at::Tensor out = at::empty(per_row.sizes(), at::TensorOptions().dtype(at::kInt).device(p.device));
  int code;
  Py_BEGIN_ALLOW_THREADS
  code = csd_accept(p.handle, tokens, length, targets, L, int_data(out), p.stream);
  Py_END_ALLOW_THREADS
  return Py_BuildValue("(iN)", code, THPVariable_Wrap(out));
  END_HANDLE_TH_ERRORS
}

// step(pool, n, query_len, draft_len, scores, tokens, probs, counts, targets, accept_out) and
// replay(pool, n_steps, query_len, draft_len, scores, tokens, probs, fused, targets, accept_out)
template <bool REPLAY>
PyObject* step(PyObject*, PyObject* const* args, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  Call c{args, n_args};
  const Pool p(c);
  const int32_t n = c.small(), k = c.small(), L = c.small();   // tokens a path, or steps of one token
  const bool scores = c.truth();
  if (!c.usual || L < 0 || n < 0) Py_RETURN_NONE;
  const int64_t steps = REPLAY ? n : -1, rows = REPLAY ? p.rows * n : p.rows;
  const int32_t* tokens = c.ints(p.rows * n);
  const float* probs = c.floats(p.rows * n);
  const int32_t* counts = REPLAY ? nullptr : c.ints(p.rows, true);
  const bool fused = REPLAY ? c.truth() : true;
  const int32_t* targets = c.ints(rows * L, true);
  PyObject* given = c.at < c.n ? c.args[c.at] : Py_None;
  int32_t* accepted = const_cast<int32_t*>(c.ints(rows, true));
  if (!c.usual) Py_RETURN_NONE;
  const Outputs o(p, steps, L, scores, targets && given == Py_None);
  if (o.accept.defined()) accepted = int_data(o.accept);
  int code;
  Py_BEGIN_ALLOW_THREADS
  code = REPLAY ? csd_replay(p.handle, n, tokens, probs, k, L, int_data(o.tokens), int_data(o.length),
                             float_data(o.token_scores), float_data(o.path_scores), targets, accepted, fused ? 1 : 0,
                             p.stream)
                : csd_step(p.handle, tokens, probs, counts, n, k, L, int_data(o.tokens), int_data(o.length),
                           float_data(o.token_scores), float_data(o.path_scores), targets, accepted, p.stream);
  Py_END_ALLOW_THREADS
  return o.result(code, true, given == Py_None ? nullptr : given);
  END_HANDLE_TH_ERRORS
}

template <class F>
PyCFunction fast(F f) {
  return reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(f));
}
PyMethodDef methods[] = {
    {"reset", fast(reset), METH_FASTCALL, nullptr},
    {"append", fast(append), METH_FASTCALL, nullptr},
    {"draft", fast(draft), METH_FASTCALL, nullptr},
    {"accept", fast(accept), METH_FASTCALL, nullptr},
    {"step", fast(step<false>), METH_FASTCALL, nullptr},
    {"replay", fast(step<true>), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_csd_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject* PyInit__csd_torch() { return PyModule_Create(&module); }
