// Regular calls of the C ABI from Python: checks the tensors and takes their addresses in native code.
//
// A call of the smallest workloads takes the GPU 8 us.  The two launches take the host about 4; checking shapes and types, asking
// some twenty tensors for their addresses and converting as many arguments one by one in Python took it another 4-5, so that the
// host was what bounded such calls.  Here that takes 0.7 (6.8 in Python, both timed on one slower machine).  us per call: one greedy chain of 9 x 32 000
// fp32 10.2 -> 7.9, 3 trees of 14 x 2 692 with seven thresholds 11.3 -> 8.5, margin statistics of 93 rows of 2 747 10.1 -> 7.6.
//
// A function here handles a call only if all of it is as the binding asks for: plain tensors of the right types and shapes, contiguous.  For anything
// else it returns None, having done nothing, and the binding goes its general way, which says what is wrong.  Nothing is kept from
// one call to the next but the addresses of the library's functions.  As with ctypes, the interpreter's lock is not held while the
// library runs.
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/mars.h"

namespace {

using at::Tensor;
struct Irregular {};

decltype(&mars_verify) f_verify;
decltype(&mars_verify_ex) f_verify_ex;
decltype(&mars_margin_stats) f_margin;
decltype(&mars_lmhead_verify) f_lmhead;
decltype(&mars_lmhead_verify_sampling) f_lmhead_sampling;

// Attributes of the binding's VerifyOutputs.
enum Field { kMask, kLen, kPath, kBonus, kDecision, kStatus, kStats, kDiag, kOutTokens, kOutLen, kKeepRows, kKeepOffsets, kThetas, kFields };
const char* const kNames[kFields] = {"accept_mask", "accept_len", "path_idx", "bonus_token", "decision", "request_status", "stats",
                                     "diag", "out_tokens", "out_len", "keep_rows", "keep_offsets", "n_theta"};
PyObject* g_names[kFields];

// A plain tensor (no subclass, whose own ways Python knows).
const Tensor& tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) throw Irregular();
  return THPVariable_Unpack(o);
}
// (data_ptr() throws where a tensor has no memory of its own)
template <typename T> T* address(const Tensor& t) { return static_cast<T*>(t.data_ptr()); }
void require(bool ok) { if (!ok) throw Irregular(); }
// An attribute, held until it has been looked at: it may have been made when it was asked for (a property that returns a view of
// a larger buffer), and then nobody else holds it.
struct Attribute {
  PyObject* o;
  Attribute(PyObject* of, Field f) : o(PyObject_GetAttr(of, g_names[f])) { require(o != nullptr); }
  ~Attribute() { Py_DECREF(o); }
  Attribute(const Attribute&) = delete;
  Attribute& operator=(const Attribute&) = delete;
};
template <typename T> T* field(PyObject* out, Field f, bool optional = false) {
  const Attribute a(out, f);
  if (a.o == Py_None) {
    require(optional);
    return nullptr;
  }
  return address<T>(tensor(a.o));
}
int code(const Tensor& t) {
  const auto s = t.scalar_type();
  if (s == at::kFloat) return MARS_F32;
  require(s == at::kBFloat16 || s == at::kUInt16 || s == at::kShort);
  return MARS_BF16;
}
bool shaped(const Tensor& t, int64_t a, int64_t b) { return t.dim() == 2 && t.size(0) == a && t.size(1) == b && t.is_contiguous(); }
bool shaped(const Tensor& t, int64_t a, int64_t b, int64_t c) {
  return t.dim() == 3 && t.size(0) == a && t.size(1) == b && t.size(2) == c && t.is_contiguous();
}
int narrow(int64_t x) {
  require(x >= 0 && x <= 0x7FFFFFFF);
  return static_cast<int>(x);
}
float number(PyObject* o) {
  require(PyFloat_CheckExact(o) || PyLong_CheckExact(o));
  const double x = PyFloat_AsDouble(o);
  require(!PyErr_Occurred());
  return static_cast<float>(x);
}
int integer(PyObject* o) {
  require(PyLong_CheckExact(o));
  int over = 0;
  const long x = PyLong_AsLongAndOverflow(o, &over);
  require(!over && x >= -0x7FFFFFFFL - 1 && x <= 0x7FFFFFFFL);
  return static_cast<int>(x);
}
// (asked for last, when everything else is as it should be)
void* stream_of(PyObject* ask) {
  PyObject* o = PyObject_CallNoArgs(ask);
  require(o != nullptr);
  void* s = PyLong_AsVoidPtr(o);
  Py_DECREF(o);
  require(!PyErr_Occurred());
  return s;
}
// What the calls have in common: the request's tables, shapes [B, N].
struct Requests {
  const int32_t *tok, *par;
  const float *theta, *u = nullptr;
  const void* q = nullptr;
  int qcode = 0;
  Requests(PyObject* tokens, PyObject* parents, PyObject* thetas, PyObject* uniforms, PyObject* probs, int64_t B, int64_t N, int64_t V, int K,
           bool whole_theta) {
    const Tensor &t = tensor(tokens), &p = tensor(parents), &th = tensor(thetas);
    require(t.scalar_type() == at::kInt && shaped(t, B, N) && p.scalar_type() == at::kInt && shaped(p, B, N));
    require(th.scalar_type() == at::kFloat && th.numel() == K * B && (!whole_theta || th.is_contiguous()));
    tok = address<int32_t>(t); par = address<int32_t>(p); theta = address<float>(th);
    if (uniforms != Py_None) {
      const Tensor& x = tensor(uniforms);
      require(x.scalar_type() == at::kFloat && shaped(x, B, N + 1));
      u = address<float>(x);
    }
    if (probs != Py_None) {
      const Tensor& x = tensor(probs);
      require(shaped(x, B, N, V));
      qcode = code(x);
      q = address<void>(x);
    }
  }
};
mars_verify_options options_of(PyObject* out, PyObject* indicator, int K, PyObject* spin_limit, PyObject* stages) {
  require(integer(Attribute(out, kThetas).o) == K);
  mars_verify_options o = {};
  o.indicator = integer(indicator); o.n_theta = K; o.spin_limit = integer(spin_limit); o.stages = integer(stages);
  o.out_tokens = field<int32_t>(out, kOutTokens, true); o.out_len = field<int32_t>(out, kOutLen, true);
  o.keep_rows = field<int32_t>(out, kKeepRows, true); o.keep_offsets = field<int32_t>(out, kKeepOffsets, true);
  return o;
}
// What a call writes, of VerifyOutputs.
struct Results {
  uint8_t *mask, *dec;
  int32_t *len, *path, *bonus, *status;
  mars_row_stat* stats;
  explicit Results(PyObject* out)
      : mask(field<uint8_t>(out, kMask)), dec(field<uint8_t>(out, kDecision, true)), len(field<int32_t>(out, kLen)),
        path(field<int32_t>(out, kPath)), bonus(field<int32_t>(out, kBonus)), status(field<int32_t>(out, kStatus, true)),
        stats(field<mars_row_stat>(out, kStats, true)) {}
};

// A call, or None where it is not a regular one (nothing has been done then).
template <typename Call>
PyObject* regular(Call call) {
  try {
    return PyLong_FromLong(call());
  } catch (...) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}
template <typename Run>
int unlocked(Run run) {
  PyThreadState* s = PyEval_SaveThread();
  const int rc = run();
  PyEval_RestoreThread(s);
  return rc;
}

// logits, draft_tokens, tree_parent, theta, temperature, uniforms, draft_probs, out, workspace, stream
PyObject* verify(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return regular([&]() -> int {
    require(n == 10);
    const Tensor &z = tensor(a[0]), &ws = tensor(a[8]);
    require(z.dim() == 3 && z.is_contiguous());
    const int B = narrow(z.size(0)), N = narrow(z.size(1)), V = narrow(z.size(2));
    const Requests r(a[1], a[2], a[3], a[5], a[6], B, N, V, 1, false);
    const Results o(a[7]);
    const float T = number(a[4]);
    const int zcode = code(z);
    const void* logits = address<void>(z);
    auto* diag = field<mars_req_diag>(a[7], kDiag, true);
    void *w = address<void>(ws), *stream = stream_of(a[9]);
    const size_t bytes = static_cast<size_t>(ws.numel());
    return unlocked([&]() {
      return f_verify(logits, zcode, r.tok, r.par, r.q, r.qcode, r.theta, T, r.u, B, N, V, o.mask, o.len, o.path, o.bonus, o.dec, o.status,
                      o.stats, diag, w, bytes, stream);
    });
  });
}
// ..., indicator, n_theta, spin_limit, stages, stream
PyObject* verify_ex(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return regular([&]() -> int {
    require(n == 14);
    const Tensor &z = tensor(a[0]), &ws = tensor(a[8]);
    require(z.dim() == 3 && z.is_contiguous());
    const int B = narrow(z.size(0)), N = narrow(z.size(1)), V = narrow(z.size(2)), K = integer(a[10]);
    const Requests r(a[1], a[2], a[3], a[5], a[6], B, N, V, K, true);
    const mars_verify_options opt = options_of(a[7], a[9], K, a[11], a[12]);
    const Results o(a[7]);
    const float T = number(a[4]);
    const int zcode = code(z);
    const void* logits = address<void>(z);
    auto* diag = field<mars_req_diag>(a[7], kDiag, true);
    void *w = address<void>(ws), *stream = stream_of(a[13]);
    const size_t bytes = static_cast<size_t>(ws.numel());
    return unlocked([&]() {
      return f_verify_ex(logits, zcode, r.tok, r.par, r.q, r.qcode, r.theta, T, r.u, B, N, V, o.mask, o.len, o.path, o.bonus, o.dec,
                         o.status, o.stats, diag, w, bytes, stream, &opt);
    });
  });
}
// logits, theta, temperature, ranges, bins, rows_out, counts, workspace, stream
PyObject* margin_stats(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return regular([&]() -> int {
    require(n == 9);
    const Tensor &z = tensor(a[0]), &th = tensor(a[1]), &ws = tensor(a[7]);
    require(z.dim() == 3 && z.is_contiguous());
    const int B = narrow(z.size(0)), N = narrow(z.size(1)), V = narrow(z.size(2));
    require(th.scalar_type() == at::kFloat && th.numel() == B);
    require(PyTuple_CheckExact(a[3]) && PyTuple_GET_SIZE(a[3]) == 6 && PyTuple_CheckExact(a[4]) && PyTuple_GET_SIZE(a[4]) == 3);
    float range[6];
    int32_t bins[3];
    for (int i = 0; i < 6; ++i) range[i] = number(PyTuple_GET_ITEM(a[3], i));
    for (int i = 0; i < 3; ++i) bins[i] = integer(PyTuple_GET_ITEM(a[4], i));
    const float T = number(a[2]);
    const int zcode = code(z);
    const void* logits = address<void>(z);
    const float* theta = address<float>(th);
    auto* rows = a[5] == Py_None ? nullptr : address<mars_margin_row>(tensor(a[5]));
    auto* counts = address<uint32_t>(tensor(a[6]));
    void *w = address<void>(ws), *stream = stream_of(a[8]);
    const size_t bytes = static_cast<size_t>(ws.numel());
    return unlocked([&]() { return f_margin(logits, zcode, theta, T, B, N, V, range, bins, rows, counts, w, bytes, stream); });
  });
}
// hidden, weight, draft_tokens, tree_parent, theta, out, workspace, indicator, n_theta, stages, stream
PyObject* lmhead_verify(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return regular([&]() -> int {
    require(n == 11);
    const Tensor &h = tensor(a[0]), &w = tensor(a[1]), &ws = tensor(a[6]);
    require(h.dim() == 3 && h.is_contiguous() && w.dim() == 2 && w.is_contiguous() && w.size(1) == h.size(2));
    require(code(h) == MARS_BF16 && code(w) == MARS_BF16);
    const int B = narrow(h.size(0)), N = narrow(h.size(1)), H = narrow(h.size(2)), V = narrow(w.size(0)), K = integer(a[8]);
    const Requests r(a[2], a[3], a[4], Py_None, Py_None, B, N, V, K, true);
    mars_verify_options opt = options_of(a[5], a[7], K, a[9], a[9]);
    opt.spin_limit = 0;
    const Results o(a[5]);
    const void *hp = address<void>(h), *wp = address<void>(w);
    void *work = address<void>(ws), *stream = stream_of(a[10]);
    const size_t bytes = static_cast<size_t>(ws.numel());
    return unlocked([&]() {
      return f_lmhead(hp, wp, H, r.tok, r.par, r.theta, B, N, V, o.mask, o.len, o.path, o.bonus, o.dec, o.status, o.stats, work, bytes,
                      stream, &opt);
    });
  });
}
// hidden, weight, draft_tokens, tree_parent, theta, temperature, uniforms, draft_probs, logits_out, out, workspace, indicator, n_theta,
// spin_limit, stages, stream
PyObject* lmhead_verify_sampling(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return regular([&]() -> int {
    require(n == 16 && a[6] != Py_None);
    const Tensor &h = tensor(a[0]), &w = tensor(a[1]), &lo = tensor(a[8]), &ws = tensor(a[10]);
    require(h.dim() == 3 && h.is_contiguous() && w.dim() == 2 && w.is_contiguous() && w.size(1) == h.size(2));
    require(code(h) == MARS_BF16 && code(w) == MARS_BF16 && code(lo) == MARS_BF16);
    const int B = narrow(h.size(0)), N = narrow(h.size(1)), H = narrow(h.size(2)), V = narrow(w.size(0)), K = integer(a[12]);
    require(shaped(lo, B, N, V));
    const Requests r(a[2], a[3], a[4], a[6], a[7], B, N, V, K, true);
    const mars_verify_options opt = options_of(a[9], a[11], K, a[13], a[14]);
    const Results o(a[9]);
    const float T = number(a[5]);
    const void *hp = address<void>(h), *wp = address<void>(w);
    void* lp = address<void>(lo);
    auto* diag = field<mars_req_diag>(a[9], kDiag, true);
    void *work = address<void>(ws), *stream = stream_of(a[15]);
    const size_t bytes = static_cast<size_t>(ws.numel());
    return unlocked([&]() {
      return f_lmhead_sampling(hp, wp, H, r.tok, r.par, r.q, r.qcode, r.theta, T, r.u, B, N, V, lp, o.mask, o.len, o.path, o.bonus, o.dec,
                               o.status, o.stats, diag, work, bytes, stream, &opt);
    });
  });
}

// The addresses of the library's functions, in the order of the functions above.
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void* at[5];
  if (n != 5) { PyErr_SetString(PyExc_TypeError, "bind: five addresses"); return nullptr; }
  for (int i = 0; i < 5; ++i) {
    at[i] = PyLong_AsVoidPtr(a[i]);
    if (PyErr_Occurred()) return nullptr;
  }
  f_verify = reinterpret_cast<decltype(f_verify)>(at[0]);
  f_verify_ex = reinterpret_cast<decltype(f_verify_ex)>(at[1]);
  f_margin = reinterpret_cast<decltype(f_margin)>(at[2]);
  f_lmhead = reinterpret_cast<decltype(f_lmhead)>(at[3]);
  f_lmhead_sampling = reinterpret_cast<decltype(f_lmhead_sampling)>(at[4]);
  Py_RETURN_NONE;
}

#define MARS_METHOD(F) {#F, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(F)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {MARS_METHOD(bind),          MARS_METHOD(verify),        MARS_METHOD(verify_ex),
                           MARS_METHOD(margin_stats),  MARS_METHOD(lmhead_verify), MARS_METHOD(lmhead_verify_sampling),
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() {
  for (int i = 0; i < kFields; ++i)
    if (!(g_names[i] = PyUnicode_InternFromString(kNames[i]))) return nullptr;
  PyObject* m = PyModule_Create(&g_module);
  // (what it was built against: the binding looks at no tensor through another version's layout)
  if (m && PyModule_AddStringConstant(m, "torch_version", MARS_TORCH_VERSION) != 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
