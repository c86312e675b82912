// The calls of binding.py that a training or serving step makes many times, in native code: tensors in, C ABI out.  Host
// code only.  With small batches the host's time per call is what bounds a step: in Python a call cost 1.5 to 4 us on top of
// the launch, most of it for looking at tensors (data_ptr, shape, stride) one method call at a time.
//
// One object (`Calls`) per imported binding: it holds the addresses of the C functions, the binding's error class and how to
// find the current stream.  Its methods take what the binding documents, by position or by name, and do what the C ABI does
// not: defaults, allocation of what is not given, and the checks of shapes and strides that are left once a tensor is a pointer.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include <cstdint>
#include <utility>

#include "mosaic_attn.h"

namespace {

// Thrown with the Python error set.
struct Raised {};

[[noreturn]] void raise(PyObject* type, const char* text) {
  PyErr_SetString(type, text);
  throw Raised();
}
void require(bool ok, const char* text) {
  if (!ok) raise(PyExc_AssertionError, text);
}

struct Calls {
  PyObject_HEAD
  PyObject* error;        // the binding's exception class: (status, message)
  PyObject* device;       // () -> current device
  PyObject* raw_stream;   // (device) -> stream handle, or None
  PyObject* stream;       // () -> stream handle, where there is no raw_stream
  decltype(&mb_last_error) last_error;
  decltype(&mb_unpad_index) unpad_index;
  decltype(&mb_unpad) unpad;
  decltype(&mb_pad) pad;
  decltype(&mb_zero_padding) zero_padding;
  decltype(&mb_alibi_attn_fwd) attn_fwd;
  decltype(&mb_alibi_attn_fwd_workspace_bytes) attn_fwd_bytes;
  decltype(&mb_alibi_attn_bwd) attn_bwd;
  decltype(&mb_alibi_attn_bwd_workspace_bytes) attn_bwd_bytes;
  decltype(&mb_add_layernorm_fwd) layernorm_fwd;
  decltype(&mb_add_layernorm_bwd) layernorm_bwd;
  decltype(&mb_add_layernorm_bwd_workspace_bytes) layernorm_bwd_bytes;
  decltype(&mb_geglu_fwd) geglu_fwd;
  decltype(&mb_geglu_bwd) geglu_bwd;
  decltype(&mb_geglu_bwd_workspace_bytes) geglu_bwd_bytes;
  decltype(&mb_linear_fwd) linear_fwd;
};

// ---------------------------------------------------------------------------------------------------- arguments
// The parameters of a call: keywords arrive as interned strings, so that looking for one is comparing pointers.
template <int N>
struct Names {
  const char* text[N];
  PyObject* interned[N];
  template <typename... T>
  explicit Names(T... t) : text{t...}, interned{PyUnicode_InternFromString(t)...} {
    static_assert(sizeof...(T) == N, "as many names as parameters");
  }
  int find(PyObject* key) const {
    for (int i = 0; i < N; ++i)
      if (key == interned[i]) return i;
    for (int i = 0; i < N; ++i)
      if (PyUnicode_CompareWithASCIIString(key, text[i]) == 0) return i;
    return N;
  }
};
template <typename... T>
Names(T...) -> Names<sizeof...(T)>;

// What x.name() gives: the calls below take a bare pointer from any object that has the method.
PyObject* asked(PyObject* x, const char* name) {
  PyObject* r = PyObject_CallMethod(x, name, nullptr);
  if (!r) throw Raised();
  return r;
}

// The arguments of a call by their place in `names` (nullptr where not given).
template <int N>
struct Args {
  PyObject* v[N] = {};
  Args(const char* call, const Names<N>& names, int required, PyObject* const* args, Py_ssize_t n, PyObject* kw) {
    if (n > N) {
      PyErr_Format(PyExc_TypeError, "%s() takes %d arguments but %zd were given", call, N, n);
      throw Raised();
    }
    for (Py_ssize_t i = 0; i < n; ++i) v[i] = args[i];
    const Py_ssize_t nk = kw ? PyTuple_GET_SIZE(kw) : 0;
    for (Py_ssize_t j = 0; j < nk; ++j) {
      PyObject* key = PyTuple_GET_ITEM(kw, j);
      const int at = names.find(key);
      if (at == N) {
        PyErr_Format(PyExc_TypeError, "%s() got an unexpected keyword argument '%U'", call, key);
        throw Raised();
      }
      if (v[at]) {
        PyErr_Format(PyExc_TypeError, "%s() got multiple values for argument '%s'", call, names.text[at]);
        throw Raised();
      }
      v[at] = args[n + j];
    }
    for (int i = 0; i < required; ++i)
      if (!v[i]) {
        PyErr_Format(PyExc_TypeError, "%s() missing required argument '%s'", call, names.text[i]);
        throw Raised();
      }
  }
  bool given(int i) const { return v[i] && v[i] != Py_None; }
  const at::Tensor& tensor(int i) const {
    if (!THPVariable_Check(v[i])) {
      PyErr_Format(PyExc_TypeError, "argument %d must be a tensor, not %s", i + 1, Py_TYPE(v[i])->tp_name);
      throw Raised();
    }
    return THPVariable_Unpack(v[i]);
  }
  void* ptr(int i) const {
    if (!given(i)) return nullptr;
    if (THPVariable_Check(v[i])) return THPVariable_Unpack(v[i]).data_ptr();
    PyObject* r = asked(v[i], "data_ptr");
    void* p = r == Py_None ? nullptr : PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    if (!p && PyErr_Occurred()) throw Raised();
    return p;
  }
  int64_t numel(int i) const {
    if (THPVariable_Check(v[i])) return THPVariable_Unpack(v[i]).numel();
    PyObject* r = asked(v[i], "numel");
    const int64_t n = PyLong_AsLongLong(r);
    Py_DECREF(r);
    if (n == -1 && PyErr_Occurred()) throw Raised();
    return n;
  }
  bool contiguous(int i) const {
    if (THPVariable_Check(v[i])) return THPVariable_Unpack(v[i]).is_contiguous();
    PyObject* r = asked(v[i], "is_contiguous");
    const int yes = PyObject_IsTrue(r);
    Py_DECREF(r);
    if (yes < 0) throw Raised();
    return yes;
  }
  int integer(int i) const {   // as ctypes converts to a C int
    PyObject* x = PyNumber_Index(v[i]);
    if (!x) throw Raised();
    const unsigned long u = PyLong_AsUnsignedLongMask(x);
    Py_DECREF(x);
    if (u == (unsigned long)-1 && PyErr_Occurred()) throw Raised();
    return (int)u;
  }
  int integer_or(int i, int64_t otherwise) const { return given(i) ? integer(i) : (int)otherwise; }
  float number(int i) const {
    PyObject* x = PyNumber_Float(v[i]);
    if (!x) throw Raised();
    const double d = PyFloat_AS_DOUBLE(x);
    Py_DECREF(x);
    return (float)d;
  }
};

// A result: the object that was given, or a tensor made here.
struct Result {
  PyObject* object = nullptr;   // borrowed, if given
  at::Tensor made;
  void* ptr = nullptr;
  template <typename A, typename Make>
  Result(const A& a, int i, Make make) {
    if (a.given(i)) {
      object = a.v[i];
      ptr = a.ptr(i);
    } else {
      made = make();
      ptr = made.data_ptr();
    }
  }
  template <typename A>
  const at::Tensor& tensor(const A& a, int i) const { return object ? a.tensor(i) : made; }
  template <typename A>
  size_t numel(const A& a, int i) const { return (size_t)(object ? a.numel(i) : made.numel()); }
  PyObject* take() {
    if (object) {
      Py_INCREF(object);
      return object;
    }
    return THPVariable_Wrap(std::move(made));
  }
};

template <typename... R>
PyObject* tuple_of(R&&... results) {
  PyObject* t = PyTuple_New(sizeof...(results));
  if (!t) throw Raised();
  Py_ssize_t i = 0;
  auto put = [&](PyObject* x) {
    if (!x) {
      Py_DECREF(t);
      throw Raised();
    }
    PyTuple_SET_ITEM(t, i++, x);
  };
  (put(results), ...);
  return t;
}

int dtype_code(const at::Tensor& t) {
  if (t.scalar_type() == at::kBFloat16) return MB_BF16;
  if (t.scalar_type() == at::kFloat) return MB_F32;
  const std::string text = std::string("unsupported dtype ") + c10::toString(t.scalar_type());
  raise(PyExc_TypeError, text.c_str());
}

// [T, H, D] view with dense (H, D): the token stride in elements.
int64_t row_stride(const at::Tensor& t) {
  require(t.dim() == 3 && t.stride(2) == 1 && t.stride(1) == t.size(2), "need [T, H, D] with dense (H, D)");
  return t.size(0) > 1 ? t.stride(0) : std::max(t.stride(0), t.size(1) * t.size(2));
}

at::Tensor new_like(const at::Tensor& like, at::IntArrayRef sizes, at::ScalarType type) {
  return at::empty(sizes, like.options().dtype(type).requires_grad(false));
}
at::Tensor new_bytes(const at::Tensor& like, size_t n) { return new_like(like, {(int64_t)n}, at::kByte); }

void* current_stream(const Calls* s) {
  PyObject* handle;
  if (s->raw_stream == Py_None) {
    handle = PyObject_CallNoArgs(s->stream);
  } else {
    PyObject* device = PyObject_CallNoArgs(s->device);
    if (!device) throw Raised();
    handle = PyObject_CallOneArg(s->raw_stream, device);
    Py_DECREF(device);
  }
  if (!handle) throw Raised();
  void* p = handle == Py_None ? nullptr : PyLong_AsVoidPtr(handle);
  Py_DECREF(handle);
  if (!p && PyErr_Occurred()) throw Raised();
  return p;
}

// Runs the C function without the interpreter's lock, as ctypes does.
template <typename F, typename... A>
void run(const Calls* s, F function, A... args) {
  mb_status status;
  Py_BEGIN_ALLOW_THREADS
  status = function(args...);
  Py_END_ALLOW_THREADS
  if (status == MB_OK) return;
  PyObject* e = PyObject_CallFunction(s->error, "is", (int)status, s->last_error());
  if (e) {
    PyErr_SetObject(s->error, e);
    Py_DECREF(e);
  }
  throw Raised();
}

// ---------------------------------------------------------------------------------------------------- the calls
using Self = const Calls*;
using Argv = PyObject* const*;

PyObject* unpad_index(Self s, Argv argv, Py_ssize_t n, PyObject* kw) {
  static const Names names("mask");
  const Args<1> a("mb_unpad_index", names, 1, argv, n, kw);
  const at::Tensor& mask = a.tensor(0);
  require(mask.scalar_type() == at::kInt && mask.dim() == 2 && mask.is_contiguous(), "need a contiguous [B, L] int32 mask");
  const int64_t B = mask.size(0), L = mask.size(1);
  auto make = [&](int64_t count) { return new_like(mask, {count}, at::kInt); };
  at::Tensor seqlens = B > 0 ? make(B) : make(1).slice(0, 0, 0), cu = make(B + 1),
             indices = B * L > 0 ? make(B * L) : make(1).slice(0, 0, 0), meta = make(2);
  void* const stream = current_stream(s);
  run(s, s->unpad_index, (const int32_t*)mask.data_ptr(), (int)B, (int)L, (int32_t*)seqlens.data_ptr(),
      (int32_t*)cu.data_ptr(), (int32_t*)indices.data_ptr(), (int32_t*)meta.data_ptr(), stream);
  return tuple_of(THPVariable_Wrap(std::move(seqlens)), THPVariable_Wrap(std::move(cu)), THPVariable_Wrap(std::move(indices)),
                  THPVariable_Wrap(std::move(meta)));
}

PyObject* unpad(Self s, Argv argv, Py_ssize_t n, PyObject* kw) {
  static const Names names("padded", "indices", "T_cap", "meta", "out");
  const Args<5> a("mb_unpad", names, 4, argv, n, kw);
  const at::Tensor& padded = a.tensor(0);
  require(padded.dim() == 2 && padded.is_contiguous(), "padded must be a contiguous matrix");
  const int64_t W = padded.size(1);
  const int T_cap = a.integer(2);
  Result out(a, 4, [&] { return new_like(padded, {T_cap, W}, padded.scalar_type()); });
  const at::Tensor& o = out.tensor(a, 4);
  require(o.is_contiguous() && o.dim() >= 2 && o.size(1) == W && o.size(0) >= T_cap, "out must be contiguous, [>= T_cap, W]");
  const mb_dtype dt = (mb_dtype)dtype_code(padded);
  void* const stream = current_stream(s);
  run(s, s->unpad, padded.data_ptr(), (const int32_t*)a.ptr(1), T_cap, (const int32_t*)a.ptr(3), (int)W,
      dt, out.ptr, stream);
  return out.take();
}

PyObject* pad(Self s, Argv argv, Py_ssize_t n, PyObject* kw) {
  static const Names names("packed", "indices", "T_cap", "meta", "B", "L", "out");
  const Args<7> a("mb_pad", names, 6, argv, n, kw);
  const at::Tensor& packed = a.tensor(0);
  require(packed.dim() == 2 && packed.is_contiguous(), "packed must be a contiguous matrix");
  const int64_t W = packed.size(1);
  const int B = a.integer(4), L = a.integer(5);
  Result out(a, 6, [&] { return new_like(packed, {(int64_t)B * L, W}, packed.scalar_type()); });
  const at::Tensor& o = out.tensor(a, 6);
  require(o.is_contiguous() && o.dim() == 2 && o.size(0) == (int64_t)B * L && o.size(1) == W, "out must be contiguous, [B * L, W]");
  const mb_dtype dt = (mb_dtype)dtype_code(packed);
  void* const stream = current_stream(s);
  run(s, s->pad, packed.data_ptr(), (const int32_t*)a.ptr(1), a.integer(2), (const int32_t*)a.ptr(3), B, L, (int)W,
      dt, out.ptr, stream);
  return out.take();
}

PyObject* zero_padding(Self s, Argv argv, Py_ssize_t n, PyObject* kw) {
  static const Names names("padded", "indices", "T_cap", "meta", "B", "L");
  const Args<6> a("mb_zero_padding", names, 6, argv, n, kw);
  const at::Tensor& padded = a.tensor(0);
  const int B = a.integer(4), L = a.integer(5);
  require(padded.dim() == 2 && padded.is_contiguous() && padded.size(0) == (int64_t)B * L, "padded must be contiguous, [B * L, W]");
  const mb_dtype dt = (mb_dtype)dtype_code(padded);
  void* const stream = current_stream(s);
  run(s, s->zero_padding, (const int32_t*)a.ptr(1), a.integer(2), (const int32_t*)a.ptr(3), B, L, (int)padded.size(1),
      dt, padded.data_ptr(), stream);
  Py_INCREF(a.v[0]);
  return a.v[0];
}

// [T, H, D] of q: what an attention call takes its sizes from.
void attention_sizes(const at::Tensor& q, int64_t* R, int64_t* H, int64_t* D) {
  if (q.dim() != 3) raise(PyExc_ValueError, "q must be [T, H, D]");
  *R = q.size(0);
  *H = q.size(1);
  *D = q.size(2);
}

PyObject* attn_fwd(Self s, Argv argv, Py_ssize_t n, PyObject* kw) {
  static const Names names("q", "k", "v", "cu_seqlens", "max_seqlen", "slopes", "softmax_scale", "out", "lse",
                                      "token_rows", "T", "workspace", "key_lens", "plan");
  const Args<14> a("mb_alibi_attn_fwd", names, 7, argv, n, kw);
  const at::Tensor &q = a.tensor(0), &k = a.tensor(1), &v = a.tensor(2);
  int64_t R, H, D;
  attention_sizes(q, &R, &H, &D);
  const int T = a.integer_or(10, R), max_seqlen = a.integer(4), B = (int)(a.numel(3) - 1);
  Result out(a, 7, [&] { return new_like(q, {R, H, D}, q.scalar_type()); });
  Result lse(a, 8, [&] { return new_like(q, {H, T}, at::kFloat); });
  const mb_dtype dt = (mb_dtype)dtype_code(q);
  at::Tensor own;
  void* workspace = a.ptr(11);
  size_t workspace_bytes = a.given(11) ? (size_t)a.numel(11) : 0;
  if (!a.given(11) && !a.given(13)) {
    workspace_bytes = s->attn_fwd_bytes(B, T, max_seqlen, (int)H, (int)D, dt);
    if (workspace_bytes > 0) {
      own = new_bytes(q, workspace_bytes);
      workspace = own.data_ptr();
    }
  }
  void* const stream = current_stream(s);
  run(s, s->attn_fwd, (const void*)q.data_ptr(), (const void*)k.data_ptr(), (const void*)v.data_ptr(), row_stride(q),
      row_stride(k), row_stride(v), (const int32_t*)a.ptr(3), B, T, max_seqlen, (int)H, (int)D,
      (const float*)a.ptr(5), a.number(6), dt, out.ptr, row_stride(out.tensor(a, 7)), (float*)lse.ptr, workspace, workspace_bytes,
      (const int32_t*)a.ptr(12), (const int32_t*)a.ptr(9), (const void*)a.ptr(13), stream);
  return tuple_of(out.take(), lse.take());
}

PyObject* attn_bwd(Self s, Argv argv, Py_ssize_t n, PyObject* kw) {
  static const Names names("dout", "q", "k", "v", "o", "lse", "cu_seqlens", "max_seqlen", "slopes",
                                      "softmax_scale", "dq", "dk", "dv", "workspace", "token_rows", "T", "key_lens", "plan");
  const Args<18> a("mb_alibi_attn_bwd", names, 10, argv, n, kw);
  const at::Tensor &dout = a.tensor(0), &q = a.tensor(1), &k = a.tensor(2), &v = a.tensor(3), &o = a.tensor(4);
  int64_t R, H, D;
  attention_sizes(q, &R, &H, &D);
  const int T = a.integer_or(15, R), max_seqlen = a.integer(7), B = (int)(a.numel(6) - 1);
  auto make = [&] { return new_like(q, {R, H, D}, q.scalar_type()); };
  Result dq(a, 10, make), dk(a, 11, make), dv(a, 12, make);
  const mb_dtype dt = (mb_dtype)dtype_code(q);
  Result workspace(a, 13, [&] {
    return new_bytes(q, std::max<size_t>(s->attn_bwd_bytes(B, T, max_seqlen, (int)H, (int)D, dt), 16));
  });
  void* const stream = current_stream(s);
  run(s, s->attn_bwd, (const void*)dout.data_ptr(), (const void*)q.data_ptr(), (const void*)k.data_ptr(),
      (const void*)v.data_ptr(), (const void*)o.data_ptr(), (const float*)a.ptr(5), row_stride(dout), row_stride(q),
      row_stride(k), row_stride(v), row_stride(o), (const int32_t*)a.ptr(6), B, T, max_seqlen, (int)H, (int)D,
      (const float*)a.ptr(8), a.number(9), dt, dq.ptr, dk.ptr, dv.ptr, row_stride(dq.tensor(a, 10)), row_stride(dk.tensor(a, 11)),
      row_stride(dv.tensor(a, 12)), workspace.ptr, workspace.numel(a, 13), (const int32_t*)a.ptr(16),
      (const int32_t*)a.ptr(14), (const void*)a.ptr(17), stream);
  return tuple_of(dq.take(), dk.take(), dv.take());
}

PyObject* layernorm_fwd(Self s, Argv argv, Py_ssize_t n, PyObject* kw) {
  static const Names names("x", "r", "gamma", "beta", "eps", "T_cap", "meta", "y", "s", "mean", "rstd", "y_rows");
  const Args<12> a("mb_add_layernorm_fwd", names, 5, argv, n, kw);
  const at::Tensor& x = a.tensor(0);
  require(x.dim() == 2 && x.is_contiguous(), "x must be a contiguous matrix");
  require(!a.given(11) || a.given(7), "y_rows needs y");
  const int64_t rows = x.size(0), W = x.size(1);
  auto like = [&] { return new_like(x, {rows, W}, x.scalar_type()); };
  auto per_row = [&] { return new_like(x, {rows}, at::kFloat); };
  const bool add = a.given(1);
  Result y(a, 7, like);
  Result sum(a, add ? 8 : 0, like);   // without r the sum is x itself
  Result mean(a, 9, per_row), rstd(a, 10, per_row);
  const mb_dtype dt = (mb_dtype)dtype_code(x);
  void* const stream = current_stream(s);
  run(s, s->layernorm_fwd, (const void*)x.data_ptr(), (const void*)a.ptr(1), (const void*)a.ptr(2), (const void*)a.ptr(3),
      a.integer_or(5, rows), (const int32_t*)a.ptr(6), (int)W, a.number(4), dt, y.ptr,
      add ? sum.ptr : nullptr, (float*)mean.ptr, (float*)rstd.ptr, (const int32_t*)a.ptr(11), stream);
  return tuple_of(y.take(), sum.take(), mean.take(), rstd.take());
}

PyObject* layernorm_bwd(Self s, Argv argv, Py_ssize_t n, PyObject* kw) {
  static const Names names("dy", "s", "gamma", "mean", "rstd", "T_cap", "meta", "ds", "dgamma", "dbeta",
                                      "workspace", "dy_rows");
  const Args<12> a("mb_add_layernorm_bwd", names, 5, argv, n, kw);
  const at::Tensor& sum = a.tensor(1);
  if (sum.dim() != 2) raise(PyExc_ValueError, "s must be a matrix");
  const int64_t rows = sum.size(0), W = sum.size(1);
  auto column = [&] { return new_like(sum, {W}, at::kFloat); };
  Result ds(a, 7, [&] { return at::empty_like(sum, sum.options().requires_grad(false)); });
  Result dgamma(a, 8, column), dbeta(a, 9, column);
  Result workspace(a, 10, [&] { return new_bytes(sum, s->layernorm_bwd_bytes((int)W)); });
  const mb_dtype dt = (mb_dtype)dtype_code(sum);
  void* const stream = current_stream(s);
  run(s, s->layernorm_bwd, (const void*)a.ptr(0), (const void*)sum.data_ptr(), (const void*)a.ptr(2), (const float*)a.ptr(3),
      (const float*)a.ptr(4), a.integer_or(5, rows), (const int32_t*)a.ptr(6), (int)W, dt, ds.ptr,
      (float*)dgamma.ptr, (float*)dbeta.ptr, workspace.ptr, workspace.numel(a, 10), (const int32_t*)a.ptr(11),
      stream);
  return tuple_of(ds.take(), dgamma.take(), dbeta.take());
}

PyObject* geglu_fwd(Self s, Argv argv, Py_ssize_t n, PyObject* kw) {
  static const Names names("x", "w1v", "w2", "T_cap", "meta", "act", "y");
  const Args<7> a("mb_geglu_fwd", names, 3, argv, n, kw);
  const at::Tensor &x = a.tensor(0), &w1v = a.tensor(1), &w2 = a.tensor(2);
  require(x.dim() == 2 && x.is_contiguous() && w1v.is_contiguous() && w2.is_contiguous(), "x, w1v and w2 must be contiguous");
  require(w1v.dim() == 2 && w2.dim() == 2, "w1v and w2 must be matrices");
  const int64_t rows = x.size(0), hidden = x.size(1), inter = w2.size(1);
  require(w1v.size(0) == 2 * inter && w1v.size(1) == hidden && w2.size(0) == hidden, "w1v [2 inter, hidden], w2 [hidden, inter]");
  Result act(a, 5, [&] { return new_like(x, {rows, inter}, x.scalar_type()); });
  Result y(a, 6, [&] { return new_like(x, {rows, hidden}, x.scalar_type()); });
  const mb_dtype dt = (mb_dtype)dtype_code(x);
  void* const stream = current_stream(s);
  run(s, s->geglu_fwd, (const void*)x.data_ptr(), (const void*)w1v.data_ptr(), (const void*)w2.data_ptr(),
      a.integer_or(3, rows), (const int32_t*)a.ptr(4), (int)hidden, (int)inter, dt, act.ptr, y.ptr,
      stream);
  return tuple_of(y.take(), act.take());
}

PyObject* geglu_bwd(Self s, Argv argv, Py_ssize_t n, PyObject* kw) {
  static const Names names("dy", "x", "w1v", "w2", "act", "hg", "T_cap", "meta", "dx", "dw1v", "dw2", "workspace");
  const Args<12> a("mb_geglu_bwd", names, 5, argv, n, kw);
  require(!a.given(5) || a.contiguous(5), "hg must be contiguous");
  const at::Tensor &x = a.tensor(1), &w2 = a.tensor(3);
  if (x.dim() != 2) raise(PyExc_ValueError, "x must be a matrix");
  if (w2.dim() < 2) raise(PyExc_IndexError, "w2 must be a matrix");
  const int64_t rows = x.size(0), hidden = x.size(1), inter = w2.size(1);
  const int T_cap = a.integer_or(6, rows);
  const mb_dtype dt = (mb_dtype)dtype_code(x);
  Result dx(a, 8, [&] { return at::empty_like(x, x.options().requires_grad(false)); });
  Result dw1v(a, 9, [&] { return new_like(x, {2 * inter, hidden}, at::kFloat); });
  Result dw2(a, 10, [&] { return new_like(x, {hidden, inter}, at::kFloat); });
  Result workspace(a, 11, [&] {
    return new_bytes(x, std::max<size_t>(s->geglu_bwd_bytes(T_cap, (int)hidden, (int)inter, dt), 256));
  });
  void* const stream = current_stream(s);
  run(s, s->geglu_bwd, (const void*)a.ptr(0), (const void*)x.data_ptr(), (const void*)a.ptr(2), (const void*)w2.data_ptr(),
      (const void*)a.ptr(4), (const void*)a.ptr(5), T_cap, (const int32_t*)a.ptr(7), (int)hidden, (int)inter, dt, dx.ptr,
      (float*)dw1v.ptr, (float*)dw2.ptr, workspace.ptr, workspace.numel(a, 11), stream);
  return tuple_of(dx.take(), dw1v.take(), dw2.take());
}

PyObject* linear_fwd(Self s, Argv argv, Py_ssize_t n, PyObject* kw) {
  static const Names names("x", "wt", "T_cap", "meta", "y");
  const Args<5> a("mb_linear_fwd", names, 2, argv, n, kw);
  const at::Tensor &x = a.tensor(0), &wt = a.tensor(1);
  require(x.dim() == 2 && x.is_contiguous() && wt.is_contiguous() && wt.dim() >= 2 && wt.size(1) == x.size(1),
          "x and wt must be contiguous, with as many columns");
  const int64_t rows = x.size(0), n_in = x.size(1), n_out = wt.size(0);
  Result y(a, 4, [&] { return new_like(x, {rows, n_out}, x.scalar_type()); });
  const mb_dtype dt = (mb_dtype)dtype_code(x);
  void* const stream = current_stream(s);
  run(s, s->linear_fwd, (const void*)x.data_ptr(), (const void*)wt.data_ptr(), a.integer_or(2, rows), (const int32_t*)a.ptr(3),
      (int)n_in, (int)n_out, dt, y.ptr, stream);
  return y.take();
}

// ---------------------------------------------------------------------------------------------------- the object
// No C++ exception leaves a method.
template <PyObject* (*F)(Self, Argv, Py_ssize_t, PyObject*)>
PyObject* guarded(PyObject* self, PyObject* const* args, Py_ssize_t n, PyObject* kw) {
  HANDLE_TH_ERRORS
  try {
    return F(reinterpret_cast<const Calls*>(self), args, n, kw);
  } catch (const Raised&) {
    return nullptr;
  }
  END_HANDLE_TH_ERRORS
}
template <PyObject* (*F)(Self, Argv, Py_ssize_t, PyObject*)>
PyCFunction method() {
  return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&guarded<F>));
}
#define MB_METHOD(name, f, doc) {name, method<f>(), METH_FASTCALL | METH_KEYWORDS, doc}

PyMethodDef methods[] = {
    MB_METHOD("mb_unpad_index", unpad_index,
              "mb_unpad_index($self, mask)\n--\n\n"
              "mask [B, L] int32 on the GPU -> (seqlens [B], cu_seqlens [B+1], indices [B*L] (first T valid), meta [2])."),
    MB_METHOD("mb_unpad", unpad,
              "mb_unpad($self, padded, indices, T_cap, meta, out=None)\n--\n\n"
              "padded [B*L, W] (any leading shape flattened by the caller) -> packed [T_cap, W]; rows < T written."),
    MB_METHOD("mb_pad", pad,
              "mb_pad($self, packed, indices, T_cap, meta, B, L, out=None)\n--\n\n"
              "packed [>=T, W] -> padded [B*L, W], zero at padded positions."),
    MB_METHOD("mb_zero_padding", zero_padding,
              "mb_zero_padding($self, padded, indices, T_cap, meta, B, L)\n--\n\n"
              "Zero the rows of padded [B*L, W] that `indices` does not list."),
    MB_METHOD("mb_alibi_attn_fwd", attn_fwd,
              "mb_alibi_attn_fwd($self, q, k, v, cu_seqlens, max_seqlen, slopes, softmax_scale, out=None, lse=None, "
              "token_rows=None, T=None, workspace=None, key_lens=None, plan=None)\n--\n\n"
              "q, k, v: [T, H, D] views (token stride free).  Returns (o [T, H, D], lse [H, T] float32).\n"
              "With token_rows the views are over a padded batch ([B*L, H, D]) and T (the lse pitch) must be given."),
    MB_METHOD("mb_alibi_attn_bwd", attn_bwd,
              "mb_alibi_attn_bwd($self, dout, q, k, v, o, lse, cu_seqlens, max_seqlen, slopes, softmax_scale, dq=None, "
              "dk=None, dv=None, workspace=None, token_rows=None, T=None, key_lens=None, plan=None)\n--\n\n"
              "Returns (dq, dk, dv), each [T, H, D] (padded-batch views when token_rows is given)."),
    MB_METHOD("mb_add_layernorm_fwd", layernorm_fwd,
              "mb_add_layernorm_fwd($self, x, r, gamma, beta, eps, T_cap=None, meta=None, y=None, s=None, mean=None, "
              "rstd=None, y_rows=None)\n--\n\n"
              "x, r: [rows, W] (r may be None).  Returns (y, s, mean, rstd); s is x itself when r is None.\n"
              "With y_rows, y must be given: a padded batch whose row y_rows[t] receives the result of token t."),
    MB_METHOD("mb_add_layernorm_bwd", layernorm_bwd,
              "mb_add_layernorm_bwd($self, dy, s, gamma, mean, rstd, T_cap=None, meta=None, ds=None, dgamma=None, "
              "dbeta=None, workspace=None, dy_rows=None)\n--\n\n"
              "Returns (ds [rows, W], dgamma [W] float32, dbeta [W] float32).\n"
              "With dy_rows, dy is a padded batch and token t's row is dy[dy_rows[t]]."),
    MB_METHOD("mb_geglu_fwd", geglu_fwd,
              "mb_geglu_fwd($self, x, w1v, w2, T_cap=None, meta=None, act=None, y=None)\n--\n\n"
              "x [rows, hidden]; w1v [2*inter, hidden] (W1 transposed over V transposed); w2 [hidden, inter] (W2\n"
              "transposed).  Returns (y [rows, hidden], act [rows, inter])."),
    MB_METHOD("mb_geglu_bwd", geglu_bwd,
              "mb_geglu_bwd($self, dy, x, w1v, w2, act, hg=None, T_cap=None, meta=None, dx=None, dw1v=None, dw2=None, "
              "workspace=None)\n--\n\n"
              "Returns (dx [rows, hidden], dw1v [2*inter, hidden] float32, dw2 [hidden, inter] float32).  hg: the stored\n"
              "[rows, 2*inter] projections of the unfused forward, or None to have them computed again."),
    MB_METHOD("mb_linear_fwd", linear_fwd,
              "mb_linear_fwd($self, x, wt, T_cap=None, meta=None, y=None)\n--\n\n"
              "y = x @ wt.T for x [rows, n_in], wt [n_out, n_in]."),
    {nullptr, nullptr, 0, nullptr}};

// Calls(addresses, error, device, raw_stream, stream): `addresses` maps names of the C ABI to function addresses.
PyObject* calls_new(PyTypeObject* type, PyObject* args, PyObject*) {
  PyObject *addresses, *error, *device, *raw_stream, *stream;
  if (!PyArg_ParseTuple(args, "O!OOOO", &PyDict_Type, &addresses, &error, &device, &raw_stream, &stream)) return nullptr;
  Calls* c = reinterpret_cast<Calls*>(type->tp_alloc(type, 0));
  if (!c) return nullptr;
  auto keep = [](PyObject*& to, PyObject* x) {
    Py_INCREF(x);
    to = x;
  };
  keep(c->error, error);
  keep(c->device, device);
  keep(c->raw_stream, raw_stream);
  keep(c->stream, stream);
  bool ok = true;
  auto find = [&](auto& to, const char* name) {
    PyObject* x = ok ? PyDict_GetItemString(addresses, name) : nullptr;
    void* p = x ? PyLong_AsVoidPtr(x) : nullptr;
    if (ok && !p) {
      if (!PyErr_Occurred()) PyErr_Format(PyExc_KeyError, "no address of %s", name);
      ok = false;
    }
    to = reinterpret_cast<std::remove_reference_t<decltype(to)>>(p);
  };
  find(c->last_error, "mb_last_error");
  find(c->unpad_index, "mb_unpad_index");
  find(c->unpad, "mb_unpad");
  find(c->pad, "mb_pad");
  find(c->zero_padding, "mb_zero_padding");
  find(c->attn_fwd, "mb_alibi_attn_fwd");
  find(c->attn_fwd_bytes, "mb_alibi_attn_fwd_workspace_bytes");
  find(c->attn_bwd, "mb_alibi_attn_bwd");
  find(c->attn_bwd_bytes, "mb_alibi_attn_bwd_workspace_bytes");
  find(c->layernorm_fwd, "mb_add_layernorm_fwd");
  find(c->layernorm_bwd, "mb_add_layernorm_bwd");
  find(c->layernorm_bwd_bytes, "mb_add_layernorm_bwd_workspace_bytes");
  find(c->geglu_fwd, "mb_geglu_fwd");
  find(c->geglu_bwd, "mb_geglu_bwd");
  find(c->geglu_bwd_bytes, "mb_geglu_bwd_workspace_bytes");
  find(c->linear_fwd, "mb_linear_fwd");
  if (!ok) {
    Py_DECREF(c);
    return nullptr;
  }
  return reinterpret_cast<PyObject*>(c);
}

void calls_dealloc(PyObject* self) {
  Calls* c = reinterpret_cast<Calls*>(self);
  Py_XDECREF(c->error);
  Py_XDECREF(c->device);
  Py_XDECREF(c->raw_stream);
  Py_XDECREF(c->stream);
  PyTypeObject* type = Py_TYPE(self);
  type->tp_free(self);
  Py_DECREF(type);
}

PyType_Slot slots[] = {{Py_tp_new, (void*)calls_new},
                       {Py_tp_dealloc, (void*)calls_dealloc},
                       {Py_tp_methods, methods},
                       {0, nullptr}};
PyType_Spec spec = {"_mosaic_marshal.Calls", sizeof(Calls), 0, Py_TPFLAGS_DEFAULT, slots};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_mosaic_marshal", nullptr, 0, nullptr, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject* PyInit__mosaic_marshal() {
  PyObject* m = PyModule_Create(&module_def);
  if (!m) return nullptr;
  PyObject* type = PyType_FromSpec(&spec);
  if (!type || PyModule_AddObject(m, "Calls", type) < 0) {
    Py_XDECREF(type);
    Py_DECREF(m);
    return nullptr;
  }
  if (PyModule_AddStringConstant(m, "torch_version", TORCH_VERSION) < 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
