// Marshalling of the calls that a forward pass is made of, without the interpreter: tensor checks, sizes, the output's allocation
// and the call of the C entry point.  The Python functions in __init__.py are the reference for every check: a call that this file does
// not take as it is (another tensor class, a host tensor, strides, mixed types, sizes that do not fit) comes back as None and
// goes through them, so what is refused, and how, is written once.
//
// Per call, us (marshalling in Python -> here; of both 3.5 are the launch): linear 5.3 to 5.9 -> 3.8 with an output given, 7.5 -> 4.6 with one allocated; conv2d 8.2 -> 4.7.
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cmath>
#include <exception>

#include "../../include/netfuse.h"

namespace {

decltype(&netfuse_linear) f_linear, f_packed;
decltype(&netfuse_layernorm) f_layernorm;
decltype(&netfuse_attention) f_attention;
decltype(&netfuse_attention_relpos) f_relpos;
decltype(&netfuse_conv2d) f_conv2d;
PyObject* g_error;                           // callable (entry point, status) that raises

const c10::DispatchKeySet kWrapped({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                    c10::DispatchKey::Functionalize});

// A tensor whose data pointer is what the kernels may read: cuda, contiguous, float32 or bfloat16, not a wrapper.
const at::Tensor* plain(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || t.key_set().has_any(kWrapped) || !t.has_storage() || !t.is_contiguous()) return nullptr;
  const auto st = t.scalar_type();
  return st == at::kFloat || st == at::kBFloat16 ? &t : nullptr;
}
// An optional operand of type `st`: false if it is neither None nor that.
bool operand(PyObject* o, at::ScalarType st, void** p) {
  *p = nullptr;
  if (o == Py_None) return true;
  const at::Tensor* t = plain(o);
  if (!t || t->scalar_type() != st) return false;
  *p = t->data_ptr();
  return true;
}
bool whole(PyObject* o, int* v) {
  if (!PyLong_CheckExact(o)) return false;
  int over = 0;
  const long x = PyLong_AsLongAndOverflow(o, &over);
  *v = (int)x;
  return !over && x == *v;
}
bool size(int64_t n, int* v) {
  *v = (int)n;
  return n == *v;
}
bool stream_of(PyObject* o, void** s) {
  if (!PyLong_CheckExact(o)) return false;
  *s = PyLong_AsVoidPtr(o);
  return !PyErr_Occurred();
}
nf_dtype type_of(const at::Tensor& t) { return t.scalar_type() == at::kFloat ? NF_F32 : NF_BF16; }

PyObject* not_taken() {
  PyErr_Clear();
  Py_RETURN_NONE;
}
PyObject* done(const char* fn, nf_status st, PyObject* given, at::Tensor& made) {
  if (st != NF_OK) {
    PyObject* r = PyObject_CallFunction(g_error, "si", fn, (int)st);
    Py_XDECREF(r);
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, fn);
    return nullptr;
  }
  if (given != Py_None) {
    Py_INCREF(given);
    return given;
  }
  return THPVariable_Wrap(std::move(made));
}

// The interpreter's lock is not held while this lives.
struct Unlocked {
  PyThreadState* const state = PyEval_SaveThread();
  Unlocked() = default;
  Unlocked(const Unlocked&) = delete;
  ~Unlocked() noexcept(false) { PyEval_RestoreThread(state); }   // a daemon thread may end here when the interpreter does
};
// The output and the call: call(y) on the tensor given, or on a new one.  The allocation may wait for memory and the launch for room
// in its queue, for as long as the work in front of it takes, so other Python threads run meanwhile, a host callback that the queue
// waits for among them (0.05 us).  `call` takes no Python object: every operand is a pointer by then.
template <class F>
PyObject* produce(const char* fn, PyObject* given, at::IntArrayRef shape, const at::TensorOptions& like, F&& call) {
  void* y = nullptr;
  if (!operand(given, at::typeMetaToScalarType(like.dtype()), &y)) return not_taken();
  at::Tensor made;
  nf_status st;
  {
    Unlocked unlocked;
    if (given == Py_None) {
      made = at::empty(shape, like);
      y = made.data_ptr();
    }
    st = call(y);
  }
  return done(fn, st, given, made);
}

// A C++ error (an allocation that fails) is met again, and raised as torch raises it, by the Python path.
template <class F>
PyObject* guarded(F&& f) {
  try {
    return f();
  } catch (const std::exception&) {
    return not_taken();
  }
}

// X, W, bias, residual, act, out, stream
PyObject* matmul(decltype(f_linear) f, const char* name, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 7) return not_taken();
    const at::Tensor *X = plain(a[0]), *W = plain(a[1]);
    if (!X || !W || X->dim() != 3 || W->dim() != 3 || W->scalar_type() != X->scalar_type()) return not_taken();
    int M, N, K, No, act;
    void *b, *r, *s;
    if (!size(X->size(0), &M) || !size(X->size(1), &N) || !size(X->size(2), &K) || !size(W->size(2), &No) || W->size(0) != M ||
        W->size(1) != K || !operand(a[2], at::kFloat, &b) || !operand(a[3], X->scalar_type(), &r) || !whole(a[4], &act) || !stream_of(a[6], &s))
      return not_taken();
    const void *x = X->data_ptr(), *w = W->data_ptr();
    const nf_dtype dt = type_of(*X);
    return produce(name, a[5], {M, N, No}, X->options(), [=](void* y) { return f(x, w, (const float*)b, r, y, M, N, K, No, dt, (nf_act)act, s); });
  });
}
PyObject* linear(PyObject*, PyObject* const* a, Py_ssize_t n) { return matmul(f_linear, "netfuse_linear", a, n); }
PyObject* linear_packed(PyObject*, PyObject* const* a, Py_ssize_t n) { return matmul(f_packed, "netfuse_linear_packed", a, n); }

// x, gamma, beta, M, residual, eps, layout, out, stream
PyObject* layernorm(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 9) return not_taken();
    const at::Tensor* x = plain(a[0]);
    int M, layout, rows, H;
    void *g, *b, *r, *s;
    if (!x || !whole(a[3], &M) || M <= 0 || !whole(a[6], &layout) || !PyFloat_CheckExact(a[5]) || !operand(a[1], at::kFloat, &g) ||
        !operand(a[2], at::kFloat, &b) || !operand(a[4], x->scalar_type(), &r) || !stream_of(a[8], &s))
      return not_taken();
    if (layout == NF_MERGE_BATCH) {
      if (x->dim() != 3 || !size(x->size(1), &rows) || !size(x->size(2), &H)) return not_taken();
    } else if (x->dim() != 2 || !size(x->size(0), &rows) || !size(x->size(1) / M, &H)) {
      return not_taken();
    }
    const void* in = x->data_ptr();
    const float eps = (float)PyFloat_AS_DOUBLE(a[5]);
    const nf_dtype dt = type_of(*x);
    const at::DimVector shape(x->sizes());
    return produce("netfuse_layernorm", a[7], shape, x->options(), [=](void* y) {
      return f_layernorm(in, r, (const float*)g, (const float*)b, y, M, rows, H, eps, (nf_merge_dim)layout, dt, s);
    });
  });
}

// QKV[M][B*S][3 heads d] with its scale: the shape checks of both attentions
bool packed_qkv(const at::Tensor& t, PyObject* B_, PyObject* S_, PyObject* heads_, PyObject* scale_, int* M, int* B, int* S, int* heads, int* d,
                float* scale) {
  int N, H3;
  if (t.dim() != 3 || !whole(B_, B) || !whole(S_, S) || !whole(heads_, heads) || *heads <= 0 || !size(t.size(0), M) || !size(t.size(1), &N) ||
      !size(t.size(2), &H3))
    return false;
  *d = H3 / 3 / *heads;
  if (N != (int64_t)*B * *S || H3 != 3LL * *heads * *d || *d <= 0) return false;
  if (scale_ == Py_None) *scale = (float)std::pow((double)*d, -0.5);
  else if (PyFloat_CheckExact(scale_)) *scale = (float)PyFloat_AS_DOUBLE(scale_);
  else return false;
  return true;
}
// QKV, B, S, heads, scale, mask, out, stream
PyObject* attention_packed(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 8) return not_taken();
    const at::Tensor* Q = plain(a[0]);
    int M, B, S, heads, d;
    float scale;
    void *mask, *s;
    if (!Q || !packed_qkv(*Q, a[1], a[2], a[3], a[4], &M, &B, &S, &heads, &d, &scale) || !operand(a[5], at::kFloat, &mask) || !stream_of(a[7], &s))
      return not_taken();
    const long Hd = (long)heads * d, N = (long)B * S;
    const char* base = (const char*)Q->data_ptr();
    const long step = Hd * (long)Q->element_size();
    const nf_dtype dt = type_of(*Q);
    return produce("netfuse_attention", a[6], {M, N, Hd}, Q->options(), [=](void* y) {
      return f_attention(base, base + step, base + 2 * step, (const float*)mask, y, M, B, S, heads, d, N * 3 * Hd, 3 * Hd, scale, dt, s);
    });
  });
}
// QKV, Kr, B, S, heads, bias_w, bias_r, scale, mask, out, stream
PyObject* attention_relpos_packed(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 11) return not_taken();
    const at::Tensor *Q = plain(a[0]), *Kr = plain(a[1]);
    int M, B, S, heads, d;
    float scale;
    void *bw, *br, *mask, *s;
    if (!Q || !Kr || Kr->scalar_type() != Q->scalar_type() || !packed_qkv(*Q, a[2], a[3], a[4], a[7], &M, &B, &S, &heads, &d, &scale) ||
        !operand(a[5], at::kFloat, &bw) || !operand(a[6], at::kFloat, &br) || !operand(a[8], at::kFloat, &mask) || !stream_of(a[10], &s))
      return not_taken();
    const long Hd = (long)heads * d, N = (long)B * S;
    if (Kr->dim() != 3 || Kr->size(0) != M || Kr->size(1) != 2LL * S || Kr->size(2) != Hd) return not_taken();
    const char* base = (const char*)Q->data_ptr();
    const void* kr = Kr->data_ptr();
    const long step = Hd * (long)Q->element_size();
    const nf_dtype dt = type_of(*Q);
    return produce("netfuse_attention_relpos", a[9], {M, N, Hd}, Q->options(), [=](void* y) {
      return f_relpos(base, base + step, base + 2 * step, kr, (const float*)bw, (const float*)br, (const float*)mask, y, M, B, S, heads, d,
                      N * 3 * Hd, 3 * Hd, scale, dt, s);
    });
  });
}

// x, w, M, g, bias, scale, shift, residual, stride, pad, dil, act, out, stream
PyObject* conv2d(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 14) return not_taken();
    const at::Tensor *x = plain(a[0]), *w = plain(a[1]);
    int M, g, stride, pad, dil, act, B, Ct, H, W, Co, cig, KH, KW;
    void *bias, *scale, *shift, *r, *s;
    if (!x || !w || x->dim() != 4 || w->dim() != 4 || w->scalar_type() != x->scalar_type() || !whole(a[2], &M) || M <= 0 || !whole(a[3], &g) || g <= 0 ||
        !operand(a[4], at::kFloat, &bias) || !operand(a[5], at::kFloat, &scale) || !operand(a[6], at::kFloat, &shift) ||
        !operand(a[7], x->scalar_type(), &r) || !whole(a[8], &stride) || stride <= 0 || !whole(a[9], &pad) || pad < 0 || !whole(a[10], &dil) || dil <= 0 ||
        !whole(a[11], &act) || !stream_of(a[13], &s))
      return not_taken();
    if (!size(x->size(0), &B) || !size(x->size(1), &Ct) || !size(x->size(2), &H) || !size(x->size(3), &W) || !size(w->size(0), &Co) ||
        !size(w->size(1), &cig) || !size(w->size(2), &KH) || !size(w->size(3), &KW) || Ct % M || Co % M || (int64_t)cig * g != Ct / M)
      return not_taken();
    const int64_t eh = (int64_t)H + 2LL * pad - (int64_t)dil * (KH - 1) - 1, ew = (int64_t)W + 2LL * pad - (int64_t)dil * (KW - 1) - 1;
    if (eh < 0 || ew < 0) return not_taken();
    const void *in = x->data_ptr(), *wt = w->data_ptr();
    const nf_dtype dt = type_of(*x);
    return produce("netfuse_conv2d", a[12], {B, Co, eh / stride + 1, ew / stride + 1}, x->options(), [=](void* y) {
      return f_conv2d(in, wt, (const float*)bias, (const float*)scale, (const float*)shift, r, y, M, B, Ct / M, Co / M, g, H, W, KH, KW, stride, pad,
                      dil, dt, (nf_act)act, s);
    });
  });
}

// bind(error, linear, linear_packed, layernorm, attention, attention_relpos, conv2d): the addresses of the entry points
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 7) {
    PyErr_SetString(PyExc_TypeError, "bind takes a callable and six addresses");
    return nullptr;
  }
  void* p[7];
  for (int i = 1; i < 7; ++i) {
    p[i] = PyLong_AsVoidPtr(a[i]);
    if (PyErr_Occurred()) return nullptr;
  }
  Py_INCREF(a[0]);
  Py_XSETREF(g_error, a[0]);
  f_linear = (decltype(f_linear))p[1];
  f_packed = (decltype(f_packed))p[2];
  f_layernorm = (decltype(f_layernorm))p[3];
  f_attention = (decltype(f_attention))p[4];
  f_relpos = (decltype(f_relpos))p[5];
  f_conv2d = (decltype(f_conv2d))p[6];
  Py_RETURN_NONE;
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(bind), FAST(linear), FAST(linear_packed), FAST(layernorm), FAST(attention_packed), FAST(attention_relpos_packed),
                         FAST(conv2d), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: the Python and torch whose headers are compiled in; the package uses the module with no other.
PyMODINIT_FUNC PyInit__binding() {
  PyObject* m = PyModule_Create(&module);
  if (m && PyModule_AddStringConstant(m, "built_for", NETFUSE_BUILT_FOR) < 0) Py_CLEAR(m);
  return m;
}
