// Native marshalling of the Python binding's hot entry points: argument checks,
// output allocation, current stream and the call into the C ABI of
// include/resonator.h, in one C call each (about 4 us of host time a call where
// the same steps in Python take 15 to 40; a block training step of float32
// [1, 777, 128] was bound by them: 247 us of host time for 22 launches).
//
// Each function takes every argument of the Python function of the same name, in
// order, and serves the plain case only: exact torch.Tensor (or Parameter)
// arguments on the GPU, contiguous, of the documented types and shapes.  For
// anything else it returns None without having done anything, and the Python
// function goes on with its own checks and messages.  A non-zero error code of
// the library comes back as an int.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/Functions.h>
#include <c10/core/DeviceGuard.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/resonator.h"

namespace {

using at::Tensor;

const c10::DispatchKeySet kWrapped({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched,
                                    c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize,
                                    c10::DispatchKey::Negative, c10::DispatchKey::Conjugate,
                                    c10::DispatchKey::ZeroTensor, c10::DispatchKey::BatchedNestedTensor});

// A plain contiguous GPU tensor (borrowed from the caller's reference).
const Tensor* plain(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage() ||
      t.key_set().has_any(kWrapped) || !t.is_contiguous())
    return nullptr;
  return &t;
}
int code(const Tensor& t) {  // activation type code, -1 for other types
  return t.scalar_type() == at::kFloat ? RES_F32 : t.scalar_type() == at::kBFloat16 ? RES_BF16 : -1;
}
bool f32(const Tensor& t) { return t.scalar_type() == at::kFloat; }
bool shape(const Tensor& t, std::initializer_list<int64_t> s) { return t.sizes() == at::IntArrayRef(s); }
const float* fp(const Tensor& t) { return static_cast<const float*>(t.data_ptr()); }
float* fpm(const Tensor& t) { return static_cast<float*>(t.data_ptr()); }
// The launch context of a call on t's GPU: that device current until the end of the
// scope (a device's default stream is the null stream, which means the current
// device) and its current stream.
struct OnDevice {
  c10::OptionalDeviceGuard guard;
  void* stream;
  explicit OnDevice(const Tensor& t) : stream(c10::hip::getCurrentHIPStream(t.device().index()).stream()) {
    // (the count is kept by c10: a process with one GPU asks nothing, 0.15 us a call)
    if (c10::hip::device_count() > 1 && t.device().index() != c10::hip::current_device())
      guard.reset_device(t.device());
  }
};
Tensor empty(at::IntArrayRef s, const Tensor& like, at::ScalarType dt) {
  return at::empty(s, at::TensorOptions().device(like.device()).dtype(dt));
}
PyObject* none() { Py_RETURN_NONE; }
bool truth(PyObject* o, bool* v) {
  if (o != Py_True && o != Py_False) return false;
  *v = o == Py_True;
  return true;
}
bool integer(PyObject* o, int64_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  int over = 0;
  *v = PyLong_AsLongLongAndOverflow(o, &over);
  return over == 0;
}
bool number(PyObject* o, float* v) {
  if (!PyFloat_CheckExact(o)) return false;
  *v = static_cast<float>(PyFloat_AS_DOUBLE(o));
  return true;
}

struct Params {
  const float *gamma, *omega, *amp, *phase;
  int64_t D, M;
};
// the four parameter tensors, float32 [D, M]
bool params(PyObject* const* o, Params* p) {
  const Tensor* t[4];
  for (int i = 0; i < 4; ++i) {
    t[i] = plain(o[i]);
    if (!t[i] || !f32(*t[i]) || t[i]->dim() != 2 || t[i]->sizes() != t[0]->sizes()) return false;
  }
  *p = Params{fp(*t[0]), fp(*t[1]), fp(*t[2]), fp(*t[3]), t[0]->size(0), t[0]->size(1)};
  return true;
}

// Calls the library without the interpreter lock (as a ctypes call does).
template <typename F>
int call(F&& f) {
  int rc;
  Py_BEGIN_ALLOW_THREADS rc = f();
  Py_END_ALLOW_THREADS return rc;
}

PyObject* pack(std::initializer_list<Tensor> ts) {
  PyObject* r = PyTuple_New(static_cast<Py_ssize_t>(ts.size()));
  if (!r) throw python_error();
  Py_ssize_t i = 0;
  for (const Tensor& t : ts) {
    PyObject* w = t.defined() ? THPVariable_Wrap(t) : Py_NewRef(Py_None);
    if (!w) {
      Py_DECREF(r);
      throw python_error();
    }
    PyTuple_SET_ITEM(r, i++, w);
  }
  return r;
}

// (x, gamma, omega, amp, phase, h0, out_dtype, return_state, out, ws, h_out)
PyObject* mix_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 11) return none();
  const Tensor* x = plain(a[0]);
  Params p;
  bool want_state;
  if (!x || x->dim() != 3 || code(*x) < 0 || !params(a + 1, &p) || p.D != x->size(2) || !truth(a[7], &want_state))
    return none();
  const int64_t B = x->size(0), L = x->size(1), D = p.D, M = p.M;
  const size_t nb = resonator_workspace_bytes(RES_OP_FWD, (res_dtype_t)code(*x), B, L, D, M);
  if (nb == 0) return none();
  const Tensor* h0 = nullptr;
  if (a[5] != Py_None) {
    h0 = plain(a[5]);
    if (!h0 || !f32(*h0) || !shape(*h0, {B, D, M, 2})) return none();
  }
  Tensor y, ws, ho;
  if (a[8] != Py_None) {
    const Tensor* o = plain(a[8]);
    if (!o || code(*o) < 0 || o->numel() < x->numel()) return none();
    y = *o;
  }
  at::ScalarType odt = x->scalar_type();
  if (a[6] != Py_None) {
    if (!THPDtype_Check(a[6])) return none();
    odt = reinterpret_cast<THPDtype*>(a[6])->scalar_type;
    if (odt != at::kFloat && odt != at::kBFloat16) return none();
  }
  if (a[9] != Py_None) {
    const Tensor* w = plain(a[9]);
    if (!w || w->numel() * (int64_t)w->element_size() < (int64_t)nb) return none();
    ws = *w;
  }
  if (a[10] != Py_None) {
    const Tensor* o = plain(a[10]);
    if (!o || !f32(*o) || !shape(*o, {B, D, M, 2})) return none();
    ho = *o;
  }
  if (!y.defined()) y = empty(x->sizes(), *x, odt);
  if (!ho.defined() && want_state) ho = empty({B, D, M, 2}, *x, at::kFloat);
  const bool own = !ws.defined();  // a workspace of this call alone
  if (own) ws = empty({(int64_t)std::max<size_t>(nb, 256)}, *x, at::kByte);
  const OnDevice on(*x);
  const int rc = call([&] {
    if (own) {
      const int e = resonator_fwd_workspace_init((res_dtype_t)code(*x), B, L, D, M, ws.data_ptr(), nb, on.stream);
      if (e) return e;
    }
    return resonator_mix_fwd(x->data_ptr(), (res_dtype_t)code(*x), y.data_ptr(), (res_dtype_t)code(y), B, L, D, M,
                             p.gamma, p.omega, p.amp, p.phase, h0 ? fp(*h0) : nullptr,
                             ho.defined() ? fpm(ho) : nullptr, ws.data_ptr(), nb, on.stream);
  });
  if (rc) return PyLong_FromLong(rc);
  return want_state ? pack({y, ho}) : THPVariable_Wrap(y);
  END_HANDLE_TH_ERRORS
}

// (x, dy, gamma, omega, amp, phase, h0, want_dh0, ws) -> (dx, dgamma, domega, damp, dphase, dh0 or None)
PyObject* mix_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 9) return none();
  const Tensor *x = plain(a[0]), *dy = plain(a[1]);
  Params p;
  bool want;
  if (!x || !dy || x->dim() != 3 || code(*x) < 0 || x->sizes() != dy->sizes() ||
      x->scalar_type() != dy->scalar_type() || !params(a + 2, &p) || p.D != x->size(2) || !truth(a[7], &want))
    return none();
  const int64_t B = x->size(0), L = x->size(1), D = p.D, M = p.M;
  const size_t nb = resonator_workspace_bytes(RES_OP_BWD, (res_dtype_t)code(*x), B, L, D, M);
  if (nb == 0) return none();
  const Tensor* h0 = nullptr;
  if (a[6] != Py_None) {
    h0 = plain(a[6]);
    if (!h0 || !f32(*h0) || !shape(*h0, {B, D, M, 2})) return none();
  }
  Tensor ws;
  if (a[8] != Py_None) {
    const Tensor* w = plain(a[8]);
    if (!w || w->numel() * (int64_t)w->element_size() < (int64_t)nb) return none();
    ws = *w;
  }
  const Tensor dx = empty(x->sizes(), *x, x->scalar_type());
  Tensor g[4], dh0;
  for (Tensor& t : g) t = empty({D, M}, *x, at::kFloat);
  if (want) dh0 = empty({B, D, M, 2}, *x, at::kFloat);
  if (!ws.defined()) ws = empty({(int64_t)std::max<size_t>(nb, 256)}, *x, at::kByte);
  const OnDevice on(*x);
  const int rc = call([&] {
    return resonator_mix_bwd(x->data_ptr(), dy->data_ptr(), (res_dtype_t)code(*x), dx.data_ptr(), B, L, D, M, p.gamma,
                             p.omega, p.amp, p.phase, h0 ? fp(*h0) : nullptr, fpm(g[0]), fpm(g[1]), fpm(g[2]),
                             fpm(g[3]), want ? fpm(dh0) : nullptr, ws.data_ptr(), nb, on.stream);
  });
  if (rc) return PyLong_FromLong(rc);
  return pack({dx, g[0], g[1], g[2], g[3], dh0});
  END_HANDLE_TH_ERRORS
}

// (x_prompt, gamma, omega, amp, phase)
PyObject* state_init(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 5) return none();
  const Tensor* x = plain(a[0]);
  Params p;
  if (!x || x->dim() != 3 || code(*x) < 0 || !params(a + 1, &p) || p.D != x->size(2)) return none();
  const int64_t B = x->size(0), L = x->size(1), D = p.D, M = p.M;
  const size_t nb = L > 0 ? resonator_workspace_bytes(RES_OP_STATE_INIT, (res_dtype_t)code(*x), B, L, D, M) : 0;
  if (nb == 0) return none();
  const Tensor h = empty({B, D, M, 2}, *x, at::kFloat);
  const Tensor ws = empty({(int64_t)std::max<size_t>(nb, 256)}, *x, at::kByte);
  const OnDevice on(*x);
  const int rc = call([&] {
    return resonator_state_init(x->data_ptr(), (res_dtype_t)code(*x), B, L, D, M, p.gamma, p.omega, p.amp, p.phase,
                                fpm(h), ws.data_ptr(), nb, on.stream);
  });
  return rc ? PyLong_FromLong(rc) : THPVariable_Wrap(h);
  END_HANDLE_TH_ERRORS
}

// (x, gamma, omega, amp, phase, state): x [B, N, D] (steps) or [B, D] (one step)
template <bool STEPS>
PyObject* decode(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 6) return none();
  const Tensor *x = plain(a[0]), *s = plain(a[5]);
  Params p;
  if (!x || !s || x->dim() != (STEPS ? 3 : 2) || code(*x) < 0 || !params(a + 1, &p) || p.D != x->size(-1))
    return none();
  const int64_t B = x->size(0), N = STEPS ? x->size(1) : 1;
  if (!f32(*s) || !shape(*s, {B, p.D, p.M, 2})) return none();
  const Tensor y = empty(x->sizes(), *x, x->scalar_type());
  const auto dt = (res_dtype_t)code(*x);
  const OnDevice on(*x);
  const int rc = call([&] {
    return STEPS ? resonator_decode_steps(x->data_ptr(), dt, y.data_ptr(), dt, B, N, p.D, p.M, p.gamma, p.omega, p.amp,
                                          p.phase, fpm(*s), on.stream)
                 : resonator_decode_step(x->data_ptr(), dt, y.data_ptr(), dt, B, p.D, p.M, p.gamma, p.omega, p.amp,
                                         p.phase, fpm(*s), on.stream);
  });
  return rc ? PyLong_FromLong(rc) : THPVariable_Wrap(y);
  END_HANDLE_TH_ERRORS
}

// (x, gamma, omega, amp, phase, state, y): N steps of time-major drives x [N, B, D] into y; True when done
PyObject* decode_steps_tm(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 7) return none();
  const Tensor *x = plain(a[0]), *s = plain(a[5]), *y = plain(a[6]);
  Params p;
  if (!x || !s || !y || x->dim() != 3 || code(*x) < 0 || code(*y) < 0 || y->sizes() != x->sizes() ||
      !params(a + 1, &p) || p.D != x->size(2) || !f32(*s) || !shape(*s, {x->size(1), p.D, p.M, 2}))
    return none();
  const OnDevice on(*x);
  const int rc = call([&] {
    return resonator_decode_steps_tm(x->data_ptr(), (res_dtype_t)code(*x), y->data_ptr(), (res_dtype_t)code(*y),
                                     x->size(1), x->size(0), p.D, p.M, p.gamma, p.omega, p.amp, p.phase, fpm(*s),
                                     on.stream);
  });
  if (rc) return PyLong_FromLong(rc);
  Py_RETURN_TRUE;
  END_HANDLE_TH_ERRORS
}

// A grouped weight [G, d_in/G, d_out/G] of type dt.
const Tensor* weight(PyObject* o, at::ScalarType dt) {
  const Tensor* w = plain(o);
  return w && w->dim() == 3 && w->scalar_type() == dt ? w : nullptr;
}

// (x, W)
PyObject* grouped_linear(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 2) return none();
  const Tensor* x = plain(a[0]);
  if (!x || x->dim() < 1 || code(*x) < 0) return none();
  const Tensor* W = weight(a[1], x->scalar_type());
  const int64_t d_in = x->size(-1);
  if (!W || d_in < 1 || W->size(0) * W->size(1) != d_in) return none();
  const int64_t G = W->size(0), d_out = G * W->size(2), N = x->numel() / d_in;
  auto s = x->sizes().vec();
  s.back() = d_out;
  const Tensor y = empty(s, *x, x->scalar_type());
  const OnDevice on(*x);
  const int rc = call([&] {
    return resonator_grouped_linear(x->data_ptr(), W->data_ptr(), (res_dtype_t)code(*x), y.data_ptr(), N, d_in, d_out,
                                    G, on.stream);
  });
  return rc ? PyLong_FromLong(rc) : THPVariable_Wrap(y);
  END_HANDLE_TH_ERRORS
}

// (x, W0, W1)
PyObject* grouped_linear2(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 3) return none();
  const Tensor* x = plain(a[0]);
  if (!x || x->dim() < 1 || code(*x) < 0) return none();
  const Tensor *W0 = weight(a[1], x->scalar_type()), *W1 = weight(a[2], x->scalar_type());
  const int64_t d_in = x->size(-1);
  if (!W0 || !W1 || d_in < 1 || W0->sizes() != W1->sizes() || W0->size(0) * W0->size(1) != d_in) return none();
  const int64_t G = W0->size(0), d_out = G * W0->size(2), N = x->numel() / d_in;
  auto s = x->sizes().vec();
  s.back() = d_out;
  const Tensor y0 = empty(s, *x, x->scalar_type()), y1 = empty(s, *x, x->scalar_type());
  const OnDevice on(*x);
  const int rc = call([&] {
    return resonator_grouped_linear2(x->data_ptr(), W0->data_ptr(), W1->data_ptr(), (res_dtype_t)code(*x),
                                     y0.data_ptr(), y1.data_ptr(), N, d_in, d_out, G, on.stream);
  });
  return rc ? PyLong_FromLong(rc) : pack({y0, y1});
  END_HANDLE_TH_ERRORS
}

// A list or tuple of 1 to most plain tensors; 0 if it is not one.
int tensors(PyObject* o, const Tensor** t, int most) {
  if (!PyList_CheckExact(o) && !PyTuple_CheckExact(o)) return 0;
  const Py_ssize_t n = PySequence_Fast_GET_SIZE(o);
  if (n < 1 || n > most) return 0;
  for (Py_ssize_t i = 0; i < n; ++i)
    if (!(t[i] = plain(PySequence_Fast_GET_ITEM(o, i)))) return 0;
  return (int)n;
}

// (dys, Ws): a new dx
PyObject* bwd_data_sum(PyObject*, PyObject* const* a, Py_ssize_t na) {
  HANDLE_TH_ERRORS
  if (na != 2) return none();
  const Tensor *d[3], *w[3];
  const int n = tensors(a[0], d, 3);
  if (n == 0 || tensors(a[1], w, 3) != n || d[0]->dim() < 1 || code(*d[0]) < 0 || w[0]->dim() != 3) return none();
  const int64_t G = w[0]->size(0), di = w[0]->size(1), d_out = d[0]->size(-1);
  if (d_out < 1 || G * w[0]->size(2) != d_out) return none();
  const void *dp[3], *wp[3];
  for (int i = 0; i < n; ++i) {
    if (d[i]->scalar_type() != d[0]->scalar_type() || d[i]->sizes() != d[0]->sizes() ||
        w[i]->scalar_type() != d[0]->scalar_type() || w[i]->sizes() != w[0]->sizes())
      return none();
    dp[i] = d[i]->data_ptr();
    wp[i] = w[i]->data_ptr();
  }
  auto s = d[0]->sizes().vec();
  s.back() = G * di;
  const Tensor dx = empty(s, *d[0], d[0]->scalar_type());
  const OnDevice on(*d[0]);
  const int rc = call([&] {
    return resonator_grouped_linear_bwd_data_sum(n, dp, wp, (res_dtype_t)code(*d[0]), dx.data_ptr(),
                                                 d[0]->numel() / d_out, G * di, d_out, G, 0, on.stream);
  });
  return rc ? PyLong_FromLong(rc) : THPVariable_Wrap(dx);
  END_HANDLE_TH_ERRORS
}

// (x, dys, outs, dWs): into the given dWs; True when done
PyObject* bwd_weight_sum(PyObject*, PyObject* const* a, Py_ssize_t na) {
  HANDLE_TH_ERRORS
  if (na != 4) return none();
  const Tensor *x = plain(a[0]), *d[3], *w[2];
  if (!x || x->dim() < 1 || code(*x) < 0) return none();
  const int n = tensors(a[1], d, 3), m = tensors(a[3], w, 2);
  if (n == 0 || m == 0 || (!PyList_CheckExact(a[2]) && !PyTuple_CheckExact(a[2])) ||
      PySequence_Fast_GET_SIZE(a[2]) != n)
    return none();
  int outs[3];
  bool used[2] = {false, false};
  for (int i = 0; i < n; ++i) {
    int64_t v;
    if (!integer(PySequence_Fast_GET_ITEM(a[2], i), &v) || v < 0 || v >= m) return none();
    outs[i] = (int)v;
    used[v] = true;
  }
  if (!used[0] || (m == 2 && !used[1])) return none();
  const int64_t d_in = x->size(-1), d_out = d[0]->dim() < 1 ? 0 : d[0]->size(-1);
  if (d_in < 1 || d_out < 1 || w[0]->dim() != 3) return none();
  const int64_t N = x->numel() / d_in, G = w[0]->size(0);
  const void* dp[3];
  for (int i = 0; i < n; ++i) {
    if (d[i]->scalar_type() != x->scalar_type() || d[i]->dim() < 1 || d[i]->size(-1) != d_out ||
        d[i]->numel() != N * d_out)
      return none();
    dp[i] = d[i]->data_ptr();
  }
  if (G < 1 || d_in % G || d_out % G) return none();
  for (int i = 0; i < m; ++i)
    if (!f32(*w[i]) || !shape(*w[i], {G, d_in / G, d_out / G})) return none();
  const auto dt = (res_dtype_t)code(*x);
  const size_t nb = resonator_grouped_linear_bwd_weight_sum_workspace_bytes(n, m, N, d_in, d_out, G, dt);
  const Tensor ws = empty({(int64_t)std::max<size_t>(nb, 256)}, *x, at::kByte);
  const OnDevice on(*x);
  const int rc = call([&] {
    return resonator_grouped_linear_bwd_weight_sum(n, x->data_ptr(), dp, outs, dt, fpm(*w[0]),
                                                   m == 2 ? fpm(*w[1]) : nullptr, N, d_in, d_out, G, 0, ws.data_ptr(),
                                                   (size_t)ws.numel(), on.stream);
  });
  if (rc) return PyLong_FromLong(rc);
  Py_RETURN_TRUE;
  END_HANDLE_TH_ERRORS
}

// (x, dy, dW, accumulate): the grouped weight gradient into dW; True when done
PyObject* bwd_weight(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 4) return none();
  const Tensor *x = plain(a[0]), *dy = plain(a[1]), *w = plain(a[2]);
  bool acc;
  if (!x || !dy || !w || x->dim() < 1 || dy->dim() < 1 || code(*x) < 0 || x->scalar_type() != dy->scalar_type() ||
      !f32(*w) || w->dim() != 3 || !truth(a[3], &acc))
    return none();
  const int64_t d_in = x->size(-1), d_out = dy->size(-1), G = w->size(0);
  if (d_in < 1 || d_out < 1 || G < 1 || d_in % G || d_out % G || !shape(*w, {G, d_in / G, d_out / G})) return none();
  const int64_t N = dy->numel() / d_out;
  if (x->numel() != N * d_in) return none();
  const OnDevice on(*x);
  const int rc = call([&] {
    return resonator_grouped_linear_bwd_weight(x->data_ptr(), dy->data_ptr(), (res_dtype_t)code(*x), fpm(*w), N, d_in,
                                               d_out, G, acc, on.stream);
  });
  if (rc) return PyLong_FromLong(rc);
  Py_RETURN_TRUE;
  END_HANDLE_TH_ERRORS
}

// The epilogue's arguments after the activations: (Ct, lambda_c, w, s, H) at a.
struct EpiArgs {
  int64_t B, L, D, H, K;
  float lc;
  const float *Ct, *w, *s;
};
bool epi_args(const Tensor& y, PyObject* const* a, EpiArgs* e) {
  const Tensor* Ct = plain(a[0]);
  if (!Ct || y.dim() != 3 || code(y) < 0 || !number(a[1], &e->lc) || !integer(a[4], &e->H)) return false;
  e->B = y.size(0);
  e->L = y.size(1);
  e->D = y.size(2);
  if (e->H < 1 || e->D % e->H || !f32(*Ct) || !shape(*Ct, {e->H, e->H})) return false;
  e->Ct = fp(*Ct);
  e->K = 0;
  e->w = e->s = nullptr;
  if (a[2] != Py_None) {
    const Tensor* w = plain(a[2]);
    if (!w || !f32(*w) || w->dim() != 2 || w->size(0) != e->D) return false;
    e->K = w->size(1);
    if (e->K > 0) {
      const Tensor* s = plain(a[3]);
      if (!s || !f32(*s) || !shape(*s, {e->D})) return false;
      e->w = fp(*w);
      e->s = fp(*s);
    }
  }
  return true;
}
const Tensor* like(PyObject* o, const Tensor& y) {
  const Tensor* t = plain(o);
  return t && t->sizes() == y.sizes() && t->scalar_type() == y.scalar_type() ? t : nullptr;
}

// (y, gate, v, Ct, lambda_c, w, s, H)
PyObject* epilogue_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 8) return none();
  const Tensor* y = plain(a[0]);
  EpiArgs e;
  if (!y || !epi_args(*y, a + 3, &e)) return none();
  const Tensor *g = like(a[1], *y), *v = e.K ? like(a[2], *y) : nullptr;
  if (!g || (e.K && !v)) return none();
  const Tensor z = empty(y->sizes(), *y, y->scalar_type());
  const OnDevice on(*y);
  const int rc = call([&] {
    return resonator_epilogue_fwd(y->data_ptr(), g->data_ptr(), v ? v->data_ptr() : nullptr, (res_dtype_t)code(*y),
                                  z.data_ptr(), e.B, e.L, e.H, e.D / e.H, e.K, e.Ct, e.lc, e.w, e.s, on.stream);
  });
  return rc ? PyLong_FromLong(rc) : THPVariable_Wrap(z);
  END_HANDLE_TH_ERRORS
}

// (y, gate, v, Ct, lambda_c, w, s, H, Wo, z)
PyObject* epilogue_proj_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 10) return none();
  const Tensor* y = plain(a[0]);
  EpiArgs e;
  if (!y || !epi_args(*y, a + 3, &e)) return none();
  const Tensor *g = like(a[1], *y), *v = e.K ? like(a[2], *y) : nullptr, *W = weight(a[8], y->scalar_type());
  if (!g || (e.K && !v) || !W || W->size(0) != e.H || W->size(1) != e.D / e.H) return none();
  const Tensor* z = nullptr;
  if (a[9] != Py_None && !(z = like(a[9], *y))) return none();
  const int64_t d_out = e.H * W->size(2);
  const Tensor o = empty({e.B, e.L, d_out}, *y, y->scalar_type());
  const OnDevice on(*y);
  const int rc = call([&] {
    return resonator_epilogue_proj_fwd(y->data_ptr(), g->data_ptr(), v ? v->data_ptr() : nullptr, (res_dtype_t)code(*y),
                                       W->data_ptr(), o.data_ptr(), z ? z->data_ptr() : nullptr, e.B, e.L, e.H,
                                       e.D / e.H, e.K, d_out, e.Ct, e.lc, e.w, e.s, on.stream);
  });
  return rc ? PyLong_FromLong(rc) : THPVariable_Wrap(o);
  END_HANDLE_TH_ERRORS
}

// (y, gate, v, dz, Ct, lambda_c, w, s, H) -> (dy, dgate, dv, dCt, dlambda_c, dw, ds)
PyObject* epilogue_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 9) return none();
  const Tensor* y = plain(a[0]);
  EpiArgs e;
  if (!y || !epi_args(*y, a + 4, &e)) return none();
  const Tensor *g = like(a[1], *y), *v = e.K ? like(a[2], *y) : nullptr, *dz = like(a[3], *y);
  if (!g || !dz || (e.K && !v)) return none();
  const Tensor dy = empty(y->sizes(), *y, y->scalar_type()), dg = empty(y->sizes(), *y, y->scalar_type());
  const Tensor dCt = empty({e.H, e.H}, *y, at::kFloat), dl = empty({1}, *y, at::kFloat);
  Tensor dv, dw, ds;
  if (e.K) {
    dv = empty(y->sizes(), *y, y->scalar_type());
    dw = empty({e.D, e.K}, *y, at::kFloat);
    ds = empty({e.D}, *y, at::kFloat);
  }
  const size_t nb = resonator_epilogue_workspace_bytes(e.B, e.L, e.H, e.D / e.H, e.K);
  const Tensor ws = empty({(int64_t)nb}, *y, at::kByte);
  const OnDevice on(*y);
  const int rc = call([&] {
    return resonator_epilogue_bwd(y->data_ptr(), g->data_ptr(), v ? v->data_ptr() : nullptr, dz->data_ptr(),
                                  (res_dtype_t)code(*y), dy.data_ptr(), dg.data_ptr(),
                                  e.K ? dv.data_ptr() : nullptr, e.B, e.L, e.H, e.D / e.H, e.K, e.Ct, e.lc, e.w, e.s,
                                  fpm(dCt), fpm(dl), e.K ? fpm(dw) : nullptr, e.K ? fpm(ds) : nullptr, ws.data_ptr(),
                                  nb, on.stream);
  });
  return rc ? PyLong_FromLong(rc) : pack({dy, dg, dv, dCt, dl, dw, ds});
  END_HANDLE_TH_ERRORS
}

#define RES_FN(name, f) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {RES_FN("mix_fwd", mix_fwd),
                         RES_FN("mix_bwd", mix_bwd),
                         RES_FN("state_init", state_init),
                         RES_FN("decode_steps", decode<true>),
                         RES_FN("decode_step", decode<false>),
                         RES_FN("decode_steps_tm", decode_steps_tm),
                         RES_FN("grouped_linear", grouped_linear),
                         RES_FN("grouped_linear2", grouped_linear2),
                         RES_FN("bwd_data_sum", bwd_data_sum),
                         RES_FN("bwd_weight_sum", bwd_weight_sum),
                         RES_FN("bwd_weight", bwd_weight),
                         RES_FN("epilogue_fwd", epilogue_fwd),
                         RES_FN("epilogue_proj_fwd", epilogue_proj_fwd),
                         RES_FN("epilogue_bwd", epilogue_bwd),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_host", "Native marshalling of the hot entry points.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host() { return PyModule_Create(&module); }
