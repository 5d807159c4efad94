// Native call path of the torch binding: the ordinary calls (plain contiguous
// GPU tensors) from argument checks to launch without
// going through Python and ctypes. Every function takes exactly the arguments
// of its Python namesake and answers None for whatever it does not handle
// itself (other tensor types, subclasses, wrapped tensors, a bad shape, a failing
// call): the Python function then takes the call from the
// start, with its own checks and errors. Host code only.
//
// What it is for: a call through the Python checks and ctypes costs 8 - 20 us of
// host time, several times the GPU time of a small problem (4096 quadruples:
// 3.3 us).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/Functions.h>
#include <ATen/TensorSubclassLikeUtils.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>
#include <exception>
#include <limits>
#include <optional>

#include "homog.h"

namespace {

using at::ScalarType;
using at::Tensor;

// The tensor behind a Python object if it is an ordinary GPU tensor of type st.
const Tensor *plain(PyObject *o, ScalarType st) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const Tensor &t = THPVariable_Unpack(o);
  if (!t.is_cuda() || t.scalar_type() != st || at::isTensorSubclassLike(t)) return nullptr;
  return &t;
}

const Tensor *packed(PyObject *o, ScalarType st) {
  const Tensor *t = plain(o, st);
  return t && t->is_contiguous() ? t : nullptr;
}

// (k, n) float planes with contiguous rows; their plane stride in ld.
const Tensor *planes(PyObject *o, int64_t k, int64_t &ld) {
  const Tensor *t = plain(o, ScalarType::Float);
  if (!t || t->dim() != 2 || t->size(0) != k || (t->size(1) > 1 && t->stride(1) != 1))
    return nullptr;
  ld = k > 1 ? t->stride(0) : t->size(1);
  return t;
}

// The stream of a call: the current one (None), or that of an object with a
// cuda_stream handle. While it lives, tensors are allocated from that stream's pool
// (_pool in __init__.py has the reason).
class CallStream {
 public:
  void *raw = nullptr;

  bool take(PyObject *o, const Tensor &like) {
    if (o == Py_None) {
      raw = c10::hip::getCurrentHIPStream().stream();
      return true;
    }
    PyObject *handle = PyObject_GetAttrString(o, "cuda_stream");
    const bool ok = handle && PyLong_CheckExact(handle);
    raw = ok ? PyLong_AsVoidPtr(handle) : nullptr;
    Py_XDECREF(handle);
    if (!ok || PyErr_Occurred()) {
      PyErr_Clear();
      return false;
    }
    const c10::DeviceIndex device = like.device().index();
    const c10::hip::HIPStream here = c10::hip::getCurrentHIPStream(device);
    if (raw != here.stream()) {
      c10::hip::setCurrentHIPStream(
          raw ? c10::hip::getStreamFromExternal(static_cast<hipStream_t>(raw), device)
              : c10::hip::getDefaultHIPStream(device));
      here_ = here;
    }
    return true;
  }

  // A new output, which the caller will use on the current stream.
  Tensor lend(Tensor t) const {
    if (here_) c10::hip::HIPCachingAllocator::recordStream(t.storage().data_ptr(), *here_);
    return t;
  }

  CallStream() = default;
  CallStream(const CallStream &) = delete;
  ~CallStream() {
    if (here_) c10::hip::setCurrentHIPStream(*here_);
  }

 private:
  std::optional<c10::hip::HIPStream> here_;   // the current stream, where it is another
};

Tensor empty(at::IntArrayRef size, ScalarType st, const Tensor &like) {
  return at::empty(size, at::TensorOptions().dtype(st).device(like.device()));
}

template <class T>
T *ptr(const Tensor &t) {
  return static_cast<T *>(t.data_ptr());
}

// An output: the caller's tensor, or a new one.
struct Out {
  PyObject *given = nullptr;
  Tensor t;
  PyObject *take() const {
    if (given) return Py_NewRef(given);
    return THPVariable_Wrap(t);
  }
};

PyObject *tuple(std::initializer_list<PyObject *> v) {
  PyObject *r = PyTuple_New(static_cast<Py_ssize_t>(v.size()));
  Py_ssize_t i = 0;
  for (PyObject *o : v) {
    if (!o || !r) {
      Py_XDECREF(r);
      return nullptr;
    }
    PyTuple_SET_ITEM(r, i++, o);
  }
  return r;
}

// Runs a library call without the GIL; true if it succeeded. The GIL is taken again
// on every way out: reading a tensor's pointer may throw (one without storage).
struct NoGil {
  PyThreadState *state = PyEval_SaveThread();
  ~NoGil() { PyEval_RestoreThread(state); }
};

template <class F>
bool launch(F &&f) {
  const NoGil released;
  return f() == HG_OK;
}

#define DECLINE Py_RETURN_NONE
#define NEED(cond) \
  if (!(cond)) DECLINE

// H (9 or 6 planes at stride ld) and flags of the solvers.
bool solver_out(PyObject *Ho, PyObject *fo, int64_t rows, int64_t ld, int64_t n, const Tensor &like,
                const CallStream &st, Out &H, Out &flags) {
  if (Ho == Py_None) {
    H.t = st.lend(empty({rows, ld}, ScalarType::Float, like));
    if (ld != n) H.t = H.t.slice(1, 0, n);
  } else {
    int64_t l;
    const Tensor *t = planes(Ho, rows, l);
    if (!t || l != ld) return false;
    H.given = Ho;
    H.t = *t;
  }
  if (fo == Py_None) {
    flags.t = st.lend(empty({n}, ScalarType::Byte, like));
  } else {
    const Tensor *t = plain(fo, ScalarType::Byte);
    if (!t) return false;
    flags.given = fo;
    flags.t = *t;
  }
  return true;
}

// solve4(src, dst, method, H, flags, stream) -> (H, flags)
PyObject *solve4(PyObject *const *a) {
  int method;
  if (PyLong_CheckExact(a[2])) {
    int over;   // without an error where the number does not fit
    const long m = PyLong_AsLongAndOverflow(a[2], &over);
    NEED(!over && (m == HG_ACA || m == HG_SKS));
    method = static_cast<int>(m);
  } else {
    NEED(PyUnicode_CheckExact(a[2]));
    if (PyUnicode_CompareWithASCIIString(a[2], "aca") == 0) {
      method = HG_ACA;
    } else {
      NEED(PyUnicode_CompareWithASCIIString(a[2], "sks") == 0);
      method = HG_SKS;
    }
  }
  int64_t ld, ld2;
  const Tensor *s = planes(a[0], 8, ld), *d = planes(a[1], 8, ld2);
  NEED(s && d && ld == ld2);
  const int64_t n = s->size(1);
  Out H, flags;
  CallStream st;
  NEED(st.take(a[5], *s) && solver_out(a[3], a[4], 9, ld, n, *s, st, H, flags));
  NEED(launch([&] {
    return hg_solve4(method, ptr<float>(*s), ptr<float>(*d), n, ld, ptr<float>(H.t),
                     ptr<uint8_t>(flags.t), st.raw);
  }));
  return tuple({H.take(), flags.take()});
}

// solve3_affine(src, dst, A, flags, stream) -> (A, flags)
PyObject *solve3_affine(PyObject *const *a) {
  int64_t ld, ld2;
  const Tensor *s = planes(a[0], 6, ld), *d = planes(a[1], 6, ld2);
  NEED(s && d && ld == ld2);
  const int64_t n = s->size(1);
  Out A, flags;
  CallStream st;
  NEED(st.take(a[4], *s) && solver_out(a[2], a[3], 6, ld, n, *s, st, A, flags));
  NEED(launch([&] {
    return hg_solve3_affine(ptr<float>(*s), ptr<float>(*d), n, ld, ptr<float>(A.t),
                            ptr<uint8_t>(flags.t), st.raw);
  }));
  return tuple({A.take(), flags.take()});
}

// solve_sk(obj, dst, H, flags, stream) -> (H, flags, 9 numbers of H_S1)
PyObject *solve_sk(PyObject *const *a) {
  NEED(PyTuple_CheckExact(a[0]) && PyTuple_GET_SIZE(a[0]) == 8);
  double obj[8], frame[9];
  for (int k = 0; k < 8; ++k) {
    PyObject *v = PyTuple_GET_ITEM(a[0], k);
    NEED(PyFloat_CheckExact(v));
    obj[k] = PyFloat_AS_DOUBLE(v);
  }
  int64_t ld;
  const Tensor *d = planes(a[1], 8, ld);
  NEED(d);
  const int64_t n = d->size(1);
  Out H, flags;
  CallStream st;
  NEED(st.take(a[4], *d) && solver_out(a[2], a[3], 9, ld, n, *d, st, H, flags));
  NEED(launch([&] {
    return hg_solve_sk(obj, ptr<float>(*d), n, ld, ptr<float>(H.t), ptr<uint8_t>(flags.t), frame,
                       st.raw);
  }));
  PyObject *f = PyTuple_New(9);
  if (!f) return nullptr;
  for (int k = 0; k < 9; ++k) PyTuple_SET_ITEM(f, k, PyFloat_FromDouble(frame[k]));
  return tuple({H.take(), flags.take(), f});
}

// ransac(plain, corr, n_hyp, thresh, seed, want_counts, ws, stream) -> dict
PyObject *ransac(PyObject *const *a) {
  NEED(PyLong_CheckExact(a[2]) && PyFloat_CheckExact(a[3]) && PyLong_CheckExact(a[4]));
  int64_t ld;
  const Tensor *c = planes(a[1], 4, ld);
  NEED(c);
  const int64_t n = c->size(1);
  const long nh = PyLong_AsLong(a[2]);
  if (nh == -1 && PyErr_Occurred()) {
    PyErr_Clear();
    DECLINE;
  }
  constexpr int64_t kMax = std::numeric_limits<int32_t>::max();
  NEED(n >= 4 && n <= kMax && nh >= 1 && nh <= kMax);
  const uint64_t seed = PyLong_AsUnsignedLongLongMask(a[4]);
  const float thresh = static_cast<float>(PyFloat_AS_DOUBLE(a[3]));
  const int counts = PyObject_IsTrue(a[5]);
  if (counts < 0) return nullptr;
  const size_t bytes = hg_ransac_ws_bytes(static_cast<int32_t>(n), static_cast<int32_t>(nh));
  CallStream st;
  NEED(st.take(a[7], *c));
  Tensor ws;
  if (a[6] == Py_None) {
    ws = empty({static_cast<int64_t>(bytes)}, ScalarType::Byte, *c);
  } else {
    const Tensor *w = plain(a[6], ScalarType::Byte);
    NEED(w && w->numel() >= static_cast<int64_t>(bytes));
    ws = *w;
  }
  const Tensor H = st.lend(empty({9}, ScalarType::Float, *c)),
               cnt = st.lend(empty({1}, ScalarType::Int, *c)),
               hyp = st.lend(empty({1}, ScalarType::Int, *c)),
               mask = st.lend(empty({n}, ScalarType::Byte, *c));
  Tensor hc;
  if (counts) hc = st.lend(empty({nh}, ScalarType::Int, *c));
  auto *fn = PyObject_IsTrue(a[0]) ? hg_ransac_plain : hg_ransac;
  NEED(launch([&] {
    return fn(ptr<float>(*c), static_cast<int32_t>(n), ld, static_cast<int32_t>(nh), thresh, seed,
              ptr<float>(H), ptr<int32_t>(cnt), ptr<int32_t>(hyp), ptr<uint8_t>(mask),
              counts ? ptr<int32_t>(hc) : nullptr, ws.data_ptr(),
              static_cast<size_t>(ws.numel()), st.raw);
  }));
  PyObject *r = PyDict_New();
  if (!r) return nullptr;
  bool ok = true;
  auto put = [&](const char *key, PyObject *v) {
    ok = ok && v && PyDict_SetItemString(r, key, v) == 0;
    Py_XDECREF(v);
  };
  put("best_H", THPVariable_Wrap(H));
  put("best_count", THPVariable_Wrap(cnt));
  put("best_hyp", THPVariable_Wrap(hyp));
  put("mask", THPVariable_Wrap(mask));
  put("hyp_counts", counts ? THPVariable_Wrap(hc) : Py_NewRef(Py_None));
  if (ok) return r;
  Py_DECREF(r);
  return nullptr;
}

// Whether the host copy of pair offsets (an int64 array or CPU tensor) has m
// entries, non-decreasing within [0, total].
bool offsets_fit(PyObject *o, int64_t m, int64_t total) {
  auto fit = [&](const int64_t *v) {
    if (v[0] < 0 || v[m - 1] > total) return false;
    int64_t bad = 0;
    for (int64_t i = 1; i < m; ++i) bad |= v[i] - v[i - 1];
    return bad >= 0;   // the sign bit of every difference is clear
  };
  if (THPVariable_CheckExact(o)) {
    const Tensor &t = THPVariable_Unpack(o);
    return t.is_cpu() && t.scalar_type() == ScalarType::Long && !at::isTensorSubclassLike(t) &&
           t.dim() == 1 && t.is_contiguous() && t.numel() == m && fit(ptr<int64_t>(t));
  }
  Py_buffer b;
  if (!PyObject_CheckBuffer(o) || PyObject_GetBuffer(o, &b, PyBUF_FORMAT | PyBUF_C_CONTIGUOUS)) {
    PyErr_Clear();
    return false;
  }
  const bool ok = b.ndim == 1 && b.itemsize == 8 && b.format && std::strcmp(b.format, "l") == 0 &&
                  b.len == 8 * m && fit(static_cast<const int64_t *>(b.buf));
  PyBuffer_Release(&b);
  return ok;
}

bool refit_out(PyObject *o, ScalarType type, at::IntArrayRef size, int64_t numel,
               const Tensor &like, const CallStream &st, Out &out) {
  if (o == Py_None) {
    out.t = st.lend(empty(size, type, like));
    return true;
  }
  const Tensor *t = packed(o, type);
  if (!t || t->numel() < numel || t->device() != like.device()) return false;
  out.given = o;
  out.t = *t;
  return true;
}

// refit_ho(corr, off, mask, H, n_used, flags, stream, off_host) -> (H, n_used, flags)
PyObject *refit_ho(PyObject *const *a) {
  NEED(a[7] != Py_None);
  int64_t ld;
  const Tensor *c = planes(a[0], 4, ld), *off = packed(a[1], ScalarType::Long);
  NEED(c && off && off->dim() == 1 && off->numel() >= 1);
  const int64_t total = c->size(1), pairs = off->numel() - 1;
  NEED(pairs <= std::numeric_limits<int32_t>::max() && offsets_fit(a[7], pairs + 1, total));
  const Tensor *mask = nullptr;
  if (a[2] != Py_None) {
    mask = packed(a[2], ScalarType::Byte);
    NEED(mask && mask->numel() >= total);
  }
  Out H, used, flags;
  CallStream st;
  NEED(st.take(a[6], *c));
  NEED(refit_out(a[3], ScalarType::Float, {pairs, 9}, 9 * pairs, *c, st, H));
  NEED(refit_out(a[4], ScalarType::Int, {pairs}, pairs, *c, st, used));
  NEED(refit_out(a[5], ScalarType::Byte, {pairs}, pairs, *c, st, flags));
  NEED(launch([&] {
    return hg_refit_ho(ptr<float>(*c), ld, ptr<int64_t>(*off), static_cast<int32_t>(pairs),
                       mask ? ptr<uint8_t>(*mask) : nullptr, ptr<float>(H.t),
                       ptr<int32_t>(used.t), ptr<uint8_t>(flags.t), st.raw);
  }));
  return tuple({H.take(), used.take(), flags.take()});
}

// (B, 8) or (B, 4, 2) float rows.
const Tensor *quads(PyObject *o) {
  const Tensor *t = packed(o, ScalarType::Float);
  if (!t || t->size(0) > (1 << 30)) return nullptr;
  if (t->dim() == 2 && t->size(1) == 8) return t;
  if (t->dim() == 3 && t->size(1) * t->size(2) == 8) return t;
  return nullptr;
}

// aca_fwd(src, dst, stream) -> H
PyObject *aca_fwd(PyObject *const *a) {
  const Tensor *s = quads(a[0]), *d = quads(a[1]);
  NEED(s && d && s->size(0) == d->size(0));
  const int64_t B = s->size(0);
  CallStream st;
  NEED(st.take(a[2], *s));
  const Tensor H = st.lend(empty({B, 9}, ScalarType::Double, *s));
  NEED(launch([&] {
    return hg_aca_fwd(ptr<float>(*s), ptr<float>(*d), static_cast<int32_t>(B), ptr<double>(H),
                      st.raw);
  }));
  return THPVariable_Wrap(H);
}

// aca_bwd(src, dst, grad_H, want_src, want_dst, stream) -> (grad_src, grad_dst)
PyObject *aca_bwd(PyObject *const *a) {
  const Tensor *s = quads(a[0]), *d = quads(a[1]), *g = packed(a[2], ScalarType::Double);
  NEED(s && d && g && s->size(0) == d->size(0) && g->numel() == 9 * s->size(0));
  NEED(PyBool_Check(a[3]) && PyBool_Check(a[4]));
  const bool ws = a[3] == Py_True, wd = a[4] == Py_True;
  Tensor gs, gd;
  CallStream st;
  NEED(st.take(a[5], *s));
  if (ws) gs = st.lend(at::empty_like(s->detach()));
  if (wd) gd = st.lend(at::empty_like(d->detach()));
  NEED(launch([&] {
    return hg_aca_bwd(ptr<float>(*s), ptr<float>(*d), ptr<double>(*g),
                      static_cast<int32_t>(s->size(0)), ws ? ptr<float>(gs) : nullptr,
                      wd ? ptr<float>(gd) : nullptr, st.raw);
  }));
  return tuple({ws ? THPVariable_Wrap(gs) : Py_NewRef(Py_None),
                wd ? THPVariable_Wrap(gd) : Py_NewRef(Py_None)});
}

// The images of a photometric call and its batch's workspace.
struct Images {
  const Tensor *img = nullptr, *tgt = nullptr;
  int32_t B = 0, h = 0, w = 0;
  Tensor ws;
  bool take(PyObject *io, PyObject *to) {
    img = packed(io, ScalarType::Float);
    tgt = packed(to, ScalarType::Float);
    if (!img || !tgt || img->dim() != 3 || img->sizes() != tgt->sizes()) return false;
    for (int k = 0; k < 3; ++k)
      if (img->size(k) > (1 << 27)) return false;
    B = static_cast<int32_t>(img->size(0));
    h = static_cast<int32_t>(img->size(1));
    w = static_cast<int32_t>(img->size(2));
    return true;
  }
  void workspace() {
    const size_t n = hg_photometric_ws_bytes(B, h, w);
    if (n) ws = empty({static_cast<int64_t>(n)}, ScalarType::Byte, *img);
  }
  void *wp() const { return ws.defined() ? ws.data_ptr() : nullptr; }
  size_t wb() const { return ws.defined() ? static_cast<size_t>(ws.numel()) : 0; }
};

const Tensor *sized(PyObject *o, ScalarType st, int64_t numel) {
  const Tensor *t = packed(o, st);
  return t && t->numel() == numel ? t : nullptr;
}

// photometric_fwd(offsets, img, tgt, stream) -> loss
PyObject *photometric_fwd(PyObject *const *a) {
  Images im;
  CallStream st;
  NEED(im.take(a[1], a[2]) && st.take(a[3], *im.img));
  const Tensor *o = sized(a[0], ScalarType::Float, 8ll * im.B);
  NEED(o);
  const Tensor loss = st.lend(empty({im.B}, ScalarType::Float, *im.img));
  im.workspace();
  NEED(launch([&] {
    return hg_photometric_fwd_ws(ptr<float>(*o), ptr<float>(*im.img), ptr<float>(*im.tgt), im.B,
                                 im.h, im.w, ptr<float>(loss), im.wp(), im.wb(), st.raw);
  }));
  return THPVariable_Wrap(loss);
}

// photometric_bwd(offsets, img, tgt, grad_loss, stream) -> grad_offsets
PyObject *photometric_bwd(PyObject *const *a) {
  Images im;
  CallStream st;
  NEED(im.take(a[1], a[2]) && st.take(a[4], *im.img));
  const Tensor *o = sized(a[0], ScalarType::Float, 8ll * im.B),
               *gl = sized(a[3], ScalarType::Float, im.B);
  NEED(o && gl);
  const Tensor g = st.lend(empty({im.B, 4, 2}, ScalarType::Float, *im.img));
  im.workspace();
  NEED(launch([&] {
    return hg_photometric_bwd_ws(ptr<float>(*o), ptr<float>(*im.img), ptr<float>(*im.tgt),
                                 ptr<float>(*gl), im.B, im.h, im.w, ptr<float>(g), im.wp(),
                                 im.wb(), st.raw);
  }));
  return THPVariable_Wrap(g);
}

// photometric_fwd_grad(offsets, img, tgt, stream) -> (loss, grad_unit)
PyObject *photometric_fwd_grad(PyObject *const *a) {
  Images im;
  CallStream st;
  NEED(im.take(a[1], a[2]) && st.take(a[3], *im.img));
  const Tensor *o = sized(a[0], ScalarType::Float, 8ll * im.B);
  NEED(o);
  const Tensor loss = st.lend(empty({im.B}, ScalarType::Float, *im.img)),
               g = st.lend(empty({im.B, 4, 2}, ScalarType::Float, *im.img));
  im.workspace();
  NEED(launch([&] {
    return hg_photometric_fwd_grad_ws(ptr<float>(*o), ptr<float>(*im.img), ptr<float>(*im.tgt),
                                      im.B, im.h, im.w, ptr<float>(loss), ptr<float>(g), im.wp(),
                                      im.wb(), st.raw);
  }));
  return tuple({THPVariable_Wrap(loss), THPVariable_Wrap(g)});
}

// scale_grad(grad_unit, grad_loss, stream) -> grad_offsets
PyObject *scale_grad(PyObject *const *a) {
  const Tensor *u = packed(a[0], ScalarType::Float);
  NEED(u && u->dim() == 3 && u->size(1) == 4 && u->size(2) == 2 && u->size(0) <= (1 << 27));
  const Tensor *gl = sized(a[1], ScalarType::Float, u->size(0));
  NEED(gl);
  CallStream st;
  NEED(st.take(a[2], *u));
  const Tensor g = st.lend(at::empty_like(u->detach()));
  NEED(launch([&] {
    return hg_scale_grad(ptr<float>(*u), ptr<float>(*gl), static_cast<int32_t>(u->size(0)),
                         ptr<float>(g), st.raw);
  }));
  return THPVariable_Wrap(g);
}

// warp_l1_fwd(H, img, tgt, stream) -> loss
PyObject *warp_l1_fwd(PyObject *const *a) {
  Images im;
  CallStream st;
  NEED(im.take(a[1], a[2]) && st.take(a[3], *im.img));
  const Tensor *H = sized(a[0], ScalarType::Double, 9ll * im.B);
  NEED(H);
  const Tensor loss = st.lend(empty({im.B}, ScalarType::Float, *im.img));
  im.workspace();
  NEED(launch([&] {
    return hg_warp_l1_fwd_ws(ptr<double>(*H), ptr<float>(*im.img), ptr<float>(*im.tgt), im.B, im.h,
                             im.w, ptr<float>(loss), im.wp(), im.wb(), st.raw);
  }));
  return THPVariable_Wrap(loss);
}

// warp_l1_bwd(H, img, tgt, grad_loss, stream) -> grad_H
PyObject *warp_l1_bwd(PyObject *const *a) {
  Images im;
  CallStream st;
  NEED(im.take(a[1], a[2]) && st.take(a[4], *im.img));
  const Tensor *H = sized(a[0], ScalarType::Double, 9ll * im.B),
               *gl = sized(a[3], ScalarType::Float, im.B);
  NEED(H && gl);
  const Tensor g = st.lend(empty({im.B, 9}, ScalarType::Double, *im.img));
  im.workspace();
  NEED(launch([&] {
    return hg_warp_l1_bwd_ws(ptr<double>(*H), ptr<float>(*im.img), ptr<float>(*im.tgt),
                             ptr<float>(*gl), im.B, im.h, im.w, ptr<double>(g), im.wp(), im.wb(),
                             st.raw);
  }));
  return THPVariable_Wrap(g);
}

// The four rectangle arguments as floats.
bool rect(PyObject *const *a, float v[4]) {
  for (int k = 0; k < 4; ++k) {
    if (!PyFloat_CheckExact(a[k])) return false;
    v[k] = static_cast<float>(PyFloat_AS_DOUBLE(a[k]));
  }
  return true;
}

// aca_rect_fwd(offsets, x0, y0, w, r, stream) -> H
PyObject *aca_rect_fwd(PyObject *const *a) {
  float v[4];
  const Tensor *o = packed(a[0], ScalarType::Float);
  CallStream st;
  NEED(o && o->dim() >= 1 && rect(a + 1, v) && st.take(a[5], *o));
  const int64_t B = o->size(0);
  NEED(B <= (1 << 27) && o->numel() == 8 * B);
  const Tensor H = st.lend(empty({B, 9}, ScalarType::Double, *o));
  NEED(launch([&] {
    return hg_aca_rect_fwd(ptr<float>(*o), static_cast<int32_t>(B), v[0], v[1], v[2], v[3],
                           ptr<double>(H), st.raw);
  }));
  return THPVariable_Wrap(H);
}

// aca_rect_bwd(offsets, grad_H, x0, y0, w, r, stream) -> grad_offsets
PyObject *aca_rect_bwd(PyObject *const *a) {
  float v[4];
  const Tensor *o = packed(a[0], ScalarType::Float);
  CallStream st;
  NEED(o && o->dim() >= 1 && rect(a + 2, v) && st.take(a[6], *o));
  const int64_t B = o->size(0);
  const Tensor *g = sized(a[1], ScalarType::Double, 9 * B);
  NEED(g && B <= (1 << 27) && o->numel() == 8 * B);
  const Tensor go = st.lend(empty({B, 4, 2}, ScalarType::Float, *o));
  NEED(launch([&] {
    return hg_aca_rect_bwd(ptr<float>(*o), ptr<double>(*g), static_cast<int32_t>(B), v[0], v[1],
                           v[2], v[3], ptr<float>(go), st.raw);
  }));
  return THPVariable_Wrap(go);
}

// Entry with a fixed number of arguments. A C++ exception (an allocation that
// failed, say) also leaves the call to the Python function, which raises it.
template <PyObject *(*F)(PyObject *const *), Py_ssize_t N>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t n) {
  if (n != N) {
    PyErr_Format(PyExc_TypeError, "%zd arguments expected, got %zd", N, n);
    return nullptr;
  }
  try {
    return F(args);
  } catch (const std::exception &) {
    PyErr_Clear();
    DECLINE;
  }
}

#define ENTRY(name, n) \
  {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(entry<name, n>)), METH_FASTCALL, nullptr}

PyMethodDef methods[] = {ENTRY(solve4, 6),
                         ENTRY(solve3_affine, 5),
                         ENTRY(solve_sk, 5),
                         ENTRY(ransac, 8),
                         ENTRY(refit_ho, 8),
                         ENTRY(aca_fwd, 3),
                         ENTRY(aca_bwd, 6),
                         ENTRY(photometric_fwd, 4),
                         ENTRY(photometric_bwd, 5),
                         ENTRY(photometric_fwd_grad, 4),
                         ENTRY(scale_grad, 3),
                         ENTRY(warp_l1_fwd, 4),
                         ENTRY(warp_l1_bwd, 5),
                         ENTRY(aca_rect_fwd, 6),
                         ENTRY(aca_rect_bwd, 7),
                         {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&module); }
