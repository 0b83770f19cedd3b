// The calls a serving loop makes, from Python objects straight to the C ABI: checks of device, type, shape and
// strides, and addresses.  binding.py allocates what was not given and turns return codes into exceptions; here the
// arguments are positional and complete, the last one torch's current stream.  A step of small tensors is bound by the
// host, where checking twenty tensors and building a ctypes call in Python took longer than the launches: a step of
// two heads of 1024 tokens (five launches, 3 us each) 32.9 -> 20.6 us of host time, 32.0 -> 23.9 us a pass.
#include <Python.h>

#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "heart.h"

namespace {

using at::Tensor;
using Sizes = c10::IntArrayRef;

[[noreturn]] void raise(PyObject *type, const std::string &msg) {
  PyErr_SetString(type, msg.c_str());
  throw python_error();
}
[[noreturn]] void type_error(const std::string &msg) { raise(PyExc_TypeError, msg); }
[[noreturn]] void value_error(const std::string &msg) { raise(PyExc_ValueError, msg); }

const char *torch_name(at::ScalarType t) {
  switch (t) {
    case at::kBFloat16: return "torch.bfloat16";
    case at::kFloat: return "torch.float32";
    case at::kDouble: return "torch.float64";
    case at::kInt: return "torch.int32";
    case at::kByte: return "torch.uint8";
    default: return c10::toString(t);
  }
}

const Tensor *tensor(PyObject *o, const char *name) {
  if (o == Py_None) return nullptr;
  if (!THPVariable_Check(o)) type_error(std::string(name) + " must be a GPU tensor");
  return &THPVariable_Unpack(o);
}

// address of a GPU tensor of the given type (nullptr for None)
void *dev(PyObject *o, at::ScalarType type, const char *name, bool contiguous = true) {
  const Tensor *t = tensor(o, name);
  if (!t) return nullptr;
  if (!t->is_cuda()) type_error(std::string(name) + " must be a GPU tensor");
  if (t->scalar_type() != type)
    type_error(std::string(name) + " must have dtype " + torch_name(type) + ", got " + torch_name(t->scalar_type()));
  if (contiguous && !t->is_contiguous()) value_error(std::string(name) + " must be contiguous");
  return t->data_ptr();
}
template <typename T>
T *dev(PyObject *o, const char *name) {
  return static_cast<T *>(dev(o, c10::CppTypeToScalarType<T>::value, name));
}
void *dev_bf16(PyObject *o, const char *name) { return dev(o, at::kBFloat16, name, false); }

const Tensor &some(PyObject *o, const char *name) {
  const Tensor *t = tensor(o, name);
  if (!t) type_error(std::string(name) + " must be a GPU tensor");
  return *t;
}
void check_sizes(PyObject *o, const char *name, Sizes want, const char *msg) {
  const Tensor *t = tensor(o, name);
  if (t && t->sizes() != want) value_error(msg);
}
// `t` is read or written as `n` contiguous elements: fewer would leave it (more are left alone)
void check_numel(const Tensor *t, int64_t n, const char *msg) {
  if (t && t->numel() < n) value_error(msg);
}
// scratch memory: any type
void *scratch(PyObject *o, size_t *bytes) {
  const Tensor &t = some(o, "workspace");
  if (!t.is_cuda() || !t.is_contiguous()) value_error("workspace must be a contiguous GPU tensor");
  *bytes = t.nbytes();
  return t.data_ptr();
}

void strides(const Tensor &t, const char *name, long long out[3]) {
  if (t.dim() != 4 || t.stride(3) != 1) value_error(std::string(name) + " must be [B,H,N,D] with a contiguous D axis");
  for (int i = 0; i < 3; ++i) out[i] = t.stride(i);
}
heart_shape shape_of(const Tensor &q, const Tensor &k, long block, const Tensor *v = nullptr, const Tensor *o = nullptr) {
  if (q.dim() != 4) value_error("q must be [B,H,N,D] with a contiguous D axis");
  if (block == 0) raise(PyExc_ZeroDivisionError, "block must not be zero");
  if (block > INT_MAX || block < -INT_MAX) value_error("block is too large");  // (negative ones: the library's error)
  for (int i = 0; i < 4; ++i)
    if (q.size(i) > INT_MAX) value_error("q is too large");
  heart_shape s{};
  s.B = (int)q.size(0), s.H = (int)q.size(1), s.N = (int)q.size(2), s.D = (int)q.size(3), s.block = (int)block;
  strides(q, "q", s.q_stride);
  strides(k, "k", s.k_stride);
  strides(v ? *v : k, v ? "v" : "k", s.v_stride);
  strides(o ? *o : q, o ? "out" : "q", s.o_stride);
  return s;
}
int64_t blocks(const heart_shape &s) { return ((int64_t)s.N + s.block - 1) / s.block; }

long integer(PyObject *o) {
  const long v = PyLong_Check(o) ? PyLong_AsLong(o) : [&] {
    PyObject *i = PyNumber_Long(o);
    if (!i) throw python_error();
    const long r = PyLong_AsLong(i);
    Py_DECREF(i);
    return r;
  }();
  if (v == -1 && PyErr_Occurred()) throw python_error();
  return v;
}
int integer32(PyObject *o) {
  const long v = integer(o);
  if (v > INT_MAX || v < INT_MIN) value_error("integer argument out of range");
  return (int)v;
}
// tokens per block: a whole number, not one with a fraction cut off
long block_of(PyObject *o) {
  if (!PyIndex_Check(o)) type_error("block must be an integer");
  return integer(o);
}
double real(PyObject *o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw python_error();
  return v;
}
void *handle(PyObject *o) {
  void *p = PyLong_AsVoidPtr(o);
  if (!p && PyErr_Occurred()) throw python_error();
  return p;
}

// the call, other Python threads running meanwhile
template <typename F>
PyObject *call(F &&f) {
  int rc;
  Py_BEGIN_ALLOW_THREADS;
  rc = f();
  Py_END_ALLOW_THREADS;
  return PyLong_FromLong(rc);
}

void check_count(Py_ssize_t n, Py_ssize_t want) {
  if (n != want) type_error("wrong number of arguments");
}

PyObject *pool_drift(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  check_count(n, 18);
  const Tensor &q = some(a[0], "q"), &k = some(a[1], "k");
  if (q.sizes() != k.sizes()) value_error("q and k must have the same shape");
  const heart_shape s = shape_of(q, k, block_of(a[2]));
  const int64_t means[3] = {s.B, s.H, s.D}, heads[2] = {s.B, s.H};
  if (some(a[6], "delta").numel() != s.H) value_error("delta must have H entries");
  const char *names[4] = {"qanchor", "kanchor", "qmean", "kmean"};
  PyObject *const vecs[4] = {a[3], a[4], a[13], a[14]};
  for (int i = 0; i < 4; ++i) check_sizes(vecs[i], names[i], means, (std::string(names[i]) + " must be [B,H,D]").c_str());
  const int64_t n_blk = (int64_t)s.B * s.H * blocks(s) * s.D;
  check_numel(tensor(a[11], "qblk"), n_blk, "qblk must hold [B,H,Nb,D]");
  check_numel(tensor(a[12], "kblk"), n_blk, "kblk must hold [B,H,Nb,D]");
  PyObject *const flags[3] = {a[5], a[15], a[16]};
  for (PyObject *f : flags) check_sizes(f, "has_anchor, drift, refresh", heads, "has_anchor, drift, refresh must be [B,H]");
  size_t ws_bytes;
  void *ws = scratch(a[7], &ws_bytes);
  const void *qp = dev_bf16(a[0], "q"), *kp = dev_bf16(a[1], "k");
  float *qblk = dev<float>(a[11], "qblk"), *kblk = dev<float>(a[12], "kblk"), *qmean = dev<float>(a[13], "qmean"),
        *kmean = dev<float>(a[14], "kmean"), *qa = dev<float>(a[3], "qanchor"), *ka = dev<float>(a[4], "kanchor");
  unsigned char *has = dev<uint8_t>(a[5], "has_anchor"), *refresh = dev<uint8_t>(a[16], "refresh");
  const float *delta = dev<float>(a[6], "delta");
  float *drift = dev<float>(a[15], "drift");
  const float lo = (float)real(a[8]), hi = (float)real(a[9]);
  const int commit = PyObject_IsTrue(a[10]);
  if (commit < 0) throw python_error();
  void *st = handle(a[17]);
  return call([&] {
    return heart_pool_drift(&s, qp, kp, qblk, kblk, qmean, kmean, qa, ka, has, delta, lo, hi, commit, drift, refresh, ws,
                            ws_bytes, st);
  });
  END_HANDLE_TH_ERRORS
}

PyObject *mask_topp(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  check_count(n, 14);
  const Tensor *qblk = tensor(a[0], "qblk"), *scores = tensor(a[4], "scores_in");
  const Tensor &from = scores ? *scores : some(a[0], "qblk");
  if (from.dim() != 4) value_error(scores ? "scores_in must be [B,H,Nb,Nb]" : "qblk must be [B,H,Nb,D]");
  for (int i = 0; i < 4; ++i)
    if (from.size(i) > INT_MAX) value_error("tensor is too large");
  const int B = (int)from.size(0), H = (int)from.size(1), Nb = (int)from.size(2);
  const int D = scores ? (qblk ? (int)qblk->size(-1) : 0) : (int)from.size(3);
  const int64_t square[4] = {B, H, Nb, Nb}, heads[2] = {B, H}, means[4] = {B, H, Nb, D};
  if (some(a[2], "tau").numel() != H) value_error("tau must have H entries");
  check_sizes(a[8], "mask", square, "mask must have shape [B,H,Nb,Nb]");
  check_sizes(a[9], "kept_idx", square, "kept_idx must have shape [B,H,Nb,Nb]");
  check_sizes(a[10], "kept_count", Sizes(square, 3), "kept_count must have shape [B,H,Nb]");
  check_sizes(a[11], "scores_out", square, "scores_out must be [B,H,Nb,Nb]");
  check_sizes(a[3], "refresh", heads, "refresh must be [B,H]");
  if (!scores && some(a[1], "kblk").sizes() != Sizes(means)) value_error("kblk must match qblk");
  check_numel(scores, (int64_t)B * H * Nb * Nb, "scores_in must be [B,H,Nb,Nb]");
  const float *qp = dev<float>(a[0], "qblk"), *kp = dev<float>(a[1], "kblk"), *sp = dev<float>(a[4], "scores_in"),
              *tau = dev<float>(a[2], "tau");
  const unsigned char *refresh = dev<uint8_t>(a[3], "refresh");
  unsigned char *mask = dev<uint8_t>(a[8], "mask");
  int *idx = dev<int>(a[9], "kept_idx"), *cnt = dev<int>(a[10], "kept_count");
  float *out = dev<float>(a[11], "scores_out");
  const int n_kv = integer32(a[5]), n_q = integer32(a[6]), keep = integer32(a[7]);
  void *st = handle(a[13]);
  if (a[12] == Py_None)
    return call([&] { return heart_mask_topp(B, H, Nb, D, qp, kp, sp, tau, refresh, n_kv, n_q, keep, mask, idx, cnt, out, st); });
  size_t ws_bytes;
  void *ws = scratch(a[12], &ws_bytes);
  return call([&] {
    return heart_mask_topp_ws(B, H, Nb, D, qp, kp, sp, tau, refresh, n_kv, n_q, keep, mask, idx, cnt, out, ws, ws_bytes, st);
  });
  END_HANDLE_TH_ERRORS
}

PyObject *block_sparse_attn(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  check_count(n, 12);
  const Tensor &q = some(a[0], "q"), &k = some(a[1], "k"), &v = some(a[2], "v"), &out = some(a[8], "out");
  if (q.sizes() != k.sizes() || q.sizes() != v.sizes()) value_error("q, k, v must have the same shape");
  const heart_shape s = shape_of(q, k, block_of(a[3]), &v, &out);
  const int64_t Nb = blocks(s), square[4] = {s.B, s.H, Nb, Nb}, rows[3] = {s.B, s.H, s.N};
  if (some(a[4], "kept_idx").sizes() != Sizes(square) || some(a[5], "kept_count").sizes() != Sizes(square, 3))
    value_error("kept_idx must be [B,H,Nb,Nb] and kept_count [B,H,Nb]");
  for (int i = 0; i < 4; ++i)
    if (out.size(i) < q.size(i)) value_error("out must hold the [B,H,N,D] of q");
  check_sizes(a[9], "lse", rows, "lse must be [B,H,N]");
  size_t ws_bytes = 0;
  void *ws = a[10] == Py_None ? nullptr : scratch(a[10], &ws_bytes);
  const void *qp = dev_bf16(a[0], "q"), *kp = dev_bf16(a[1], "k"), *vp = dev_bf16(a[2], "v");
  const int *idx = dev<int>(a[4], "kept_idx"), *cnt = dev<int>(a[5], "kept_count");
  const float scale = (float)real(a[6]);
  const unsigned flags = (unsigned)integer(a[7]);
  void *op = dev_bf16(a[8], "out");
  float *lse = dev<float>(a[9], "lse");
  void *st = handle(a[11]);
  return call([&] { return heart_block_sparse_attn_flags(&s, qp, kp, vp, idx, cnt, scale, flags, op, lse, ws, ws_bytes, st); });
  END_HANDLE_TH_ERRORS
}

PyObject *scores_antidiag(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  check_count(n, 8);
  const Tensor &q = some(a[0], "q"), &k = some(a[1], "k");
  if (q.sizes() != k.sizes()) value_error("q and k must have the same shape");
  const heart_shape s = shape_of(q, k, block_of(a[2]));
  const int stride = integer32(a[3]);
  const int64_t Nb = blocks(s), square[4] = {s.B, s.H, Nb, Nb}, heads[2] = {s.B, s.H};
  check_sizes(a[6], "refresh", heads, "refresh must be [B,H]");
  check_sizes(a[4], "scores", square, "scores must be [B,H,Nb,Nb]");
  size_t ws_bytes;
  void *ws = scratch(a[5], &ws_bytes);
  const void *qp = dev_bf16(a[0], "q"), *kp = dev_bf16(a[1], "k");
  const unsigned char *refresh = dev<uint8_t>(a[6], "refresh");
  float *scores = dev<float>(a[4], "scores");
  void *st = handle(a[7]);
  return call([&] { return heart_scores_antidiag(&s, qp, kp, stride, refresh, scores, ws, ws_bytes, st); });
  END_HANDLE_TH_ERRORS
}

PyObject *ebc_band_error(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  check_count(n, 10);
  const Tensor &err = some(a[0], "err"), &dense = some(a[1], "dense"), &w = some(a[7], "workspace");
  if (err.sizes() != dense.sizes() || err.dim() < 3) value_error("err and dense must have the same shape [..., T, Y, X]");
  check_numel(&some(a[8], "out"), 6, "out must hold six values");
  int axis[3];
  for (int i = 0; i < 3; ++i) {
    if (err.size(i - 3) > INT_MAX) value_error("err is too large");
    axis[i] = (int)err.size(i - 3);
  }
  const int64_t plane = (int64_t)axis[0] * axis[1] * axis[2];
  if (plane == 0) raise(PyExc_ZeroDivisionError, "err has an empty axis");
  const long long C = err.numel() / plane;
  double weights[4];
  for (int i = 0; i < 4; ++i) weights[i] = real(a[2 + i]);
  const double epsilon = real(a[6]);
  const float *ep = dev<float>(a[0], "err"), *dp = dev<float>(a[1], "dense");
  void *ws = dev(a[7], w.scalar_type(), "workspace");
  const size_t ws_bytes = w.nbytes();
  double *out = dev<double>(a[8], "out");
  void *st = handle(a[9]);
  return call([&] {
    return heart_ebc_band_error(C, axis[0], axis[1], axis[2], ep, dp, weights, epsilon, ws, ws_bytes, out, st);
  });
  END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"pool_drift", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(pool_drift)), METH_FASTCALL, nullptr},
    {"mask_topp", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(mask_topp)), METH_FASTCALL, nullptr},
    {"block_sparse_attn", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(block_sparse_attn)), METH_FASTCALL, nullptr},
    {"scores_antidiag", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(scores_antidiag)), METH_FASTCALL, nullptr},
    {"ebc_band_error", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(ebc_band_error)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", HEART_TORCH, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
