// Argument marshalling of the per-operator entry points for Python: tensors -> device pointers, sizes and types, one call of the C ABI.
//
// What bounds a small layer is the host: through ctypes a convolution's nineteen arguments cost 5 us of marshalling (1.9 us of conversions,
// 0.28 us for each of nine tensors) beside 2 to 3 us of the launch itself; here 0.6 us.  The entry points are bound by address, so that the
// library is loaded in one place (wmdec.py).  Every function returns the library's status; what torch throws (a tensor without storage has no
// address) becomes a Python error at the entry.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>

#include "../../include/wmdec.h"

namespace {

decltype(&wmdec_gn_stats) g_gn_stats;
decltype(&wmdec_gn_silu_conv3x3) g_conv3x3;
decltype(&wmdec_gn_conv1x1) g_conv1x1;
decltype(&wmdec_gn_silu_conv3x3_shortcut) g_shortcut;
decltype(&wmdec_gn_silu_conv3x3_stats) g_conv_stats;
decltype(&wmdec_upsample2x_conv3x3) g_upconv;
decltype(&wmdec_attention) g_attention;
decltype(&wmdec_adaln_fused_projection) g_adaln;

constexpr Py_ssize_t kBind = 8;   // arguments of bind(): as many as no other function has

// Reads the arguments; the first one that is not what it should be leaves a Python error and `ok` false.
struct Reader {
  PyObject* const* args;
  bool ok;
  Reader(const char* who, PyObject* const* a, Py_ssize_t given, Py_ssize_t wanted) : args(a), ok(given == wanted) {
    if (!ok) PyErr_Format(PyExc_TypeError, "%s: %zd arguments expected, got %zd", who, wanted, given);
    else if (wanted != kBind && !g_adaln) { ok = false; PyErr_SetString(PyExc_RuntimeError, "the entry points have not been bound"); }
  }
  const at::Tensor* tensor(int i) {
    if (!ok) return nullptr;
    if (!THPVariable_Check(args[i])) { ok = false; PyErr_Format(PyExc_TypeError, "argument %d: tensor expected", i); return nullptr; }
    const at::Tensor& t = THPVariable_Unpack(args[i]);
    if (!t.is_cuda() || !t.is_contiguous()) { ok = false; PyErr_SetString(PyExc_AssertionError, "device-resident contiguous tensor expected"); return nullptr; }
    return &t;
  }
  void* ptr(int i) {   // of a tensor, null for None
    if (!ok || args[i] == Py_None) return nullptr;
    const at::Tensor* t = tensor(i);
    return t ? t->data_ptr() : nullptr;
  }
  int dtype(int i) {
    const at::Tensor* t = tensor(i);
    if (!t) return 0;
    switch (t->scalar_type()) {
      case at::kFloat: return WMDEC_F32;
      case at::kBFloat16: return WMDEC_BF16;
      case at::kHalf: return WMDEC_F16;
      default: ok = false; PyErr_SetString(PyExc_KeyError, "tensor type is none of float32, bfloat16, float16"); return 0;
    }
  }
  int size(int i, int dim, int dims, bool more = false) {   // of a tensor of `dims` dimensions, or of more
    const at::Tensor* t = tensor(i);
    if (!t) return 0;
    if (t->dim() < dims || (t->dim() > dims && !more)) { ok = false; PyErr_Format(PyExc_ValueError, "argument %d: %d dimensions expected, got %d", i, dims, (int)t->dim()); return 0; }
    return (int)t->size(dim);
  }
  size_t bytes(int i) { const at::Tensor* t = tensor(i); return t ? (size_t)t->nbytes() : 0; }
  int integer(int i) {   // the low bits of what can stand for an index, as ctypes passes it
    if (!ok) return 0;
    const unsigned long v = PyLong_AsUnsignedLongMask(args[i]);
    if (v == (unsigned long)-1 && PyErr_Occurred()) ok = false;
    return (int)v;
  }
  int flag(int i) {   // int() of the argument: None and texts that are no number are refused, 0.5 is 0
    if (!ok) return 0;
    PyObject* whole = PyNumber_Long(args[i]);
    const unsigned long v = whole ? PyLong_AsUnsignedLongMask(whole) : 0;
    Py_XDECREF(whole);
    if (PyErr_Occurred()) ok = false;
    return (int)v;
  }
  float real(int i) {
    if (!ok) return 0.f;
    const double v = PyFloat_AsDouble(args[i]);
    if (v == -1.0 && PyErr_Occurred()) ok = false;
    return (float)v;
  }
  void* address(int i) {
    if (!ok) return nullptr;
    void* v = PyLong_AsVoidPtr(args[i]);
    if (!v && PyErr_Occurred()) ok = false;
    return v;
  }
};
// Other threads run Python until its end, also where that is an exception: the handler in entry() sets a Python error.
struct ThreadsAllowed {
  PyThreadState* state = PyEval_SaveThread();
  ~ThreadsAllowed() { PyEval_RestoreThread(state); }
};
#define WMDEC_RETURN(call_)                    \
  do {                                         \
    if (!r.ok) return nullptr;                 \
    int status;                                \
    {                                          \
      ThreadsAllowed threads;                  \
      status = call_;                          \
    }                                          \
    return PyLong_FromLong(status);            \
  } while (0)

// x, groups, eps, mean, rstd, workspace, stream
PyObject* gn_stats(PyObject*, PyObject* const* a, Py_ssize_t na) {
  Reader r("gn_stats", a, na, 7);
  const void* x = r.ptr(0);
  const int dt = r.dtype(0), n = r.size(0, 0, 4), h = r.size(0, 1, 4), w = r.size(0, 2, 4), c = r.size(0, 3, 4), groups = r.integer(1);
  const float eps = r.real(2);
  float *mean = (float*)r.ptr(3), *rstd = (float*)r.ptr(4);
  void* ws = r.ptr(5);
  const size_t bytes = r.bytes(5);
  void* stream = r.address(6);
  WMDEC_RETURN(g_gn_stats(x, dt, n, h, w, c, groups, eps, mean, rstd, ws, bytes, stream));
}

// the arguments that the convolutions share: x, mean, rstd, gamma, beta, groups, apply_silu, w_packed, bias
struct ConvHead {
  const void *x, *w;
  const float *mean, *rstd, *gamma, *beta, *bias;
  int dt, groups, silu, cin;
  ConvHead(Reader& r, int at)
      : x(r.ptr(at)), w(nullptr), dt(r.dtype(at)), cin(r.size(at, 3, 4, true)) {
    mean = (const float*)r.ptr(at + 1); rstd = (const float*)r.ptr(at + 2); gamma = (const float*)r.ptr(at + 3); beta = (const float*)r.ptr(at + 4);
    groups = r.integer(at + 5); silu = r.flag(at + 6);
    w = r.ptr(at + 7); bias = (const float*)r.ptr(at + 8);
  }
};
struct Output { void* y; int dt, n, h, w, c; Output(Reader& r, int i) : y(r.ptr(i)), dt(r.dtype(i)), n(r.size(i, 0, 4)), h(r.size(i, 1, 4)), w(r.size(i, 2, 4)), c(r.size(i, 3, 4)) {} };

// ksize, <head>, residual, y, stream
PyObject* conv(PyObject*, PyObject* const* a, Py_ssize_t na) {
  Reader r("conv", a, na, 13);
  if (!r.ok) return nullptr;
  const int k = r.integer(0);
  const ConvHead c(r, 1);
  const void* res = r.ptr(10);
  const Output y(r, 11);
  void* stream = r.address(12);
  WMDEC_RETURN((k == 3 ? g_conv3x3 : g_conv1x1)(c.x, c.dt, c.mean, c.rstd, c.gamma, c.beta, c.groups, c.silu, c.w, c.bias, res, y.y, y.dt, y.n, y.h, y.w, c.cin, y.c, stream));
}

// <head>, x2, w2_packed, bias2, y, stream
PyObject* conv_shortcut(PyObject*, PyObject* const* a, Py_ssize_t na) {
  Reader r("gn_silu_conv3x3_shortcut", a, na, 14);
  if (!r.ok) return nullptr;
  const ConvHead c(r, 0);
  const void *x2 = r.ptr(9), *w2 = r.ptr(10);
  const int cin2 = r.size(9, 3, 4, true);
  const float* bias2 = (const float*)r.ptr(11);
  const Output y(r, 12);
  void* stream = r.address(13);
  WMDEC_RETURN(g_shortcut(c.x, c.dt, c.mean, c.rstd, c.gamma, c.beta, c.groups, c.silu, c.w, c.bias, x2, cin2, w2, bias2, y.y, y.dt, y.n, y.h, y.w, c.cin, y.c, stream));
}

// <head>, residual, y, out_groups, out_eps, mean_out, rstd_out, workspace, stream
PyObject* conv_stats(PyObject*, PyObject* const* a, Py_ssize_t na) {
  Reader r("gn_silu_conv3x3_stats", a, na, 17);
  if (!r.ok) return nullptr;
  const ConvHead c(r, 0);
  const void* res = r.ptr(9);
  const Output y(r, 10);
  const int groups = r.integer(11);
  const float eps = r.real(12);
  float *mean = (float*)r.ptr(13), *rstd = (float*)r.ptr(14);
  void* ws = r.ptr(15);
  const size_t bytes = r.bytes(15);
  void* stream = r.address(16);
  WMDEC_RETURN(g_conv_stats(c.x, c.dt, c.mean, c.rstd, c.gamma, c.beta, c.groups, c.silu, c.w, c.bias, res, y.y, y.dt, y.n, y.h, y.w, c.cin, y.c, groups, eps, mean, rstd, ws,
                            bytes, stream));
}

// x, w_packed, bias, y, stream
PyObject* upconv(PyObject*, PyObject* const* a, Py_ssize_t na) {
  Reader r("upsample2x_conv3x3", a, na, 5);
  if (!r.ok) return nullptr;
  const Output x(r, 0);   // (a tensor's pointer, type and sizes)
  const void* w = r.ptr(1);
  const float* bias = (const float*)r.ptr(2);
  const Output y(r, 3);
  void* stream = r.address(4);
  WMDEC_RETURN(g_upconv(x.y, x.dt, w, bias, y.y, y.dt, x.n, x.h, x.w, x.c, y.c, stream));
}

// x, mean, rstd, gamma, beta, groups, wqkv_packed, bqkv, wo_packed, bo, y, workspace, stream
PyObject* attention(PyObject*, PyObject* const* a, Py_ssize_t na) {
  Reader r("attention", a, na, 13);
  if (!r.ok) return nullptr;
  const Output x(r, 0);
  const float *mean = (const float*)r.ptr(1), *rstd = (const float*)r.ptr(2), *gamma = (const float*)r.ptr(3), *beta = (const float*)r.ptr(4);
  const int groups = r.integer(5);
  const void* wqkv = r.ptr(6);
  const float* bqkv = (const float*)r.ptr(7);
  const void* wo = r.ptr(8);
  const float* bo = (const float*)r.ptr(9);
  void *y = r.ptr(10), *ws = r.ptr(11);
  const size_t bytes = r.bytes(11);
  void* stream = r.address(12);
  WMDEC_RETURN(g_attention(x.y, x.dt, mean, rstd, gamma, beta, groups, wqkv, bqkv, wo, bo, y, x.n, x.h, x.w, x.c, ws, bytes, stream));
}

// c, w_fused, bias, out, apply_silu, stream
PyObject* adaln(PyObject*, PyObject* const* a, Py_ssize_t na) {
  Reader r("adaln_fused_projection", a, na, 6);
  if (!r.ok) return nullptr;
  const void *c = r.ptr(0), *w = r.ptr(1);
  const int cdt = r.dtype(0), wdt = r.dtype(1), batch = r.size(0, 0, 2), d = r.size(0, 1, 2);
  const at::Tensor* wt = r.tensor(1);
  const int rows = wt && wt->dim() > 0 ? (int)wt->size(0) : 0;
  const float* bias = (const float*)r.ptr(2);
  float* out = (float*)r.ptr(3);
  const int silu = r.flag(4);
  void* stream = r.address(5);
  WMDEC_RETURN(g_adaln(c, cdt, w, wdt, bias, out, batch, d, rows, silu, stream));
}

// the addresses of the entry points, in the order of wmdec.py
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t na) {
  Reader r("bind", a, na, kBind);
  void* f[kBind];
  for (int i = 0; i < kBind; ++i) f[i] = r.address(i);
  if (!r.ok) return nullptr;
  g_gn_stats = (decltype(g_gn_stats))f[0]; g_conv3x3 = (decltype(g_conv3x3))f[1]; g_conv1x1 = (decltype(g_conv1x1))f[2];
  g_shortcut = (decltype(g_shortcut))f[3]; g_conv_stats = (decltype(g_conv_stats))f[4]; g_upconv = (decltype(g_upconv))f[5];
  g_attention = (decltype(g_attention))f[6]; g_adaln = (decltype(g_adaln))f[7];
  Py_RETURN_NONE;
}

template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)> PyObject* entry(PyObject* self, PyObject* const* a, Py_ssize_t na) {
  try {
    return F(self, a, na);
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}
#define WMDEC_METHOD(name_) {#name_, (PyCFunction)(void (*)())entry<name_>, METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {WMDEC_METHOD(gn_stats), WMDEC_METHOD(conv), WMDEC_METHOD(conv_shortcut), WMDEC_METHOD(conv_stats), WMDEC_METHOD(upconv),
                           WMDEC_METHOD(attention), WMDEC_METHOD(adaln), WMDEC_METHOD(bind), {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&g_module); }
