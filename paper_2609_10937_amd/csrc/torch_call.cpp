// The calls of capi.py that a program makes per launch, from torch tensors
// straight to libattn.so: shapes, types and pointers are read from the tensor
// objects in C++ instead of through a dozen Python attribute calls and ctypes
// conversions, which cost more than the launch itself (one small attn_fwd 5.9 us
// of host time, 2.4 of them in the binding).
//
// Each function takes the plain case only (exact tensors on one GPU,
// contiguous, types and shapes that the C entry takes) and returns the entry's
// status; for anything else it returns None, and capi.py's own path checks and
// raises as it always did.  No C++ exception leaves a function here.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

using FwdFn = int (*)(const void*, const void*, const void*, void*, int, int, int, int, float, int, int, void*);
using SoftmaxFn = int (*)(const void*, void*, int64_t, int64_t, int, int, void*);
using GemmFn = int (*)(const void*, const void*, float*, int64_t, int64_t, int64_t, int, void*);

FwdFn g_fwd, g_fwd_noalloc;
SoftmaxFn g_softmax;
GemmFn g_gemm;
PyObject* g_raw_stream;  // torch's getter of a device's current stream handle

constexpr int kBf16 = 0, kF16 = 1, kF32 = 2;  // the library's type codes

int type_code(const at::Tensor& t) {
  switch (t.scalar_type()) {
    case at::kBFloat16: return kBf16;
    case at::kHalf: return kF16;
    case at::kFloat: return kF32;
    default: return -1;
  }
}

// The tensor of an exact torch.Tensor or Parameter that lies contiguous on a GPU,
// else null (subclasses and wrapped tensors keep their own rules).
const at::Tensor* plain(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.is_contiguous()) return nullptr;
  return &t;
}

// A Python bool or int as 0 or 1; -1 for anything else.
int truth(PyObject* o) {
  if (o == Py_True) return 1;
  if (o == Py_False) return 0;
  return -1;
}

// The current stream of t's device; false with a Python error set.
bool stream_of(const at::Tensor& t, void** out) {
  PyObject* d = PyLong_FromLong(t.get_device());
  if (!d) return false;
  PyObject* r = PyObject_CallOneArg(g_raw_stream, d);
  Py_DECREF(d);
  if (!r) return false;
  *out = PyLong_AsVoidPtr(r);
  Py_DECREF(r);
  return !PyErr_Occurred();
}

PyObject* status(int rc) { return PyLong_FromLong(rc); }

PyObject* fwd_call(FwdFn fn, PyObject* const* a, Py_ssize_t n) {
  if (!fn || n != 6 || !PyFloat_CheckExact(a[4])) Py_RETURN_NONE;
  const int causal = truth(a[5]);
  if (causal < 0) Py_RETURN_NONE;
  try {
    const at::Tensor* t[4];
    for (int i = 0; i < 4; ++i)
      if (!(t[i] = plain(a[i]))) Py_RETURN_NONE;
    const int code = type_code(*t[0]);
    if (t[0]->dim() != 4 || (code != kBf16 && code != kF16)) Py_RETURN_NONE;
    int s[4];
    for (int i = 0; i < 4; ++i) {
      const int64_t v = t[0]->size(i);
      if (v < 0 || v > INT32_MAX) Py_RETURN_NONE;
      s[i] = (int)v;
    }
    for (int i = 1; i < 4; ++i)
      if (t[i]->sizes() != t[0]->sizes() || t[i]->scalar_type() != t[0]->scalar_type()) Py_RETURN_NONE;
    const void* q = t[0]->data_ptr();
    const void* k = t[1]->data_ptr();
    const void* v = t[2]->data_ptr();
    void* o = t[3]->data_ptr();
    void* stream = nullptr;
    if (!stream_of(*t[0], &stream)) return nullptr;
    const float scale = (float)PyFloat_AS_DOUBLE(a[4]);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = fn(q, k, v, o, s[0], s[1], s[2], s[3], scale, causal, code, stream);
    Py_END_ALLOW_THREADS
    return status(rc);
  } catch (...) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

PyObject* attn_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) { return fwd_call(g_fwd, a, n); }
PyObject* attn_fwd_noalloc(PyObject*, PyObject* const* a, Py_ssize_t n) { return fwd_call(g_fwd_noalloc, a, n); }

PyObject* attn_softmax(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!g_softmax || n != 3) Py_RETURN_NONE;
  const int causal = truth(a[2]);
  if (causal < 0) Py_RETURN_NONE;
  try {
    const at::Tensor *x = plain(a[0]), *y = plain(a[1]);
    if (!x || !y || x->dim() < 1 || x->sizes() != y->sizes() || x->scalar_type() != y->scalar_type()) Py_RETURN_NONE;
    const int code = type_code(*x);
    const int64_t cols = x->size(-1);
    if ((code != kBf16 && code != kF16) || cols < 1) Py_RETURN_NONE;
    const int64_t rows = x->numel() / cols;
    const void* xp = x->data_ptr();
    void* yp = y->data_ptr();
    void* stream = nullptr;
    if (!stream_of(*x, &stream)) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_softmax(xp, yp, rows, cols, causal, code, stream);
    Py_END_ALLOW_THREADS
    return status(rc);
  } catch (...) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

PyObject* attn_gemm(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!g_gemm || n != 3) Py_RETURN_NONE;
  try {
    const at::Tensor *x = plain(a[0]), *y = plain(a[1]), *z = plain(a[2]);
    if (!x || !y || !z || x->dim() != 2 || y->dim() != 2 || z->dim() != 2) Py_RETURN_NONE;
    const int code = type_code(*x);
    if (code < 0 || y->scalar_type() != x->scalar_type() || z->scalar_type() != at::kFloat) Py_RETURN_NONE;
    const int64_t M = x->size(0), K = x->size(1), N = y->size(1);
    if (y->size(0) != K || z->size(0) != M || z->size(1) != N) Py_RETURN_NONE;
    const void* xp = x->data_ptr();
    const void* yp = y->data_ptr();
    float* zp = static_cast<float*>(z->data_ptr());
    void* stream = nullptr;
    if (!stream_of(*x, &stream)) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_gemm(xp, yp, zp, M, N, K, code, stream);
    Py_END_ALLOW_THREADS
    return status(rc);
  } catch (...) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

// bind(attn_fwd, attn_fwd_noalloc, attn_softmax, attn_gemm, raw_stream): the C
// entries' addresses and torch's stream getter.
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 5) {
    PyErr_SetString(PyExc_TypeError, "bind takes four addresses and the stream getter");
    return nullptr;
  }
  void* p[4];
  for (int i = 0; i < 4; ++i) {
    p[i] = PyLong_AsVoidPtr(a[i]);
    if (PyErr_Occurred()) return nullptr;
  }
  g_fwd = reinterpret_cast<FwdFn>(p[0]);
  g_fwd_noalloc = reinterpret_cast<FwdFn>(p[1]);
  g_softmax = reinterpret_cast<SoftmaxFn>(p[2]);
  g_gemm = reinterpret_cast<GemmFn>(p[3]);
  Py_INCREF(a[4]);
  Py_XSETREF(g_raw_stream, a[4]);
  Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    {"attn_fwd", (PyCFunction)(void (*)(void))attn_fwd, METH_FASTCALL, nullptr},
    {"attn_fwd_noalloc", (PyCFunction)(void (*)(void))attn_fwd_noalloc, METH_FASTCALL, nullptr},
    {"attn_softmax", (PyCFunction)(void (*)(void))attn_softmax, METH_FASTCALL, nullptr},
    {"attn_gemm", (PyCFunction)(void (*)(void))attn_gemm, METH_FASTCALL, nullptr},
    {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_torch_call", nullptr, -1, kMethods};

}  // namespace

PyMODINIT_FUNC PyInit__torch_call(void) { return PyModule_Create(&kModule); }
