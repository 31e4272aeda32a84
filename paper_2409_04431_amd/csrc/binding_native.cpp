// The hot half of the Python binding: checks the tensors, reads their pointers and strides and calls
// the C entry points without a Python object per argument.  Small problems are bound by this host
// work: a call through ctypes with its Python checks takes 10 to 17 us (one struct object per tensor
// and a conversion per argument), the launches in it 2 to 3 each; from here 3 to 4 altogether.
// Passes among others, us: norm forward + backward of 255 tokens 21.0 -> 6.4, one new token per
// sequence against 213 keys 12.6 -> 4.9, forward + backward of 100 tokens 27.4 -> 15.2 (then bound by
// the kernels).
//
// Every function returns the entry point's status, or None where a tensor is not a plain CUDA tensor
// of the expected form: the caller then takes the ctypes path, which raises for what is wrong (and
// serves tensor subclasses).
#include <ATen/ops/empty.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/sattn.h"

namespace {

PyObject* g_current_device;  // () -> index of the current device
PyObject* g_raw_stream;      // index -> torch's current stream of that device, as an integer

struct Arg {
  void* ptr;
  sattn_strides st;
};

const at::Tensor* plain_cuda(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  return t.is_cuda() && t.layout() == at::kStrided ? &t : nullptr;
}

// Attention operands a[0..n): bf16 or fp32 of one dtype, `dim` dimensions, the last one contiguous.
// Tensors whose bit is set in `kv` share the second shape, the others the first.
struct Operands {
  Arg arg[8];
  const at::Tensor* q = nullptr;
  const at::Tensor* k = nullptr;
  sattn_dtype dtype = SATTN_BF16;

  bool read(PyObject* const* a, int n, int dim, unsigned kv = 0) {
    for (int i = 0; i < n; ++i) {
      const at::Tensor* t = plain_cuda(a[i]);
      if (!t || t->dim() != dim || t->stride(dim - 1) != 1) return false;
      const at::Tensor*& ref = (kv >> i & 1) ? k : q;
      if (!ref) ref = t;
      if (t->scalar_type() != a0_type(t, i) || t->sizes() != ref->sizes()) return false;
      if (dim == 4) arg[i].st = {t->stride(0), t->stride(1), t->stride(2)};
      else arg[i].st = {0, t->stride(1), t->stride(0)};
      arg[i].ptr = t->data_ptr();
    }
    if (type != at::kBFloat16 && type != at::kFloat) return false;
    dtype = type == at::kBFloat16 ? SATTN_BF16 : SATTN_F32;
    for (int i = 0; i < dim; ++i)
      if (q->size(i) > INT32_MAX || (k && k->size(i) > INT32_MAX)) return false;
    return true;
  }
  int size(int i) const { return (int)q->size(i); }

 private:
  at::ScalarType type = at::kFloat;
  at::ScalarType a0_type(const at::Tensor* t, int i) {
    if (i == 0) type = t->scalar_type();
    return type;
  }
};

// Optional contiguous CUDA tensor of `type` with `numel` elements (and the given shape): its pointer.
bool vector_ptr(PyObject* o, at::ScalarType type, int64_t numel, void** out) {
  *out = nullptr;
  if (o == Py_None) return true;
  const at::Tensor* t = plain_cuda(o);
  if (!t || t->scalar_type() != type || t->numel() != numel || !t->is_contiguous()) return false;
  *out = t->data_ptr();
  return true;
}
bool shaped_ptr(PyObject* o, at::IntArrayRef shape, void** out) {
  const at::Tensor* t = plain_cuda(o);
  if (!t || t->scalar_type() != at::kFloat || t->sizes() != shape || !t->is_contiguous()) return false;
  *out = t->data_ptr();
  return true;
}
// Workspace: any tensor on the GPU; where the caller gave None, `need` bytes from torch's allocator, on
// the device of `like` (given back with this object, after the launch: the allocator orders its
// reuse by the stream).
struct Workspace {
  at::Tensor own;
  void* ptr = nullptr;
  size_t bytes = 0;
  bool get(PyObject* o, size_t need, const at::Tensor& like) {
    const at::Tensor* t = &own;
    if (o == Py_None) {
      if (!need) return true;
      own = at::empty({(int64_t)need}, like.options().dtype(at::kByte));
    } else if (!(t = plain_cuda(o))) {
      return false;
    }
    ptr = t->data_ptr();
    bytes = (size_t)t->numel() * t->element_size();
    return true;
  }
};

bool number(PyObject* o, float* out) {
  const double x = PyFloat_AsDouble(o);
  if (x == -1.0 && PyErr_Occurred()) return false;
  *out = (float)x;
  return true;
}
bool integer(PyObject* o, int* out) {
  if (!PyLong_CheckExact(o)) return false;
  const long x = PyLong_AsLong(o);
  if ((x == -1 && PyErr_Occurred()) || x > INT32_MAX || x < INT32_MIN) return false;
  *out = (int)x;
  return true;
}
bool flag(PyObject* o, int* out) {
  *out = PyObject_IsTrue(o);
  return *out >= 0;
}
bool stream(void** out) {
  PyObject* dev = PyObject_CallNoArgs(g_current_device);
  if (!dev) return false;
  PyObject* s = PyObject_CallOneArg(g_raw_stream, dev);
  Py_DECREF(dev);
  if (!s) return false;
  *out = PyLong_AsVoidPtr(s);
  Py_DECREF(s);
  return !PyErr_Occurred();
}

// Runs `body`, which returns false where the call is not for this path, and then the entry point
// without the interpreter lock, as ctypes does.
template <typename Body, typename Call>
PyObject* run(Body body, Call call) {
  bool ok = false;
  try {
    ok = body();
  } catch (...) {
  }
  if (!ok) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

// What the attention calls share after their tensors.
struct Common {
  float bias;
  int causal;
  void *slopes, *st;
  bool read(PyObject* b, PyObject* c, PyObject* s, int64_t H) {
    return number(b, &bias) && flag(c, &causal) && vector_ptr(s, at::kFloat, H, &slopes) && stream(&st);
  }
};
#define SATTN_ARGS(n_) \
  if (n != n_) { PyErr_SetString(PyExc_TypeError, "wrong number of arguments"); return nullptr; }

// (q, k, v, o, bias, causal, slopes)
PyObject* fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  SATTN_ARGS(7)
  Operands t; Common c;
  return run([&] { return t.read(a, 4, 4) && c.read(a[4], a[5], a[6], t.q->size(1)); },
             [&] { return sigmoid_attn_fwd(t.arg[0].ptr, t.arg[1].ptr, t.arg[2].ptr, t.arg[3].ptr, t.size(0), t.size(1),
                                           t.size(2), t.size(3), t.dtype, c.bias, c.causal, (const float*)c.slopes,
                                           &t.arg[0].st, &t.arg[1].st, &t.arg[2].st, &t.arg[3].st, c.st); });
}

#define SATTN_BWD_PTRS t.arg[0].ptr, t.arg[1].ptr, t.arg[2].ptr, t.arg[3].ptr, t.arg[4].ptr, t.arg[5].ptr, t.arg[6].ptr
#define SATTN_BWD_STRIDES &t.arg[0].st, &t.arg[1].st, &t.arg[2].st, &t.arg[3].st, &t.arg[4].st, &t.arg[5].st, &t.arg[6].st

// (q, k, v, dout, dq, dk, dv, bias, causal, slopes): no workspace (the entry point needs none)
PyObject* bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  SATTN_ARGS(10)
  Operands t; Common c;
  return run([&] { return t.read(a, 7, 4) && c.read(a[7], a[8], a[9], t.q->size(1)); },
             [&] { return sigmoid_attn_bwd(SATTN_BWD_PTRS, t.size(0), t.size(1), t.size(2), t.size(3), t.dtype, c.bias,
                                           c.causal, (const float*)c.slopes, SATTN_BWD_STRIDES, nullptr, 0, c.st); });
}

// (q, k, v, dout, dq, dk, dv, db_rows, db, bias, causal, slopes)
PyObject* bwd_bias_grad(PyObject*, PyObject* const* a, Py_ssize_t n) {
  SATTN_ARGS(12)
  Operands t; Common c;
  void *rows, *db = nullptr;
  return run([&] { return t.read(a, 7, 4) && shaped_ptr(a[7], t.q->sizes().slice(0, 3), &rows) &&
                          (a[8] == Py_None || shaped_ptr(a[8], t.q->sizes().slice(0, 2), &db)) &&
                          c.read(a[9], a[10], a[11], t.q->size(1)); },
             [&] { return sigmoid_attn_bwd_bias_grad(SATTN_BWD_PTRS, (float*)rows, (float*)db, t.size(0), t.size(1),
                                                     t.size(2), t.size(3), t.dtype, c.bias, c.causal,
                                                     (const float*)c.slopes, SATTN_BWD_STRIDES, c.st); });
}

// Packed sequences: (cu_seqlens, max_seqlen, bias_per_seq) at a[0..3)
struct Packed {
  void *cu, *bias_vec;
  int longest, B;
  bool read(PyObject* const* a) {
    const at::Tensor* t = plain_cuda(a[0]);
    if (!t || t->scalar_type() != at::kInt || t->dim() != 1 || !t->is_contiguous() || t->numel() > INT32_MAX) return false;
    cu = t->data_ptr();
    B = (int)t->numel() - 1;
    return integer(a[1], &longest) && vector_ptr(a[2], at::kFloat, B, &bias_vec);
  }
};

// (q, k, v, o, cu_seqlens, max_seqlen, bias_per_seq, bias, causal, slopes)
PyObject* varlen_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  SATTN_ARGS(10)
  Operands t; Common c; Packed s;
  return run([&] { return t.read(a, 4, 3) && s.read(a + 4) && c.read(a[7], a[8], a[9], t.q->size(1)); },
             [&] { return sigmoid_attn_varlen_fwd(t.arg[0].ptr, t.arg[1].ptr, t.arg[2].ptr, t.arg[3].ptr,
                                                  (const int32_t*)s.cu, (const float*)s.bias_vec, s.B, t.size(1), s.longest,
                                                  t.size(2), t.dtype, c.bias, c.causal, (const float*)c.slopes,
                                                  &t.arg[0].st, &t.arg[1].st, &t.arg[2].st, &t.arg[3].st, c.st); });
}

// (q, k, v, dout, dq, dk, dv, cu_seqlens, max_seqlen, bias_per_seq, bias, causal, slopes)
PyObject* varlen_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  SATTN_ARGS(13)
  Operands t; Common c; Packed s;
  return run([&] { return t.read(a, 7, 3) && s.read(a + 7) && c.read(a[10], a[11], a[12], t.q->size(1)); },
             [&] { return sigmoid_attn_varlen_bwd(SATTN_BWD_PTRS, (const int32_t*)s.cu, (const float*)s.bias_vec, s.B,
                                                  t.size(1), s.longest, t.size(2), t.dtype, c.bias, c.causal,
                                                  (const float*)c.slopes, SATTN_BWD_STRIDES, c.st); });
}

// (q, k, v, dout, dq, dk, dv, cu_seqlens, max_seqlen, bias_per_seq, bias, causal, slopes, db_rows, db)
PyObject* varlen_bwd_bias_grad(PyObject*, PyObject* const* a, Py_ssize_t n) {
  SATTN_ARGS(15)
  Operands t; Common c; Packed s;
  void *rows, *db = nullptr;
  return run([&] {
               if (!t.read(a, 7, 3) || !s.read(a + 7) || !c.read(a[10], a[11], a[12], t.q->size(1))) return false;
               const int64_t rs[2] = {t.q->size(1), t.q->size(0)}, bs[2] = {s.B, t.q->size(1)};
               return shaped_ptr(a[13], rs, &rows) && (a[14] == Py_None || shaped_ptr(a[14], bs, &db));
             },
             [&] { return sigmoid_attn_varlen_bwd_bias_grad(SATTN_BWD_PTRS, (float*)rows, (float*)db, (const int32_t*)s.cu,
                                                            (const float*)s.bias_vec, s.B, t.size(1), s.longest, t.size(0),
                                                            t.size(2), t.dtype, c.bias, c.causal, (const float*)c.slopes,
                                                            SATTN_BWD_STRIDES, c.st); });
}

// q and k share batch, tokens and features; k's heads divide q's
bool shared_heads(const Operands& t) {
  const int64_t Hkv = t.k->size(1);
  return t.k->size(0) == t.q->size(0) && t.k->size(2) == t.q->size(2) && t.k->size(3) == t.q->size(3) && Hkv > 0 &&
         t.q->size(1) % Hkv == 0;
}

// (q, k, v, o, bias, causal, slopes)
PyObject* mqa_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  SATTN_ARGS(7)
  Operands t; Common c;
  return run([&] { return t.read(a, 4, 4, 0b0110) && shared_heads(t) && c.read(a[4], a[5], a[6], t.q->size(1)); },
             [&] { return sigmoid_attn_mqa_fwd(t.arg[0].ptr, t.arg[1].ptr, t.arg[2].ptr, t.arg[3].ptr, t.size(0), t.size(1),
                                               (int)t.k->size(1), t.size(2), t.size(3), t.dtype, c.bias, c.causal,
                                               (const float*)c.slopes, &t.arg[0].st, &t.arg[1].st, &t.arg[2].st,
                                               &t.arg[3].st, c.st); });
}

// (q, k, v, dout, dq, dk, dv, bias, causal, slopes, workspace)
PyObject* mqa_bwd_split(PyObject*, PyObject* const* a, Py_ssize_t n) {
  SATTN_ARGS(11)
  Operands t; Common c; Workspace ws;
  return run([&] { return t.read(a, 7, 4, 0b1100110) && shared_heads(t) && c.read(a[7], a[8], a[9], t.q->size(1)) &&
                          ws.get(a[10], sigmoid_attn_mqa_bwd_workspace_bytes(t.size(0), t.size(1), (int)t.k->size(1),
                                                                             t.size(2), t.size(3), t.dtype, c.causal), *t.q); },
             [&] { return sigmoid_attn_mqa_bwd_split(SATTN_BWD_PTRS, t.size(0), t.size(1), (int)t.k->size(1), t.size(2),
                                                     t.size(3), t.dtype, c.bias, c.causal, (const float*)c.slopes,
                                                     SATTN_BWD_STRIDES, ws.ptr, ws.bytes, c.st); });
}

// (q, k, v, o, bias, causal, slopes, workspace)
PyObject* cross_aligned_fwd_split(PyObject*, PyObject* const* a, Py_ssize_t n) {
  SATTN_ARGS(8)
  Operands t; Common c; Workspace ws;
  return run([&] {
               if (!t.read(a, 4, 4, 0b0110) || t.k->size(0) != t.q->size(0) || t.k->size(1) != t.q->size(1) ||
                   t.k->size(3) != t.q->size(3) || t.k->size(2) <= 0 || !c.read(a[4], a[5], a[6], t.q->size(1))) return false;
               return ws.get(a[7], sigmoid_attn_cross_aligned_fwd_workspace_bytes(t.size(0), t.size(1), t.size(2),
                                                                                  (int)t.k->size(2), t.size(3), t.dtype), *t.q);
             },
             [&] { return sigmoid_attn_cross_aligned_fwd_split(
                       t.arg[0].ptr, t.arg[1].ptr, t.arg[2].ptr, t.arg[3].ptr, t.size(0), t.size(1), t.size(2),
                       (int)t.k->size(2), t.size(3), t.dtype, c.bias, c.causal, (const float*)c.slopes, &t.arg[0].st,
                       &t.arg[1].st, &t.arg[2].st, &t.arg[3].st, ws.ptr, ws.bytes, c.st); });
}

bool stats_ptr(PyObject* o, const Operands& t, void** out) {
  const int64_t shape[3] = {t.q->size(0), t.q->size(2), 2};
  return shaped_ptr(o, shape, out);
}

// (x, y, stats, kind, eps)
PyObject* norm_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  SATTN_ARGS(5)
  Operands t;
  void *stats, *st; int kind; float eps;
  return run([&] { return t.read(a, 2, 4) && stats_ptr(a[2], t, &stats) && integer(a[3], &kind) && number(a[4], &eps) && stream(&st); },
             [&] { return sattn_headconcat_norm_fwd(t.arg[0].ptr, t.arg[1].ptr, (float*)stats, t.size(0), t.size(1), t.size(2),
                                                    t.size(3), t.dtype, kind, eps, &t.arg[0].st, &t.arg[1].st, st); });
}

// (x, dy, dx, stats, kind)
PyObject* norm_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  SATTN_ARGS(5)
  Operands t;
  void *stats, *st; int kind;
  return run([&] { return t.read(a, 3, 4) && stats_ptr(a[3], t, &stats) && integer(a[4], &kind) && stream(&st); },
             [&] { return sattn_headconcat_norm_bwd(t.arg[0].ptr, t.arg[1].ptr, (const float*)stats, t.arg[2].ptr, t.size(0),
                                                    t.size(1), t.size(2), t.size(3), t.dtype, kind, &t.arg[0].st,
                                                    &t.arg[1].st, &t.arg[2].st, st); });
}

#define SATTN_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    SATTN_METHOD(fwd), SATTN_METHOD(bwd), SATTN_METHOD(bwd_bias_grad), SATTN_METHOD(varlen_fwd), SATTN_METHOD(varlen_bwd),
    SATTN_METHOD(varlen_bwd_bias_grad), SATTN_METHOD(mqa_fwd), SATTN_METHOD(mqa_bwd_split),
    SATTN_METHOD(cross_aligned_fwd_split), SATTN_METHOD(norm_fwd), SATTN_METHOD(norm_bwd), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) {
  PyObject* torch_c = PyImport_ImportModule("torch._C");
  if (!torch_c) return nullptr;
  g_current_device = PyObject_GetAttrString(torch_c, "_cuda_getDevice");
  g_raw_stream = PyObject_GetAttrString(torch_c, "_cuda_getCurrentRawStream");
  Py_DECREF(torch_c);
  if (!g_current_device || !g_raw_stream) return nullptr;
  return PyModule_Create(&module);
}
