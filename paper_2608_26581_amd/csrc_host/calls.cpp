// The common form of the binding's calls in native code: checks on plain
// device tensors, allocation of the outputs and the call into librfq.
//
// At decode sizes a call's kernel takes 4 to 13 us, and checking its tensors
// and marshalling 12 to 14 arguments through ctypes in Python took as long (9 us
// a call, 14 with a workspace).  Each function here takes the binding's
// arguments and returns its result, or None where anything is not the common
// form (a tensor subclass, another device, a wrong shape or type) or the
// library refused an argument: the caller then goes through the Python path,
// which accepts the rest and words the errors.  Any other failure comes back
// as the library's status and is not tried again.
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

#include "rfq.h"

namespace {

// Entry points of the librfq that the binding has loaded (bind()).
struct Lib {
  int (*quantize_act)(const void *, int, int64_t, int64_t, void *, void *, void *, void *, void *);
  int (*gemm)(const void *, const void *, const void *, const void *, const void *, const void *,
              int64_t, int64_t, int64_t, void *, int, void *);
  int (*gemm_split)(const void *, const void *, const void *, const void *, const void *,
                    const void *, int64_t, int64_t, int64_t, void *, int, void *, int64_t, void *);
  int64_t (*gemm_workspace_bytes)(int64_t, int64_t, int64_t);
  int (*gemm_stream)(const void *, int, int, const void *, const void *, int64_t, int64_t, int64_t,
                     void *, int, void *);
  int (*hif4_quantize)(const void *, int, int64_t, int64_t, void *, void *, void *, void *, void *);
  decltype(gemm) hif4_gemm;
  decltype(gemm_split) hif4_gemm_split;
  decltype(gemm_workspace_bytes) hif4_gemm_workspace_bytes;
  int (*gemm_phi)(const void *, const void *, const void *, const void *, const void *,
                  const void *, const void *, int64_t, int64_t, int64_t, void *, int, void *);
  int (*fallback_map)(const void *, const void *, int64_t, int64_t, int, int, void *, void *);
  int (*gemm_swiglu_quantize)(const void *, const void *, const void *, const void *, const void *,
                              const void *, int64_t, int64_t, int64_t, void *, void *, void *,
                              void *, void *, void *);
} lib;

// A plain torch.Tensor (no subclass), contiguous, strided, 2-D, on device dev.
const at::Tensor *plain(PyObject *o, int dev) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor &t = THPVariable_Unpack(o);
  if (!t.is_cuda() || t.layout() != at::kStrided || t.dim() != 2 || !t.is_contiguous() ||
      t.get_device() != dev)
    return nullptr;
  return &t;
}

bool is(const at::Tensor *t, at::ScalarType type, int64_t rows, int64_t cols) {
  return t && t->scalar_type() == type && t->size(0) == rows && t->size(1) == cols;
}

// dtype code (0 fp32, 1 bf16) of a floating tensor, -1 of another.
int float_code(const at::Tensor &t) {
  return t.scalar_type() == at::kBFloat16 ? 1 : (t.scalar_type() == at::kFloat ? 0 : -1);
}

// Releases the interpreter lock for its lifetime: an allocation may have to
// wait for the driver and a launch for room in a full queue, and a host
// callback that the queue waits for may need the lock.
class NoGil {
 public:
  NoGil() : state_(PyEval_SaveThread()) {}
  ~NoGil() { PyEval_RestoreThread(state_); }
  NoGil(const NoGil &) = delete;
  NoGil &operator=(const NoGil &) = delete;

 private:
  PyThreadState *state_;
};

// A new tensor on like's device (called without the interpreter lock).
at::Tensor empty(const at::Tensor &like, at::IntArrayRef sizes, at::ScalarType type) {
  return at::empty(sizes, like.options().dtype(type).requires_grad(false));
}

// A library call without the interpreter lock; its arguments are read from
// the tensors before.
template <class F, class... A>
int call(F f, A... a) {
  const NoGil unlocked;
  return f(a...);
}

void *stream_of(int dev) { return c10::hip::getCurrentHIPStream((c10::DeviceIndex)dev).stream(); }

PyObject *none() { Py_RETURN_NONE; }

// What a call returns for status st other than RFQ_OK.  The argument errors
// are found on the host before anything runs; after a failed launch part of
// the call may have run, and the launch's error has been read (and so
// cleared), so that a second try could report success.
PyObject *failed(int st) {
  const bool argument = st == RFQ_ERR_NULL || st == RFQ_ERR_SHAPE || st == RFQ_ERR_DTYPE ||
                        st == RFQ_ERR_ALIGN;
  return argument ? none() : PyLong_FromLong(st);
}

// The current device, or -1 where o is not a device tensor.
int device_for(PyObject *o) {
  return THPVariable_CheckExact(o) && THPVariable_Unpack(o).is_cuda() ? c10::hip::current_device()
                                                                       : -1;
}

// An operand: codes [rows][K/2] and scales (MXFP4: uint8 [rows][K/32]) or
// metadata (HiF4: int32 [rows][K/64]).
struct Operand {
  const at::Tensor *codes = nullptr, *scales = nullptr;
  const void *c() const { return codes ? codes->data_ptr() : nullptr; }
  const void *s() const { return scales ? scales->data_ptr() : nullptr; }
};

template <bool HIF4>
bool operand(PyObject *codes, PyObject *scales, int64_t rows, int64_t K, int dev, Operand &o) {
  constexpr int64_t kBlock = HIF4 ? 64 : 32;
  o.codes = plain(codes, dev);
  o.scales = plain(scales, dev);
  return is(o.codes, at::kByte, rows, K / 2) &&
         is(o.scales, HIF4 ? at::kInt : at::kByte, rows, K / kBlock);
}

// (t[0], .., t[n-1]), None for the undefined ones.
PyObject *tuple(const at::Tensor *t, int n) {
  PyObject *r = PyTuple_New(n);
  if (!r) return nullptr;
  for (int i = 0; i < n; ++i) {
    PyObject *v = t[i].defined() ? THPVariable_Wrap(t[i]) : none();
    if (!v) {
      Py_DECREF(r);
      return nullptr;
    }
    PyTuple_SET_ITEM(r, i, v);
  }
  return r;
}

// quantize(x, residual) -> (codes, scales, residual codes, residual scales).
template <bool HIF4>
PyObject *quantize(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  const int dev = n != 2 ? -1 : device_for(a[0]);
  if (dev < 0) return none();
  const at::Tensor *x = plain(a[0], dev);
  if (!x || float_code(*x) < 0) return none();
  const int residual = PyObject_IsTrue(a[1]);
  if (residual < 0) return nullptr;
  const int64_t rows = x->size(0), K = x->size(1);
  at::Tensor t[4];
  {
    const NoGil unlocked;
    for (int i = 0; i < (residual ? 4 : 2); i += 2) {
      t[i] = empty(*x, {rows, K / 2}, at::kByte);
      t[i + 1] = HIF4 ? empty(*x, {rows, K / 64}, at::kInt) : empty(*x, {rows, K / 32}, at::kByte);
    }
  }
  void *p[4];
  for (int i = 0; i < 4; ++i) p[i] = t[i].defined() ? t[i].data_ptr() : nullptr;
  const int st = call(HIF4 ? lib.hif4_quantize : lib.quantize_act, x->data_ptr(), float_code(*x),
                      rows, K, p[0], p[1], p[2], p[3], stream_of(dev));
  return st ? failed(st) : tuple(t, 4);
  END_HANDLE_TH_ERRORS
}

// out (given and fitting) or a new [M][N] tensor of dtype code `code`;
// undefined where neither fits.
at::Tensor output(PyObject *out, int code, const at::Tensor &like, int64_t M, int64_t N, int dev) {
  if (out != Py_None) {
    const at::Tensor *t = plain(out, dev);
    return t && float_code(*t) >= 0 && t->size(0) == M && t->size(1) == N ? *t : at::Tensor();
  }
  if (code != 0 && code != 1) return at::Tensor();
  const NoGil unlocked;
  return empty(like, {M, N}, code ? at::kBFloat16 : at::kFloat);
}

// What a call with `out` returns: that object, or the new tensor.
PyObject *result(PyObject *out, const at::Tensor &z) {
  if (out == Py_None) return THPVariable_Wrap(z);
  Py_INCREF(out);
  return out;
}

// Operands of a product (q, qs, r, rs, w, ws): its sizes, or false.
struct Product {
  int64_t M, N, K;
  Operand q, r, w;
};
template <bool HIF4>
bool product(PyObject *const *a, int dev, Product &p) {
  const at::Tensor *q = plain(a[0], dev), *w = plain(a[4], dev);
  if (!q || !w) return false;
  p.M = q->size(0);
  p.K = q->size(1) * 2;
  p.N = w->size(0);
  return operand<HIF4>(a[0], a[1], p.M, p.K, dev, p.q) &&
         operand<HIF4>(a[4], a[5], p.N, p.K, dev, p.w) &&
         (a[2] == Py_None ? a[3] == Py_None : operand<HIF4>(a[2], a[3], p.M, p.K, dev, p.r));
}

// gemm(q, qs, r, rs, w, ws, dtype code, out, split) -> Z.
template <bool HIF4>
PyObject *gemm(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  const int dev = n != 9 ? -1 : device_for(a[0]);
  if (dev < 0) return none();
  Product p;
  if (!product<HIF4>(a, dev, p)) return none();
  const int split = PyObject_IsTrue(a[8]);
  const long code = PyLong_AsLong(a[6]);
  if (split < 0 || (code == -1 && PyErr_Occurred())) return nullptr;
  const at::Tensor z = output(a[7], (int)code, *p.q.codes, p.M, p.N, dev);
  if (!z.defined()) return none();
  int64_t bytes = 0;
  if (split)
    bytes = (HIF4 ? lib.hif4_gemm_workspace_bytes : lib.gemm_workspace_bytes)(p.M, p.N, p.K);
  int st;
  if (bytes > 0) {
    at::Tensor work;
    {
      const NoGil unlocked;
      work = empty(*p.q.codes, {bytes}, at::kByte);
    }
    st = call(HIF4 ? lib.hif4_gemm_split : lib.gemm_split, p.q.c(), p.q.s(), p.r.c(), p.r.s(),
              p.w.c(), p.w.s(), p.M, p.N, p.K, z.data_ptr(), float_code(z), work.data_ptr(),
              bytes, stream_of(dev));
  } else {
    st = call(HIF4 ? lib.hif4_gemm : lib.gemm, p.q.c(), p.q.s(), p.r.c(), p.r.s(), p.w.c(),
              p.w.s(), p.M, p.N, p.K, z.data_ptr(), float_code(z), stream_of(dev));
  }
  return st ? failed(st) : result(a[7], z);
  END_HANDLE_TH_ERRORS
}

// gemm_phi(q, qs, r, rs, w, ws, phi or None, dtype code, out) -> Z.
PyObject *gemm_phi(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  const int dev = n != 9 ? -1 : device_for(a[0]);
  if (dev < 0) return none();
  Product p;
  if (!product<false>(a, dev, p)) return none();
  const at::Tensor *phi = nullptr;
  if (a[6] != Py_None) {
    phi = plain(a[6], dev);
    if (!is(phi, at::kByte, (p.M + 63) / 64, (p.K + 255) / 256)) return none();
  }
  const long code = PyLong_AsLong(a[7]);
  if (code == -1 && PyErr_Occurred()) return nullptr;
  const at::Tensor z = output(a[8], (int)code, *p.q.codes, p.M, p.N, dev);
  if (!z.defined()) return none();
  const int st = call(lib.gemm_phi, p.q.c(), p.q.s(), p.r.c(), p.r.s(), p.w.c(), p.w.s(),
                      phi ? phi->data_ptr() : nullptr, p.M, p.N, p.K, z.data_ptr(), float_code(z),
                      stream_of(dev));
  return st ? failed(st) : result(a[8], z);
  END_HANDLE_TH_ERRORS
}

// fallback_map(r or None, qs, rule, threshold) -> phi.  Both tensors are
// checked here, also the one that the rule does not read (else: Python).
PyObject *fallback_map(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  const int dev = n != 4 ? -1 : device_for(a[1]);
  if (dev < 0) return none();
  const at::Tensor *qs = plain(a[1], dev);
  if (!qs || qs->scalar_type() != at::kByte) return none();
  const int64_t M = qs->size(0), K = qs->size(1) * 32;
  const at::Tensor *r = nullptr;
  if (a[0] != Py_None) {
    r = plain(a[0], dev);
    if (!is(r, at::kByte, M, K / 2)) return none();
  }
  if (!PyLong_CheckExact(a[2]) || !PyLong_CheckExact(a[3])) return none();
  int over = 0;
  const long rule = PyLong_AsLongAndOverflow(a[2], &over);
  const long threshold = over ? 0 : PyLong_AsLongAndOverflow(a[3], &over);
  if (over || (rule != 0 && rule != 1) || threshold != (int)threshold || (rule == 0 && !r))
    return none();
  at::Tensor phi;
  {
    const NoGil unlocked;
    phi = empty(*qs, {(M + 63) / 64, (K + 255) / 256}, at::kByte);
  }
  const int st = call(lib.fallback_map, r ? r->data_ptr() : nullptr, qs->data_ptr(), M, K,
                      (int)rule, (int)threshold, phi.data_ptr(), stream_of(dev));
  return st ? failed(st) : THPVariable_Wrap(phi);
  END_HANDLE_TH_ERRORS
}

// gemm_swiglu_quantize(q, qs, r, rs, wgu, wgus, residual) -> (codes, scales,
// residual codes, residual scales, None).
PyObject *gemm_swiglu_quantize(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  const int dev = n != 7 ? -1 : device_for(a[0]);
  if (dev < 0) return none();
  Product p;
  if (!product<false>(a, dev, p) || p.N % 2) return none();
  const int residual = PyObject_IsTrue(a[6]);
  if (residual < 0) return nullptr;
  const int64_t Nh = p.N / 2;
  at::Tensor t[5];
  {
    const NoGil unlocked;
    for (int i = 0; i < (residual ? 4 : 2); i += 2) {
      t[i] = empty(*p.q.codes, {p.M, Nh / 2}, at::kByte);
      t[i + 1] = empty(*p.q.codes, {p.M, Nh / 32}, at::kByte);
    }
  }
  const int st = call(lib.gemm_swiglu_quantize, p.q.c(), p.q.s(), p.r.c(), p.r.s(), p.w.c(),
                      p.w.s(), p.M, Nh, p.K, t[0].data_ptr(), t[1].data_ptr(),
                      residual ? t[2].data_ptr() : nullptr, residual ? t[3].data_ptr() : nullptr,
                      nullptr, stream_of(dev));
  return st ? failed(st) : tuple(t, 5);
  END_HANDLE_TH_ERRORS
}

// gemm_stream(x, w, ws, residual, dtype code, out) -> Z.
PyObject *gemm_stream(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  const int dev = n != 6 ? -1 : device_for(a[0]);
  if (dev < 0) return none();
  const at::Tensor *x = plain(a[0], dev), *w = plain(a[1], dev);
  if (!x || !w || float_code(*x) < 0) return none();
  const int64_t M = x->size(0), K = x->size(1), N = w->size(0);
  Operand ow;
  if (K % 2 || !operand<false>(a[1], a[2], N, K, dev, ow)) return none();
  const int residual = PyObject_IsTrue(a[3]);
  const long code = PyLong_AsLong(a[4]);
  if (residual < 0 || (code == -1 && PyErr_Occurred())) return nullptr;
  const at::Tensor z = output(a[5], (int)code, *x, M, N, dev);
  if (!z.defined()) return none();
  const int st = call(lib.gemm_stream, x->data_ptr(), float_code(*x), residual, ow.c(), ow.s(), M,
                      N, K, z.data_ptr(), float_code(z), stream_of(dev));
  return st ? failed(st) : result(a[5], z);
  END_HANDLE_TH_ERRORS
}

// bind(addresses): the entry points, in Lib's order.
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n) {
  void **slot = reinterpret_cast<void **>(&lib);
  if (n != (Py_ssize_t)(sizeof(Lib) / sizeof(void *))) {
    PyErr_SetString(PyExc_TypeError, "bind: one address per entry point");
    return nullptr;
  }
  for (Py_ssize_t i = 0; i < n; ++i) {
    void *p = PyLong_AsVoidPtr(a[i]);
    if (!p) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "bind: null address");
      return nullptr;
    }
    slot[i] = p;
  }
  Py_RETURN_NONE;
}

#define RFQ_METHOD(name, fn) \
  {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(fn)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {RFQ_METHOD("bind", bind),
                         RFQ_METHOD("quantize_act", quantize<false>),
                         RFQ_METHOD("gemm", gemm<false>),
                         RFQ_METHOD("gemm_stream", gemm_stream),
                         RFQ_METHOD("gemm_phi", gemm_phi),
                         RFQ_METHOD("fallback_map", fallback_map),
                         RFQ_METHOD("gemm_swiglu_quantize", gemm_swiglu_quantize),
                         RFQ_METHOD("hif4_quantize", quantize<true>),
                         RFQ_METHOD("hif4_gemm", gemm<true>),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_rfq_calls", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

// torch_version: the torch that the module was compiled against (its C++
// interface changes between versions; the binding uses the module only with
// the same one).
PyMODINIT_FUNC PyInit__rfq_calls() {
  PyObject *m = PyModule_Create(&module);
  if (m && PyModule_AddStringConstant(m, "torch_version", RFQ_TORCH_VERSION) < 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
