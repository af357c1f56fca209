// The host path of the Python entry points for the calls that need nothing unusual: argument checks,
// output allocation and the C-ABI call in one native function per direction (CPython extension
// `_spark_host`, used by binding.py).
//
// Small problems are bound by the host: a training step of 2 heads x 128 tokens took 33 us a pass with its
// marshalling in Python through ctypes (nine tensors checked and six allocated in the interpreter, arguments
// converted one by one), here 18 us with the same three launches, 14.4 us with two and 13.8 us with the allocations
// below (10.7 us of kernels).
//
// Nothing is refused or reported here.  Whatever is not an ordinary call (a wrong shape, type, device or
// layout, a tensor subclass or transform wrapper, an active dispatch mode, a number that is not a plain
// float or int) returns None before anything has been allocated or launched, and binding.py's general
// path, which accepts or raises as documented there, takes the call.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/ops/empty.h>
#include <ATen/record_function.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>

#include <limits.h>

#include "../../include/spark_mha.h"

namespace {

enum Kind { SELF = 0, CROSS = 1, STRIDED = 2 };

constexpr c10::DispatchKeySet kWrappers({c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot,
                                         c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                         c10::DispatchKey::Functionalize, c10::DispatchKey::Conjugate,
                                         c10::DispatchKey::Negative, c10::DispatchKey::ZeroTensor});

// An ordinary dense device tensor of dtype `st` and rank `rank`, or nullptr.
const at::Tensor* plain(PyObject* o, int rank) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || t.dim() != rank) return nullptr;
  if (t.key_set().has_any(kWrappers) || !t.has_storage() || t.unsafeGetTensorImpl()->has_symbolic_sizes_strides())
    return nullptr;
  return &t;
}

bool shaped(const at::Tensor& t, at::ScalarType st, int64_t B, int64_t H, int64_t N, int64_t d, int kind) {
  return t.scalar_type() == st && t.size(0) == B && t.size(1) == H && t.size(2) == N && t.size(3) == d &&
         (kind == STRIDED ? t.stride(3) == 1 : t.is_contiguous());
}

bool stats_shaped(const at::Tensor& t, int64_t B, int64_t H, int64_t N) {
  return t.scalar_type() == at::kFloat && t.size(0) == B && t.size(1) == H && t.size(2) == N && t.is_contiguous();
}

// A contiguous tensor may have any stride in a dimension of size one: those of its sizes are passed then.
spark_strides_t strides(const at::Tensor& t, int kind) {
  if (kind == STRIDED) return spark_strides_t{t.stride(0), t.stride(1), t.stride(2)};
  return spark_strides_t{t.size(1) * t.size(2) * t.size(3), t.size(2) * t.size(3), t.size(3)};
}

// torch._C._cuda_getDevice and torch._C._cuda_getCurrentRawStream, handed over once by bind()
PyObject *get_device = nullptr, *get_raw_stream = nullptr;

// The current stream of the current device; false with a Python error set if torch cannot say.
bool current_stream(void** out) {
  PyObject* dev = PyObject_CallNoArgs(get_device);
  if (!dev) return false;
  PyObject* raw = PyObject_CallOneArg(get_raw_stream, dev);
  Py_DECREF(dev);
  if (!raw) return false;
  *out = PyLong_AsVoidPtr(raw);
  Py_DECREF(raw);
  return !PyErr_Occurred();
}

struct Numbers {
  float scale, p_drop;
  int causal, kind;
  unsigned long long seed;
  unsigned offset;
};

// scale, causal, p_drop, seed, offset, kind
bool numbers(PyObject* const* a, Numbers* n) {
  if (!PyFloat_Check(a[0]) || !PyBool_Check(a[1]) || !PyFloat_Check(a[2]) || !PyLong_Check(a[3]) ||
      !PyLong_Check(a[4]) || !PyLong_Check(a[5]))
    return false;
  n->scale = (float)PyFloat_AS_DOUBLE(a[0]);
  n->causal = a[1] == Py_True;
  n->p_drop = (float)PyFloat_AS_DOUBLE(a[2]);
  n->seed = PyLong_AsUnsignedLongLongMask(a[3]);  // modulo 2^64 and 2^32, as ctypes converts them
  n->offset = (unsigned)PyLong_AsUnsignedLongLongMask(a[4]);
  n->kind = (int)PyLong_AsLong(a[5]);
  return true;
}

bool modes_active() {
  return c10::impl::TorchDispatchModeTLS::any_modes_set() || at::impl::torch_function_mode_enabled();
}

// Allocations of a call.  With nothing in the thread's dispatch state that wants to see them (a tracer, a transform, a
// profiler) they go to the device's kernel directly: a step of 2 heads x 128 tokens makes six of them, and the way there
// through the dispatcher, and through empty_like's choice of a layout, took 0.6 of its 14.4 us (both ways in alternating
// blocks of one process, whose medians vary by 0.1 us; from process to process a pass varies by 1 us).
class Allocator {
 public:
  explicit Allocator(const at::Tensor& like)
      : direct_((c10::impl::tls_local_dispatch_key_set().included_ - c10::default_included_set).empty() &&
                !at::hasCallbacks()),
        like_(like) {}
  at::Tensor contiguous(at::IntArrayRef sizes, at::ScalarType st) const {
    if (!direct_) return at::empty(sizes, like_.options().dtype(st));
    return at::_ops::empty_memory_format::redispatch(c10::DispatchKeySet(c10::DispatchKey::CUDA),
                                                     c10::fromIntArrayRefSlow(sizes), st, c10::Layout::Strided,
                                                     like_.device(), std::nullopt, std::nullopt);
  }
  // sizes, type, layout and names of `t`, as torch.empty_like
  at::Tensor same(const at::Tensor& t) const {
    if (t.has_names()) return at::empty_like(t);
    int64_t stride = 1;
    for (int i = 3; i >= 0; stride *= t.size(i--))
      if (t.stride(i) != stride || t.size(i) < 1) return at::empty_like(t);
    return contiguous(t.sizes(), t.scalar_type());
  }

 private:
  const bool direct_;
  const at::Tensor& like_;
};

// Sizes of the problem as ints and its dtype; false if they do not fit.
struct Sizes {
  int B, H, Nq, Nk, d;
  spark_dtype_t code;
};
bool sizes(const at::Tensor& Q, const at::Tensor& K, int kind, Sizes* s) {
  for (int i = 0; i < 4; ++i)
    if (Q.size(i) > INT_MAX) return false;
  if (K.size(2) > INT_MAX || (kind == SELF && K.size(2) != Q.size(2))) return false;
  if (Q.scalar_type() != at::kHalf && Q.scalar_type() != at::kBFloat16) return false;
  *s = Sizes{(int)Q.size(0), (int)Q.size(1), (int)Q.size(2), (int)K.size(2), (int)Q.size(3),
             Q.scalar_type() == at::kHalf ? SPARK_F16 : SPARK_BF16};
  return true;
}

// fwd(Q, K, V, O | None, LSE | None, scale, causal, p_drop, seed, offset, kind)
//   -> (O, LSE), a status other than 0, or None (not taken)
PyObject* host_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Numbers x;
  Sizes s;
  if (n != 11 || !get_device || !numbers(a + 5, &x) || modes_active()) Py_RETURN_NONE;
  const at::Tensor *Q = plain(a[0], 4), *K = plain(a[1], 4), *V = plain(a[2], 4);
  if (!Q || !K || !V || !sizes(*Q, *K, x.kind, &s)) Py_RETURN_NONE;
  const at::ScalarType st = Q->scalar_type();
  if (!shaped(*Q, st, s.B, s.H, s.Nq, s.d, x.kind) || !shaped(*K, st, s.B, s.H, s.Nk, s.d, x.kind) ||
      !shaped(*V, st, s.B, s.H, s.Nk, s.d, x.kind))
    Py_RETURN_NONE;
  const at::Tensor* Og = a[3] == Py_None ? nullptr : plain(a[3], 4);
  const at::Tensor* Lg = a[4] == Py_None ? nullptr : plain(a[4], 3);
  if ((a[3] != Py_None && (!Og || !shaped(*Og, st, s.B, s.H, s.Nq, s.d, x.kind))) ||
      (a[4] != Py_None && (!Lg || !stats_shaped(*Lg, s.B, s.H, s.Nq))))
    Py_RETURN_NONE;
  const Allocator fresh(*Q);
  const at::Tensor O = Og ? *Og : fresh.same(*Q);
  const at::Tensor L = Lg ? *Lg : fresh.contiguous({s.B, s.H, s.Nq}, at::kFloat);
  const size_t need = spark_mha_fwd_workspace_bytes(s.B, s.H, s.Nq, s.Nk, s.d, x.causal, s.code);
  at::Tensor ws;
  if (need) ws = fresh.contiguous({(int64_t)need}, at::kByte);
  const void *q = Q->data_ptr(), *k = K->data_ptr(), *v = V->data_ptr();
  void *o = O.data_ptr(), *work = need ? ws.data_ptr() : nullptr;
  float* lse = static_cast<float*>(L.data_ptr());
  void* stream;
  if (!current_stream(&stream)) return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS;
  const spark_strides_t sq = strides(*Q, x.kind), sk = strides(*K, x.kind), sv = strides(*V, x.kind),
                        so = strides(O, x.kind);
  rc = spark_mha_workspace_fwd(q, k, v, o, lse, &sq, &sk, &sv, &so, work, need, s.B, s.H, s.Nq, s.Nk, s.d, x.scale,
                               x.causal, x.p_drop, x.seed, x.offset, s.code, stream);
  Py_END_ALLOW_THREADS;
  if (rc != SPARK_OK) return PyLong_FromLong(rc);
  PyObject* out = PyTuple_New(2);
  if (!out) return nullptr;
  PyTuple_SET_ITEM(out, 0, THPVariable_Wrap(O));
  PyTuple_SET_ITEM(out, 1, THPVariable_Wrap(L));
  return out;
  END_HANDLE_TH_ERRORS
}

// bwd(Q, K, V, O, LSE, dO, dQ | None, dK | None, dV | None, scale, causal, p_drop, seed, offset, kind)
//   -> (dQ, dK, dV), a status other than 0, or None (not taken)
PyObject* host_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Numbers x;
  Sizes s;
  if (n != 15 || !get_device || !numbers(a + 9, &x) || modes_active()) Py_RETURN_NONE;
  const at::Tensor *Q = plain(a[0], 4), *K = plain(a[1], 4), *V = plain(a[2], 4), *O = plain(a[3], 4),
                   *L = plain(a[4], 3), *dO = plain(a[5], 4);
  if (!Q || !K || !V || !O || !L || !dO || !sizes(*Q, *K, x.kind, &s)) Py_RETURN_NONE;
  const at::ScalarType st = Q->scalar_type();
  auto q_like = [&](const at::Tensor& t) { return shaped(t, st, s.B, s.H, s.Nq, s.d, x.kind); };
  auto k_like = [&](const at::Tensor& t) { return shaped(t, st, s.B, s.H, s.Nk, s.d, x.kind); };
  if (!q_like(*Q) || !q_like(*O) || !q_like(*dO) || !k_like(*K) || !k_like(*V) || !stats_shaped(*L, s.B, s.H, s.Nq))
    Py_RETURN_NONE;
  const at::Tensor* given[3];
  for (int i = 0; i < 3; ++i) {
    given[i] = a[6 + i] == Py_None ? nullptr : plain(a[6 + i], 4);
    if (a[6 + i] != Py_None && (!given[i] || !(i == 0 ? q_like(*given[i]) : k_like(*given[i])))) Py_RETURN_NONE;
  }
  const size_t need = spark_mha_cross_bwd_workspace_bytes(s.B, s.H, s.Nq, s.Nk, s.d, s.code);
  const Allocator fresh(*Q);
  const at::Tensor dQ = given[0] ? *given[0] : fresh.same(*Q), dK = given[1] ? *given[1] : fresh.same(*K),
                   dV = given[2] ? *given[2] : fresh.same(*V);
  const int64_t wbytes = need > 16 ? (int64_t)need : 16;
  const at::Tensor ws = fresh.contiguous({wbytes}, at::kByte);
  const void *q = Q->data_ptr(), *k = K->data_ptr(), *v = V->data_ptr(), *o = O->data_ptr(), *dout = dO->data_ptr();
  const float* lse = static_cast<const float*>(L->data_ptr());
  void *dq = dQ.data_ptr(), *dk = dK.data_ptr(), *dv = dV.data_ptr(), *work = ws.data_ptr();
  void* stream;
  if (!current_stream(&stream)) return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS;
  if (x.kind == STRIDED) {
    const int st4 = STRIDED;
    const spark_strides_t sq = strides(*Q, st4), sk = strides(*K, st4), sv = strides(*V, st4), so = strides(*O, st4),
                          sdo = strides(*dO, st4), sdq = strides(dQ, st4), sdk = strides(dK, st4),
                          sdv = strides(dV, st4);
    rc = spark_mha_strided_bwd(q, k, v, o, lse, dout, dq, dk, dv, &sq, &sk, &sv, &so, &sdo, &sdq, &sdk, &sdv, work,
                               (size_t)wbytes, s.B, s.H, s.Nq, s.Nk, s.d, x.scale, x.causal, x.p_drop, x.seed, x.offset,
                               s.code, stream);
  } else {
    rc = spark_mha_dropout_bwd(q, k, v, o, lse, dout, dq, dk, dv, work, (size_t)wbytes, s.B, s.H, s.Nq, s.Nk, s.d,
                               x.scale, x.causal, x.p_drop, x.seed, x.offset, s.code, stream);
  }
  Py_END_ALLOW_THREADS;
  if (rc != SPARK_OK) return PyLong_FromLong(rc);
  PyObject* out = PyTuple_New(3);
  if (!out) return nullptr;
  PyTuple_SET_ITEM(out, 0, THPVariable_Wrap(dQ));
  PyTuple_SET_ITEM(out, 1, THPVariable_Wrap(dK));
  PyTuple_SET_ITEM(out, 2, THPVariable_Wrap(dV));
  return out;
  END_HANDLE_TH_ERRORS
}

// bind(get_device, get_raw_stream)
PyObject* host_bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 2 || !PyCallable_Check(a[0]) || !PyCallable_Check(a[1])) {
    PyErr_SetString(PyExc_TypeError, "bind(get_device, get_raw_stream)");
    return nullptr;
  }
  Py_INCREF(a[0]);
  Py_INCREF(a[1]);
  Py_XSETREF(get_device, a[0]);
  Py_XSETREF(get_raw_stream, a[1]);
  Py_RETURN_NONE;
}

#define SPARK_FASTCALL(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(f)), METH_FASTCALL
PyMethodDef methods[] = {
    {"bind", SPARK_FASTCALL(host_bind), "the two torch functions that name the current stream"},
    {"fwd", SPARK_FASTCALL(host_fwd), "forward"},
    {"bwd", SPARK_FASTCALL(host_bwd), "backward"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_spark_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__spark_host() { return PyModule_Create(&module); }
