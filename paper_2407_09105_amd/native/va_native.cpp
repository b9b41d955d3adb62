// The calls of `binding` that a training step makes per layer, without their Python: the checks, the output allocations and
// the library call of one pass in one C++ call each.
//
// A pass over 16 tokens (boundaries, forward, backward: four kernels of 3 to 6 us) took 38 us of host time: 14 us for the
// launches themselves, the rest in Python checks, seven torch.empty of 1.3 us and ctypes calls of up to 21 arguments.
//
// Each function handles the plain case - exact torch.Tensor arguments that satisfy every check of its counterpart in
// binding.py, outputs not given - and returns None for anything else before it has done anything; the caller then goes on
// in Python, where every error is raised.  Tensors are allocated in the same order, by the same operators, and the library is
// reached through the addresses of the C functions that binding.py loaded.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/python_headers.h>
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>

#include <algorithm>

#include "varlen_attn.h"

namespace {

struct Library {
  decltype(&va_plan_bytes) plan_bytes;
  decltype(&va_segments_bind) segments_bind;
  decltype(&va_pack_to_cu_seqlens) pack;
  decltype(&va_attn_workspace_bytes) workspace_bytes;
  decltype(&va_varlen_attn_fwd) fwd;
  decltype(&va_varlen_attn_bwd) bwd;
};
Library lib = {};

// Other Python threads run while a tensor is allocated (which can wait for the GPU) and kernels are launched (which can wait
// for room in their queue), as they do around torch's own allocations and around ctypes calls.  A 16-token pass takes 23.0 us
// with it and without.
struct WithoutGil {
  PyThreadState *state = PyEval_SaveThread();
  ~WithoutGil() { PyEval_RestoreThread(state); }
};

template <class F> void set_address(F &f, PyObject *address) { f = (F)PyLong_AsVoidPtr(address); }

// The tensor behind `x`, or nullptr where it is no plain one that lives contiguously on the GPU, or where a mode asks to see
// the Python calls that create tensors.
const at::Tensor *plain(PyObject *x) {
  if (!THPVariable_CheckExact(x) || at::impl::torch_function_mode_enabled()) return nullptr;
  const at::Tensor &t = THPVariable_Unpack(x);
  return t.layout() == at::kStrided && t.is_cuda() && t.is_contiguous() ? &t : nullptr;
}

int element_type(at::ScalarType t) {
  return t == at::kFloat ? VA_F32 : t == at::kBFloat16 ? VA_BF16 : t == at::kHalf ? VA_F16 : -1;
}

struct Sizes {
  int64_t n, hq, hkv, d;
};
// Q [N, Hq, d], K and V [N, Hkv, d] of one element type the library has, for a stream of rows * T tokens
bool sizes(const at::Tensor *q, const at::Tensor *k, const at::Tensor *v, int64_t tokens, Sizes &s) {
  if (!q || !k || !v || q->dim() != 3 || k->dim() != 3 || v->sizes() != k->sizes()) return false;
  s = {q->size(0), q->size(1), k->size(1), q->size(2)};
  return k->size(0) == s.n && k->size(2) == s.d && s.n == tokens && q->scalar_type() == k->scalar_type() &&
         q->scalar_type() == v->scalar_type() && element_type(q->scalar_type()) >= 0;
}

// connect(plan_bytes, segments_bind, pack, workspace_bytes, fwd, bwd): addresses of the library's functions
PyObject *connect(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 6) return PyErr_Format(PyExc_TypeError, "connect takes 6 addresses");
  set_address(lib.plan_bytes, a[0]);
  set_address(lib.segments_bind, a[1]);
  set_address(lib.pack, a[2]);
  set_address(lib.workspace_bytes, a[3]);
  set_address(lib.fwd, a[4]);
  set_address(lib.bwd, a[5]);
  if (PyErr_Occurred()) return nullptr;
  Py_RETURN_NONE;
}

// pack(position_ids, address of a va_segments, stream) -> (rows, tokens_per_row, plan) | status | None
PyObject *pack(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  const at::Tensor *pos = n == 3 ? plain(a[0]) : nullptr;
  if (!pos || pos->dim() != 2 || (pos->scalar_type() != at::kLong && pos->scalar_type() != at::kInt)) Py_RETURN_NONE;
  const int64_t rows = pos->size(0), T = pos->size(1);
  if (rows <= 0 || T <= 0 || rows >= INT32_MAX || T >= INT32_MAX) Py_RETURN_NONE;
  va_segments *seg = (va_segments *)PyLong_AsVoidPtr(a[1]);
  void *stream = PyLong_AsVoidPtr(a[2]);
  if (PyErr_Occurred()) return nullptr;
  const size_t bytes = lib.plan_bytes((int32_t)rows, (int32_t)T);
  if (bytes == 0) Py_RETURN_NONE;
  at::Tensor plan;
  va_status bound, s = VA_OK;
  {
    WithoutGil free;
    plan = at::empty({(int64_t)(bytes / 4)}, pos->options().dtype(at::kInt));
    bound = lib.segments_bind(plan.data_ptr(), bytes, (int32_t)rows, (int32_t)T, seg);
    if (bound == VA_OK)
      s = lib.pack(pos->data_ptr(), pos->scalar_type() == at::kLong ? VA_I64 : VA_I32, (int32_t)rows, (int32_t)T, seg, stream);
  }
  if (bound != VA_OK) Py_RETURN_NONE;
  if (s != VA_OK) return PyLong_FromLong(s);
  return Py_BuildValue("LLN", (long long)rows, (long long)T, THPVariable_Wrap(std::move(plan)));
  END_HANDLE_TH_ERRORS
}

// fwd(q, k, v, address of the va_segments, rows, tokens_per_row, softmax_scale, stream) -> (o, lse) | status | None
PyObject *fwd(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 8) Py_RETURN_NONE;
  const va_segments *seg = (const va_segments *)PyLong_AsVoidPtr(a[3]);
  const int64_t rows = PyLong_AsLongLong(a[4]), T = PyLong_AsLongLong(a[5]);
  const float scale = (float)PyFloat_AsDouble(a[6]);
  void *stream = PyLong_AsVoidPtr(a[7]);
  if (PyErr_Occurred()) return nullptr;
  const at::Tensor *q = plain(a[0]), *k = plain(a[1]), *v = plain(a[2]);
  Sizes s;
  if (!sizes(q, k, v, rows * T, s)) Py_RETURN_NONE;
  at::Tensor o, lse;
  va_status status;
  {
    WithoutGil free;
    o = at::empty_like(*q), lse = at::empty({s.hq, s.n}, q->options().dtype(at::kFloat));
    status = lib.fwd(q->data_ptr(), k->data_ptr(), v->data_ptr(), o.data_ptr(), (float *)lse.data_ptr(), seg, (int32_t)rows,
                     (int32_t)T, (int32_t)s.hq, (int32_t)s.hkv, (int32_t)s.d, (va_dtype)element_type(q->scalar_type()), scale, nullptr,
                     0, stream);
  }
  if (status != VA_OK) return PyLong_FromLong(status);
  return Py_BuildValue("NN", THPVariable_Wrap(std::move(o)), THPVariable_Wrap(std::move(lse)));
  END_HANDLE_TH_ERRORS
}

// bwd(do, q, k, v, o, lse, address of the va_segments, rows, tokens_per_row, softmax_scale, gradients in float32, stream)
// -> (dq, dk, dv) | status | None.  Gradients in float32, or else in the inputs' type.
PyObject *bwd(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 12) Py_RETURN_NONE;
  const va_segments *seg = (const va_segments *)PyLong_AsVoidPtr(a[6]);
  const int64_t rows = PyLong_AsLongLong(a[7]), T = PyLong_AsLongLong(a[8]);
  const float scale = (float)PyFloat_AsDouble(a[9]);
  const bool f32_grads = a[10] == Py_True;
  void *stream = PyLong_AsVoidPtr(a[11]);
  if (PyErr_Occurred()) return nullptr;
  const at::Tensor *g = plain(a[0]), *q = plain(a[1]), *k = plain(a[2]), *v = plain(a[3]), *o = plain(a[4]), *lse = plain(a[5]);
  Sizes s;
  if (!g || !o || !lse || !sizes(q, k, v, rows * T, s) || g->scalar_type() != q->scalar_type() || o->scalar_type() != q->scalar_type() ||
      lse->scalar_type() != at::kFloat || lse->sizes() != at::IntArrayRef({s.hq, s.n}) || g->numel() < q->numel() || o->numel() < q->numel())
    Py_RETURN_NONE;
  const at::TensorOptions like = q->options(), grads = f32_grads ? like.dtype(at::kFloat) : like;
  at::Tensor dq, dk, dv;
  va_status status;
  {
    WithoutGil free;
    dq = at::empty(q->sizes(), grads), dk = at::empty(k->sizes(), grads), dv = at::empty(v->sizes(), grads);
    const size_t bytes = lib.workspace_bytes((int32_t)s.n, (int32_t)s.hq, (int32_t)s.hkv, (int32_t)s.d, 1);
    const int64_t floats = (int64_t)(std::max<size_t>(bytes, 4) / 4);
    at::Tensor ws = at::empty({floats}, like.dtype(at::kFloat));
    status = lib.bwd(g->data_ptr(), q->data_ptr(), k->data_ptr(), v->data_ptr(), o->data_ptr(), (const float *)lse->data_ptr(),
                     dq.data_ptr(), dk.data_ptr(), dv.data_ptr(), f32_grads ? VA_F32 : (va_dtype)element_type(q->scalar_type()), seg,
                     (int32_t)rows, (int32_t)T, (int32_t)s.hq, (int32_t)s.hkv, (int32_t)s.d, (va_dtype)element_type(q->scalar_type()),
                     scale, ws.data_ptr(), (size_t)floats * 4, stream);
  }
  if (status != VA_OK) return PyLong_FromLong(status);
  return Py_BuildValue("NNN", THPVariable_Wrap(std::move(dq)), THPVariable_Wrap(std::move(dk)), THPVariable_Wrap(std::move(dv)));
  END_HANDLE_TH_ERRORS
}

#define VA_METHOD(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {VA_METHOD(connect), VA_METHOD(pack), VA_METHOD(fwd), VA_METHOD(bwd), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_va_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__va_native() {
  PyObject *m = PyModule_Create(&module);
  // the torch whose headers this was compiled with: objects of another one may lie differently in memory
  if (m && PyModule_AddStringConstant(m, "torch_version", VA_TORCH_VERSION) < 0) Py_CLEAR(m);
  return m;
}
