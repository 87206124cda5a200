// Argument marshalling of the hot entry points, as a CPython extension (module _call).
//
// A short clip's step is eight small calls and a generated token one call per layer: the GPU needs 3-15 us for each,
// and marshalling them through Python and ctypes took the host 11-12 us per call (tensor attributes one by one, the
// stream object, eleven ctypes conversions), so the host, not the GPU, set the time.  Here a call reads its tensors
// through at::Tensor and asks c10 for the current stream.  A refused tensor raises the type and text that the binding's
// own checks raise (TypeError; AssertionError for the fp32 and int32 ones, here with a text), an exception of torch's
// C++ code the type that torch's Python functions raise for it (OutOfMemoryError, IndexError, ...).  The C ABI's functions
// are called through pointers handed over by the binding (`bind`), so that whatever library it loaded is the one that
// runs.  The GIL is released around every C call, as ctypes does.
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/device_lazy_init.h>

#include <algorithm>
#include <cstring>
#include <exception>
#include <new>
#include <sstream>
#include <string>
#include <utility>
#include <vector>

#include "purekv.h"

namespace {

// The C ABI, in the order `bind` receives the addresses.
struct Abi {
  decltype(&purekv_workspace_bytes) workspace_bytes;
  decltype(&purekv_workspace_init) workspace_init;
  decltype(&purekv_st_spattn_prefill) prefill;
  decltype(&purekv_st_spattn_prefill_vnorm) prefill_vnorm;
  decltype(&purekv_lowlayer_importance) importance;
  decltype(&purekv_topk_select) topk_select;
  decltype(&purekv_kv_compact) kv_compact;
  decltype(&purekv_kv_append) kv_append;
  decltype(&purekv_decode_attn) decode_attn;
  decltype(&purekv_decode_step) decode_step;
};
constexpr Py_ssize_t kAbiFunctions = sizeof(Abi) / sizeof(void*);
Abi abi{};
PyObject* raise_status = nullptr;   // the binding's check(status, where): raises PureKVError

// A Python error is set.
struct Raised {};

[[noreturn]] void raise(PyObject* type, const std::string& what) {
  PyErr_SetString(type, what.c_str());
  throw Raised{};
}

// Device scratch of one plan: one buffer per (operation, stream), kept for the plan's life.  Calls on one stream are
// ordered and may share a buffer; another stream gets its own.
struct Workspace {
  int op;
  hipStream_t stream;
  at::Tensor t;
};

struct PlanObject {
  PyObject_HEAD
  purekv_plan_t* plan;
  int64_t Hq, Hkv, N, d;
  int64_t q_st[2], kv_st[2], o_st[2];
  std::vector<Workspace>* ws;
};

PlanObject* as_plan(PyObject* o);

// torch's own initialisation comes first, as in torch.cuda.current_stream(): it refuses, with a RuntimeError, a process
// without a GPU and one that was forked after its parent had initialised the GPU.
hipStream_t current_stream() {
  torch::utils::device_lazy_init(at::kCUDA);
  return c10::hip::getCurrentHIPStream().stream();
}

bool is_none(PyObject* o) { return o == Py_None; }

const at::Tensor& tensor(PyObject* o, const char* name) {
  if (!THPVariable_Check(o)) raise(PyExc_TypeError, std::string(name) + " must be a tensor");
  return THPVariable_Unpack(o);
}

int32_t integer(PyObject* o) {
  const long x = PyLong_AsLong(o);
  if (x == -1 && PyErr_Occurred()) throw Raised{};
  if (x != (long)(int32_t)x) raise(PyExc_OverflowError, "integer argument out of range");
  return (int32_t)x;
}

// A contiguous bf16 device tensor.
const at::Tensor& dev_bf16(PyObject* o, const char* name) {
  const at::Tensor& t = tensor(o, name);
  if (!t.is_cuda() || t.scalar_type() != at::kBFloat16 || !t.is_contiguous())
    raise(PyExc_TypeError, std::string(name) + " must be a contiguous bf16 device tensor");
  return t;
}

void print(std::ostream& s, at::IntArrayRef x) {   // as Python prints a tuple
  s << '(';
  for (size_t i = 0; i < x.size(); ++i) s << (i ? ", " : "") << x[i];
  s << (x.size() == 1 ? ",)" : ")");
}

// A (..., heads, n, d) bf16 device view with the given head and token strides and contiguous channels.
const at::Tensor& strided_bf16(PyObject* o, const char* name, int64_t heads, int64_t n, int64_t d, const int64_t* st) {
  const at::Tensor& t = tensor(o, name);
  if (!t.is_cuda() || t.scalar_type() != at::kBFloat16) raise(PyExc_TypeError, std::string(name) + " must be a bf16 device tensor");
  const auto size = t.sizes(), stride = t.strides();
  const size_t r = size.size();
  if (r < 3 || size[r - 3] != heads || size[r - 2] != n || size[r - 1] != d || stride[r - 1] != 1 ||
      stride[r - 3] != st[0] || stride[r - 2] != st[1]) {
    std::ostringstream s;
    s << name << ": shape ";
    print(s, size);
    s << " / strides ";
    print(s, stride);
    s << " do not match the plan ((" << heads << ", " << n << ", " << d << "), head stride " << st[0] << ", token stride "
      << st[1] << ", channel stride 1)";
    raise(PyExc_TypeError, s.str());
  }
  return t;
}

const at::Tensor& dense_of(PyObject* o, const char* name, at::ScalarType type, const char* type_name) {
  const at::Tensor& t = tensor(o, name);
  if (!t.is_cuda() || t.scalar_type() != type || !t.is_contiguous())
    raise(PyExc_AssertionError, std::string(name) + " must be a contiguous " + type_name + " device tensor");
  return t;
}

// Owned reference to the caller's tensor, or to a new one made by `make` when the caller passed None.
template <class F>
PyObject* given_or(PyObject* o, F make) {
  if (is_none(o)) return THPVariable_Wrap(make());
  Py_INCREF(o);
  return o;
}

struct Ref {   // owns one reference
  PyObject* o;
  explicit Ref(PyObject* x) : o(x) {
    if (o == nullptr) throw Raised{};
  }
  Ref(const Ref&) = delete;
  ~Ref() { Py_XDECREF(o); }
  PyObject* release() { return std::exchange(o, nullptr); }
};

void* ptr(PyObject* o, const char* name) { return is_none(o) ? nullptr : tensor(o, name).data_ptr(); }

template <class F, class... A>
int unlocked(F f, A... args) {
  int rc;
  Py_BEGIN_ALLOW_THREADS rc = f(args...);
  Py_END_ALLOW_THREADS return rc;
}

void check(int status, const char* where) {
  if (status == PUREKV_OK) return;
  PyObject* r = PyObject_CallFunction(raise_status, "is", status, where);
  Py_XDECREF(r);
  if (r != nullptr) PyErr_SetString(PyExc_RuntimeError, where);
  throw Raised{};
}

Workspace* find_workspace(PlanObject* p, int op, hipStream_t stream) {
  for (Workspace& x : *p->ws)
    if (x.op == op && x.stream == stream) return &x;
  return nullptr;
}

// The plan's scratch for `op` on `stream` (undefined if it needs none); a fresh buffer goes through purekv_workspace_init
// once.  The caller holds the buffer until its launch is queued: while it is without the GIL, a call of another thread
// that needs a larger one may replace it in the list.
at::Tensor workspace(PlanObject* p, int op, hipStream_t stream, size_t nbytes, const at::Device& device, int32_t n_layers,
                     int32_t w, int32_t cap) {
  if (nbytes == 0) return {};
  if (const Workspace* x = find_workspace(p, op, stream))
    if ((size_t)x->t.numel() >= nbytes && x->t.device() == device) return x->t;
  at::Tensor t = at::empty({(int64_t)nbytes}, at::TensorOptions().dtype(at::kByte).device(device));
  check(abi.workspace_init(p->plan, op, t.data_ptr(), nbytes, n_layers, w, cap, stream), "purekv_workspace_init");
  // The allocation may have run Python code (a dispatch mode sees it), and with it other calls on this plan: the entry
  // is looked up again, the list may have moved.
  if (Workspace* x = find_workspace(p, op, stream)) x->t = t;
  else p->ws->push_back({op, stream, t});
  return t;
}

void* address(const at::Tensor& ws) { return ws.defined() ? ws.data_ptr() : nullptr; }

at::TensorOptions like(const at::Tensor& t, at::ScalarType type) { return at::TensorOptions().dtype(type).device(t.device()); }

// ---- entry points: (plan, arguments of the Python function in order) -----------------------------------------------

PyObject* prefill(PlanObject* p, PyObject* const* a) {   // q, k, v, out, want_lse, lse, vnorm2
  const at::Tensor& q = strided_bf16(a[0], "q", p->Hq, p->N, p->d, p->q_st);
  const at::Tensor& k = strided_bf16(a[1], "k", p->Hkv, p->N, p->d, p->kv_st);
  const at::Tensor& v = strided_bf16(a[2], "v", p->Hkv, p->N, p->d, p->kv_st);
  Ref out(given_or(a[3], [&] {
    const int64_t span = (p->Hq - 1) * p->o_st[0] + (p->N - 1) * p->o_st[1] + p->d;
    return at::empty({span}, like(q, at::kBFloat16)).as_strided({p->Hq, p->N, p->d}, {p->o_st[0], p->o_st[1], 1});
  }));
  void* const o = strided_bf16(out.o, "out", p->Hq, p->N, p->d, p->o_st).data_ptr();
  const int want = PyObject_IsTrue(a[4]);
  if (want < 0) throw Raised{};
  Ref lse(want && is_none(a[5]) ? THPVariable_Wrap(at::empty({p->Hq, p->N}, like(q, at::kFloat))) : Py_NewRef(a[5]));
  float* const l = static_cast<float*>(ptr(lse.o, "lse"));
  hipStream_t st = current_stream();
  const size_t nb = abi.workspace_bytes(p->plan, PUREKV_OP_PREFILL, 0, 0, 0);
  const at::Tensor ws = workspace(p, PUREKV_OP_PREFILL, st, nb, q.device(), 0, 0, 0);
  if (is_none(a[6])) {
    check(unlocked(abi.prefill, p->plan, q.data_ptr(), k.data_ptr(), v.data_ptr(), o, l, address(ws), nb, (void*)st),
          "purekv_st_spattn_prefill");
  } else {
    const at::Tensor& n2 = dense_of(a[6], "vnorm2", at::kFloat, "fp32");
    if (n2.dim() != 2 || n2.size(0) != p->Hkv || n2.size(1) != p->N) raise(PyExc_AssertionError, "vnorm2 must be [Hkv, N]");
    check(unlocked(abi.prefill_vnorm, p->plan, q.data_ptr(), k.data_ptr(), v.data_ptr(), o, l,
                   static_cast<float*>(n2.data_ptr()), address(ws), nb, (void*)st),
          "purekv_st_spattn_prefill_vnorm");
  }
  return is_none(lse.o) ? out.release() : PyTuple_Pack(2, out.o, lse.o);
}

PyObject* importance(PlanObject* p, PyObject* const* a) {   // q, k, lse, w, c_out
  const at::Tensor& q = strided_bf16(a[0], "q", p->Hq, p->N, p->d, p->q_st);
  const at::Tensor& k = strided_bf16(a[1], "k", p->Hkv, p->N, p->d, p->kv_st);
  const at::Tensor& lse = dense_of(a[2], "lse", at::kFloat, "fp32");
  if (lse.dim() != 2 || lse.size(0) != p->Hq || lse.size(1) != p->N) raise(PyExc_AssertionError, "lse must be [Hq, N]");
  const int32_t w = integer(a[3]);
  Ref c(given_or(a[4], [&] { return at::empty({p->Hkv, std::max<int64_t>(p->N - w, 0)}, like(q, at::kFloat)); }));
  check(unlocked(abi.importance, p->plan, q.data_ptr(), k.data_ptr(), static_cast<float*>(lse.data_ptr()), w,
                 static_cast<float*>(ptr(c.o, "c_out")), (void*)nullptr, (size_t)0, (void*)current_stream()),
        "purekv_lowlayer_importance");
  return c.release();
}

// The layer axis of an optional leading dimension is taken off again for callers whose tensors have none.
PyObject* without_layer_axis(PyObject* o, bool layered) {
  if (layered) return Py_NewRef(o);
  return THPVariable_Wrap(THPVariable_Unpack(o).select(0, 0));
}

PyObject* topk_select(PlanObject* p, PyObject* const* a) {   // c, v, w, h, want_scores, idx_out
  const at::Tensor& c = dense_of(a[0], "c", at::kFloat, "fp32");
  const at::Tensor* v = is_none(a[1]) ? nullptr : &strided_bf16(a[1], "v", p->Hkv, p->N, p->d, p->kv_st);
  const int32_t w = integer(a[2]), h = integer(a[3]);
  const bool layered = v != nullptr && v->dim() == 4;
  const int64_t n_layers = layered ? v->size(0) : 1, stride = layered ? v->stride(0) : 0;
  Ref idx(given_or(a[5], [&] { return at::empty({n_layers, p->Hkv, (int64_t)h + w}, like(c, at::kInt)); }));
  const int want = PyObject_IsTrue(a[4]);
  if (want < 0) throw Raised{};
  Ref s(want ? THPVariable_Wrap(at::empty({n_layers, p->Hkv, p->N - w}, like(c, at::kFloat))) : Py_NewRef(Py_None));
  hipStream_t st = current_stream();
  const size_t nb = v != nullptr && !want ? abi.workspace_bytes(p->plan, PUREKV_OP_TOPK, (int32_t)n_layers, w, 0) : 0;
  const at::Tensor ws = workspace(p, PUREKV_OP_TOPK, st, nb, c.device(), (int32_t)n_layers, w, 0);
  check(unlocked(abi.topk_select, p->plan, static_cast<float*>(c.data_ptr()), v != nullptr ? v->data_ptr() : nullptr,
                 stride, (int32_t)n_layers, w, h, static_cast<int32_t*>(ptr(idx.o, "idx_out")),
                 static_cast<float*>(ptr(s.o, "scores")), address(ws), nb, (void*)st),
        "purekv_topk_select");
  Ref i(without_layer_axis(idx.o, layered));
  if (!want) return i.release();
  Ref sc(without_layer_axis(s.o, layered));
  return PyTuple_Pack(2, i.o, sc.o);
}

PyObject* kv_compact(PlanObject* p, PyObject* const* a) {   // k, v, idx, cap, kc, vc
  const at::Tensor& k = strided_bf16(a[0], "k", p->Hkv, p->N, p->d, p->kv_st);
  const at::Tensor& v = strided_bf16(a[1], "v", p->Hkv, p->N, p->d, p->kv_st);
  const at::Tensor& idx = dense_of(a[2], "idx", at::kInt, "int32");
  const bool layered = k.dim() == 4;
  const int64_t n_layers = layered ? k.size(0) : 1, stride = layered ? k.stride(0) : 0;
  if (layered && (v.dim() != 4 || v.stride(0) != stride)) raise(PyExc_AssertionError, "k and v must share their layer stride");
  const int64_t n_keep = idx.size(-1);
  const int32_t cap = is_none(a[3]) ? (int32_t)n_keep : integer(a[3]);
  auto cache = [&] {
    return layered ? at::empty({n_layers, p->Hkv, cap, p->d}, like(k, at::kBFloat16))
                   : at::empty({p->Hkv, cap, p->d}, like(k, at::kBFloat16));
  };
  Ref kc(given_or(a[4], cache)), vc(given_or(a[5], cache));
  check(unlocked(abi.kv_compact, p->plan, k.data_ptr(), v.data_ptr(), stride, (int32_t)n_layers,
                 static_cast<int32_t*>(idx.data_ptr()), (int32_t)n_keep, ptr(kc.o, "kc"), ptr(vc.o, "vc"), cap,
                 (void*)current_stream()),
        "purekv_kv_compact");
  return PyTuple_Pack(2, kc.o, vc.o);
}

PyObject* kv_append(PlanObject* p, PyObject* const* a) {   // k_new, v_new, kc, vc, n_cached
  const at::Tensor &k = dev_bf16(a[0], "k_new"), &v = dev_bf16(a[1], "v_new"), &kc = dev_bf16(a[2], "kc"), &vc = dev_bf16(a[3], "vc");
  const int32_t n = integer(a[4]);
  check(unlocked(abi.kv_append, p->plan, k.data_ptr(), v.data_ptr(), kc.data_ptr(), vc.data_ptr(), n,
                 (int32_t)kc.size(-2), (void*)current_stream()),
        "purekv_kv_append");
  return PyLong_FromLong((long)n + 1);
}

// q_new, kc, vc, n_cached, out
PyObject* decode_attn(PlanObject* p, PyObject* const* a) {
  const at::Tensor &q = dev_bf16(a[0], "q_new"), &kc = dev_bf16(a[1], "kc"), &vc = dev_bf16(a[2], "vc");
  const int32_t n = integer(a[3]), cap = (int32_t)kc.size(-2);
  Ref out(given_or(a[4], [&] { return at::empty_like(q); }));
  hipStream_t st = current_stream();
  const size_t nb = abi.workspace_bytes(p->plan, PUREKV_OP_DECODE, 0, 0, cap);
  const at::Tensor ws = workspace(p, PUREKV_OP_DECODE, st, nb, q.device(), 0, 0, cap);
  check(unlocked(abi.decode_attn, p->plan, q.data_ptr(), kc.data_ptr(), vc.data_ptr(), n, cap, ptr(out.o, "out"), address(ws),
                 nb, (void*)st),
        "purekv_decode_attn");
  return out.release();
}

// q_new, k_new, v_new, kc, vc, n_cached, out
PyObject* decode_step(PlanObject* p, PyObject* const* a) {
  const at::Tensor &q = dev_bf16(a[0], "q_new"), &k = dev_bf16(a[1], "k_new"), &v = dev_bf16(a[2], "v_new"),
                   &kc = dev_bf16(a[3], "kc"), &vc = dev_bf16(a[4], "vc");
  const int32_t n = integer(a[5]), cap = (int32_t)kc.size(-2);
  Ref out(given_or(a[6], [&] { return at::empty_like(q); }));
  hipStream_t st = current_stream();
  const size_t nb = abi.workspace_bytes(p->plan, PUREKV_OP_DECODE, 0, 0, cap);
  const at::Tensor ws = workspace(p, PUREKV_OP_DECODE, st, nb, q.device(), 0, 0, cap);
  check(unlocked(abi.decode_step, p->plan, q.data_ptr(), k.data_ptr(), v.data_ptr(), kc.data_ptr(), vc.data_ptr(), n, cap,
                 ptr(out.o, "out"), address(ws), nb, (void*)st),
        "purekv_decode_step");
  return out.release();
}

// ---- module --------------------------------------------------------------------------------------------------------

template <class F>
PyObject* guarded(F f) {
  try {
    return f();
  } catch (const Raised&) {
  } catch (const std::exception&) {
    torch::translate_exception_to_python(std::current_exception());
  }
  return nullptr;
}

template <PyObject* (*Fn)(PlanObject*, PyObject* const*), int Args>
PyObject* entry(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != Args + 1) {
    PyErr_Format(PyExc_TypeError, "%d arguments expected", Args + 1);
    return nullptr;
  }
  return guarded([&] { return Fn(as_plan(a[0]), a + 1); });
}

PyObject* bind(PyObject*, PyObject* args) {   // bind(addresses, check)
  PyObject *addresses, *fn;
  if (!PyArg_ParseTuple(args, "O!O", &PyTuple_Type, &addresses, &fn)) return nullptr;
  if (PyTuple_GET_SIZE(addresses) != kAbiFunctions) {
    PyErr_SetString(PyExc_TypeError, "one address per C function expected");
    return nullptr;
  }
  void* f[kAbiFunctions];
  for (Py_ssize_t i = 0; i < kAbiFunctions; ++i) {
    f[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(addresses, i));
    if (f[i] == nullptr) return PyErr_Occurred() ? nullptr : (PyErr_SetString(PyExc_ValueError, "null address"), nullptr);
  }
  std::memcpy(&abi, f, sizeof(abi));
  Py_INCREF(fn);
  Py_XSETREF(raise_status, fn);
  Py_RETURN_NONE;
}

PyObject* plan_new(PyTypeObject* type, PyObject* args, PyObject*) {
  // Plan(handle, Hq, Hkv, N, d, (q strides), (kv strides), (o strides))
  unsigned long long handle;
  long long Hq, Hkv, N, d, q0, q1, kv0, kv1, o0, o1;
  if (!PyArg_ParseTuple(args, "KLLLL(LL)(LL)(LL)", &handle, &Hq, &Hkv, &N, &d, &q0, &q1, &kv0, &kv1, &o0, &o1)) return nullptr;
  auto* p = reinterpret_cast<PlanObject*>(type->tp_alloc(type, 0));
  if (p == nullptr) return nullptr;
  p->plan = reinterpret_cast<purekv_plan_t*>(static_cast<uintptr_t>(handle));
  p->Hq = Hq, p->Hkv = Hkv, p->N = N, p->d = d;
  p->q_st[0] = q0, p->q_st[1] = q1, p->kv_st[0] = kv0, p->kv_st[1] = kv1, p->o_st[0] = o0, p->o_st[1] = o1;
  p->ws = new (std::nothrow) std::vector<Workspace>();
  if (p->ws == nullptr) {
    Py_DECREF(p);
    return PyErr_NoMemory();
  }
  return reinterpret_cast<PyObject*>(p);
}

void plan_dealloc(PyObject* o) {
  delete reinterpret_cast<PlanObject*>(o)->ws;
  Py_TYPE(o)->tp_free(o);
}

PyObject* plan_close(PyObject* o, PyObject*) {   // the plan itself belongs to the binding
  auto* p = reinterpret_cast<PlanObject*>(o);
  p->plan = nullptr;
  p->ws->clear();
  Py_RETURN_NONE;
}

PyObject* plan_workspace(PyObject* o, PyObject* args) {   // workspace(op, nbytes, tensor on the device, n_layers, w, cap) -> buffer or None
  int op, n_layers, w, cap;
  unsigned long long nbytes;
  PyObject* t;
  if (!PyArg_ParseTuple(args, "iKOiii", &op, &nbytes, &t, &n_layers, &w, &cap)) return nullptr;
  return guarded([&]() -> PyObject* {
    const at::Tensor ws = workspace(reinterpret_cast<PlanObject*>(o), op, current_stream(), (size_t)nbytes,
                               tensor(t, "tensor").device(), n_layers, w, cap);
    return ws.defined() ? THPVariable_Wrap(ws) : Py_NewRef(Py_None);
  });
}

PyMethodDef plan_methods[] = {{"close", plan_close, METH_NOARGS, nullptr},
                              {"workspace", plan_workspace, METH_VARARGS, nullptr},
                              {nullptr, nullptr, 0, nullptr}};

PyTypeObject plan_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

PlanObject* as_plan(PyObject* o) {
  if (Py_TYPE(o) != &plan_type) raise(PyExc_TypeError, "a plan is expected");
  return reinterpret_cast<PlanObject*>(o);
}

PyObject* stream(PyObject*, PyObject*) {
  return guarded([] { return PyLong_FromVoidPtr(current_stream()); });
}

template <PyObject* (*Fn)(PlanObject*, PyObject* const*), int Args>
PyCFunction fast() {
  return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<Fn, Args>));
}

PyMethodDef methods[] = {{"bind", bind, METH_VARARGS, nullptr},
                         {"stream", stream, METH_NOARGS, "address of the current stream"},
                         {"prefill", fast<prefill, 7>(), METH_FASTCALL, nullptr},
                         {"importance", fast<importance, 5>(), METH_FASTCALL, nullptr},
                         {"topk_select", fast<topk_select, 6>(), METH_FASTCALL, nullptr},
                         {"kv_compact", fast<kv_compact, 6>(), METH_FASTCALL, nullptr},
                         {"kv_append", fast<kv_append, 5>(), METH_FASTCALL, nullptr},
                         {"decode_attn", fast<decode_attn, 5>(), METH_FASTCALL, nullptr},
                         {"decode_step", fast<decode_step, 7>(), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", "Argument marshalling of the hot entry points.", -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__call() {
  plan_type.tp_name = "paper_2510_25600_amd._call.Plan";
  plan_type.tp_basicsize = sizeof(PlanObject);
  plan_type.tp_flags = Py_TPFLAGS_DEFAULT;
  plan_type.tp_new = plan_new;
  plan_type.tp_dealloc = plan_dealloc;
  plan_type.tp_methods = plan_methods;
  if (PyType_Ready(&plan_type) < 0) return nullptr;
  PyObject* m = PyModule_Create(&module);
  if (m == nullptr) return nullptr;
  Py_INCREF(&plan_type);
  if (PyModule_AddObject(m, "Plan", reinterpret_cast<PyObject*>(&plan_type)) < 0) return nullptr;
  return m;
}
