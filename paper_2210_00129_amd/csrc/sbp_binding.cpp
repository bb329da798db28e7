// The calls of a layer's every step - draw, cache, linear backward - between Python and the C ABI, in native code: checks of the
// tensors, allocation of the outputs and the workspace, the current stream, the call.  A small layer is bound by the host: its three
// calls (64 -> 256 channels on two 14 x 14 maps, fp32) took 28.7 us, of which the three C calls, a kernel launch each, are 12; seven
// torch.empty calls at 1.4 us and the argument marshalling of ctypes were most of the rest.
// The C functions come as addresses from the package's loaded libsbp.so (bind), so this module has no library of its own to find.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/DynamicTypes.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/device_lazy_init.h>

#include "sbp.h"

namespace {

decltype(&sbp_keep_count) f_keep_count = nullptr;
decltype(&sbp_sample_indices) f_sample = nullptr;
decltype(&sbp_forward_cache) f_cache = nullptr;
decltype(&sbp_backward_linear_workspace) f_workspace = nullptr;
decltype(&sbp_backward_linear) f_linear = nullptr;
PyObject* f_check = nullptr;          // _lib.check: raises for a negative status
PyObject* f_stream = nullptr;         // device index -> handle of torch's current stream there

struct PyFail {};                     // a Python error is set

[[noreturn]] void fail(PyObject* type, const char* fmt, const char* what) {
  PyErr_Format(type, fmt, what);
  throw PyFail{};
}

// the tensor of an argument, or nullptr for None
const at::Tensor* tensor(PyObject* o, const char* name) {
  if (o == Py_None) return nullptr;
  if (!THPVariable_Check(o)) fail(PyExc_TypeError, "%s must be a tensor", name);
  return &THPVariable_Unpack(o);
}
const at::Tensor& needed(PyObject* o, const char* name) {
  const at::Tensor* t = tensor(o, name);
  if (!t) fail(PyExc_TypeError, "%s must be a tensor", name);
  return *t;
}

void* dev(const at::Tensor* t, const char* name) {
  if (!t) return nullptr;
  if (!t->is_cuda()) fail(PyExc_ValueError, "%s must live in GPU memory", name);
  if (!t->is_contiguous()) fail(PyExc_ValueError, "%s must be contiguous", name);
  return t->data_ptr();
}

int32_t dtype_code(const at::Tensor& t) {
  if (t.scalar_type() == at::kFloat) return SBP_F32;
  if (t.scalar_type() == at::kBFloat16) return SBP_BF16;
  PyErr_Format(PyExc_TypeError, "unsupported dtype %S; use float32 or bfloat16", reinterpret_cast<PyObject*>(torch::getTHPDtype(t.scalar_type())));
  throw PyFail{};
}

// Other Python threads run while memory is allocated or work is enqueued (either may block).
struct WithoutGil {
  PyThreadState* state = PyEval_SaveThread();
  ~WithoutGil() { PyEval_RestoreThread(state); }
};

// as torch.empty: a process that has not used the GPU yet gets torch.cuda's initialization (and with it the fork check), a child
// forked from one that has gets torch's error
at::Tensor empty(at::IntArrayRef sizes, at::ScalarType type, c10::Device device) {
  if (device.is_cuda()) torch::utils::device_lazy_init(at::kCUDA);
  WithoutGil no_gil;
  return at::empty(sizes, at::TensorOptions().dtype(type).device(device));
}

void* stream_of(c10::Device device) {
  PyObject* index = PyLong_FromLong(device.index());
  if (!index) throw PyFail{};
  PyObject* h = PyObject_CallFunctionObjArgs(f_stream, index, nullptr);
  Py_DECREF(index);
  if (!h) throw PyFail{};
  void* s = PyLong_AsVoidPtr(h);
  Py_DECREF(h);
  if (!s && PyErr_Occurred()) throw PyFail{};
  return s;
}

void check(int64_t status) {
  if (status >= 0) return;
  PyObject* r = PyObject_CallFunction(f_check, "L", (long long)status);
  Py_XDECREF(r);
  if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, "libsbp call failed");
  throw PyFail{};
}

template <class F>
int32_t enqueue(F&& f) {
  WithoutGil no_gil;
  return f();
}

int64_t integer(PyObject* o, bool whole = false) {                   // whole: numbers that int() would round are refused
  PyObject* n = whole ? PyNumber_Index(o) : PyNumber_Long(o);
  if (!n) throw PyFail{};
  const long long v = PyLong_AsLongLong(n);
  Py_DECREF(n);
  if (v == -1 && PyErr_Occurred()) throw PyFail{};
  return v;
}
int32_t integer32(PyObject* o) { return (int32_t)integer(o); }       // (as a C int field takes it: the low 32 bits)
uint64_t bits64(PyObject* o, bool whole = false) {
  PyObject* n = whole ? PyNumber_Index(o) : PyNumber_Long(o);
  if (!n) throw PyFail{};
  const unsigned long long v = PyLong_AsUnsignedLongLongMask(n);
  Py_DECREF(n);
  if (v == (unsigned long long)-1 && PyErr_Occurred()) throw PyFail{};
  return v;
}

PyObject* wrap(const at::Tensor& t) { return THPVariable_Wrap(t); }
PyObject* keep_or_wrap(PyObject* given, const at::Tensor& made) {
  if (given != Py_None) { Py_INCREF(given); return given; }
  if (!made.defined()) Py_RETURN_NONE;
  return wrap(made);
}

PyObject* pack(std::initializer_list<PyObject*> items) {
  bool ok = true;
  for (PyObject* o : items) ok = ok && o;
  PyObject* r = ok ? PyTuple_New((Py_ssize_t)items.size()) : nullptr;
  Py_ssize_t i = 0;
  for (PyObject* o : items) {
    if (r) PyTuple_SET_ITEM(r, i++, o);
    else Py_XDECREF(o);
  }
  return r;
}

void count(Py_ssize_t n, Py_ssize_t want) {
  if (n != want) fail(PyExc_TypeError, "%s", "wrong number of arguments");
}

// (address of sbp_keep_count, sbp_sample_indices, sbp_forward_cache, sbp_backward_linear_workspace, sbp_backward_linear, check, stream)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  try {
    count(n, 7);
    f_keep_count = reinterpret_cast<decltype(f_keep_count)>(bits64(a[0]));
    f_sample = reinterpret_cast<decltype(f_sample)>(bits64(a[1]));
    f_cache = reinterpret_cast<decltype(f_cache)>(bits64(a[2]));
    f_workspace = reinterpret_cast<decltype(f_workspace)>(bits64(a[3]));
    f_linear = reinterpret_cast<decltype(f_linear)>(bits64(a[4]));
    Py_INCREF(a[5]);
    Py_XDECREF(f_check);
    f_check = a[5];
    Py_INCREF(a[6]);
    Py_XDECREF(f_stream);
    f_stream = a[6];
    Py_RETURN_NONE;
  } catch (const PyFail&) { return nullptr; }
}

// (B, P, H, W, cell, k, mode, per_sample, seed, stream_id, want_inv, device index, idx_out, inv_out) -> (idx, inv)
PyObject* sample_indices(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  try {
    count(n, 14);
    sbp_sample_desc d{};
    d.B = integer32(a[0]); d.P = integer32(a[1]); d.H = integer32(a[2]); d.W = integer32(a[3]);
    d.cell = integer32(a[4]); d.k = integer32(a[5]); d.mode = integer32(a[6]); d.per_sample = integer32(a[7]);
    d.seed = bits64(a[8]); d.stream_id = bits64(a[9]);
    const int64_t K = f_keep_count(&d);
    check(K);
    const c10::Device device(c10::DeviceType::CUDA, (c10::DeviceIndex)integer(a[11]));
    const at::Tensor *idx_out = tensor(a[12], "idx"), *inv_out = tensor(a[13], "inv");
    at::Tensor idx, inv;
    if (!idx_out) idx = empty({K}, at::kInt, device);
    const int want_inv = PyObject_IsTrue(a[10]);
    if (want_inv < 0) throw PyFail{};
    if (!inv_out && want_inv) inv = empty({(int64_t)d.B * (d.P + (int64_t)d.H * d.W)}, at::kInt, device);
    const at::Tensor& i = idx_out ? *idx_out : idx;
    void* const ip = dev(&i, "idx");
    void* const vp = dev(inv_out ? inv_out : (inv.defined() ? &inv : nullptr), "inv");
    void* const stream = stream_of(i.device());
    const int64_t capacity = i.numel();
    check(enqueue([&] { return f_sample(&d, static_cast<int32_t*>(ip), capacity, static_cast<int32_t*>(vp), stream); }));
    return pack({keep_or_wrap(a[12], idx), keep_or_wrap(a[13], inv)});
  } catch (const PyFail&) { return nullptr; }
  END_HANDLE_TH_ERRORS
}

// (X, idx, out) -> X_k
PyObject* forward_cache(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  try {
    count(n, 3);
    const at::Tensor &X = needed(a[0], "X"), &idx = needed(a[1], "idx");
    const at::Tensor* out = tensor(a[2], "X_k");
    if (X.dim() != 2) fail(PyExc_ValueError, "%s", "X must be [M, C]");
    const int64_t K = idx.numel();
    at::Tensor made;
    if (!out) made = empty({K, X.size(1)}, X.scalar_type(), X.device());
    void *const xp = dev(&X, "X"), *const ip = dev(&idx, "idx");
    const int32_t code = dtype_code(X);
    void *const op = dev(out ? out : &made, "X_k"), *const stream = stream_of(X.device());
    const int64_t M = X.size(0), C = X.size(1);
    check(enqueue([&] { return f_cache(xp, static_cast<const int32_t*>(ip), M, K, (int32_t)C, code, op, stream); }));
    return keep_or_wrap(a[2], made);
  } catch (const PyFail&) { return nullptr; }
  END_HANDLE_TH_ERRORS
}

// (dY, idx, X_k, W, M, flags, want (1 dW, 2 db, 4 dX), dW, db, dX, workspace, inv) -> (dW, db, dX)
PyObject* backward_linear(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  try {
    count(n, 12);
    const at::Tensor &dY = needed(a[0], "dY"), &W = needed(a[3], "W");
    const at::Tensor *idx = tensor(a[1], "idx"), *Xk = tensor(a[2], "X_k");
    const at::Tensor *dW = tensor(a[7], "dW"), *db = tensor(a[8], "db"), *dX = tensor(a[9], "dX"), *ws = tensor(a[10], "workspace"), *inv = tensor(a[11], "inv");
    if (W.dim() != 2) fail(PyExc_ValueError, "%s", "W must be [Cout, Cin]");
    const int64_t Cout = W.size(0), Cin = W.size(1);
    const uint32_t flags = (uint32_t)bits64(a[5], true), want = (uint32_t)integer(a[6]);
    if (!idx && dY.dim() < 1) fail(PyExc_ValueError, "%s", "dY must be [rows, Cout]");
    const int64_t K = idx ? idx->numel() : dY.size(0);
    int64_t M;
    if (a[4] != Py_None) M = integer(a[4], true);
    else {
      if (flags & SBP_FLAG_DY_COMPACT) fail(PyExc_ValueError, "%s", "M is required when dY is compact");
      if (dY.dim() < 1) fail(PyExc_ValueError, "%s", "dY must be [rows, Cout]");
      M = dY.size(0);
    }
    const int32_t code = dtype_code(W);
    const c10::Device device = W.device();
    const at::ScalarType dw_type = flags & SBP_FLAG_DW_OUT_BF16 ? at::kBFloat16 : at::kFloat;
    at::Tensor made_dW, made_db, made_dX, made_ws;
    if ((want & 1) && !dW) { made_dW = empty({Cout, Cin}, dw_type, device); dW = &made_dW; }
    if (dW && dW->scalar_type() != dw_type) fail(PyExc_ValueError, "%s", "dW must be bfloat16 with FLAG_DW_OUT_BF16 and float32 without");
    if ((want & 2) && !db) { made_db = empty({Cout}, at::kFloat, device); db = &made_db; }
    if ((want & 4) && !dX) { made_dX = empty({flags & SBP_FLAG_DX_COMPACT ? K : M, Cin}, W.scalar_type(), device); dX = &made_dX; }
    if (!ws) {
      const int64_t need = (int64_t)f_workspace(M, K, (int32_t)Cin, (int32_t)Cout, code, flags);
      made_ws = empty({std::max<int64_t>(need, 256)}, at::kByte, device);
      ws = &made_ws;
    }
    const void *const dYp = dev(&dY, "dY"), *const idxp = dev(idx, "idx"), *const invp = dev(inv, "inv"), *const Xkp = dev(Xk, "X_k"), *const Wp = dev(&W, "W");
    void *const dWp = dev(dW, "dW"), *const dbp = dev(db, "db"), *const dXp = dev(dX, "dX"), *const wsp = dev(ws, "workspace");
    void* const stream = stream_of(device);
    const size_t ws_bytes = (size_t)ws->numel();
    check(enqueue([&] {
      return f_linear(dYp, static_cast<const int32_t*>(idxp), static_cast<const int32_t*>(invp), Xkp, Wp, M, K, (int32_t)Cin, (int32_t)Cout, code, dWp,
                      static_cast<float*>(dbp), dXp, wsp, ws_bytes, flags, stream);
    }));
    return pack({keep_or_wrap(a[7], made_dW), keep_or_wrap(a[8], made_db), keep_or_wrap(a[9], made_dX)});
  } catch (const PyFail&) { return nullptr; }
  END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {{"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(bind)), METH_FASTCALL, nullptr},
                         {"sample_indices", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(sample_indices)), METH_FASTCALL, nullptr},
                         {"forward_cache", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(forward_cache)), METH_FASTCALL, nullptr},
                         {"backward_linear", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(backward_linear)), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
