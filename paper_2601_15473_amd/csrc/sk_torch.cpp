// The PyTorch layers' autograd functions in native code: what nn.py's SKLinearFunction and
// SKLinearTwoSidedFunction do, for the calls that need nothing of Python.
//
// A small layer's step is host time (64 tokens, 256 -> 256, R = 16, fp32: 134 us through the Python
// functions, 67 here; a sentence of 131 tokens through 768 -> 3072, R = 128, 16.5 : 9.0), most of it
// interpreting the two functions and marshalling their arguments.  Here a forward pass is one call
// from Python and a backward pass none.  `linear` and `linear_two_sided` return None for whatever they
// do not take -- subclasses of Tensor, functorch transforms, dispatch and function modes, tracing,
// forward-mode gradients, arguments that are to be refused -- and the Python functions go on from there.
#include <Python.h>

#include <dlfcn.h>
#include <stdlib.h>

#include <list>
#include <mutex>
#include <string>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/DeviceGuard.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/pybind.h>

#define __HIP_PLATFORM_AMD__ 1
#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>

#include "../../include/sk.h"

namespace {

using at::Tensor;
using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

// One scratch buffer per (device, stream), grown to the largest request; the least recently used of more
// than MAX_STREAMS goes back to the allocator, which keeps it until the work queued on it is done.
// Calls queue their kernels under the lock: two threads that share a stream share its buffer.
struct Workspaces {
  static constexpr size_t MAX_STREAMS = 8;
  // Most that a pass keeps here beside its workspace: an allocation a pass is 1 us of host, 1 to 2 % of a small two-sided layer's step, and the sums
  // of a large one (4096 -> 11008, 2048 columns: 107 MB) would stay on every stream.
  static constexpr size_t MAX_SUMS = 4 << 20;
  struct Entry {
    c10::DeviceIndex device;
    void* stream;
    Tensor buffer;
  };
  std::mutex mutex;
  std::list<Entry> entries;   // most recently used first

  const Tensor& get(const at::Device& device, void* stream, size_t bytes) {   // (with the lock held)
    auto it = entries.begin();
    while (it != entries.end() && !(it->device == device.index() && it->stream == stream)) ++it;
    if (it == entries.end()) entries.push_front(Entry{device.index(), stream, Tensor()});
    else if (it != entries.begin()) entries.splice(entries.begin(), entries, it);
    Entry& e = entries.front();
    if (!e.buffer.defined() || (size_t)e.buffer.numel() < bytes)
      e.buffer = at::empty({(int64_t)(bytes < 256 ? 256 : bytes)}, at::TensorOptions().dtype(at::kByte).device(device));
    if (entries.size() > MAX_STREAMS) entries.pop_back();
    return e.buffer;
  }
};
// (never destroyed: the allocator may be gone before this library's own destructors run)
Workspaces& workspaces() {
  static Workspaces* w = new Workspaces;
  return *w;
}

sk_dtype dtype_of(const Tensor& t) { return t.scalar_type() == at::kFloat ? SK_F32 : SK_BF16; }

void* stream_of(const at::Device& device) {
  return static_cast<hipStream_t>(c10::hip::getCurrentHIPStreamMasqueradingAsCUDA(device.index()).stream());
}

PyObject* g_error = nullptr;   // libsk.SkError, which nn.py hands over

// As libsk.check: raises SkError with its status.  (Not under the workspaces' lock: it takes the GIL and runs Python.)
void check(sk_status s) {
  if (s == SK_OK) return;
  pybind11::gil_scoped_acquire gil;
  PyObject* const e = g_error != nullptr ? PyObject_CallFunction(g_error, "i", (int)s) : nullptr;
  if (e != nullptr) {
    PyErr_SetObject(g_error, e);
    Py_DECREF(e);
  } else if (!PyErr_Occurred()) {
    PyErr_SetString(PyExc_RuntimeError, sk_status_string(s));
  }
  python_error error;
  error.persist();   // (a backward pass is on another thread than its caller)
  throw error;
}

Tensor rows(const Tensor& x, int64_t width) {
  if (x.dim() == 2 && x.is_contiguous()) return x;
  return x.reshape({-1, width}).contiguous();
}

// What the first pass leaves for the second beside its tensors: x's shape where that is not the rows'
// own, and l and k, with the bias in the sign.
void keep(AutogradContext* ctx, const Tensor& x, int64_t l, int64_t k, bool bias) {
  ctx->saved_data["lk"] = (l << 32 | k) * (bias ? 1 : -1);
  if (x.dim() != 2) ctx->saved_data["shape"] = x.sizes().vec();
}
struct Kept {
  int32_t l, k;
  bool bias;
  explicit Kept(AutogradContext* ctx) {
    const int64_t lk = ctx->saved_data["lk"].toInt();
    bias = lk > 0;
    l = (int32_t)((bias ? lk : -lk) >> 32);
    k = (int32_t)((bias ? lk : -lk) & 0xffffffff);
  }
};
Tensor in_shape(AutogradContext* ctx, const Tensor& dX) {
  const auto it = ctx->saved_data.find("shape");
  return it == ctx->saved_data.end() || !dX.defined() ? dX : dX.reshape(it->second.toIntVector());
}

Tensor forward_pass(const Tensor& x, const Tensor& x2, const Tensor& S, const Tensor& U, const std::optional<Tensor>& bias, int32_t l, int32_t k) {
  const int64_t tokens = x2.size(0), in = x2.size(1), out = U.size(1);
  const sk_dtype dt = dtype_of(S);
  const c10::DeviceGuard guard(x2.device());
  Tensor y = at::empty({tokens, out}, x2.options());
  void* const stream = stream_of(x2.device());
  const size_t need = sk_linear_workspace_bytes(SK_OP_FWD, tokens, in, out, l, k, dt);
  Workspaces& w = workspaces();
  sk_status st;
  {
    const std::lock_guard<std::mutex> lock(w.mutex);
    const Tensor& ws = w.get(x2.device(), stream, need);
    st = sk_linear_fwd(x2.data_ptr(), S.data_ptr(), U.data_ptr(), bias.has_value() ? bias->data_ptr() : nullptr, y.data_ptr(), tokens, in,
                       out, l, k, dt, ws.data_ptr(), (size_t)ws.numel(), stream);
  }
  check(st);
  if (x.dim() == 2) return y;
  std::vector<int64_t> shape = x.sizes().vec();
  shape.back() = out;
  return y.reshape(shape);
}

Tensor rows_of_gradient(const Tensor& g, const Tensor& like, int64_t width) {
  TORCH_CHECK(g.is_cuda(), "SKLinear: the gradient of y is on ", g.device(), "; libsk runs on the GPU only");
  return rows(g.scalar_type() == like.scalar_type() ? g : g.to(like.scalar_type()), width);
}

// fp32 gradients in the layer's type, each a tensor of its own, in one launch
struct Rounding {
  const float* from[3];
  void* to[3];
  int64_t n[3];
  int count = 0;
  Tensor add(const Tensor& g, const at::TensorOptions& options) {
    Tensor t = at::empty(g.sizes(), options);
    from[count] = g.data_ptr<float>(); to[count] = t.data_ptr(); n[count] = g.numel();
    ++count;
    return t;
  }
};

struct Linear : torch::autograd::Function<Linear> {
  static Tensor forward(AutogradContext* ctx, const Tensor& x, const Tensor& S, const Tensor& U, const std::optional<Tensor>& bias, int64_t l, int64_t k) {
    const Tensor x2 = rows(x, S.size(0));
    const Tensor y = forward_pass(x, x2, S, U, bias, (int32_t)l, (int32_t)k);
    ctx->save_for_backward({x2, S, U});
    keep(ctx, x, l, k, bias.has_value());
    return y;
  }

  static variable_list backward(AutogradContext* ctx, variable_list grads) {
    const variable_list saved = ctx->get_saved_variables();
    const Tensor &x2 = saved[0], &S = saved[1], &U = saved[2];
    const Kept kept(ctx);
    const int64_t tokens = x2.size(0), in = x2.size(1), out = U.size(1);
    const sk_dtype dt = dtype_of(S);
    const bool need_dx = ctx->needs_input_grad(0), need_du = ctx->needs_input_grad(2), need_db = kept.bias && ctx->needs_input_grad(3);
    const bool need_w = need_du || need_db;
    Tensor dX, dU, db;
    if (need_dx || need_w) {
      const c10::DeviceGuard guard(x2.device());
      const Tensor dY = rows_of_gradient(grads[0], S, out);
      const auto f32 = x2.options().dtype(at::kFloat);
      if (need_dx) dX = at::empty({tokens, in}, x2.options());
      if (need_w) {
        dU = at::empty({U.size(0), out}, f32);
        if (kept.bias) db = at::empty({out}, f32);
      }
      Rounding round;
      Tensor dU_out = dU, db_out = db;
      if (dt != SK_F32) {
        if (need_du) dU_out = round.add(dU, U.options());
        if (need_db) db_out = round.add(db, U.options());
      }
      void* const stream = stream_of(x2.device());
      const size_t need = sk_linear_workspace_bytes(SK_OP_BWD, tokens, in, out, kept.l, kept.k, dt);
      float* const du = need_w ? dU.data_ptr<float>() : nullptr;
      float* const dbias = db.defined() ? db.data_ptr<float>() : nullptr;
      Workspaces& w = workspaces();
      sk_status st;
      {
        const std::lock_guard<std::mutex> lock(w.mutex);
        const Tensor& ws = w.get(x2.device(), stream, need);
        void* const wp = ws.data_ptr();
        const size_t wn = (size_t)ws.numel();
        if (need_dx && need_w && round.count > 0)
          st = sk_linear_bwd_rounded(x2.data_ptr(), dY.data_ptr(), S.data_ptr(), U.data_ptr(), dX.data_ptr(), du, dbias, nullptr,
                                     need_du ? dU_out.data_ptr() : nullptr, U.size(0), need_db ? db_out.data_ptr() : nullptr, nullptr, tokens, in, out, kept.l,
                                     kept.k, dt, wp, wn, stream);
        else if (need_dx && need_w)
          st = sk_linear_bwd(x2.data_ptr(), dY.data_ptr(), S.data_ptr(), U.data_ptr(), dX.data_ptr(), du, dbias, tokens, in, out, kept.l,
                             kept.k, dt, wp, wn, stream);
        else if (need_dx)
          st = sk_linear_bwd_input(dY.data_ptr(), S.data_ptr(), U.data_ptr(), dX.data_ptr(), tokens, in, out, kept.l, kept.k, dt, wp, wn, stream);
        else
          st = sk_linear_bwd_weight(x2.data_ptr(), S.data_ptr(), dY.data_ptr(), du, dbias, tokens, in, out, kept.l, kept.k, dt, wp, wn, stream);
        if (st == SK_OK && round.count > 0 && !need_dx) st = sk_round_gradients(round.from, round.to, round.n, round.count, stream);
      }
      check(st);
      dU = need_du ? dU_out : Tensor();
      db = need_db ? db_out : Tensor();
    }
    return {in_shape(ctx, dX), Tensor(), dU, db, Tensor(), Tensor()};
  }
};

// x, U1, U2, bias, then A = [S1 | U2] and B = [U1 ; S2^T] (nn.py keeps those two), which the passes run on; l: terms per side
struct LinearTwoSided : torch::autograd::Function<LinearTwoSided> {
  static Tensor forward(AutogradContext* ctx, const Tensor& x, const Tensor& U1, const Tensor& U2, const std::optional<Tensor>& bias, const Tensor& A,
                        const Tensor& B, int64_t l, int64_t k) {
    const Tensor x2 = rows(x, A.size(0));
    const Tensor y = forward_pass(x, x2, A, B, bias, (int32_t)(2 * l), (int32_t)k);
    ctx->save_for_backward({x2, A, B});
    keep(ctx, x, l, k, bias.has_value());
    return y;
  }

  static variable_list backward(AutogradContext* ctx, variable_list grads) {
    const variable_list saved = ctx->get_saved_variables();
    const Tensor &x2 = saved[0], &A = saved[1], &B = saved[2];
    const Kept kept(ctx);
    const int64_t tokens = x2.size(0), in = x2.size(1), out = B.size(1), half = B.size(0) / 2;
    const sk_dtype dt = dtype_of(A);
    const c10::DeviceGuard guard(x2.device());
    const Tensor dY = rows_of_gradient(grads[0], A, out);
    // (rows half .. of B's gradient belong to S2^T, fixed numbers: formed by the product, given to nobody)
    Tensor dX = at::empty({tokens, in}, x2.options()), dA, dB, db;
    void* const stream = stream_of(x2.device());
    const int32_t l2 = 2 * kept.l;
    const size_t need = sk_linear_workspace_bytes(SK_OP_BWD_TWO_SIDED, tokens, in, out, l2, kept.k, dt);
    Workspaces& w = workspaces();
    sk_status st;
    const auto f32 = x2.options().dtype(at::kFloat);
    if (dt != SK_F32) {   // results each a tensor of its own; their fp32 sums behind the workspace while they are small, else in one that goes back with the pass
      dB = at::empty({half, out}, A.options());
      dA = at::empty({in, half}, A.options());
      if (kept.bias) db = at::empty({out}, A.options());
      const int64_t sums = 2 * half * out + in * half + out;
      const bool behind = (size_t)sums * 4 <= Workspaces::MAX_SUMS;
      const Tensor own = behind ? Tensor() : at::empty({sums}, f32);
      const size_t at_sums = (need + 255) / 256 * 256;
      const std::lock_guard<std::mutex> lock(w.mutex);
      unsigned char* const ws = static_cast<unsigned char*>(w.get(x2.device(), stream, behind ? at_sums + (size_t)sums * 4 : need).data_ptr());
      float* const sum_dB = behind ? reinterpret_cast<float*>(ws + at_sums) : own.data_ptr<float>();
      float* const sum_dA = sum_dB + 2 * half * out;
      st = sk_linear_bwd_rounded(x2.data_ptr(), dY.data_ptr(), A.data_ptr(), B.data_ptr(), dX.data_ptr(), sum_dB, kept.bias ? sum_dA + in * half : nullptr, sum_dA,
                                 dB.data_ptr(), half, kept.bias ? db.data_ptr() : nullptr, dA.data_ptr(), tokens, in, out, l2, kept.k, dt, ws, need, stream);
    } else {
      const Tensor whole = at::empty({2 * half, out}, f32);
      dA = at::empty({in, half}, f32);
      dB = whole.narrow(0, 0, half);
      if (kept.bias) db = at::empty({out}, f32);
      const std::lock_guard<std::mutex> lock(w.mutex);
      const Tensor& ws = w.get(x2.device(), stream, need);
      st = sk_linear_bwd_two_sided(x2.data_ptr(), dY.data_ptr(), A.data_ptr(), B.data_ptr(), dX.data_ptr(), whole.data_ptr<float>(),
                                   kept.bias ? db.data_ptr<float>() : nullptr, dA.data_ptr<float>(), tokens, in, out, l2, kept.k, dt, ws.data_ptr(),
                                   (size_t)ws.numel(), stream);
    }
    check(st);
    return {in_shape(ctx, dX), dB, dA, db, Tensor(), Tensor(), Tensor(), Tensor()};
  }
};

PyTypeObject* g_parameter = nullptr;   // torch.nn.Parameter

// A plain tensor or parameter on `device` (any, if null) with the given type and dense rows
const Tensor* plain(PyObject* o) {
  PyTypeObject* const type = Py_TYPE(o);
  if (type != reinterpret_cast<PyTypeObject*>(THPVariableClass) && type != g_parameter) return nullptr;
  const Tensor& t = THPVariable_Unpack(o);
  return t.defined() && t.is_cuda() && t.layout() == at::kStrided && !t.is_conj() && !t.is_neg() ? &t : nullptr;
}

// Nothing is watching that the native functions would pass by.
bool unwatched() {
  using at::DispatchKey;
  for (DispatchKey k : {DispatchKey::FuncTorchDynamicLayerFrontMode, DispatchKey::FuncTorchDynamicLayerBackMode, DispatchKey::Tracer, DispatchKey::Functionalize})
    if (c10::impl::tls_is_dispatch_key_included(k)) return false;
  return !c10::impl::TorchDispatchModeTLS::any_modes_set() && !at::impl::torch_function_mode_enabled();
}
bool no_tangent(const Tensor& t) { return !t._fw_grad(0).defined(); }

// Tensors of one layer: of x's type and device, without forward-mode gradients
bool same(const Tensor& x, const Tensor& t) { return t.scalar_type() == x.scalar_type() && t.device() == x.device() && no_tangent(t); }
bool takes(const Tensor& x, int64_t in, int64_t out, int64_t l, int64_t k) {
  if ((x.scalar_type() != at::kFloat && x.scalar_type() != at::kBFloat16) || x.dim() < 1 || x.size(-1) != in || x.numel() == 0 || !no_tangent(x)) return false;
  if (l < 1 || k < 1 || l > INT32_MAX / 2 || k > INT32_MAX) return false;
  return sk_linear_workspace_bytes(SK_OP_FWD, x.numel() / in, in, out, (int32_t)l, (int32_t)k, dtype_of(x)) != (size_t)-1;
}
bool aligned(const Tensor& t) { return (reinterpret_cast<uintptr_t>(t.data_ptr()) & 15) == 0; }

PyObject* linear(PyObject*, PyObject* const* a, Py_ssize_t n) {   // x, S, U, bias or None, l, k
  HANDLE_TH_ERRORS
  if (n != 6 || !PyLong_Check(a[4]) || !PyLong_Check(a[5]) || !unwatched()) Py_RETURN_NONE;
  const Tensor *x = plain(a[0]), *S = plain(a[1]), *U = plain(a[2]), *b = a[3] == Py_None ? nullptr : plain(a[3]);
  if (!x || !S || !U || (a[3] != Py_None && !b)) Py_RETURN_NONE;
  const int64_t l = PyLong_AsLongLong(a[4]), k = PyLong_AsLongLong(a[5]);
  if (PyErr_Occurred()) { PyErr_Clear(); Py_RETURN_NONE; }
  if (S->dim() != 2 || U->dim() != 2 || !S->is_contiguous() || !U->is_contiguous() || U->size(0) != S->size(1) ||
      !takes(*x, S->size(0), U->size(1), l, k) || S->size(1) != l * k || !same(*x, *S) || !same(*x, *U) || !aligned(*x) || !aligned(*S) || !aligned(*U))
    Py_RETURN_NONE;
  if (b && (b->dim() != 1 || b->size(0) != U->size(1) || !b->is_contiguous() || !same(*x, *b) || !aligned(*b))) Py_RETURN_NONE;
  Tensor y;
  {
    pybind11::gil_scoped_release no_gil;
    const std::optional<Tensor> bias = b ? std::optional<Tensor>(*b) : std::nullopt;
    if (at::GradMode::is_enabled() && (x->requires_grad() || S->requires_grad() || U->requires_grad() || (b && b->requires_grad())))
      y = Linear::apply(*x, *S, *U, bias, l, k);
    else
      y = forward_pass(*x, rows(*x, S->size(0)), *S, *U, bias, (int32_t)l, (int32_t)k);
  }
  return THPVariable_Wrap(std::move(y));
  END_HANDLE_TH_ERRORS
}

PyObject* linear_two_sided(PyObject*, PyObject* const* a, Py_ssize_t n) {   // x, S1, U1, U2, S2^T, bias or None, A, B, l, k
  HANDLE_TH_ERRORS
  if (n != 10 || !PyLong_Check(a[8]) || !PyLong_Check(a[9]) || !unwatched()) Py_RETURN_NONE;
  const Tensor* t[8];
  for (int i = 0; i < 8; ++i) {
    t[i] = i == 5 && a[i] == Py_None ? nullptr : plain(a[i]);
    if (!t[i] && !(i == 5 && a[i] == Py_None)) Py_RETURN_NONE;
  }
  const Tensor &x = *t[0], &S1 = *t[1], &U1 = *t[2], &U2 = *t[3], &S2T = *t[4], &A = *t[6], &B = *t[7];
  const int64_t l = PyLong_AsLongLong(a[8]), k = PyLong_AsLongLong(a[9]);
  if (PyErr_Occurred()) { PyErr_Clear(); Py_RETURN_NONE; }
  for (int i = 1; i < 8; ++i)
    if (t[i] && (t[i]->dim() != (i == 5 ? 1 : 2) || !same(x, *t[i]))) Py_RETURN_NONE;
  const int64_t in = S1.size(0), half = S1.size(1), out = U1.size(1);
  if (l < 1 || k < 1 || half != l * k || U1.size(0) != half || U2.size(0) != in || U2.size(1) != half || S2T.size(0) != half || S2T.size(1) != out ||
      A.size(0) != in || A.size(1) != 2 * half || B.size(0) != 2 * half || B.size(1) != out || (t[5] && (t[5]->size(0) != out || !t[5]->is_contiguous())) ||
      !A.is_contiguous() || !B.is_contiguous() || !takes(x, in, out, 2 * l, k) || half % 16 != 0 || !aligned(x) || !aligned(A) || !aligned(B) || (t[5] && !aligned(*t[5])))
    Py_RETURN_NONE;
  Tensor y;
  {
    pybind11::gil_scoped_release no_gil;
    y = LinearTwoSided::apply(x, U1, U2, t[5] ? std::optional<Tensor>(*t[5]) : std::nullopt, A, B, l, k);
  }
  return THPVariable_Wrap(std::move(y));
  END_HANDLE_TH_ERRORS
}

PyObject* release_workspaces(PyObject*, PyObject*) {
  HANDLE_TH_ERRORS
  {
    pybind11::gil_scoped_release no_gil;
    Workspaces& w = workspaces();
    const std::lock_guard<std::mutex> lock(w.mutex);
    w.entries.clear();
  }
  Py_RETURN_NONE;
  END_HANDLE_TH_ERRORS
}

PyObject* raise_as(PyObject*, PyObject* type) {
  Py_INCREF(type);
  Py_XDECREF(g_error);
  g_error = type;
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"linear", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(linear)), METH_FASTCALL, "y, or None for a call it does not take"},
    {"linear_two_sided", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(linear_two_sided)), METH_FASTCALL, "y, or None for a call it does not take"},
    {"raise_as", raise_as, METH_O, "the exception type of a refused call, made from its status"},
    {"release_workspaces", release_workspaces, METH_NOARGS, "gives the scratch buffers back to the allocator"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_sktorch", "libsk under autograd, in native code", -1, methods, nullptr, nullptr, nullptr, nullptr};

// The folder of the file that `address` was loaded from, without links.
std::string folder_of(const void* address) {
  Dl_info info;
  char* const path = dladdr(address, &info) != 0 && info.dli_fname != nullptr ? realpath(info.dli_fname, nullptr) : nullptr;
  const std::string s = path != nullptr ? path : "";
  free(path);
  return s.substr(0, s.rfind('/') + 1);
}

}  // namespace

PyMODINIT_FUNC PyInit__sktorch() {
  // (the loader takes a libsk.so that the process has already, say of another copy of this package)
  const std::string here = folder_of(&module), sk = folder_of(reinterpret_cast<const void*>(&sk_linear_fwd));
  if (here != sk) {
    PyErr_Format(PyExc_ImportError, "%s_sktorch.so is bound to %slibsk.so, not to the one beside it", here.c_str(), sk.c_str());
    return nullptr;
  }
  // (torch's C++ layouts change from one version to the next, also where every symbol is still there)
  const std::string version = SK_TORCH_VERSION;
  PyObject* const torch = PyImport_ImportModule("torch");
  PyObject* const got = torch != nullptr ? PyObject_GetAttrString(torch, "__version__") : nullptr;
  Py_XDECREF(torch);
  if (got == nullptr) return nullptr;
  const char* const now = PyUnicode_AsUTF8(got);
  if (now == nullptr || now != version) {
    if (now != nullptr) PyErr_Format(PyExc_ImportError, "_sktorch.so was built for PyTorch %s, this is %s", version.c_str(), now);
    Py_DECREF(got);
    return nullptr;
  }
  Py_DECREF(got);
  PyObject* const nn = PyImport_ImportModule("torch.nn");
  if (nn == nullptr) return nullptr;
  g_parameter = reinterpret_cast<PyTypeObject*>(PyObject_GetAttrString(nn, "Parameter"));   // (kept for good)
  Py_DECREF(nn);
  return g_parameter == nullptr ? nullptr : PyModule_Create(&module);
}
