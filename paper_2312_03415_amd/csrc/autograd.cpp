// The LoRA layer's autograd node in native code (host only): RunLoRAFunction of module.py without Python in its forward and
// backward.  Same buffers, same calls into librunlora, same results; what it saves is host time.
//
// A training pass of a small layer is bound by its host work: with the Python node, forward + backward of 256 x 768 -> 768
// fp32 take 102-189 us of host time a pass for 75 us of GPU work (forward 30; the backward's body alone 68, because the
// autograd engine runs it on a thread of its own, where every Python object it touches comes over from another core).  With
// this node the host takes 14 us for the forward and at most the GPU's time in all: 194 -> 88 us a pass; 1024 x 4096 -> 4096
// r 64 196 -> 114, 1237 x 2056 -> 5464 197 -> 122.
//
// lora(...) returns None where this node does not apply, and the caller then takes the Python node: tensor subclasses, torch
// function / dispatch modes, functorch transforms and tracing (all of which have to see a Python-level function), devices
// other than the current GPU, and operands that only the Python path's checks describe properly.  Forward-mode gradients are
// refused by either node, saved-tensor hooks apply to both (the same four tensors are saved in the same order).
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/DeviceGuard.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>
#include <torch/csrc/utils/pybind.h>

#include "../../include/runlora.h"

namespace {

// entry points of librunlora (already loaded by binding.py, which hands over the addresses) and binding._check
decltype(&runlora_forward) p_forward = nullptr;
decltype(&runlora_backward) p_backward = nullptr;
decltype(&runlora_call_workspace_bytes) p_workspace_bytes = nullptr;
PyObject* g_check = nullptr;

void check(int rc) {
  if (rc == RL_OK) return;
  pybind11::gil_scoped_acquire gil;
  PyObject* r = PyObject_CallFunction(g_check, "i", rc);  // raises RunLoRAError
  Py_XDECREF(r);
  if (r == nullptr) {
    python_error e;
    e.persist();
    throw std::move(e);
  }
}

int dtype_code(at::ScalarType t) {
  return t == at::kFloat ? RL_F32 : (t == at::kHalf ? RL_F16 : (t == at::kBFloat16 ? RL_BF16 : -1));
}

rl_tensor_t desc(const at::Tensor& t, int code) {
  return rl_tensor_t{t.data_ptr(), t.size(0), t.size(1), t.stride(0), code, nullptr, 0};
}

// a saved operand as the backward gets it back: a saved-tensor hook may have changed its type, layout or device, so that
// what held in the forward is checked again (types and sizes by the library, against the descriptor's own)
rl_tensor_t saved_desc(const at::Tensor& t, const at::Tensor& x) {
  TORCH_CHECK_VALUE(t.dim() == 2 && t.stride(1) == 1, "expected a 2-D tensor with contiguous rows");
  TORCH_CHECK_VALUE(t.device() == x.device(), "a saved tensor came back on another device: ", t.device(), ", not ", x.device());
  return desc(t, dtype_code(t.scalar_type()));
}

// rows as the library takes them (the same test as the Python node's)
at::Tensor rows(const at::Tensor& t, int64_t cols) {
  at::Tensor r = t.reshape({-1, cols});
  if (r.stride(-1) != 1 || r.stride(0) % 8 != 0 || reinterpret_cast<uintptr_t>(r.data_ptr()) % 16 != 0) r = r.contiguous();
  return r;
}

// scratch of one call, given back to the caching allocator behind it (stream-ordered like every tensor)
at::Tensor scratch(size_t bytes, const at::Tensor& like) {
  return at::empty({(int64_t)(bytes < 256 ? 256 : bytes)}, like.options().dtype(at::kByte));
}

struct LoRANode : public torch::autograd::Function<LoRANode> {
  static at::Tensor forward(torch::autograd::AutogradContext* ctx, const at::Tensor& x, const at::Tensor& W, const at::Tensor& A,
                            const at::Tensor& B, const std::optional<at::Tensor>& bias, double scale, int64_t fwd, int64_t bwd,
                            bool keep_merged, double dropout_p, int64_t dropout_seed, bool keep_t) {
    const int64_t i = W.size(0), o = W.size(1), r = A.size(1);
    const int code = dtype_code(x.scalar_type());
    const at::Tensor x2 = rows(x, i);
    const int64_t n = x2.size(0);
    at::Tensor y = at::empty({n, o}, x.options());
    rl_saved_t saved{};
    at::Tensor T, M;
    const bool bwd_t = bwd == 1 || bwd == 5 || bwd == 6 || bwd == 7, bwd_m = bwd == 4 || bwd == 5 || bwd == 7 || bwd == 8;
    if (fwd == RL_FWD_DEFAULT || (keep_t && (fwd == RL_FWD1 || fwd == RL_FWD3) && bwd_t)) {
      T = at::empty({n, r}, x.options());
      saved.T = T.data_ptr();
      saved.ldt = r;
    }
    if (keep_merged && fwd == RL_FWD2 && bwd_m) {
      M = at::empty({i, o}, x.options());
      saved.M = M.data_ptr();
      saved.ldm = o;
    }
    const int choices = (T.defined() ? RL_CALL_T : 0) | (M.defined() ? RL_CALL_M : 0) | ((float)dropout_p != 0.f ? RL_CALL_DROPOUT : 0);
    const at::Tensor ws = scratch(p_workspace_bytes((int)fwd, -1, n, i, o, r, code, choices), x);
    rl_opts_t opts{};
    opts.stream = c10::hip::getCurrentHIPStream(x.device().index()).stream();
    opts.workspace = ws.data_ptr();
    opts.workspace_bytes = (size_t)ws.numel();
    opts.scale = (float)scale;
    opts.bias = bias.has_value() ? bias->data_ptr() : nullptr;
    opts.dropout_p = (float)dropout_p;
    opts.dropout_seed = (uint32_t)((uint64_t)dropout_seed & 0xFFFFFFFFu);
    const rl_tensor_t dx = desc(x2, code), dw = desc(W, code), da = desc(A, code), db = desc(B, code);
    rl_tensor_t dy = desc(y, code);
    check(p_forward((int)fwd, &dx, &dw, &da, &db, &dy, &saved, &opts));
    ctx->save_for_backward({x2, W, A, B});
    ctx->saved_data["bwd"] = bwd;
    ctx->saved_data["fwd"] = (int64_t)saved.fwd_variant;
    ctx->saved_data["scale"] = (double)saved.scale;
    ctx->saved_data["thr"] = (int64_t)saved.dropout_thr;
    ctx->saved_data["seed"] = (int64_t)saved.dropout_seed;
    ctx->saved_data["x_shape"] = x.sizes().vec();
    if (T.defined()) ctx->saved_data["T"] = T;
    if (M.defined()) ctx->saved_data["M"] = M;
    std::vector<int64_t> shape = x.sizes().vec();
    shape.back() = o;
    return y.view(shape);
  }

  static torch::autograd::variable_list backward(torch::autograd::AutogradContext* ctx, torch::autograd::variable_list grads) {
    const auto vars = ctx->get_saved_variables();
    const at::Tensor &W = vars[1], &A = vars[2], &B = vars[3];
    TORCH_CHECK_VALUE(vars[0].is_cuda(), "the saved input came back on ", vars[0].device());
    const rl_tensor_t dw = saved_desc(W, vars[0]), da = saved_desc(A, vars[0]), db = saved_desc(B, vars[0]);
    const int64_t i = W.size(0), o = W.size(1), r = A.size(1);
    const at::Tensor x2 = rows(vars[0], i);
    const int64_t n = x2.size(0);
    const int code = dtype_code(x2.scalar_type());
    const c10::OptionalDeviceGuard guard(x2.device());
    const at::Tensor dy2 = rows(grads[0], o);
    const int bwd = (int)ctx->saved_data["bwd"].toInt();
    rl_saved_t saved{};
    saved.fwd_variant = (int32_t)ctx->saved_data["fwd"].toInt();
    saved.dtype = code;
    saved.n = n; saved.i = i; saved.o = o; saved.r = r;
    saved.X = x2.data_ptr();
    saved.ldx = x2.stride(0);
    saved.scale = (float)ctx->saved_data["scale"].toDouble();
    saved.dropout_thr = (uint32_t)ctx->saved_data["thr"].toInt();
    saved.dropout_seed = (uint32_t)ctx->saved_data["seed"].toInt();
    at::Tensor T, M;
    auto it = ctx->saved_data.find("T");
    if (it != ctx->saved_data.end()) { T = it->second.toTensor(); saved.T = T.data_ptr(); saved.ldt = T.stride(0); }
    it = ctx->saved_data.find("M");
    if (it != ctx->saved_data.end()) { M = it->second.toTensor(); saved.M = M.data_ptr(); saved.ldm = M.stride(0); }
    at::Tensor dx, dA, dB;
    rl_tensor_t tx{}, ta{}, tb{};
    if (ctx->needs_input_grad(0)) { dx = at::empty({n, i}, x2.options()); tx = desc(dx, code); }
    if (ctx->needs_input_grad(2)) { dA = at::empty_like(A); ta = desc(dA, da.dtype); }
    if (ctx->needs_input_grad(3)) { dB = at::empty_like(B); tb = desc(dB, db.dtype); }
    const int choices = (T.defined() ? RL_CALL_T : 0) | (M.defined() ? RL_CALL_M : 0) | (saved.dropout_thr != 0 ? RL_CALL_DROPOUT : 0) |
                        (dx.defined() ? 0 : RL_CALL_NO_DX) | (dA.defined() ? 0 : RL_CALL_NO_DA) | (dB.defined() ? 0 : RL_CALL_NO_DB);
    const at::Tensor ws = scratch(p_workspace_bytes(-1, bwd, n, i, o, r, code, choices), x2);
    rl_opts_t opts{};
    opts.stream = c10::hip::getCurrentHIPStream(x2.device().index()).stream();
    opts.workspace = ws.data_ptr();
    opts.workspace_bytes = (size_t)ws.numel();
    const rl_tensor_t ddy = desc(dy2, dtype_code(dy2.scalar_type()));
    check(p_backward(bwd, &ddy, &saved, &dw, &da, &db, dx.defined() ? &tx : nullptr, dA.defined() ? &ta : nullptr,
                     dB.defined() ? &tb : nullptr, &opts));
    if (dx.defined()) dx = dx.view(ctx->saved_data["x_shape"].toIntVector());
    at::Tensor none;
    return {dx, none, dA, dB, none, none, none, none, none, none, none, none};
  }
};

bool plain_2d(const at::Tensor& t, const at::Tensor& x) {
  return t.dim() == 2 && t.stride(1) == 1 && t.scalar_type() == x.scalar_type() && t.device() == x.device() && t.layout() == at::kStrided;
}

// lora(x, W, A, B, bias, scale, (fwd, bwd), keep_merged, dropout=None, keep_t=False): y, or None (see above)
PyObject* py_lora(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  if (nargs < 8 || nargs > 10 || p_forward == nullptr) Py_RETURN_NONE;
  for (int k = 0; k < 4; ++k)
    if (!THPVariable_CheckExact(args[k])) Py_RETURN_NONE;
  const bool has_bias = args[4] != Py_None;
  if (has_bias && !THPVariable_CheckExact(args[4])) Py_RETURN_NONE;
  if (!PyFloat_CheckExact(args[5]) || !PyTuple_CheckExact(args[6]) || PyTuple_GET_SIZE(args[6]) != 2 || !PyBool_Check(args[7])) Py_RETURN_NONE;
  PyObject *f = PyTuple_GET_ITEM(args[6], 0), *b = PyTuple_GET_ITEM(args[6], 1);
  if (!PyLong_CheckExact(f) || !PyLong_CheckExact(b)) Py_RETURN_NONE;
  const int64_t fwd = PyLong_AsLongLong(f), bwd = PyLong_AsLongLong(b);
  double p = 0.0;
  int64_t seed = 0;
  if (nargs > 8 && args[8] != Py_None) {
    if (!PyTuple_CheckExact(args[8]) || PyTuple_GET_SIZE(args[8]) != 2) Py_RETURN_NONE;
    PyObject *dp = PyTuple_GET_ITEM(args[8], 0), *ds = PyTuple_GET_ITEM(args[8], 1);
    if (!PyFloat_CheckExact(dp) || !PyLong_CheckExact(ds)) Py_RETURN_NONE;
    p = PyFloat_AS_DOUBLE(dp);
    seed = PyLong_AsLongLong(ds);
  }
  if (PyErr_Occurred()) {  // integers beyond 64 bits: the Python path has the message
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  if (nargs > 9 && !PyBool_Check(args[9])) Py_RETURN_NONE;
  const bool keep_merged = args[7] == Py_True, keep_t = nargs > 9 && args[9] == Py_True;
  if (fwd < RL_FWD_DEFAULT || fwd > RL_FWD3 || bwd < RL_BWD_DEFAULT || bwd > RL_BWD8) Py_RETURN_NONE;
  if (torch::jit::tracer::isTracing() || at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set() ||
      c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::FuncTorchDynamicLayerFrontMode))
    Py_RETURN_NONE;
  const at::Tensor &x = THPVariable_Unpack(args[0]), &W = THPVariable_Unpack(args[1]), &A = THPVariable_Unpack(args[2]), &B = THPVariable_Unpack(args[3]);
  if (!x.is_cuda() || x.layout() != at::kStrided || x.dim() < 1 || dtype_code(x.scalar_type()) < 0 || x.numel() == 0) Py_RETURN_NONE;
  if (!plain_2d(W, x) || !plain_2d(A, x) || !plain_2d(B, x) || W.numel() == 0 || A.numel() == 0 || B.numel() == 0) Py_RETURN_NONE;
  if (x.size(-1) != W.size(0) || x.device().index() != c10::hip::current_device()) Py_RETURN_NONE;
  // (conjugate, negative and zero-tensor views carry their values lazily)
  for (const at::Tensor* t : {&x, &W, &A, &B})
    if (t->is_conj() || t->is_neg() || t->_is_zerotensor()) Py_RETURN_NONE;
  std::optional<at::Tensor> bias;
  if (has_bias) {
    const at::Tensor& t = THPVariable_Unpack(args[4]);
    if (t.dim() != 1 || t.stride(0) != 1 || t.scalar_type() != x.scalar_type() || t.numel() != W.size(1) || t.device() != x.device()) Py_RETURN_NONE;
    bias = t;
  }
  at::Tensor y;
  {
    pybind11::gil_scoped_release release;
    y = LoRANode::apply(x, W, A, B, bias, PyFloat_AS_DOUBLE(args[5]), fwd, bwd, keep_merged, p, seed, keep_t);
  }
  return THPVariable_Wrap(y);
  END_HANDLE_TH_ERRORS
}

// init(forward, backward, call_workspace_bytes addresses, check)
PyObject* py_init(PyObject*, PyObject* args) {
  unsigned long long a, b, c;
  PyObject* chk;
  if (!PyArg_ParseTuple(args, "KKKO", &a, &b, &c, &chk)) return nullptr;
  p_forward = reinterpret_cast<decltype(p_forward)>(a);
  p_backward = reinterpret_cast<decltype(p_backward)>(b);
  p_workspace_bytes = reinterpret_cast<decltype(p_workspace_bytes)>(c);
  Py_INCREF(chk);
  Py_XDECREF(g_check);
  g_check = chk;
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"lora", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(py_lora)), METH_FASTCALL, "LoRA layer as a native autograd node, or None"},
                         {"init", py_init, METH_VARARGS, "hand over librunlora's entry points"},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_autograd", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

// read by build.py without loading the library
[[gnu::used]] const char built_for[] = "built for [" RL_BUILT_FOR "]";

}  // namespace

PyMODINIT_FUNC PyInit__autograd(void) { return PyModule_Create(&module_def); }
