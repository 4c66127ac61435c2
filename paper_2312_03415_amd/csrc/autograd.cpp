// The layers' autograd nodes in native code (host only): RunLoRAFunction, RunVeRAFunction and RunDoRAFunction of module.py without
// Python in their forward and backward.  Same buffers, same calls into librunlora, same results; what they save is host time.
//
// A training pass of a small layer is bound by its host work: with the Python node, forward + backward of 256 x 768 -> 768
// fp32 take 102-189 us of host time a pass for 75 us of GPU work (forward 30; the backward's body alone 68, because the
// autograd engine runs it on a thread of its own, where every Python object it touches comes over from another core).  With
// this node the host takes 14 us for the forward and at most the GPU's time in all: 194 -> 88 us a pass; 1024 x 4096 -> 4096
// r 64 196 -> 114, 1237 x 2056 -> 5464 197 -> 122.  Likewise VeRA (448 x 768 -> 768 r 128
// 196 -> 109, 623 x 4352 -> 4096 r 64 200 -> 117) and DoRA (765 x 1280 -> 7328 r 64 216 -> 135).
//
// lora(...), vera(...) and dora(...) return None where their node does not apply, and the caller then takes the Python node: tensor subclasses, torch
// function / dispatch modes, functorch transforms and tracing (all of which have to see a Python-level function), devices
// other than the current GPU, and operands that only the Python path's checks describe properly.  Forward-mode gradients are
// refused by either node, saved-tensor hooks apply to both (the same tensors are saved in the same order).
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
decltype(&runlora_vera_forward) p_vera_forward = nullptr;
decltype(&runlora_vera_backward) p_vera_backward = nullptr;
decltype(&runlora_vera_workspace_bytes) p_vera_workspace_bytes = nullptr;
decltype(&runlora_dora_forward) p_dora_forward = nullptr;
decltype(&runlora_dora_backward) p_dora_backward = nullptr;
decltype(&runlora_dora_workspace_bytes) p_dora_workspace_bytes = nullptr;
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

// a saved vector as the backward gets it back
void* saved_vec(const at::Tensor& t, int64_t count, at::ScalarType type, const at::Tensor& x, const char* name) {
  TORCH_CHECK_VALUE(t.device() == x.device(), "a saved tensor came back on another device: ", t.device(), ", not ", x.device());
  TORCH_CHECK_VALUE(t.dim() == 1 && t.numel() == count && t.scalar_type() == type && t.stride(0) == 1, name, " must be a dense vector of ",
                    count, " elements of the activation dtype");
  return t.data_ptr();
}

rl_opts_t options(const at::Tensor& x, const at::Tensor& ws, const std::optional<at::Tensor>& bias = std::nullopt, double scale = 0.0) {
  rl_opts_t o{};
  o.stream = c10::hip::getCurrentHIPStream(x.device().index()).stream();
  o.workspace = ws.data_ptr();
  o.workspace_bytes = (size_t)ws.numel();
  o.scale = (float)scale;
  o.bias = bias.has_value() ? bias->data_ptr() : nullptr;
  return o;
}

void keep_record(torch::autograd::AutogradContext* ctx, const rl_saved_t& saved, int64_t bwd, const at::Tensor& x) {
  ctx->saved_data["bwd"] = bwd;
  ctx->saved_data["fwd"] = (int64_t)saved.fwd_variant;
  ctx->saved_data["scale"] = (double)saved.scale;
  ctx->saved_data["x_shape"] = x.sizes().vec();
}

// the forward's record for the input as autograd hands it back (no dropout, T and M by the caller)
rl_saved_t record(torch::autograd::AutogradContext* ctx, const at::Tensor& x2, int code, int64_t o, int64_t r) {
  rl_saved_t s{};
  s.fwd_variant = (int32_t)ctx->saved_data["fwd"].toInt();
  s.dtype = code;
  s.n = x2.size(0); s.i = x2.size(1); s.o = o; s.r = r;
  s.X = x2.data_ptr();
  s.ldx = x2.stride(0);
  s.scale = (float)ctx->saved_data["scale"].toDouble();
  return s;
}

at::Tensor shaped(const at::Tensor& y, const at::Tensor& x) {
  std::vector<int64_t> shape = x.sizes().vec();
  shape.back() = y.size(1);
  return y.view(shape);
}

struct VeRANode : public torch::autograd::Function<VeRANode> {
  static at::Tensor forward(torch::autograd::AutogradContext* ctx, const at::Tensor& x, const at::Tensor& W, const at::Tensor& A,
                            const at::Tensor& B, const at::Tensor& d, const at::Tensor& b, const std::optional<at::Tensor>& bias, double scale,
                            int64_t fwd, int64_t bwd) {
    const int64_t i = W.size(0), o = W.size(1), r = A.size(1);
    const int code = dtype_code(x.scalar_type());
    const at::Tensor x2 = rows(x, i);
    const int64_t n = x2.size(0);
    at::Tensor y = at::empty({n, o}, x.options()), T;
    rl_saved_t saved{};
    if (fwd == RL_FWD_DEFAULT) {
      T = at::empty({n, r}, x.options());
      saved.T = T.data_ptr();
      saved.ldt = r;
    }
    const at::Tensor ws = scratch(p_vera_workspace_bytes((int)fwd, -1, n, i, o, r, code), x);
    const rl_opts_t opts = options(x, ws, bias, scale);
    const rl_tensor_t dx = desc(x2, code), dw = desc(W, code), da = desc(A, code), db = desc(B, code);
    rl_tensor_t dy = desc(y, code);
    check(p_vera_forward((int)fwd, &dx, &dw, &da, &db, d.data_ptr(), b.data_ptr(), &dy, &saved, &opts));
    ctx->save_for_backward({x2, W, A, B, d, b});
    keep_record(ctx, saved, bwd, x);
    if (T.defined()) ctx->saved_data["T"] = T;
    return shaped(y, x);
  }

  static torch::autograd::variable_list backward(torch::autograd::AutogradContext* ctx, torch::autograd::variable_list grads) {
    const auto vars = ctx->get_saved_variables();
    TORCH_CHECK_VALUE(vars[0].is_cuda(), "the saved input came back on ", vars[0].device());
    const rl_tensor_t dw = saved_desc(vars[1], vars[0]), da = saved_desc(vars[2], vars[0]), db = saved_desc(vars[3], vars[0]);
    const int64_t i = dw.rows, o = dw.cols, r = db.rows;
    const at::Tensor x2 = rows(vars[0], i);
    const int64_t n = x2.size(0);
    const int code = dtype_code(x2.scalar_type());
    const c10::OptionalDeviceGuard guard(x2.device());
    const at::Tensor dy2 = rows(grads[0], o);
    void* const d = saved_vec(vars[4], r, dy2.scalar_type(), x2, "d");
    void* const b = saved_vec(vars[5], o, dy2.scalar_type(), x2, "b");
    const int bwd = (int)ctx->saved_data["bwd"].toInt();
    rl_saved_t saved = record(ctx, x2, code, o, r);
    at::Tensor T;
    auto it = ctx->saved_data.find("T");
    if (it != ctx->saved_data.end()) { T = it->second.toTensor(); saved.T = T.data_ptr(); saved.ldt = T.stride(0); }
    at::Tensor dx, dd, dbv;
    rl_tensor_t tx{};
    if (ctx->needs_input_grad(0)) { dx = at::empty({n, i}, x2.options()); tx = desc(dx, code); }
    if (ctx->needs_input_grad(4)) dd = at::empty_like(vars[4]);
    if (ctx->needs_input_grad(5)) dbv = at::empty_like(vars[5]);
    const at::Tensor ws = scratch(p_vera_workspace_bytes(-1, bwd, n, i, o, r, code), x2);
    const rl_opts_t opts = options(x2, ws);
    const rl_tensor_t ddy = desc(dy2, dtype_code(dy2.scalar_type()));
    check(p_vera_backward(bwd, &ddy, &saved, &dw, &da, &db, d, b, dx.defined() ? &tx : nullptr, dd.defined() ? dd.data_ptr() : nullptr,
                          dbv.defined() ? dbv.data_ptr() : nullptr, &opts));
    if (dx.defined()) dx = dx.view(ctx->saved_data["x_shape"].toIntVector());
    at::Tensor none;
    return {dx, none, none, none, dd, dbv, none, none, none, none};
  }
};

struct DoRANode : public torch::autograd::Function<DoRANode> {
  static at::Tensor forward(torch::autograd::AutogradContext* ctx, const at::Tensor& x, const at::Tensor& W, const at::Tensor& A,
                            const at::Tensor& B, const at::Tensor& m, const std::optional<at::Tensor>& bias, double scale, int64_t bwd) {
    const int64_t i = W.size(0), o = W.size(1), r = A.size(1);
    const int code = dtype_code(x.scalar_type());
    const at::Tensor x2 = rows(x, i);
    const int64_t n = x2.size(0);
    at::Tensor y = at::empty({n, o}, x.options());
    const at::Tensor c = at::empty({o}, x.options().dtype(at::kFloat));
    rl_saved_t saved{};
    const at::Tensor ws = scratch(p_dora_workspace_bytes(RL_FWD2, -1, n, i, o, r, code), x);
    const rl_opts_t opts = options(x, ws, bias, scale);
    const rl_tensor_t dx = desc(x2, code), dw = desc(W, code), da = desc(A, code), db = desc(B, code);
    rl_tensor_t dy = desc(y, code);
    check(p_dora_forward(RL_FWD2, &dx, &dw, &da, &db, m.data_ptr(), &dy, &saved, c.data_ptr<float>(), &opts));
    ctx->save_for_backward({x2, W, A, B, m, c, y});  // y is the tensor handed to the caller: no copy is kept
    keep_record(ctx, saved, bwd, x);
    if (bias.has_value()) ctx->saved_data["bias"] = *bias;
    return shaped(y, x);
  }

  static torch::autograd::variable_list backward(torch::autograd::AutogradContext* ctx, torch::autograd::variable_list grads) {
    const auto vars = ctx->get_saved_variables();
    TORCH_CHECK_VALUE(vars[0].is_cuda(), "the saved input came back on ", vars[0].device());
    const at::Tensor &A = vars[2], &B = vars[3], &m = vars[4];
    const rl_tensor_t dw = saved_desc(vars[1], vars[0]), da = saved_desc(A, vars[0]), db = saved_desc(B, vars[0]), ty = saved_desc(vars[6], vars[0]);
    const int64_t i = dw.rows, o = dw.cols, r = da.cols;
    const at::Tensor x2 = rows(vars[0], i);
    const int64_t n = x2.size(0);
    const int code = dtype_code(x2.scalar_type());
    const c10::OptionalDeviceGuard guard(x2.device());
    const at::Tensor dy2 = rows(grads[0], o);
    void* const pm = saved_vec(m, db.cols, dy2.scalar_type(), x2, "m");
    const float* const c = static_cast<const float*>(saved_vec(vars[5], db.cols, at::kFloat, x2, "c"));
    const int bwd = (int)ctx->saved_data["bwd"].toInt();
    const rl_saved_t saved = record(ctx, x2, code, o, r);
    at::Tensor dx, dA, dB, dm;
    rl_tensor_t tx{}, ta{}, tb{};
    if (ctx->needs_input_grad(0)) { dx = at::empty({n, i}, x2.options()); tx = desc(dx, code); }
    if (ctx->needs_input_grad(2)) { dA = at::empty_like(A); ta = desc(dA, da.dtype); }
    if (ctx->needs_input_grad(3)) { dB = at::empty_like(B); tb = desc(dB, db.dtype); }
    if (ctx->needs_input_grad(4)) dm = at::empty_like(m);
    std::optional<at::Tensor> bias;
    auto it = ctx->saved_data.find("bias");
    if (it != ctx->saved_data.end()) bias = it->second.toTensor();
    const at::Tensor ws = scratch(p_dora_workspace_bytes(-1, bwd, n, i, o, r, code), x2);
    const rl_opts_t opts = options(x2, ws, bias);
    const rl_tensor_t ddy = desc(dy2, dtype_code(dy2.scalar_type()));
    check(p_dora_backward(bwd, &ddy, &saved, &dw, &da, &db, pm, c, &ty, dx.defined() ? &tx : nullptr, dA.defined() ? &ta : nullptr,
                          dB.defined() ? &tb : nullptr, dm.defined() ? dm.data_ptr() : nullptr, &opts));
    if (dx.defined()) dx = dx.view(ctx->saved_data["x_shape"].toIntVector());
    at::Tensor none;
    return {dx, none, dA, dB, dm, none, none, none};
  }
};

bool plain_2d(const at::Tensor& t, const at::Tensor& x) {
  return t.dim() == 2 && t.stride(1) == 1 && t.scalar_type() == x.scalar_type() && t.device() == x.device() && t.layout() == at::kStrided;
}

bool plain_1d(const at::Tensor& t, int64_t count, const at::Tensor& x) {
  return t.dim() == 1 && t.stride(0) == 1 && t.scalar_type() == x.scalar_type() && t.numel() == count && t.device() == x.device() && t.layout() == at::kStrided;
}

// x, W, A and B (args[0 .. 3]), vectors as long as B has rows (0) or columns (1), and a bias or None as a native node takes them; nothing
// here raises
bool operands_ok(PyObject* const* args, PyObject* bias, std::initializer_list<std::pair<PyObject*, int>> vectors) {
  for (int k = 0; k < 4; ++k)
    if (!THPVariable_CheckExact(args[k])) return false;
  if (bias != Py_None && !THPVariable_CheckExact(bias)) return false;
  for (const auto& v : vectors)
    if (!THPVariable_CheckExact(v.first)) return false;
  if (torch::jit::tracer::isTracing() || at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set() ||
      c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::FuncTorchDynamicLayerFrontMode))
    return false;
  const at::Tensor &x = THPVariable_Unpack(args[0]), &W = THPVariable_Unpack(args[1]), &A = THPVariable_Unpack(args[2]), &B = THPVariable_Unpack(args[3]);
  if (!x.is_cuda() || x.layout() != at::kStrided || x.dim() < 1 || dtype_code(x.scalar_type()) < 0 || x.numel() == 0) return false;
  if (!plain_2d(W, x) || !plain_2d(A, x) || !plain_2d(B, x) || W.numel() == 0 || A.numel() == 0 || B.numel() == 0) return false;
  if (x.size(-1) != W.size(0) || x.device().index() != c10::hip::current_device()) return false;
  // (conjugate, negative and zero-tensor views carry their values lazily)
  auto lazy = [](const at::Tensor& t) { return t.is_conj() || t.is_neg() || t._is_zerotensor(); };
  for (const at::Tensor* t : {&x, &W, &A, &B})
    if (lazy(*t)) return false;
  for (const auto& v : vectors) {
    const at::Tensor& t = THPVariable_Unpack(v.first);
    if (!plain_1d(t, B.size(v.second), x) || lazy(t)) return false;
  }
  if (bias != Py_None) {
    const at::Tensor& t = THPVariable_Unpack(bias);
    if (t.dim() != 1 || t.stride(0) != 1 || t.scalar_type() != x.scalar_type() || t.numel() != W.size(1) || t.device() != x.device()) return false;
  }
  return true;
}

std::optional<at::Tensor> optional_tensor(PyObject* o) {
  return o == Py_None ? std::nullopt : std::optional<at::Tensor>(THPVariable_Unpack(o));
}

bool pair_of(PyObject* o, int64_t* fwd, int64_t* bwd) {
  if (!PyTuple_CheckExact(o) || PyTuple_GET_SIZE(o) != 2) return false;
  PyObject *f = PyTuple_GET_ITEM(o, 0), *b = PyTuple_GET_ITEM(o, 1);
  if (!PyLong_CheckExact(f) || !PyLong_CheckExact(b)) return false;
  *fwd = PyLong_AsLongLong(f);
  *bwd = PyLong_AsLongLong(b);
  if (PyErr_Occurred()) {  // integers beyond 64 bits: the Python path has the message
    PyErr_Clear();
    return false;
  }
  return *fwd >= RL_FWD_DEFAULT && *fwd <= RL_FWD3 && *bwd >= RL_BWD_DEFAULT && *bwd <= RL_BWD8;
}

// lora(x, W, A, B, bias, scale, (fwd, bwd), keep_merged, dropout=None, keep_t=False): y, or None (see above)
PyObject* py_lora(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  if (nargs < 8 || nargs > 10 || p_forward == nullptr) Py_RETURN_NONE;
  int64_t fwd = 0, bwd = 0;
  if (!PyFloat_CheckExact(args[5]) || !PyBool_Check(args[7]) || !pair_of(args[6], &fwd, &bwd)) Py_RETURN_NONE;
  double p = 0.0;
  int64_t seed = 0;
  if (nargs > 8 && args[8] != Py_None) {
    if (!PyTuple_CheckExact(args[8]) || PyTuple_GET_SIZE(args[8]) != 2) Py_RETURN_NONE;
    PyObject *dp = PyTuple_GET_ITEM(args[8], 0), *ds = PyTuple_GET_ITEM(args[8], 1);
    if (!PyFloat_CheckExact(dp) || !PyLong_CheckExact(ds)) Py_RETURN_NONE;
    p = PyFloat_AS_DOUBLE(dp);
    seed = PyLong_AsLongLong(ds);
  }
  if (PyErr_Occurred()) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  if (nargs > 9 && !PyBool_Check(args[9])) Py_RETURN_NONE;
  const bool keep_merged = args[7] == Py_True, keep_t = nargs > 9 && args[9] == Py_True;
  if (!operands_ok(args, args[4], {})) Py_RETURN_NONE;
  const at::Tensor &x = THPVariable_Unpack(args[0]), &W = THPVariable_Unpack(args[1]), &A = THPVariable_Unpack(args[2]), &B = THPVariable_Unpack(args[3]);
  const std::optional<at::Tensor> bias = optional_tensor(args[4]);
  at::Tensor y;
  {
    pybind11::gil_scoped_release release;
    y = LoRANode::apply(x, W, A, B, bias, PyFloat_AS_DOUBLE(args[5]), fwd, bwd, keep_merged, p, seed, keep_t);
  }
  return THPVariable_Wrap(y);
  END_HANDLE_TH_ERRORS
}

// vera(x, W, A, B, d, b, bias, scale, (fwd, bwd)): y, or None
PyObject* py_vera(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  int64_t fwd = 0, bwd = 0;
  if (nargs != 9 || p_vera_forward == nullptr || !PyFloat_CheckExact(args[7]) || !pair_of(args[8], &fwd, &bwd)) Py_RETURN_NONE;
  if (!operands_ok(args, args[6], {{args[4], 0}, {args[5], 1}})) Py_RETURN_NONE;
  const at::Tensor &x = THPVariable_Unpack(args[0]), &W = THPVariable_Unpack(args[1]), &A = THPVariable_Unpack(args[2]), &B = THPVariable_Unpack(args[3]);
  const at::Tensor &d = THPVariable_Unpack(args[4]), &b = THPVariable_Unpack(args[5]);
  const std::optional<at::Tensor> bias = optional_tensor(args[6]);
  at::Tensor y;
  {
    pybind11::gil_scoped_release release;
    y = VeRANode::apply(x, W, A, B, d, b, bias, PyFloat_AS_DOUBLE(args[7]), fwd, bwd);
  }
  return THPVariable_Wrap(y);
  END_HANDLE_TH_ERRORS
}

// dora(x, W, A, B, m, bias, scale, bwd): y, or None
PyObject* py_dora(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  if (nargs != 8 || p_dora_forward == nullptr || !PyFloat_CheckExact(args[6]) || !PyLong_CheckExact(args[7])) Py_RETURN_NONE;
  const int64_t bwd = PyLong_AsLongLong(args[7]);
  if (PyErr_Occurred()) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  if (bwd < RL_BWD_DEFAULT || bwd > RL_BWD8) Py_RETURN_NONE;
  if (!operands_ok(args, args[5], {{args[4], 1}})) Py_RETURN_NONE;
  const at::Tensor &x = THPVariable_Unpack(args[0]), &W = THPVariable_Unpack(args[1]), &A = THPVariable_Unpack(args[2]), &B = THPVariable_Unpack(args[3]);
  const at::Tensor& m = THPVariable_Unpack(args[4]);
  const std::optional<at::Tensor> bias = optional_tensor(args[5]);
  at::Tensor y;
  {
    pybind11::gil_scoped_release release;
    y = DoRANode::apply(x, W, A, B, m, bias, PyFloat_AS_DOUBLE(args[6]), bwd);
  }
  return THPVariable_Wrap(y);
  END_HANDLE_TH_ERRORS
}

// init((forward, backward, workspace_bytes addresses of LoRA, of VeRA, of DoRA: nine in all), check)
PyObject* py_init(PyObject*, PyObject* args) {
  unsigned long long a[9];
  PyObject* chk;
  if (!PyArg_ParseTuple(args, "(KKKKKKKKK)O", &a[0], &a[1], &a[2], &a[3], &a[4], &a[5], &a[6], &a[7], &a[8], &chk)) return nullptr;
  p_forward = reinterpret_cast<decltype(p_forward)>(a[0]);
  p_backward = reinterpret_cast<decltype(p_backward)>(a[1]);
  p_workspace_bytes = reinterpret_cast<decltype(p_workspace_bytes)>(a[2]);
  p_vera_forward = reinterpret_cast<decltype(p_vera_forward)>(a[3]);
  p_vera_backward = reinterpret_cast<decltype(p_vera_backward)>(a[4]);
  p_vera_workspace_bytes = reinterpret_cast<decltype(p_vera_workspace_bytes)>(a[5]);
  p_dora_forward = reinterpret_cast<decltype(p_dora_forward)>(a[6]);
  p_dora_backward = reinterpret_cast<decltype(p_dora_backward)>(a[7]);
  p_dora_workspace_bytes = reinterpret_cast<decltype(p_dora_workspace_bytes)>(a[8]);
  Py_INCREF(chk);
  Py_XDECREF(g_check);
  g_check = chk;
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"lora", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(py_lora)), METH_FASTCALL, "LoRA layer as a native autograd node, or None"},
                         {"vera", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(py_vera)), METH_FASTCALL, "VeRA layer as a native autograd node, or None"},
                         {"dora", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(py_dora)), METH_FASTCALL, "DoRA layer as a native autograd node, or None"},
                         {"init", py_init, METH_VARARGS, "hand over librunlora's entry points"},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_autograd", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

// read by build.py without loading the library
[[gnu::used]] const char built_for[] = "built for [" RL_BUILT_FOR "]";

}  // namespace

PyMODINIT_FUNC PyInit__autograd(void) { return PyModule_Create(&module_def); }
