// native.cpp -- argument marshalling of binding.py in C++: checks, output and workspace allocation, the C call.
//
// A call of the binding on a small batch is host-bound: attribute look-ups, a Python object per output and ctypes' conversion
// of sixteen arguments were most of it.  Host time of a call, in Python with ctypes / here: the loss at 16384 tokens 14.6 /
// 8.9 us, rewards and advantages (two calls) 13.2 / 8.7, aipo_loss 35 / 23, a whole step 192 / 147.  Each entry takes
// positional arguments (binding.py fills in defaults) and talks to the C ABI of include/llamarl.h.  Every call allocates what
// it returns; nothing is kept between calls.
//
// Errors: a check or a status that is not LLAMARL_OK raises binding.LlamarlError(status, message); C++ exceptions become the
// Python exceptions torch itself raises for them.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/hip/HIPEvent.h>
#include <c10/core/impl/VirtualGuardImpl.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cmath>
#include <optional>

#include "../../include/llamarl.h"
#include "tile_rules.h"

namespace {

PyObject* g_error = nullptr;      // binding.LlamarlError

struct Raised {};                 // a Python exception is set

[[noreturn]] void raise_status(int status, const std::string& message) {
  PyObject* e = PyObject_CallFunction(g_error, "is", status, message.c_str());
  if (e != nullptr) {
    PyErr_SetObject(g_error, e);
    Py_DECREF(e);
  }
  throw Raised{};
}
void check(llamarl_status s) {
  if (s != LLAMARL_OK) raise_status((int)s, llamarl_last_error());
}
[[noreturn]] void invalid(const std::string& message) { raise_status(LLAMARL_ERR_INVALID_ARG, message); }

const at::Tensor& tensor(PyObject* o, const char* name) {
  if (!THPVariable_Check(o)) {
    PyErr_Format(PyExc_TypeError, "%s must be a tensor, not %s", name, Py_TYPE(o)->tp_name);
    throw Raised{};
  }
  return THPVariable_Unpack(o);
}
const char* dtype_name(at::ScalarType t) {
  return t == at::kFloat ? "torch.float32" : t == at::kBFloat16 ? "torch.bfloat16" : t == at::kInt ? "torch.int32" : "torch.uint8";
}
llamarl_dtype dtype_code(const at::Tensor& t) {
  if (t.scalar_type() == at::kBFloat16) return LLAMARL_BF16;
  if (t.scalar_type() == at::kFloat) return LLAMARL_F32;
  invalid(std::string("unsupported tensor dtype ") + c10::toString(t.scalar_type()));
}
void need(const at::Tensor& t, at::ScalarType dtype, const char* name) {
  if (t.scalar_type() != dtype || !t.is_cuda() || !t.is_contiguous())
    invalid(std::string(name) + " must be a contiguous device tensor of " + dtype_name(dtype));
}
const at::Tensor& needed(PyObject* o, at::ScalarType dtype, const char* name) {
  const at::Tensor& t = tensor(o, name);
  need(t, dtype, name);
  return t;
}
at::Tensor empty(const at::Tensor& like, at::IntArrayRef sizes, at::ScalarType dtype = at::kFloat) {
  return at::empty(sizes, like.options().dtype(dtype).requires_grad(false));
}
// The kernels take sizes from H and W alone: an array that is too small for them would be read or written past its end.
void at_least(const at::Tensor& t, int64_t n, const char* name) {
  if (t.defined() && t.numel() < n) invalid(std::string(name) + " must have " + std::to_string(n) + " entries");
}
// the caller's workspace, or one for this call
at::Tensor workspace(PyObject* o, size_t bytes, const at::Tensor& like) {
  if (o != Py_None) {
    const at::Tensor& t = tensor(o, "ws");
    if (!(t.is_cuda() || t.is_pinned()) || !t.is_non_overlapping_and_dense()) invalid("ws must be a dense device tensor");
    return t;
  }
  return empty(like, {(int64_t)std::max<size_t>(bytes, 16)}, at::kByte);
}
// The stream of a call: the current one (None) or the caller's, which is the current one while the call allocates.  A workspace
// out of another stream's pool would be free again, and given to that stream's next allocation, while the kernels still run.
struct CallStream {
  std::optional<c10::Stream> before;      // the current stream, where it is another
  void* handle;
  CallStream(PyObject* o, const at::Tensor& like) {
    if (o == Py_None) {
      handle = c10::hip::getCurrentHIPStream().stream();
      return;
    }
    handle = PyLong_AsVoidPtr(o);
    if (handle == nullptr && PyErr_Occurred()) throw Raised{};
    const c10::DeviceIndex device = like.device().index();
    if (handle == c10::hip::getCurrentHIPStream(device).stream()) return;
    const c10::hip::HIPStream s = c10::hip::getStreamFromExternal(static_cast<hipStream_t>(handle), device);
    before = c10::impl::VirtualGuardImpl(c10::DeviceType::CUDA).exchangeStream(
        c10::Stream(c10::Stream::UNSAFE, like.device(), s.id()));
  }
  CallStream(const CallStream&) = delete;
  ~CallStream() {
    if (before) c10::impl::VirtualGuardImpl(c10::DeviceType::CUDA).exchangeStream(*before);
  }
  // an output may be read on the caller's current stream, and freed while it is
  template <typename... Ts>
  void returns(const Ts&... ts) const {
    if (before) (ts.record_stream(*before), ...);
  }
};
int64_t integer(PyObject* o) {
  const int64_t v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) throw Raised{};
  return v;
}
double real(PyObject* o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw Raised{};
  return v;
}
template <typename T = void>
T* ptr(const at::Tensor& t) {
  return t.defined() ? reinterpret_cast<T*>(t.data_ptr()) : nullptr;
}
at::Tensor optional(PyObject* o, at::ScalarType dtype, const char* name) {
  return o == Py_None ? at::Tensor() : needed(o, dtype, name);
}

// without the interpreter lock: a launch may wait for the driver
struct Unlocked {
  PyThreadState* state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};
template <typename F>
llamarl_status unlocked(F&& f) {
  const Unlocked u;
  return f();
}

PyObject* tuple(std::initializer_list<at::Tensor> ts) {
  PyObject* out = PyTuple_New((Py_ssize_t)ts.size());
  if (out == nullptr) throw Raised{};
  Py_ssize_t i = 0;
  for (const at::Tensor& t : ts) {
    PyObject* o = THPVariable_Wrap(t);
    if (o == nullptr) {
      Py_DECREF(out);
      throw Raised{};
    }
    PyTuple_SET_ITEM(out, i++, o);
  }
  return out;
}

struct Head {          // H [N,d], W [V,d], targets [N]
  at::Tensor H, W, targets;
  llamarl_dtype dt;
  int64_t N, d, V;
  Head(PyObject* h, PyObject* w, PyObject* t, const char* w_name) : H(tensor(h, "H")) {
    dt = dtype_code(H);
    need(H, H.scalar_type(), "H");
    W = needed(w, H.scalar_type(), w_name);
    targets = needed(t, at::kInt, "targets");
    if (H.dim() != 2 || W.dim() < 1) {
      PyErr_SetString(PyExc_ValueError, "H and W must be matrices");
      throw Raised{};
    }
    N = H.size(0);
    d = H.size(1);
    V = W.size(0);
  }
  void same_width(const char* w_name) const {
    if (W.dim() < 2 || W.size(1) != d || targets.numel() != N)
      invalid(std::string("shape mismatch between H, ") + w_name + ", targets");
  }
  // as the backward takes them
  void holds(const char* w_name, const at::Tensor& lse, const at::Tensor& coef) const {
    if (W.numel() != V * d) invalid(std::string("shape mismatch between H and ") + w_name);
    at_least(targets, N, "targets");
    at_least(lse, N, "lse");
    at_least(coef, N, "coef");
  }
};

// H, W, targets, mask, ws, stream
PyObject* token_logprobs(PyObject* const* a) {
  const Head x(a[0], a[1], a[2], "W");
  x.same_width("W");
  const at::Tensor mask = optional(a[3], at::kByte, "mask");
  if (mask.defined() && mask.numel() != x.N) invalid("mask must have N entries");
  const CallStream st(a[5], x.H);
  const at::Tensor logp = empty(x.H, {x.N}), lse = empty(x.H, {x.N});
  const at::Tensor ws = workspace(a[4], llamarl_workspace_bytes(x.N, x.d, x.V, x.dt, LLAMARL_PASS_LOGPROBS), x.H);
  check(unlocked([&] {
    return llamarl_token_logprobs(ptr(x.H), ptr(x.W), ptr<int32_t>(x.targets), ptr<uint8_t>(mask), x.N, x.d, x.V, x.dt,
                                  ptr<float>(logp), ptr<float>(lse), ptr(ws), (size_t)ws.numel(), st.handle);
  }));
  st.returns(logp, lse);
  return tuple({logp, lse});
}

// H, W_slice, targets, v0, V_total, mask, ws, stream
PyObject* token_logprobs_partial(PyObject* const* a) {
  const Head x(a[0], a[1], a[2], "W_slice");
  x.same_width("W_slice");
  const int64_t v0 = integer(a[3]), V_total = integer(a[4]);
  const at::Tensor mask = optional(a[5], at::kByte, "mask");
  at_least(mask, x.N, "mask");
  const CallStream st(a[7], x.H);
  const at::Tensor m = empty(x.H, {x.N}), s = empty(x.H, {x.N}), zt = empty(x.H, {x.N});
  const at::Tensor ws = workspace(a[6], llamarl_workspace_bytes(x.N, x.d, x.V, x.dt, LLAMARL_PASS_LOGPROBS), x.H);
  check(unlocked([&] {
    return llamarl_token_logprobs_partial(ptr(x.H), ptr(x.W), ptr<int32_t>(x.targets), ptr<uint8_t>(mask), x.N, x.d, x.V, v0,
                                          V_total, x.dt, ptr<float>(m), ptr<float>(s), ptr<float>(zt), ptr(ws),
                                          (size_t)ws.numel(), st.handle);
  }));
  st.returns(m, s, zt);
  return tuple({m, s, zt});
}

// m, s, zt, stream
PyObject* merge_partials(PyObject* const* a) {
  const at::Tensor &m = needed(a[0], at::kFloat, "m"), &s = needed(a[1], at::kFloat, "s"), &zt = needed(a[2], at::kFloat, "zt");
  if (m.dim() != 2 || m.sizes() != s.sizes() || m.sizes() != zt.sizes()) invalid("m, s, zt must be [shards, N]");
  const int64_t shards = m.size(0), N = m.size(1);
  const CallStream st(a[3], m);
  const at::Tensor logp = empty(m, {N}), lse = empty(m, {N});
  check(unlocked([&] {
    return llamarl_merge_partials(ptr<float>(m), ptr<float>(s), ptr<float>(zt), (int)shards, N, ptr<float>(logp), ptr<float>(lse),
                                  st.handle);
  }));
  st.returns(logp, lse);
  return tuple({logp, lse});
}

// logp, mu_logp, adv, mask, B, T, rho, norm_mode, clip_mode, eps_lo, eps_hi, targets, V, ws, stream
PyObject* offpolicy_loss_fwd(PyObject* const* a) {
  const at::Tensor &logp = needed(a[0], at::kFloat, "logp"), &mu = needed(a[1], at::kFloat, "mu_logp"),
                   &adv = needed(a[2], at::kFloat, "adv");
  const int64_t B = integer(a[4]), T = integer(a[5]), N = B * T;
  if (logp.numel() != N || mu.numel() != N || (adv.numel() != B && adv.numel() != N))
    invalid("shape mismatch between logp, mu_logp, adv and B*T");
  const int per_token = adv.numel() == N && N != B;
  const at::Tensor mask = optional(a[3], at::kByte, "mask");
  if (mask.defined() && mask.numel() != N) invalid("mask must have B*T entries");
  const at::Tensor targets = optional(a[11], at::kInt, "targets");
  at_least(targets, N, "targets");
  llamarl_loss_params p;
  p.rho = (float)real(a[6]);
  p.norm_mode = (int)integer(a[7]);
  p.clip_mode = (int)integer(a[8]);
  p.eps_lo = (float)real(a[9]);
  p.eps_hi = (float)real(a[10]);
  const int64_t V = integer(a[12]);
  const CallStream st(a[14], logp);
  const at::Tensor loss = empty(logp, {1}), coef = empty(logp, {N}), stats = empty(logp, {5});
  const at::Tensor ws = workspace(a[13], llamarl_workspace_bytes(N, 0, 0, LLAMARL_F32, LLAMARL_PASS_LOSS_FWD), logp);
  check(unlocked([&] {
    return llamarl_offpolicy_loss_fwd(ptr<float>(logp), ptr<float>(mu), ptr<float>(adv), per_token, ptr<uint8_t>(mask),
                                      ptr<int32_t>(targets), V, B, T, &p, ptr<float>(loss), ptr<float>(coef),
                                      ptr<float>(stats), ptr(ws), (size_t)ws.numel(), st.handle);
  }));
  st.returns(loss, coef, stats);
  return tuple({loss, coef, stats});
}

at::ScalarType storage(int64_t code, const at::Tensor& like) {      // binding's dtype code, negative: as `like`
  return code < 0 ? like.scalar_type() : code == LLAMARL_BF16 ? at::kBFloat16 : at::kFloat;
}

// H, W, targets, lse, coef, grad_loss, dW code, dW, accumulate, dH, ws, stream, max_rows (None: one pass)
PyObject* offpolicy_loss_bwd(PyObject* const* a) {
  const Head x(a[0], a[1], a[2], "W");
  const at::Tensor &lse = needed(a[3], at::kFloat, "lse"), &coef = needed(a[4], at::kFloat, "coef");
  x.holds("W", lse, coef);
  const float grad_loss = (float)real(a[5]);
  const int accumulate = PyObject_IsTrue(a[8]);
  if (accumulate < 0) throw Raised{};
  const CallStream st(a[11], x.H);
  at::Tensor dW, dH;
  if (a[7] != Py_None) dW = tensor(a[7], "dW");
  else if (accumulate) invalid("accumulate_dW needs an existing dW tensor");
  else dW = empty(x.H, {x.V, x.d}, storage(integer(a[6]), x.H));
  dH = a[9] != Py_None ? tensor(a[9], "dH") : empty(x.H, {x.N, x.d}, x.H.scalar_type());
  const llamarl_dtype dW_dt = dtype_code(dW);
  need(dW, dW.scalar_type(), "dW");
  need(dH, x.H.scalar_type(), "dH");
  at_least(dW, x.V * x.d, "dW");
  at_least(dH, x.N * x.d, "dH");
  const bool chunked = a[12] != Py_None;
  const int64_t rows = chunked ? integer(a[12]) : 0;
  const at::Tensor ws = workspace(a[10],
                                  chunked ? llamarl_bwd_workspace_bytes(x.N, x.d, x.V, x.dt, rows)
                                          : llamarl_workspace_bytes(x.N, x.d, x.V, x.dt, LLAMARL_PASS_LOSS_BWD), x.H);
  check(unlocked([&] {
    return chunked ? llamarl_offpolicy_loss_bwd_chunked(ptr(x.H), ptr(x.W), ptr<int32_t>(x.targets), ptr<float>(lse),
                                                        ptr<float>(coef), grad_loss, x.N, x.d, x.V, x.dt, ptr(dH), ptr(dW), dW_dt,
                                                        accumulate, rows, ptr(ws), (size_t)ws.numel(), st.handle)
                   : llamarl_offpolicy_loss_bwd(ptr(x.H), ptr(x.W), ptr<int32_t>(x.targets), ptr<float>(lse), ptr<float>(coef),
                                                grad_loss, x.N, x.d, x.V, x.dt, ptr(dH), ptr(dW), dW_dt, accumulate, ptr(ws),
                                                (size_t)ws.numel(), st.handle);
  }));
  if (a[9] == Py_None) st.returns(dH);
  if (a[7] == Py_None) st.returns(dW);
  return tuple({dH, dW});
}

// H, W_slice, targets, v0, lse, coef, grad_loss, dW code, ws, stream
PyObject* offpolicy_loss_bwd_slice(PyObject* const* a) {
  const Head x(a[0], a[1], a[2], "W_slice");
  const int64_t v0 = integer(a[3]);
  const at::Tensor &lse = needed(a[4], at::kFloat, "lse"), &coef = needed(a[5], at::kFloat, "coef");
  x.holds("W_slice", lse, coef);
  const float grad_loss = (float)real(a[6]);
  const CallStream st(a[9], x.H);
  const at::Tensor dH = empty(x.H, {x.N, x.d}, x.H.scalar_type()), dW = empty(x.H, {x.V, x.d}, storage(integer(a[7]), x.H));
  const at::Tensor ws = workspace(a[8], llamarl_workspace_bytes(x.N, x.d, x.V, x.dt, LLAMARL_PASS_LOSS_BWD), x.H);
  check(unlocked([&] {
    return llamarl_offpolicy_loss_bwd_slice(ptr(x.H), ptr(x.W), ptr<int32_t>(x.targets), ptr<float>(lse), ptr<float>(coef),
                                            grad_loss, x.N, x.d, x.V, v0, x.dt, ptr(dH), ptr(dW), dtype_code(dW), 0, ptr(ws),
                                            (size_t)ws.numel(), st.handle);
  }));
  st.returns(dH, dW);
  return tuple({dH, dW});
}

// H, W, targets, lse, coef, grad_loss (tensor), dW code, stream, checked.
// checked: the scalar is copied to the host on the way, the kernels are enqueued, then the copy is waited for and a scalar
// that is not finite refused (autograd.py).
PyObject* offpolicy_loss_bwd_device_scale(PyObject* const* a) {
  const Head x(a[0], a[1], a[2], "W");
  const at::Tensor &lse = needed(a[3], at::kFloat, "lse"), &coef = needed(a[4], at::kFloat, "coef"),
                   &g = needed(a[5], at::kFloat, "grad_loss");
  if (g.numel() != 1) invalid("grad_loss must have one entry");
  x.holds("W", lse, coef);
  const int checked = PyObject_IsTrue(a[8]);
  if (checked < 0) throw Raised{};
  const CallStream st(a[7], x.H);
  at::Tensor on_host;
  at::cuda::CUDAEvent copied;
  if (checked) {
    on_host = at::empty({}, at::TensorOptions().dtype(at::kFloat).pinned_memory(true));
    on_host.copy_(g.detach().reshape({}), /*non_blocking=*/true);
    copied.record();
  }
  const at::Tensor dH = empty(x.H, {x.N, x.d}, x.H.scalar_type()), dW = empty(x.H, {x.V, x.d}, storage(integer(a[6]), x.H));
  const at::Tensor ws = workspace(Py_None, llamarl_workspace_bytes(x.N, x.d, x.V, x.dt, LLAMARL_PASS_LOSS_BWD), x.H);
  check(unlocked([&] {
    return llamarl_offpolicy_loss_bwd_device_scale(ptr(x.H), ptr(x.W), ptr<int32_t>(x.targets), ptr<float>(lse), ptr<float>(coef),
                                                   ptr<float>(g), x.N, x.d, x.V, x.dt, ptr(dH), ptr(dW), dtype_code(dW), 0,
                                                   ptr(ws), (size_t)ws.numel(), st.handle);
  }));
  if (checked) {
    {
      const Unlocked u;
      copied.synchronize();
    }
    if (!std::isfinite(*on_host.data_ptr<float>())) invalid("grad_loss must be finite");
  }
  st.returns(dH, dW);
  return tuple({dH, dW});
}

// rewards, n, normalise_std, eps, stream
PyObject* group_advantages(PyObject* const* a) {
  const at::Tensor& r = needed(a[0], at::kFloat, "rewards");
  const int64_t n = integer(a[1]);
  if (n <= 0 || r.numel() % n != 0) invalid("rewards must hold P*n entries");
  const int std = PyObject_IsTrue(a[2]);
  if (std < 0) throw Raised{};
  const float eps = (float)real(a[3]);
  const CallStream st(a[4], r);
  const at::Tensor adv = empty(r, r.sizes());
  check(unlocked([&] { return llamarl_group_advantages(ptr<float>(r), r.numel() / n, n, std, eps, ptr<float>(adv), st.handle); }));
  st.returns(adv);
  return THPVariable_Wrap(adv);
}

// rewards, logp, base_logp, mask, lambda_kl, stream
PyObject* kl_shaped_rewards(PyObject* const* a) {
  const at::Tensor &r = needed(a[0], at::kFloat, "rewards"), &logp = needed(a[1], at::kFloat, "logp"),
                   &base = needed(a[2], at::kFloat, "base_logp");
  const at::Tensor mask = optional(a[3], at::kByte, "mask");
  const int64_t B = r.numel();
  if (B <= 0 || logp.numel() % B != 0 || base.numel() != logp.numel() || (mask.defined() && mask.numel() != logp.numel()))
    invalid("logp, base_logp and mask must hold B*T entries");
  const float lambda = (float)real(a[4]);
  const CallStream st(a[5], r);
  const at::Tensor shaped = empty(r, r.sizes()), kl = empty(r, r.sizes());
  check(unlocked([&] {
    return llamarl_kl_shaped_rewards(ptr<float>(r), ptr<float>(logp), ptr<float>(base), ptr<uint8_t>(mask), B, logp.numel() / B,
                                     lambda, ptr<float>(shaped), ptr<float>(kl), st.handle);
  }));
  st.returns(shaped, kl);
  return tuple({shaped, kl});
}

// The rules by which the library cuts and deals out its work (tile_rules.h), for tests.
// tiles_m, tiles_n, workgroups: the tiles (row * tiles_n + column) each workgroup of a logits kernel takes, in order
PyObject* tile_walk(PyObject* const* a) {
  const int tiles_m = (int)integer(a[0]), tiles_n = (int)integer(a[1]), workgroups = (int)integer(a[2]);
  PyObject* out = PyList_New(0);
  if (out == nullptr) throw Raised{};
  for (int b = 0; b < workgroups; ++b) {
    PyObject* walk = PyList_New(0);
    llamarl::TileSchedule<llamarl::PATCH_ROWS_LOGITS> sch;
    sch.init(tiles_m, tiles_n, b, workgroups);
    while (walk != nullptr && sch.has_tile()) {
      int tm, tn;
      sch.take(tm, tn);
      PyObject* id = PyLong_FromLongLong((int64_t)tm * tiles_n + tn);
      if (id == nullptr || PyList_Append(walk, id) != 0) Py_CLEAR(walk);
      Py_XDECREF(id);
    }
    const bool failed = walk == nullptr || PyList_Append(out, walk) != 0;
    Py_XDECREF(walk);
    if (failed) {
      Py_DECREF(out);
      throw Raised{};
    }
  }
  return out;
}

// active rows, bf16: columns of dz^T that the dW contraction reads
PyObject* dz_columns(PyObject* const* a) { return PyLong_FromLong(llamarl::dz_columns((int)integer(a[0]), integer(a[1]) != 0)); }
// N, V, d, bf16, backward: edge of a logits kernel's tiles
PyObject* logits_tile(PyObject* const* a) {
  const auto rule = integer(a[4]) ? llamarl::dz_tile : llamarl::logits_tile;
  return PyLong_FromLong(llamarl::tile_edge(rule(integer(a[0]), integer(a[1]), integer(a[2]), integer(a[3]) != 0)));
}
// M, columns, K, bf16: edge of a store contraction's tiles
PyObject* store_tile(PyObject* const* a) {
  return PyLong_FromLong(llamarl::tile_edge(llamarl::store_tile(integer(a[0]), integer(a[1]), integer(a[2]), integer(a[3]) != 0)));
}
// CUs, workgroups of the one and of the other a CU holds, whether the one and the other are long
PyObject* pair_workgroups(PyObject* const* a) {
  return PyLong_FromLong(llamarl::pair_workgroups((int)integer(a[0]), (int)integer(a[1]), (int)integer(a[2]), integer(a[3]) != 0, integer(a[4]) != 0));
}
// tiles_v, active rows, d, grid, backward: columns of the tiles of 256 vocabulary rows
PyObject* logits_width(PyObject* const* a) {
  const auto rule = integer(a[4]) ? llamarl::dz_width : llamarl::fwd_width;
  return PyLong_FromLong(rule((int)integer(a[0]), (int)integer(a[1]), integer(a[2]), (int)integer(a[3])).width);
}

template <PyObject* (*F)(PyObject* const*), int NARGS>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != NARGS) {
    PyErr_Format(PyExc_TypeError, "%d arguments expected, %zd given", NARGS, n);
    return nullptr;
  }
  try {
    return F(args);
  } catch (const Raised&) {
    return nullptr;
  }
  END_HANDLE_TH_ERRORS
}
#define ENTRY(name, nargs) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(entry<name, nargs>)), METH_FASTCALL, nullptr}

PyObject* set_error(PyObject*, PyObject* cls) {
  Py_INCREF(cls);
  Py_XDECREF(g_error);
  g_error = cls;
  Py_RETURN_NONE;
}

PyMethodDef g_methods[] = {
    ENTRY(token_logprobs, 6), ENTRY(token_logprobs_partial, 8), ENTRY(merge_partials, 4), ENTRY(offpolicy_loss_fwd, 15),
    ENTRY(offpolicy_loss_bwd, 13), ENTRY(offpolicy_loss_bwd_slice, 10), ENTRY(offpolicy_loss_bwd_device_scale, 9),
    ENTRY(group_advantages, 5), ENTRY(kl_shaped_rewards, 6), ENTRY(tile_walk, 3), ENTRY(logits_width, 5), ENTRY(dz_columns, 2), ENTRY(logits_tile, 5), ENTRY(store_tile, 4), ENTRY(pair_workgroups, 5), {"set_error", set_error, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&g_module); }
