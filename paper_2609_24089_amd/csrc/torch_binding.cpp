// Native fast path of the Python binding: the entry points with freshly
// allocated outputs on the current stream and automatic column layouts, and
// attention() as C++ autograd functions.  Every function returns None for a call
// that it does not take (a check fails, tensors of a functorch or dispatch-mode
// level, tensor subclasses, tracing, forward-mode tangents); the Python code then
// runs the call and raises what is to be raised.  Small problems are bound by the
// host: bob() on one head of 64 rows took 107 us through ctypes and Python checks,
// of which the five launches are about 15.
#include <c10/hip/HIPStream.h>
#include <dlfcn.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>
#include <torch/extension.h>

#include <string>
#include <vector>

#include "../../include/flashbob.h"

namespace {

using at::Tensor;
using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

struct Api {
  decltype(&::attn_fwd_lse_gqa) fwd = nullptr;
  decltype(&::attn_bwd_gqa_ws) bwd = nullptr;
  decltype(&::attn_bob_pass1_rows_gqa) pass1 = nullptr;
  decltype(&::attn_bob_pass2_cols_gqa_ws) pass2 = nullptr;
  decltype(&::bob_bwd_workspace_bytes) bwd_bytes = nullptr;
  decltype(&::bob_pass2_workspace_bytes) pass2_bytes = nullptr;
  decltype(&::bob_status_string) status = nullptr;
} api;

// Take the entry points from the library at `path`.
void bind(const std::string& path) {
  void* lib = dlopen(path.c_str(), RTLD_NOW | RTLD_LOCAL);
  if (lib == nullptr) throw std::runtime_error(dlerror());
  auto take = [&](auto& fn, const char* name) {
    fn = reinterpret_cast<std::decay_t<decltype(fn)>>(dlsym(lib, name));
    if (fn == nullptr) throw std::runtime_error(std::string("missing symbol ") + name);
  };
  Api a;
  take(a.fwd, "attn_fwd_lse_gqa");
  take(a.bwd, "attn_bwd_gqa_ws");
  take(a.pass1, "attn_bob_pass1_rows_gqa");
  take(a.pass2, "attn_bob_pass2_cols_gqa_ws");
  take(a.bwd_bytes, "bob_bwd_workspace_bytes");
  take(a.pass2_bytes, "bob_pass2_workspace_bytes");
  take(a.status, "bob_status_string");
  api = a;
}

void ok(int32_t rc) {
  if (rc != BOB_OK) throw std::runtime_error(api.status(rc));
}

// Keys of tensors whose storage is not theirs to read (functorch levels,
// subclasses and modes with a Python dispatch, functionalization).
const c10::DispatchKeySet kWrapped({c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                    c10::DispatchKey::FuncTorchDynamicLayerFrontMode,
                                    c10::DispatchKey::FuncTorchDynamicLayerBackMode, c10::DispatchKey::Functionalize,
                                    c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot});

bool outside_modes() {
  return !c10::impl::tls_local_dispatch_key_set().included_.has_any(kWrapped) && !torch::jit::tracer::isTracing();
}

bool plain(const Tensor& t) {
  return t.defined() && t.is_cuda() && t.layout() == c10::kStrided && !t.key_set().has_any(kWrapped) &&
         t.is_contiguous() && !t.is_neg() && !t.is_conj();
}

struct Dims {
  int32_t code = 0;
  int64_t B = 0, H = 0, Hkv = 0, N = 0, d = 0;
};

using Refs = std::initializer_list<const Tensor*>;

// The checks of the Python binding; false: not for this path.
bool check(Refs qside, Refs kside, Refs rows, Dims& m) {
  const Tensor& q = **qside.begin();
  const Tensor& k = **kside.begin();
  if (!plain(q) || !plain(k) || q.dim() != 4 || k.dim() != 4) return false;
  if (q.scalar_type() == at::kBFloat16)
    m.code = BOB_BF16;
  else if (q.scalar_type() == at::kFloat)
    m.code = BOB_F32;
  else
    return false;
  m.B = q.size(0), m.H = q.size(1), m.N = q.size(2), m.d = q.size(3), m.Hkv = k.size(1);
  if (k.size(0) != m.B || k.size(2) != m.N || k.size(3) != m.d) return false;
  if (m.Hkv == 0 ? m.H != 0 : m.H % m.Hkv != 0) return false;
  auto same = [&](const Tensor& t, const Tensor& like) {
    return plain(t) && t.sizes() == like.sizes() && t.scalar_type() == q.scalar_type() && t.device() == q.device();
  };
  for (const Tensor* t : qside)
    if (!same(*t, q)) return false;
  for (const Tensor* t : kside)
    if (!same(*t, k)) return false;
  for (const Tensor* t : rows)
    if (!plain(*t) || t->scalar_type() != at::kFloat || t->sizes() != q.sizes().slice(0, 3) ||
        t->device() != q.device())
      return false;
  return true;
}

void* stream_of(const Tensor& t) {
  return (void*)c10::hip::getCurrentHIPStream(t.device().index()).stream();
}
Tensor rows_like(const Tensor& q) { return at::empty(q.sizes().slice(0, 3), q.options().dtype(at::kFloat)); }
const float* f(const Tensor& t) { return (const float*)t.const_data_ptr(); }
float* fm(const Tensor& t) { return (float*)t.mutable_data_ptr(); }
const void* p(const Tensor& t) { return t.const_data_ptr(); }
void* pm(const Tensor& t) { return t.mutable_data_ptr(); }

// The library launches on the current device: the calls below run with the
// tensors' device current.
struct Rows2 {
  Tensor O, L;
};
Rows2 run_fwd(const Dims& m, const Tensor& Q, const Tensor& K, const Tensor& V, double scale, bool causal) {
  Rows2 r{at::empty_like(Q), rows_like(Q)};
  ok(api.fwd(m.code, m.B, m.H, m.Hkv, m.N, m.d, (float)scale, causal, p(Q), p(K), p(V), pm(r.O), fm(r.L),
             stream_of(Q)));
  return r;
}

// fp32 partial sums of a split column kernel, from torch's allocator on the
// current stream.
Tensor workspace(int64_t bytes, const Tensor& q) {
  return bytes > 0 ? at::empty({bytes}, q.options().dtype(at::kByte)) : Tensor();
}

struct Bwd {
  Tensor dQ, dK, dV, D;
};
Bwd run_bwd(const Dims& m, const Tensor& Q, const Tensor& K, const Tensor& V, const Tensor& O, const Tensor& dO,
            const Tensor& L, double scale, bool causal) {
  Bwd r{at::empty_like(Q), at::empty_like(K), at::empty_like(K), rows_like(Q)};
  const int64_t bytes = api.bwd_bytes(m.code, m.B, m.H, m.Hkv, m.N, m.d, causal, nullptr);
  const Tensor ws = workspace(bytes, Q);
  ok(api.bwd(m.code, m.B, m.H, m.Hkv, m.N, m.d, (float)scale, causal, p(Q), p(K), p(V), p(O), p(dO), f(L), pm(r.dQ),
             pm(r.dK), pm(r.dV), fm(r.D), nullptr, bytes > 0 ? pm(ws) : nullptr, bytes, stream_of(Q)));
  return r;
}

struct P1 {
  Tensor Qt, dOt, alpha, E;
};
P1 run_pass1(const Dims& m, const Tensor& Q, const Tensor& K, const Tensor& V, const Tensor& O, const Tensor& dO,
             const Tensor& UQ, const Tensor& UK, const Tensor& UV, const Tensor& L, const Tensor& D, const Tensor& dQ,
             double scale, bool causal) {
  P1 r{at::empty_like(Q), at::empty_like(Q), rows_like(Q), rows_like(Q)};
  ok(api.pass1(m.code, m.B, m.H, m.Hkv, m.N, m.d, (float)scale, causal, p(Q), p(K), p(V), p(O), p(dO), p(UQ), p(UK),
               p(UV), f(L), f(D), dQ.defined() ? p(dQ) : nullptr, pm(r.Qt), pm(r.dOt), fm(r.alpha), fm(r.E),
               stream_of(Q)));
  return r;
}

struct P2 {
  Tensor Kt, Vt;
};
P2 run_pass2(const Dims& m, const Tensor& Q, const Tensor& K, const Tensor& V, const Tensor& dO, const Tensor& UQ,
             const Tensor& UK, const Tensor& UV, const Tensor& L, const Tensor& D, const Tensor& alpha,
             const Tensor& E, double scale, bool causal) {
  P2 r{at::empty_like(K), at::empty_like(K)};
  const int64_t bytes = api.pass2_bytes(m.code, m.B, m.H, m.Hkv, m.N, m.d, causal, nullptr);
  const Tensor ws = workspace(bytes, Q);
  ok(api.pass2(m.code, m.B, m.H, m.Hkv, m.N, m.d, (float)scale, causal, p(Q), p(K), p(V), p(dO), p(UQ), p(UK), p(UV),
               f(L), f(D), f(alpha), f(E), pm(r.Kt), pm(r.Vt), nullptr, bytes > 0 ? pm(ws) : nullptr, bytes,
               stream_of(Q)));
  return r;
}

// ---------------------------------------------------------------------------
// Python arguments
// ---------------------------------------------------------------------------
// Tensors and Parameters alone: another subclass has a say in the type of the
// outputs, which the Python code makes from its inputs.
bool tensors(std::initializer_list<py::handle> hs, std::vector<Tensor>& out) {
  out.reserve(hs.size());
  for (py::handle h : hs) {
    if (!THPVariable_CheckExact(h.ptr())) return false;
    out.push_back(THPVariable_Unpack(h.ptr()));
  }
  return outside_modes();
}

py::object py_fwd(py::handle q, py::handle k, py::handle v, double scale, bool causal) {
  std::vector<Tensor> t;
  Dims m;
  if (!tensors({q, k, v}, t) || !check({&t[0]}, {&t[1], &t[2]}, {}, m)) return py::none();
  Rows2 r;
  {
    py::gil_scoped_release free;
    c10::OptionalDeviceGuard guard(t[0].device());
    r = run_fwd(m, t[0], t[1], t[2], scale, causal);
  }
  return py::make_tuple(r.O, r.L);
}

py::object py_bwd(py::handle q, py::handle k, py::handle v, py::handle o, py::handle dO, py::handle L, double scale,
                  bool causal) {
  std::vector<Tensor> t;
  Dims m;
  if (!tensors({q, k, v, o, dO, L}, t) || !check({&t[0], &t[3], &t[4]}, {&t[1], &t[2]}, {&t[5]}, m)) return py::none();
  Bwd r;
  {
    py::gil_scoped_release free;
    c10::OptionalDeviceGuard guard(t[0].device());
    r = run_bwd(m, t[0], t[1], t[2], t[3], t[4], t[5], scale, causal);
  }
  return py::make_tuple(r.dQ, r.dK, r.dV, r.D);
}

py::object py_pass1(py::handle q, py::handle k, py::handle v, py::handle o, py::handle dO, py::handle uq,
                    py::handle uk, py::handle uv, py::handle L, py::handle D, double scale, bool causal,
                    py::object dq) {
  std::vector<Tensor> t;
  Dims m;
  Tensor dQ;
  if (!tensors({q, k, v, o, dO, uq, uk, uv, L, D}, t)) return py::none();
  if (!dq.is_none()) {
    if (!THPVariable_CheckExact(dq.ptr())) return py::none();
    dQ = THPVariable_Unpack(dq.ptr());
  }
  if (!check({&t[0], &t[3], &t[4], &t[5], dq.is_none() ? &t[0] : &dQ}, {&t[1], &t[2], &t[6], &t[7]}, {&t[8], &t[9]},
             m))
    return py::none();
  P1 r;
  {
    py::gil_scoped_release free;
    c10::OptionalDeviceGuard guard(t[0].device());
    r = run_pass1(m, t[0], t[1], t[2], t[3], t[4], t[5], t[6], t[7], t[8], t[9], dQ, scale, causal);
  }
  return py::make_tuple(r.Qt, r.dOt, r.alpha, r.E);
}

py::object py_pass2(py::handle q, py::handle k, py::handle v, py::handle dO, py::handle uq, py::handle uk,
                    py::handle uv, py::handle L, py::handle D, py::handle alpha, py::handle E, double scale,
                    bool causal) {
  std::vector<Tensor> t;
  Dims m;
  if (!tensors({q, k, v, dO, uq, uk, uv, L, D, alpha, E}, t) ||
      !check({&t[0], &t[3], &t[4]}, {&t[1], &t[2], &t[5], &t[6]}, {&t[7], &t[8], &t[9], &t[10]}, m))
    return py::none();
  P2 r;
  {
    py::gil_scoped_release free;
    c10::OptionalDeviceGuard guard(t[0].device());
    r = run_pass2(m, t[0], t[1], t[2], t[3], t[4], t[5], t[6], t[7], t[8], t[9], t[10], scale, causal);
  }
  return py::make_tuple(r.Kt, r.Vt);
}

// The whole path.  (O, L, dQ, dK, dV, D, Qt, dOt, alpha, E, Kt, Vt).
py::object py_bob(py::handle q, py::handle k, py::handle v, py::handle dO, py::handle uq, py::handle uk,
                  py::handle uv, double scale, bool causal, bool use_dq) {
  std::vector<Tensor> t;
  Dims m;
  if (!tensors({q, k, v, dO, uq, uk, uv}, t) ||
      !check({&t[0], &t[3], &t[4]}, {&t[1], &t[2], &t[5], &t[6]}, {}, m))
    return py::none();
  Rows2 a;
  Bwd b;
  P1 c;
  P2 e;
  {
    py::gil_scoped_release free;
    c10::OptionalDeviceGuard guard(t[0].device());
    a = run_fwd(m, t[0], t[1], t[2], scale, causal);
    b = run_bwd(m, t[0], t[1], t[2], a.O, t[3], a.L, scale, causal);
    c = run_pass1(m, t[0], t[1], t[2], a.O, t[3], t[4], t[5], t[6], a.L, b.D, use_dq ? b.dQ : Tensor(), scale, causal);
    e = run_pass2(m, t[0], t[1], t[2], t[3], t[4], t[5], t[6], a.L, b.D, c.alpha, c.E, scale, causal);
  }
  return py::make_tuple(a.O, a.L, b.dQ, b.dK, b.dV, b.D, c.Qt, c.dOt, c.alpha, c.E, e.Kt, e.Vt);
}

// ---------------------------------------------------------------------------
// attention() with two levels of reverse-mode derivatives, as the Python
// functions of autograd.py (which say what flows where): the engine runs them
// without a turn through Python.
// ---------------------------------------------------------------------------
Dims dims_or_throw(Refs qside, Refs kside, Refs rows) {
  Dims m;
  TORCH_CHECK_VALUE(check(qside, kside, rows, m),
                    "attention gradients must be contiguous and share the inputs' shape, dtype and device");
  return m;
}

struct AttentionBackward : torch::autograd::Function<AttentionBackward> {
  static variable_list forward(AutogradContext* ctx, const Tensor& q, const Tensor& k, const Tensor& v,
                               const Tensor& O, const Tensor& L, const Tensor& dO, double scale, bool causal) {
    const Dims m = dims_or_throw({&q, &O, &dO}, {&k, &v}, {&L});
    c10::OptionalDeviceGuard guard(q.device());
    Bwd r = run_bwd(m, q, k, v, O, dO, L, scale, causal);
    ctx->save_for_backward({q, k, v, O, L, dO, r.D, r.dQ});
    ctx->saved_data["scale"] = scale;
    ctx->saved_data["causal"] = causal;
    return {r.dQ, r.dK, r.dV};
  }
  static variable_list backward(AutogradContext* ctx, variable_list g) {
    const variable_list s = ctx->get_saved_variables();
    const double scale = ctx->saved_data["scale"].toDouble();
    const bool causal = ctx->saved_data["causal"].toBool();
    const Tensor &q = s[0], &k = s[1], &v = s[2], &O = s[3], &L = s[4], &dO = s[5], &D = s[6], &dQ = s[7];
    auto cotangent = [](const Tensor& t, const Tensor& like) {
      return t.defined() ? t.contiguous() : at::zeros_like(like);
    };
    const Tensor uq = cotangent(g[0], q), uk = cotangent(g[1], k), uv = cotangent(g[2], v);
    const Dims m = dims_or_throw({&q, &O, &dO, &uq, &dQ}, {&k, &v, &uk, &uv}, {&L, &D});
    c10::OptionalDeviceGuard guard(q.device());
    at::AutoGradMode no_graph(false);
    const P1 a = run_pass1(m, q, k, v, O, dO, uq, uk, uv, L, D, dQ, scale, causal);
    const P2 b = run_pass2(m, q, k, v, dO, uq, uk, uv, L, D, a.alpha, a.E, scale, causal);
    return {a.Qt, b.Kt, b.Vt, Tensor(), Tensor(), a.dOt, Tensor(), Tensor()};
  }
};

struct Attention : torch::autograd::Function<Attention> {
  static Tensor forward(AutogradContext* ctx, const Tensor& q, const Tensor& k, const Tensor& v, double scale,
                        bool causal) {
    const Dims m = dims_or_throw({&q}, {&k, &v}, {});
    c10::OptionalDeviceGuard guard(q.device());
    Rows2 r = run_fwd(m, q, k, v, scale, causal);
    ctx->save_for_backward({q, k, v, r.O, r.L});
    ctx->saved_data["scale"] = scale;
    ctx->saved_data["causal"] = causal;
    return r.O;
  }
  static variable_list backward(AutogradContext* ctx, variable_list g) {
    const variable_list s = ctx->get_saved_variables();
    const variable_list d =
        AttentionBackward::apply(s[0], s[1], s[2], s[3], s[4], g[0].contiguous(), ctx->saved_data["scale"].toDouble(),
                                 ctx->saved_data["causal"].toBool());
    return {d[0], d[1], d[2], Tensor(), Tensor()};
  }
};

py::object py_attention(py::handle q, py::handle k, py::handle v, double scale, bool causal) {
  std::vector<Tensor> t;
  Dims m;
  if (!tensors({q, k, v}, t) || !check({&t[0]}, {&t[1], &t[2]}, {}, m)) return py::none();
  for (const Tensor& x : t)
    if (x._fw_grad(0).defined()) return py::none();
  Tensor O;
  {
    py::gil_scoped_release free;
    O = Attention::apply(t[0], t[1], t[2], scale, causal);
  }
  return py::cast(O);
}

}  // namespace

PYBIND11_MODULE(TORCH_EXTENSION_NAME, m) {
  m.def("bind", &bind);
  m.def("fwd", &py_fwd);
  m.def("bwd", &py_bwd);
  m.def("pass1", &py_pass1);
  m.def("pass2", &py_pass2);
  m.def("bob", &py_bob);
  m.def("attention", &py_attention);
}
