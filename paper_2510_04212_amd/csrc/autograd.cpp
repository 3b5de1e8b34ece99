// The autograd node of attention() in C++ (host code only; every computation is behind the C ABI).
//
// What bounds a training step on short sequences is the host: one sequence of 128 tokens takes the
// GPU 15 us and took the Python node 75 to 145 us, depending on the machine (argument checks, allocations and
// ctypes conversions of both directions, and the interpreter lock the engine's thread has to wait for
// in the backward).  Forward + backward, Python node -> this one, on one machine (us): B1 H1 N128 d64
// 145 -> 76, B8 H12 N1024 d64 causal 164 -> 96 (92 of them on the GPU).
//
// apply() takes the plain case - bf16 tensors on the current GPU with shapes, strides, alignments and
// parameters the library accepts - and returns nothing for any other: the caller's Python node then
// handles it, or raises what it always raised.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/utils/pybind.h>
#include <ATen/ATen.h>
#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <c10/hip/HIPFunctions.h>
#include <cmath>
#include <optional>
#include "../../include/attn.h"
#include "row_offset.hpp"

namespace {

using at::Tensor;
using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

enum Form : int64_t { kPlain, kStrided, kGrouped, kRect };

void* current_stream(const Tensor& t) {
  return static_cast<void*>(c10::hip::getCurrentHIPStreamMasqueradingAsCUDA(t.get_device()).stream());
}

// A Python exception, thrown without the interpreter lock (in the backward on the engine's thread): it travels as
// torch's python_error.  Called with the lock held.
[[noreturn]] void raise(PyObject* type, PyObject* value) {
  PyErr_SetObject(type, value);
  python_error e;
  e.persist();
  throw e;
}

// binding.AttnError(status), as the Python node raises it.
void check(int status) {
  if (status == ATTN_OK) return;
  pybind11::gil_scoped_acquire lock;
  const auto type = pybind11::module_::import("paper_2510_04212_amd.binding").attr("AttnError");
  const pybind11::object error = type(status);
  raise(type.ptr(), error.ptr());
}

// What the backward gets from saved_tensors_hooks and hooks on the node can be anything: the ValueError of the
// Python node's checks instead of kernels on host memory or on strides that are not the tensor's.
void check_backward(Form form, const Tensor& q, const Tensor& k, const Tensor& v, const Tensor& o,
                    const Tensor& lse, const Tensor& dout) {
  auto bf16 = [&](const Tensor& t) {
    return t.defined() && t.layout() == at::kStrided && t.is_cuda() && t.device() == q.device() &&
           t.scalar_type() == at::kBFloat16 && t.dim() == 4 &&
           (form == kStrided ? t.stride(3) == 1 && t.strides() == q.strides() : t.is_contiguous());
  };
  const bool ok = bf16(q) && bf16(k) && bf16(v) && bf16(o) && bf16(dout) && o.sizes() == q.sizes() &&
                  dout.sizes() == q.sizes() && v.sizes() == k.sizes() && k.size(0) == q.size(0) &&
                  k.size(3) == q.size(3) && (form == kGrouped || k.size(1) == q.size(1)) &&
                  (form == kRect || k.size(2) == q.size(2)) && lse.defined() && lse.is_cuda() &&
                  lse.device() == q.device() && lse.scalar_type() == at::kFloat && lse.is_contiguous() &&
                  lse.numel() * q.size(3) == q.numel();
  if (ok) return;
  pybind11::gil_scoped_acquire lock;
  raise(PyExc_ValueError, pybind11::str("the tensors saved for the backward and the incoming gradient must be CUDA tensors of the "
                                        "shapes, types and layout of the forward").ptr());
}

struct Attention : torch::autograd::Function<Attention> {
  static Tensor forward(AutogradContext* ctx, const Tensor& q_in, const Tensor& k_in, const Tensor& v_in,
                        bool causal, double scale, int64_t variant, double beta, double eps) {
    Tensor q = q_in, k = k_in, v = v_in;
    Form form = k.size(1) != q.size(1) ? kGrouped : k.size(2) != q.size(2) ? kRect : kPlain;
    if (form == kPlain && !(q.is_contiguous() && k.is_contiguous() && v.is_contiguous()) &&
        q.strides() == k.strides() && q.strides() == v.strides() && q.stride(3) == 1)
      form = kStrided;
    if (form != kStrided) {
      q = q.contiguous();
      k = k.contiguous();
      v = v.contiguous();
    }
    const int B = (int)q.size(0), H = (int)q.size(1), Nq = (int)q.size(2), d = (int)q.size(3);
    const int Hkv = (int)k.size(1), Nk = (int)k.size(2);
    const bool strided = form == kStrided;
    Tensor o = strided ? at::empty_strided(q.sizes(), q.strides(), q.options()) : at::empty_like(q);
    Tensor lse = at::empty({B, H, Nq}, q.options().dtype(at::kFloat));
    Tensor ws;
    const size_t need = attn_fwd_workspace_bytes(B, H, Nq, Nk, d, causal, (int)variant);
    if (need > 0) ws = at::empty({(int64_t)need}, q.options().dtype(at::kByte));
    check(attn_fwd_ws(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), lse.data_ptr<float>(),
                      need > 0 ? ws.data_ptr() : nullptr, need, strided ? q.stride(0) : 0, strided ? q.stride(1) : 0,
                      strided ? q.stride(2) : 0, B, H, Hkv, Nq, Nk, d, causal, (float)scale, (int)variant,
                      (float)beta, (float)eps, current_stream(q)));
    ctx->save_for_backward({q, k, v, o, lse});
    ctx->saved_data["args"] = c10::IValue(std::vector<int64_t>{form, causal, variant});
    ctx->saved_data["scale"] = scale;
    return o;
  }

  static variable_list backward(AutogradContext* ctx, variable_list grads) {
    const variable_list saved = ctx->get_saved_variables();
    const Tensor &q = saved[0], &k = saved[1], &v = saved[2], &o = saved[3], &lse = saved[4];
    const auto args = ctx->saved_data["args"].toIntVector();
    const auto form = (Form)args[0];
    const int causal = (int)args[1], variant = (int)args[2];
    const float scale = (float)ctx->saved_data["scale"].toDouble();
    Tensor dout = grads[0];
    auto like = [&](const Tensor& t) {
      return form == kStrided ? at::empty_strided(t.sizes(), t.strides(), t.options()) : at::empty_like(t);
    };
    if (form != kStrided) {
      dout = dout.contiguous();
    } else if (dout.strides() != q.strides()) {
      Tensor copy = like(q);
      copy.copy_(dout);
      dout = copy;
    }
    check_backward(form, q, k, v, o, lse, dout);
    const int B = (int)q.size(0), H = (int)q.size(1), Nq = (int)q.size(2), d = (int)q.size(3);
    Tensor dq = like(q), dk = like(k), dv = like(v);
    const size_t bytes = std::max<size_t>(attn_bwd_workspace_bytes(B, H, Nq, d), 256);
    Tensor ws = at::empty({(int64_t)bytes}, q.options().dtype(at::kByte));
    void* st = current_stream(q);
    const void *Q = q.data_ptr(), *K = k.data_ptr(), *V = v.data_ptr(), *O = o.data_ptr(), *G = dout.data_ptr();
    const float* L = lse.data_ptr<float>();
    void *dQ = dq.data_ptr(), *dK = dk.data_ptr(), *dV = dv.data_ptr(), *W = ws.data_ptr();
    switch (form) {
      case kGrouped:
        check(attn_bwd_gqa(Q, K, V, O, G, L, dQ, dK, dV, W, bytes, B, H, (int)k.size(1), Nq, d, causal, scale, variant, st));
        break;
      case kRect:
        check(attn_bwd_rect(Q, K, V, O, G, L, dQ, dK, dV, W, bytes, B, H, Nq, (int)k.size(2), d, causal, scale, variant, st));
        break;
      case kStrided:
        check(attn_bwd_strided(Q, K, V, O, G, L, dQ, dK, dV, W, bytes, q.stride(0), q.stride(1), q.stride(2), B, H, Nq, d,
                               causal, scale, variant, st));
        break;
      case kPlain:
        check(attn_bwd(Q, K, V, O, G, L, dQ, dK, dV, W, bytes, B, H, Nq, d, causal, scale, variant, st));
        break;
    }
    return {dq, dk, dv, Tensor(), Tensor(), Tensor(), Tensor(), Tensor()};
  }
};

// Strides the kernels take (those of contiguous() always do).
bool strides_fit(const Tensor& t, int64_t d) {
  for (int i = 0; i < 3; ++i)
    if (t.stride(i) <= 0 || t.stride(i) % 8 != 0) return false;
  return t.stride(2) >= d && t.stride(2) < kRowStrideLimit;
}

bool plain(const Tensor& t, c10::DeviceIndex device) {
  return t.defined() && t.is_cuda() && t.layout() == at::kStrided && t.scalar_type() == at::kBFloat16 && t.dim() == 4 &&
         t.numel() > 0 && t.get_device() == device && !t.is_neg() &&
         reinterpret_cast<uintptr_t>(t.data_ptr()) % 16 == 0;
}

std::optional<Tensor> apply(const Tensor& q, const Tensor& k, const Tensor& v, bool causal, double scale,
                            int64_t variant, double beta, double eps) {
  if (!q.defined() || !q.is_cuda()) return std::nullopt;
  const auto device = c10::hip::current_device();
  if (!plain(q, device) || !plain(k, device) || !plain(v, device)) return std::nullopt;
  const int64_t d = q.size(3), H = q.size(1), Hkv = k.size(1);
  if (k.sizes() != v.sizes() || k.size(0) != q.size(0) || k.size(3) != d) return std::nullopt;
  if (Hkv != H && (k.size(2) != q.size(2) || H % Hkv != 0)) return std::nullopt;
  // the library's own limits: it refuses what is outside, and the Python node reports that
  if (attn_fwd_key_tile((int)d) == 0 || q.numel() >= (1ll << 31) || k.numel() >= (1ll << 31)) return std::nullopt;
  if (variant < ATTN_VARIANT_STANDARD || variant > ATTN_VARIANT_MITIGATED_ROW) return std::nullopt;
  const float s = (float)scale, b = (float)beta, e = (float)eps;
  if (!(s > 0.f) || !std::isfinite(s) || !(b > 1.f) || !std::isfinite(b) || !(e >= 0.f) || !std::isfinite(e)) return std::nullopt;
  if (!(q.is_contiguous() && k.is_contiguous() && v.is_contiguous()) && !strides_fit(q, d)) return std::nullopt;
  try {
    pybind11::gil_scoped_release release;
    return Attention::apply(q, k, v, causal, scale, variant, beta, eps);
  } catch (python_error& e) {        // pybind11 does not know the type
    e.restore();
    throw pybind11::error_already_set();
  }
}

}  // namespace

PYBIND11_MODULE(_autograd, m) {
  m.def("apply", &apply, "attention() with its gradient; None: not a plain case");
}
