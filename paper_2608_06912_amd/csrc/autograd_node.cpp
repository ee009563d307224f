// The autograd node of the full path in native code: p = LapSum_k(scores;
// alpha) over the last dimension and its analytical VJP, both through the C
// ABI on the caller's current stream.  A Python autograd.Function did the
// same with about 35 us more host time per forward + backward (the frames,
// the saved-tensor lists and the argument marshalling of the backward run in
// the engine's thread), which is more than the kernels of most rows take.
//
// What the two share: the forward saves p, the backward returns dL/dscores
// and, for k and alpha given as tensors that require grad, dL/dk and
// dL/dalpha summed over the rows.
#include <torch/extension.h>

#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <c10/core/DeviceGuard.h>

#include <torch/csrc/Exceptions.h>

#include <stdexcept>

#include "../../include/lapsum.h"

namespace {

using torch::Tensor;
using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

// A library call that failed, as the binding's own exception: LapsumError with
// the status and the entry point's name.
struct Failed : std::runtime_error {
  Failed(int status, const char* where) : std::runtime_error(where), status(status) {}
  int status;
};

void check(int status, const char* where) {
  if (status != LAPSUM_OK) throw Failed(status, where);
}

// Sets it as the current Python error (with the GIL held).
void set_error(const Failed& f) {
  const py::object type = py::module_::import("paper_2608_06912_amd").attr("LapsumError");
  PyErr_SetObject(type.ptr(), type(f.status, f.what()).ptr());
}

hipStream_t stream_of(const Tensor& x) {
  return c10::hip::getCurrentHIPStreamMasqueradingAsCUDA(x.device().index()).stream();
}

Tensor bytes(size_t n, const Tensor& like) {
  return n ? at::empty({static_cast<int64_t>(n)}, like.options().dtype(at::kByte)) : Tensor();
}

void* ptr(const Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; }

struct FullNode : public torch::autograd::Function<FullNode> {
  static Tensor forward(AutogradContext* ctx, const Tensor& scores,
                        const std::optional<Tensor>& k_like,
                        const std::optional<Tensor>& alpha_like, double k, double alpha, bool ste) {
    const c10::DeviceGuard guard(scores.device());
    Tensor x = scores.detach();
    if (x.scalar_type() != at::kFloat) x = x.to(at::kFloat);
    x = x.contiguous();
    const int64_t n = x.size(-1);
    const int64_t batch = n ? x.numel() / n : 0;
    Tensor p = at::empty(x.sizes(), x.options());
    Tensor b = at::empty({batch}, x.options().dtype(at::kDouble));
    const size_t need = lapsum_forward_workspace_size(batch, n, 0);
    Tensor ws = bytes(need, x);
    check(lapsum_forward(x.data_ptr<float>(), batch, n, k, alpha, p.data_ptr<float>(),
                         b.data_ptr<double>(), nullptr, ptr(ws), need, stream_of(x)),
          "lapsum_forward");
    // straight-through: the mask goes forward (p + (m - p) is m exactly in
    // float32), p's gradient backward
    Tensor out = p;
    if (ste) {
      out = at::empty(x.sizes(), x.options());
      const size_t mneed = lapsum_hard_mask_workspace_size(batch, n);
      Tensor mws = bytes(mneed, x);
      check(lapsum_hard_mask(x.data_ptr<float>(), batch, n, static_cast<int64_t>(k),
                             out.data_ptr<float>(), ptr(mws), mneed, stream_of(x)),
            "lapsum_hard_mask");
    }
    ctx->save_for_backward({p});
    ctx->saved_data["alpha"] = alpha;
    // (for their shape, dtype and device)
    if (k_like) ctx->saved_data["k_like"] = *k_like;
    if (alpha_like) ctx->saved_data["alpha_like"] = *alpha_like;
    return out;
  }

  static variable_list backward(AutogradContext* ctx, variable_list grads) {
    try {
      return vjp(ctx, grads);
    } catch (const Failed& f) {   // on the engine's thread
      const py::gil_scoped_acquire gil;
      set_error(f);
      python_error e;
      e.persist();
      throw e;
    }
  }

  static variable_list vjp(AutogradContext* ctx, const variable_list& grads) {
    const Tensor p = ctx->get_saved_variables()[0].detach();
    Tensor g = grads[0];
    if (!g.defined()) return variable_list(6);
    // (a saved-tensor hook can hand back any tensor; the kernels read p as
    // dense float32 rows in device memory)
    TORCH_CHECK_VALUE(p.is_cuda() && p.device() == g.device(),
                      "the saved p must be a CUDA (HIP) tensor on the gradient's device");
    TORCH_CHECK_VALUE(p.scalar_type() == at::kFloat, "the saved p must be float32");
    TORCH_CHECK_VALUE(p.layout() == at::kStrided && p.dim() >= 1 && p.is_contiguous(),
                      "the saved p must be contiguous");
    const c10::DeviceGuard guard(p.device());
    const at::AutoDispatchBelowADInplaceOrView below;
    if (g.scalar_type() != at::kFloat) g = g.to(at::kFloat);
    g = g.expand(p.sizes()).contiguous();
    const int64_t n = p.size(-1);
    const int64_t batch = p.numel() / n;
    auto like = [&](const char* name) {
      auto it = ctx->saved_data.find(name);
      return it == ctx->saved_data.end() ? Tensor() : it->second.toTensor();
    };
    const Tensor kl = like("k_like"), al = like("alpha_like");
    // (only the tensors given count as inputs of the node)
    const bool want_k = kl.defined() && ctx->needs_input_grad(1);
    const bool want_a = al.defined() && ctx->needs_input_grad(kl.defined() ? 2 : 1);
    Tensor params;
    double *gk = nullptr, *ga = nullptr;
    if (want_k || want_a) {
      params = at::empty({2, batch}, p.options().dtype(at::kDouble));
      gk = params.data_ptr<double>();
      ga = gk + batch;
    }
    Tensor grad = at::empty(p.sizes(), p.options());
    const double alpha = ctx->saved_data["alpha"].toDouble();
    const size_t need = lapsum_backward_workspace_size(batch, n);
    Tensor ws = bytes(need, p);
    check(lapsum_backward(g.data_ptr<float>(), p.data_ptr<float>(), nullptr, batch, n, alpha,
                          grad.data_ptr<float>(), gk, ga, ptr(ws), need, stream_of(p)),
          "lapsum_backward");
    Tensor grad_k, grad_a;
    if (params.defined()) {
      Tensor sums = batch == 1 ? params.select(1, 0) : params.sum(1);
      // one copy brings both to the host where either lives there
      const bool to_host = (want_k && kl.device().is_cpu()) || (want_a && al.device().is_cpu());
      const Tensor host = to_host ? sums.to(at::kCPU) : Tensor();
      auto pick = [&](int64_t i, const Tensor& as) {
        const Tensor& from = as.device().is_cpu() ? host : sums;
        return from.select(0, i).to(as.device(), as.scalar_type()).reshape(as.sizes()).clone();
      };
      if (want_k) grad_k = pick(0, kl);
      if (want_a) grad_a = pick(1, al);
    }
    if (!ctx->needs_input_grad(0)) grad = Tensor();
    return {grad, grad_k, grad_a, Tensor(), Tensor(), Tensor()};
  }
};

}  // namespace

PYBIND11_MODULE(TORCH_EXTENSION_NAME, m) {
  m.def("full", [](const Tensor& scores, const std::optional<Tensor>& k_like,
                   const std::optional<Tensor>& alpha_like, double k, double alpha, bool ste) {
    try {
      // without the GIL, as a ctypes call runs: an allocation or a launch can
      // wait for the device
      const py::gil_scoped_release nogil;
      return FullNode::apply(scores, k_like, alpha_like, k, alpha, ste);
    } catch (const Failed& f) {
      set_error(f);
      throw py::error_already_set();
    }
  });
}
