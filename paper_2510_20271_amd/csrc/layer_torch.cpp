// The layer's autograd function in C++: the C ABI's calls of a training step with their tensors made, saved and handed
// on by torch's C++ interface.
//
// A step of the layer was bound by the host: five kernels of 55 us in all (32 x 512^2, 128 thresholds), and up to 150 us of
// Python around them -- marshalling for four calls, and a backward pass whose Python half waits for the interpreter on the
// engine's thread.  With this file a step takes 80 us where it took 154 (16 x 217 x 181 with 512 thresholds: 157 -> 81), and
// on a quicker host as long as its kernels, 52 where it took 73.
//
// layer.py takes this path for plain contiguous float32 tensors outside function transforms and tracing; everything else
// goes through its Python functions, whose results are the same.
#include <torch/extension.h>

#include <c10/hip/HIPStream.h>

#include <string>

#include "ecc.h"

namespace {

using torch::Tensor;
using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

// What the library refuses is the Python binding's EccError, with its status, in the backward pass as well.
void check(int status) {
  if (status == ECC_OK) return;
  const std::string message = ecc_last_error();  // (of this thread)
  const py::gil_scoped_acquire gil;
  const py::object type = py::module_::import("paper_2510_20271_amd.api").attr("EccError");
  const py::object error = type(status, message);
  PyErr_SetObject(type.ptr(), error.ptr());
  throw py::error_already_set();
}
void* stream() { return c10::hip::getCurrentHIPStream().stream(); }
float* f32(const Tensor& t) { return t.defined() ? t.data_ptr<float>() : nullptr; }
// Saved tensors come back from saved-tensor hooks, upstream gradients from anywhere: what the kernels are handed is as the
// forward pass made it, or nothing (numel < 0: any number of elements).
void check_device(const Tensor& t, at::ScalarType type, int64_t numel, const at::Device& device) {
  TORCH_CHECK_VALUE(t.defined() && t.layout() == at::kStrided && t.has_storage() && t.is_contiguous() && t.device() == device,
                    "tensors must be contiguous device tensors");
  TORCH_CHECK_VALUE(t.scalar_type() == type && (numel < 0 || t.numel() == numel),
                    "a saved tensor or gradient is not of the type or size that the forward pass left");
}
int64_t padded(int64_t n) { return (n + 63) / 64 * 64; }

// One buffer of floats: the direction, then (where wanted) d chi / d tau and d chi / d u, each at a multiple of 256 bytes.
struct Kept {
  float *u, *dtau, *du;
  static int64_t size(int64_t BT, int ndim, bool tau, bool u) { return 64 + (tau ? padded(BT) : 0) + (u ? BT * ndim : 0); }
  Kept(const Tensor& t, int64_t BT, bool tau, bool want_u) {
    u = t.data_ptr<float>();
    dtau = tau ? u + 64 : nullptr;
    du = want_u ? u + 64 + (tau ? padded(BT) : 0) : nullptr;
  }
};

// What the backward pass needs beside the saved tensors (in one entry of the context: each is a search by name).
// The workspace is not owned, so that one that was replaced by a larger one is not kept by the graphs of steps before.  Where
// it is gone, or the node is run on another stream than the forward pass (with whose calls it would not be safe), room is
// allocated.
struct Step : public torch::CustomClassHolder {
  float alpha, lam;
  bool tilted, u, tau;  // u, tau: derivatives that the forward pass has left
  int ndim;
  c10::weak_intrusive_ptr<at::TensorImpl, at::UndefinedTensorImpl> kept;
  int64_t bytes;
  void* on;
  Step(double alpha, double lam, bool tilted, int ndim, bool u, bool tau, const Tensor& ws)
      : alpha((float)alpha), lam((float)lam), tilted(tilted), u(u), tau(tau), ndim(ndim), kept(ws.getIntrusivePtr()),
        bytes(ws.numel()), on(stream()) {}
  Tensor workspace(const Tensor& like) const {
    if (on == stream())
      if (auto impl = kept.lock()) return Tensor(std::move(impl));
    return at::empty({bytes}, like.options().dtype(at::kByte));
  }
};

struct Angles : public torch::autograd::Function<Angles> {
  static Tensor forward(AutogradContext* ctx, const Tensor& grid, const Tensor& theta, const Tensor& tau, double alpha,
                        double lam, bool tilted, const Tensor& workspace, bool need_x, bool need_u, bool need_tau) {
    const int ndim = (int)grid.dim() - 1;
    const int64_t batch = grid.size(0), T = tau.numel(), BT = batch * T;
    const int64_t* dims = grid.sizes().data() + 1;
    const auto opts = grid.options();
    Tensor chi = at::empty({batch, T}, opts);
    Tensor kept = at::empty({Kept::size(BT, ndim, need_tau, need_u)}, opts);
    const size_t bytes = ecc_soft_state_bytes(ndim, dims, batch);
    Tensor state = at::empty({(int64_t)std::max<size_t>(bytes, 256)}, opts.dtype(at::kByte));
    const Kept k(kept, BT, need_tau, need_u);
    check(ecc_soft_direction(f32(theta), ndim, k.u, stream()));
    check(ecc_soft_fwd_save(f32(grid), ndim, dims, batch, k.u, (float)alpha, f32(tau), (int)T, (float)lam, tilted ? 1 : 0,
                            f32(chi), k.dtau, k.du, state.data_ptr(), (size_t)state.numel(), workspace.data_ptr(),
                            (size_t)workspace.numel(), stream()));
    // (the state only for the input's gradient; the angles only where theirs is wanted: a frozen direction may be changed
    // in place before the backward pass)
    ctx->save_for_backward({grid.detach(), kept, tau.detach(), need_x ? state : Tensor(), need_u ? theta : Tensor()});
    ctx->saved_data["step"] =
        at::IValue::make_capsule(c10::make_intrusive<Step>(alpha, lam, tilted, ndim, need_u, need_tau, workspace));
    return chi;
  }

  static variable_list backward(AutogradContext* ctx, variable_list grads) {
    const variable_list saved = ctx->get_saved_variables();
    const Tensor &grid = saved[0], &kept = saved[1], &tau = saved[2], &state = saved[3], &theta = saved[4];
    const Tensor g = grads[0].contiguous().to(at::kFloat);
    const auto step = c10::static_intrusive_pointer_cast<Step>(ctx->saved_data["step"].toCapsule());
    const bool made_u = step->u, made_tau = step->tau;
    const int ndim = step->ndim;
    check_device(grid, at::kFloat, -1, grid.device());
    TORCH_CHECK_VALUE(grid.is_cuda() && grid.dim() == ndim + 1, "grid must be a device tensor [batch, *item_shape]");
    const int64_t batch = grid.size(0), T = tau.numel(), BT = batch * T;
    const int64_t* dims = grid.sizes().data() + 1;
    check_device(tau, at::kFloat, -1, grid.device());
    check_device(kept, at::kFloat, Kept::size(BT, ndim, made_tau, made_u), grid.device());
    if (made_u) check_device(theta, at::kFloat, ndim - 1, grid.device());
    if (g.has_storage()) check_device(g, at::kFloat, BT, grid.device());
    const bool need_x = ctx->needs_input_grad(0), need_u = ctx->needs_input_grad(1) && made_u,
               need_tau = ctx->needs_input_grad(2) && made_tau;
    const Kept k(kept, BT, made_tau, made_u);
    Tensor grad_x, grad_theta, grad_tau;
    const Tensor ws = step->workspace(grid);
    if (need_x) {
      TORCH_CHECK(g.has_storage(), "the gradient of the input needs an upstream gradient with memory of its own");
      check_device(state, at::kByte, -1, grid.device());  // (its size is the library's to check)
      grad_x = at::empty(grid.sizes(), grid.options());
      check(ecc_soft_bwd_saved(f32(grid), ndim, dims, batch, k.u, step->alpha, f32(tau), (int)T, step->lam,
                               step->tilted ? 1 : 0, f32(g), f32(grad_x), state.data_ptr(), (size_t)state.numel(), ws.data_ptr(),
                               (size_t)ws.numel(), stream()));
    }
    if (need_u || need_tau) {
      if (!at::GradMode::is_enabled() && g.has_storage()) {
        if (need_tau) grad_tau = at::empty({T}, grid.options());
        if (need_u) grad_theta = at::empty({ndim - 1}, grid.options());
        check(ecc_soft_contract(f32(g), need_tau ? k.dtau : nullptr, need_u ? k.du : nullptr, need_u ? f32(theta) : nullptr,
                                batch, (int)T, ndim, f32(grad_tau), f32(grad_theta), ws.data_ptr(), (size_t)ws.numel(),
                                stream()));
      } else {  // a graph of the backward pass is wanted, or it runs over a batch of upstream gradients
        if (need_tau) grad_tau = (g * kept.narrow(0, 64, BT).view({batch, T})).sum(0);
        if (need_u) {
          const Tensor du = kept.narrow(0, 64 + (made_tau ? padded(BT) : 0), BT * ndim).view({batch, T, ndim});
          const Tensor d = at::einsum("bj,bjd->d", {g, du});
          const Tensor st = theta[0].sin(), ct = theta[0].cos();
          if (ndim == 2) {
            grad_theta = at::stack({ct * d[1] - st * d[0]});
          } else {
            const Tensor sp = theta[1].sin(), cp = theta[1].cos();
            grad_theta = at::stack({sp * (ct * d[1] - st * d[0]), cp * (ct * d[0] + st * d[1]) - sp * d[2]});
          }
        }
      }
    }
    return {grad_x, grad_theta, grad_tau, Tensor(), Tensor(), Tensor(), Tensor(), Tensor(), Tensor(), Tensor()};
  }
};

// chi [batch, T] of contiguous float32 tensors on the GPU: grid [batch, (D,) H, W], theta [ndim - 1], tau [T]; workspace:
// ecc_workspace_bytes and ecc_soft_contract_bytes, of the current stream
Tensor soft_angles(const Tensor& grid, const Tensor& theta, const Tensor& tau, double alpha, double lam, bool tilted,
                   const Tensor& workspace) {
  const bool graph = at::GradMode::is_enabled();
  const bool need_x = graph && grid.requires_grad(), need_u = graph && theta.requires_grad(),
             need_tau = graph && tau.requires_grad();
  if (need_x || need_u || need_tau)
    return Angles::apply(grid, theta, tau, alpha, lam, tilted, workspace, need_x, need_u, need_tau);
  const int ndim = (int)grid.dim() - 1;
  const int64_t batch = grid.size(0), T = tau.numel();
  Tensor chi = at::empty({batch, T}, grid.options());
  Tensor u = at::empty({4}, grid.options());
  check(ecc_soft_direction(f32(theta), ndim, f32(u), stream()));
  const auto fwd = tilted ? ecc_soft_fwd_tilted : ecc_soft_fwd;
  check(fwd(f32(grid), ndim, grid.sizes().data() + 1, batch, f32(u), (float)alpha, f32(tau), (int)T, (float)lam, f32(chi),
            workspace.data_ptr(), (size_t)workspace.numel(), stream()));
  return chi;
}

}  // namespace

PYBIND11_MODULE(TORCH_EXTENSION_NAME, m) {
  // (without the interpreter's lock, as the Python function's library calls: a launch waits when the device's queue is full)
  m.def("soft_angles", &soft_angles, "Soft curves with the direction given by its angles, differentiable",
        py::call_guard<py::gil_scoped_release>());
}
