"""Differentiable ECC layer over the C ABI (the paper's "differentiable PyTorch layer").

``SoftECCFunction`` is a ``torch.autograd.Function``: forward is ``ecc_soft_fwd_save`` (Eq. 6, plus the
sums of Eq. 9-10, which share its sigmoids, and the saved list of critical vertices), backward is
``ecc_soft_bwd_saved`` (Eq. 8 over that list; appendix on analytical derivatives).  The kernels
return d chi / d tau and d chi / d u uncontracted ([batch, T] and [batch, T, ndim]); the two
small contractions with the upstream gradient that autograd needs are ``ecc_soft_contract`` (tensor
operations only where a graph of the backward pass is asked for).  ``SoftECCLayer`` holds the learnable thresholds and a direction kept on the unit
sphere by reparametrisation (an angle in 2D, two angles in 3D), as the main text suggests.  For plain tensors
it runs the same calls through the C++ twin of ``_SoftECCAngles`` (``csrc/layer_torch.cpp``), which spares a step most
of its host work.

Inputs must live on the GPU; there is no CPU path.
"""
from __future__ import annotations

import math

import torch

from . import api


def _forward(ctx, grid, u, tau, alpha, lam, tilted_c, theta=None):
    """Forward of both functions below; theta: the angles u comes from, when they are what is learned."""
    ndim = grid.dim() - 1
    grid_c = grid.detach().contiguous().float()
    tau_c = tau.detach().contiguous().float()
    ctx.alpha, ctx.lam, ctx.ndim, ctx.tilted_c = float(alpha), float(lam), ndim, bool(tilted_c)
    need_x, need_u, need_tau = ctx.needs_input_grad[:3]
    if not (need_x or need_u or need_tau):
        return api.ecc_soft_fwd(grid_c, ndim, u, alpha, tau_c, lam, tilted_c=ctx.tilted_c)
    # The forward kernel shares its sigmoids with the sums of Eq. 9 / Eq. 10 and finds the vertices
    # with c != 0 that Eq. 8 needs: it returns the former and saves the latter, so backward() neither
    # sweeps the grid again nor, with fixed inputs and learnable thresholds (the usual case), runs more
    # than the small contraction.
    want = [n for n, need in (("dchi_du", need_u), ("dchi_dtau", need_tau)) if need]
    chi, dtau, du, state = api.ecc_soft_fwd_save(grid_c, ndim, u, alpha, tau_c, lam, tilted_c=ctx.tilted_c, want=want)
    # (the angles only where their gradient is wanted: a frozen direction may be changed in place before backward())
    ctx.save_for_backward(grid_c, u, tau_c, state if need_x else None, dtau, du, theta if need_u else None)
    return chi


def _backward(ctx, grad_chi):
    """Gradients with respect to the grid, the direction (or the angles) and the thresholds."""
    grid, u, tau, state, dtau, du, theta = ctx.saved_tensors
    g = grad_chi.contiguous().float()
    need_x, need_u, need_tau = ctx.needs_input_grad[:3]
    grad_X = None
    if need_x:
        grad_X = api.ecc_soft_bwd_saved(grid, ctx.ndim, u, ctx.alpha, tau, ctx.lam, state, grad_chi=g,
                                        tilted_c=ctx.tilted_c)
    if not (need_u or need_tau):
        return grad_X, None, None
    if not torch.is_grad_enabled() and _has_memory(g):
        grad_tau, grad_dir = api.ecc_soft_contract(g, dtau, du, theta, ctx.ndim)
        return grad_X, grad_dir, grad_tau
    # a graph of the backward pass is wanted, or it runs over a batch of upstream gradients (thresholds alone)
    grad_dir = torch.einsum("bj,bjd->d", g, du) if need_u else None
    if need_u and theta is not None:
        st, ct = torch.sin(theta[0]), torch.cos(theta[0])
        if ctx.ndim == 2:
            grad_dir = torch.stack([ct * grad_dir[1] - st * grad_dir[0]])
        else:
            sp, cp = torch.sin(theta[1]), torch.cos(theta[1])
            grad_dir = torch.stack([sp * (ct * grad_dir[1] - st * grad_dir[0]),
                                    cp * (ct * grad_dir[0] + st * grad_dir[1]) - sp * grad_dir[2]])
    grad_tau = (g * dtau).sum(0) if need_tau else None
    return grad_X, grad_dir, grad_tau


def _has_memory(t) -> bool:
    """False for the wrappers that function transforms pass around."""
    try:
        t.data_ptr()
    except RuntimeError:
        return False
    return True


class SoftECCFunction(torch.autograd.Function):
    """chi[b, j] = sum_p c(p) sigmoid(lambda (tau_j - X_b(p) - alpha <u, p>)), p = (x, y[, z])."""

    @staticmethod
    def forward(ctx, grid, u, tau, alpha: float, lam: float, tilted_c: bool = False):
        return _forward(ctx, grid, u.detach().contiguous().float(), tau, alpha, lam, tilted_c)

    @staticmethod
    def backward(ctx, grad_chi):
        return *_backward(ctx, grad_chi), None, None, None


class _SoftECCAngles(torch.autograd.Function):
    """The same with the direction given by its angle(s): the gradient comes back for the angles."""

    @staticmethod
    def forward(ctx, grid, theta, tau, alpha: float, lam: float, tilted_c: bool):
        return _forward(ctx, grid, api.ecc_soft_direction(theta.detach()), tau, alpha, lam, tilted_c, theta=theta)

    @staticmethod
    def backward(ctx, grad_chi):
        return *_backward(ctx, grad_chi), None, None, None


_PLAIN = (torch.Tensor, torch.nn.Parameter)


def _native_takes(grid, theta, tau, ndim: int) -> bool:
    """What the C++ function is for: plain contiguous float32 tensors of the layer's shapes on one GPU, outside function
    transforms, dispatch modes, tracing, compilation and forward-mode differentiation."""
    return (type(grid) in _PLAIN and type(tau) in _PLAIN and grid.is_cuda and tau.is_cuda
            and grid.dtype is torch.float32 and tau.dtype is torch.float32
            and grid.dim() == ndim + 1 and tau.dim() == 1 and theta.dim() == 1
            and grid.get_device() == tau.get_device() == theta.get_device()
            and grid.is_contiguous() and tau.is_contiguous()
            and not torch._C._are_functorch_transforms_active() and torch._C._len_torch_dispatch_stack() == 0
            and torch._C._get_tracing_state() is None and not torch.compiler.is_compiling()
            and torch.autograd.forward_ad._current_level < 0)


_soft_angles = None


def _native():
    global _soft_angles
    if _soft_angles is None:
        api._lib.load()
        try:
            from . import _layer_native
        except ImportError as e:
            raise RuntimeError("_layer_native.so is missing: build it with `python -m paper_2510_20271_amd.build`") from e
        _soft_angles = _layer_native.soft_angles
    return _soft_angles


def soft_ecc(grid, u, tau, alpha: float, lam: float, tilted_c: bool = False):
    """Functional form: grid [batch, (D,) H, W] float32 on the GPU, u [ndim], tau [T].
    tilted_c: take c(p) from the tilted field X + alpha <u, p> (so that a sharp sigmoid gives
    the directional hard curve) instead of from X; c stays a constant for the derivatives."""
    return SoftECCFunction.apply(grid, u, tau, alpha, lam, tilted_c)


class SoftECCLayer(torch.nn.Module):
    """Soft directional ECC with learnable thresholds and direction.

    tau:   T thresholds, initialised evenly over [tau_min, tau_max].
    theta: the direction's angle(s): u = (cos t, sin t) in 2D; in 3D u = (sin p cos t,
           sin p sin t, cos p) with theta = (t, p).  ||u|| = 1 by construction.
    alpha (weight of the tilt) and lam (sharpness of the sigmoid) are fixed.
    tilted_c: c(p) of the tilted field instead of the field's own (see soft_ecc).
    """

    def __init__(self, ndim: int, T: int, tau_min: float, tau_max: float, alpha: float = 0.01,
                 lam: float = 20.0, theta=None, learn_tau: bool = True, learn_theta: bool = True,
                 tilted_c: bool = False):
        super().__init__()
        if ndim not in (2, 3):
            raise ValueError("ndim must be 2 or 3")
        self.ndim, self.alpha, self.lam, self.tilted_c = ndim, float(alpha), float(lam), bool(tilted_c)
        tau = torch.linspace(float(tau_min), float(tau_max), T, dtype=torch.float32)
        if theta is None:
            theta = [0.3] if ndim == 2 else [0.3, 0.5 * math.pi]
        theta = torch.as_tensor(theta, dtype=torch.float32).reshape(ndim - 1)
        self.tau = torch.nn.Parameter(tau, requires_grad=learn_tau)
        self.theta = torch.nn.Parameter(theta, requires_grad=learn_theta)

    def direction(self) -> torch.Tensor:
        t = self.theta
        if self.ndim == 2:
            return torch.stack([torch.cos(t[0]), torch.sin(t[0])])
        return torch.stack([torch.sin(t[1]) * torch.cos(t[0]), torch.sin(t[1]) * torch.sin(t[0]),
                            torch.cos(t[1])])

    def forward(self, grid: torch.Tensor) -> torch.Tensor:
        # The direction inside the autograd function: two launches instead of some fifteen small tensor operations,
        # which took most of a step's time on the host.  Only for the layer's own direction() and plain angles.
        theta = self.theta
        own = type(self).direction is SoftECCLayer.direction and "direction" not in self.__dict__
        if (own and type(theta) in (torch.nn.Parameter, torch.Tensor) and theta.is_cuda and theta.is_contiguous()
                and theta.dtype == torch.float32 and theta.numel() == self.ndim - 1):
            tau = self.tau
            if _native_takes(grid, theta, tau, self.ndim) and grid.numel() and tau.numel():
                ws = api.soft_step_workspace(tuple(grid.shape[1:]), grid.shape[0], tau.numel(), grid.device)
                return _native()(grid, theta, tau, float(self.alpha), float(self.lam), bool(self.tilted_c), ws)
            return _SoftECCAngles.apply(grid, theta, self.tau, self.alpha, self.lam, self.tilted_c)
        return soft_ecc(grid, self.direction(), self.tau, self.alpha, self.lam, self.tilted_c)
