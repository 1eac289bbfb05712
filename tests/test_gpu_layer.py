"""The autograd layer over the soft path: gradients that autograd hands back must be the
oracle's (float64) contracted with the same upstream gradient, and a toy fit must move the
direction and the thresholds towards the ones that produced the target curve."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import ecc_oracle as O
from paper_2510_20271_amd import layer, synth
from tests.gpu_util import dev, host

pytestmark = pytest.mark.gpu


from tests.test_gpu_soft import _close, _close_sum  # noqa: E402  (tolerances: see there)


@pytest.mark.parametrize("shape", [(48, 60), (10, 20, 24)])
def test_autograd_gradients_match_the_oracle(shape):
    nd = len(shape)
    B, T, alpha, lam = 3, 24, 0.02, 15.0
    X = np.stack([synth.grf(shape, 2.0, 70 + i) for i in range(B)])
    u = np.array([np.cos(0.4), np.sin(0.4)] if nd == 2 else [0.48, 0.6, 0.64], np.float32)
    tau = np.linspace(X.min(), X.max() + alpha * sum(shape), T).astype(np.float32)
    gup = np.random.default_rng(4).standard_normal((B, T)).astype(np.float32)

    g = dev(X).requires_grad_(True)
    ut = dev(u).requires_grad_(True)
    tt = dev(tau).requires_grad_(True)
    chi = layer.soft_ecc(g, ut, tt, alpha, lam)
    (chi * dev(gup)).sum().backward()

    want_chi = O.soft_fwd_batch(X, u, alpha, tau, lam)
    _close_sum(host(chi.detach()), want_chi, 1e-4, "chi")
    gX = np.zeros(X.shape)
    g_tau = np.zeros(T)
    g_u = np.zeros(nd)
    for b in range(B):
        gx_b, dtau_b, du_b = O.soft_bwd(X[b], u, alpha, tau, lam, gup[b])
        gX[b] = gx_b
        g_tau += gup[b] * dtau_b
        g_u += gup[b] @ du_b
    _close(host(g.grad), gX, 1e-3, "grad_X")
    _close_sum(host(tt.grad), g_tau, 1e-3, "grad_tau")
    _close_sum(host(ut.grad), g_u, 1e-3, "grad_u")


def _setup():
    shape = (64, 64)
    X = dev(np.stack([synth.grf(shape, 3.0, 90 + i) for i in range(4)]))
    lo, hi = float(X.min()), float(X.max()) + 0.01 * 128
    return X, lo, hi


def test_direction_gradient_through_the_angle_matches_finite_differences():
    X, lo, hi = _setup()
    target = layer.SoftECCLayer(2, 16, lo, hi, alpha=0.01, lam=12.0, theta=[0.9]).cuda()
    with torch.no_grad():
        want = target(X)

    def loss_at(theta):
        m = layer.SoftECCLayer(2, 16, lo, hi, alpha=0.01, lam=12.0, theta=[theta]).cuda()
        loss = ((m(X) - want) ** 2).sum()
        return m, loss

    m, loss = loss_at(0.5)
    loss.backward()
    g = float(m.theta.grad[0])
    h = 2e-3
    with torch.no_grad():
        fd = (float(loss_at(0.5 + h)[1]) - float(loss_at(0.5 - h)[1])) / (2 * h)
    assert abs(g - fd) <= 0.05 * max(abs(fd), 1e-6), (g, fd)
    n = m.direction()
    assert abs(float((n * n).sum().detach()) - 1.0) < 1e-6  # the direction stays on the unit circle


def test_layer_learns_its_thresholds_back():
    X, lo, hi = _setup()
    target = layer.SoftECCLayer(2, 16, lo, hi, alpha=0.01, lam=12.0)
    target.cuda()
    with torch.no_grad():
        want = target(X)
    model = layer.SoftECCLayer(2, 16, lo, hi, alpha=0.01, lam=12.0, learn_theta=False).cuda()
    with torch.no_grad():
        model.tau += 0.03
    opt = torch.optim.Adam([model.tau], lr=0.002)
    first = None
    for _ in range(200):
        opt.zero_grad()
        loss = ((model(X) - want) ** 2).mean()
        loss.backward()
        opt.step()
        first = first if first is not None else float(loss.detach())
    assert float(loss.detach()) < 0.1 * first
    assert float((model.tau - target.tau).abs().mean().detach()) < 0.015


@pytest.mark.parametrize("nd,B,T", [(2, 1, 1), (2, 3, 63), (3, 7, 65), (2, 32, 128), (3, 16, 512), (2, 2, 1500),
                                    (2, 33, 1025), (3, 600, 130), (2, 512, 64), (2, 513, 64), (3, 9000, 5),
                                    (2, 40000, 1), (2, 20011, 16), (3, 65535, 33), (2, 3001, 200), (2, 70, 4096)])
def test_contraction_with_the_upstream_gradient(nd, B, T):
    gen = torch.Generator(device="cuda").manual_seed(B * T)
    g, dtau = (torch.randn(B, T, generator=gen, device="cuda") for _ in range(2))
    du = torch.randn(B, T, nd, generator=gen, device="cuda")
    theta = torch.tensor([0.7, 1.9][:nd - 1], device="cuda")
    grad_tau, grad_u = layer.api.ecc_soft_contract(g, dtau, du, None, nd)
    _, grad_theta = layer.api.ecc_soft_contract(g, None, du, theta, nd)
    gd, t = g.double(), theta.double().requires_grad_()
    want_u = torch.einsum("bj,bjd->d", gd, du.double())
    u = [torch.cos(t[0]), torch.sin(t[0])]
    if nd == 3:
        u = [torch.sin(t[1]) * u[0], torch.sin(t[1]) * u[1], torch.cos(t[1])]
    (want_theta,) = torch.autograd.grad(torch.stack(u), t, want_u)
    # float64 sums rounded once to float32: half an ulp of the value, and nothing for the sums' own rounding
    for got, want in ((grad_tau, (gd * dtau.double()).sum(0)), (grad_u, want_u), (grad_theta, want_theta)):
        torch.testing.assert_close(got.double(), want, rtol=2.0 ** -24, atol=1e-12 * B * T)


class _Overridden(layer.SoftECCLayer):
    def direction(self):
        return super().direction()


@pytest.mark.parametrize("shape", [(20, 33), (9, 12, 17)])
@pytest.mark.parametrize("tilted", [False, True])
def test_layer_equals_its_parts_as_tensor_operations(shape, tilted):
    """The direction and the contraction inside the layer against those of the general path."""
    nd = len(shape)
    X = dev(np.stack([synth.grf(shape, 2.0, 190 + i) for i in range(3)]))
    g = torch.randn(3, 40, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    out = []
    for cls in (layer.SoftECCLayer, _Overridden):
        m = cls(nd, 40, float(X.min()), float(X.max()) + 0.4, alpha=0.02, theta=[0.3, 1.1][:nd - 1],
                tilted_c=tilted).cuda()
        x = X.clone().requires_grad_()
        chi = m(x)
        out.append((chi,) + torch.autograd.grad(chi, [x, m.tau, m.theta], g, retain_graph=True))
        # the graph of the backward pass, and a batch of upstream gradients at once
        gg = g.clone().requires_grad_()
        d_tau, d_theta = torch.autograd.grad(chi, [m.tau, m.theta], gg, create_graph=True, retain_graph=True)
        out[-1] += (d_tau, d_theta) + torch.autograd.grad(d_tau.sum() + d_theta.sum(), [gg])
        m.theta.requires_grad_(False)
        out[-1] += torch.autograd.grad(m(X), [m.tau], torch.stack([g, 2 * g]), is_grads_batched=True)
    for a, b in zip(*out):  # chi and grad_X: the same kernels; the others: float32 sums of some 100 terms
        torch.testing.assert_close(a, b, rtol=1e-4, atol=1e-4 * float(b.detach().abs().max()))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


def test_direction_is_that_of_the_tensor_operations():
    theta = torch.linspace(-7.0, 7.0, 400, device="cuda")
    for nd in (2, 3):
        m = layer.SoftECCLayer(nd, 2, 0.0, 1.0).cuda()
        for i in range(0, 400, 7):
            with torch.no_grad():
                m.theta.copy_(theta[[i, 399 - i]][:nd - 1])
            assert torch.equal(layer.api.ecc_soft_direction(m.theta.detach()), m.direction().detach())


@pytest.mark.parametrize("shape", [(20, 33), (9, 12, 17)])
def test_frozen_direction_changed_between_forward_and_backward(shape):
    """One backward pass over the curves of several directions, the layer's angle(s) set in place in between."""
    nd = len(shape)
    X = dev(np.stack([synth.grf(shape, 2.0, 290 + i) for i in range(2)]))
    m = layer.SoftECCLayer(nd, 24, float(X.min()), float(X.max()) + 0.4, alpha=0.02, learn_theta=False).cuda()
    X.requires_grad_()
    angles = [torch.tensor([a, 0.5 + a][:nd - 1], device="cuda") for a in (0.2, 0.9, 2.5)]
    alone = []
    for a in angles:
        with torch.no_grad():
            m.theta.copy_(a)
        alone.append(torch.autograd.grad(m(X).sum(), [X, m.tau]))
    outs = []
    for a in angles:
        with torch.no_grad():
            m.theta.copy_(a)
        outs.append(m(X).sum())
    for got, parts in zip(torch.autograd.grad(sum(outs), [X, m.tau]), zip(*alone)):
        # the same kernels; autograd adds the three in an order of its own, in float32
        torch.testing.assert_close(got, sum(parts), rtol=1e-5, atol=1e-6 * float(sum(p.abs().max() for p in parts)))
