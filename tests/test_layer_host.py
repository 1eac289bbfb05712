"""What the autograd functions of the layer keep for the backward pass.  The library calls are replaced by small tensor
formulas, so that this runs without a GPU."""
import pytest

torch = pytest.importorskip("torch")

from paper_2510_20271_amd import layer


@pytest.fixture
def stubbed(monkeypatch):
    def fwd_save(grid, ndim, u, alpha, tau, lam, tilted_c=False, want=()):
        batch, T = grid.shape[0], tau.numel()
        dtau = torch.ones(batch, T) if "dchi_dtau" in want else None
        du = u.repeat(batch, T, 1) if "dchi_du" in want else None
        return tau.repeat(batch, 1), dtau, du, torch.zeros(8)

    def contract(g, dtau=None, du=None, theta=None, ndim=2):
        return (None if dtau is None else (g * dtau).sum(0)), (None if du is None else theta * (g * du[..., 0]).sum())

    monkeypatch.setattr(layer.api, "ecc_soft_direction",
                        lambda t: torch.cat([torch.cos(t[:1]), torch.sin(t[:1])]), raising=True)
    monkeypatch.setattr(layer.api, "ecc_soft_fwd_save", fwd_save)
    monkeypatch.setattr(layer.api, "ecc_soft_contract", contract)
    monkeypatch.setattr(layer.api, "ecc_soft_bwd_saved", lambda grid, *a, **k: torch.ones_like(grid))


def test_a_frozen_angle_may_change_before_the_backward_pass(stubbed):
    theta, tau = torch.tensor([0.3]), torch.zeros(5, requires_grad=True)
    grid = torch.zeros(2, 4, 4, requires_grad=True)
    outs = []
    for a in (0.1, 0.7):
        theta.copy_(torch.tensor([a]))
        outs.append(layer._SoftECCAngles.apply(grid, theta, tau, 0.01, 20.0, False).sum())
    sum(outs).backward()
    assert torch.equal(tau.grad, torch.full((5,), 4.0)) and torch.equal(grid.grad, torch.full((2, 4, 4), 2.0))


def test_a_learned_angle_is_kept(stubbed):
    theta, tau = torch.tensor([0.3], requires_grad=True), torch.zeros(5)
    chi = layer._SoftECCAngles.apply(torch.zeros(2, 4, 4), theta, tau, 0.01, 20.0, False)
    chi.sum().backward()
    torch.testing.assert_close(theta.grad, 0.3 * 10 * torch.cos(torch.tensor([0.3])))
