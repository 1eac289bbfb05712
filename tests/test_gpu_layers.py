"""Soft forward in layers of blocks over the thresholds (few wave units, many thresholds): thresholds at the edges of a
layer, images and volumes, plain and saving, against the float64 oracle.  Sums of up to a few thousand float32 terms of
size <= 1 (derivatives: <= lambda / 4): 1e-4 of the largest value, 1e-3 for the derivatives, as for the other soft
tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import ecc_oracle as O
from paper_2510_20271_amd import api, synth
from tests.gpu_util import dev, host

pytestmark = pytest.mark.gpu


def _near(a, b, tol):
    assert np.max(np.abs(a - b)) <= tol * np.max(np.abs(b))


@pytest.mark.parametrize("T", [63, 64, 65, 128, 129, 255, 321, 513])
@pytest.mark.parametrize("shape", [(1, 40, 261), (3, 9, 8), (2, 7, 13, 70), (1, 31, 9, 65)])
def test_layers(T, shape):
    nd = len(shape) - 1
    X = synth.grf_batch(shape[0], shape[1:], 2.0, T)
    u = np.array([0.6, 0.8] if nd == 2 else [0.48, 0.6, 0.64], dtype=np.float32)
    lo, hi = float(X.min()), float(X.max())
    tau = np.linspace(lo, hi, T).astype(np.float32)
    alpha, lam = 0.01, 20.0
    g, ud, td = dev(X), dev(u), dev(tau)
    chi = O.soft_fwd_batch(X, u, alpha, tau, lam)
    gx, dt, du = O.soft_bwd_batch(X, u, alpha, tau, lam)
    _near(host(api.ecc_soft_fwd(g, nd, ud, alpha, td, lam)), chi, 1e-4)
    c, t, d, state = api.ecc_soft_fwd_save(g, nd, ud, alpha, td, lam)
    _near(host(c), chi, 1e-4)
    _near(host(t), dt, 1e-3)
    _near(host(d), du, 1e-3)
    _near(host(api.ecc_soft_bwd_saved(g, nd, ud, alpha, td, lam, state)), gx, 1e-3)
    a, t, d = api.ecc_soft_bwd(g, nd, ud, alpha, td, lam, grad_X=torch.full_like(g, float("nan")))
    _near(host(a), gx, 1e-3)  # (every element written, by the sweep's own clearing where c = 0)
    _near(host(t), dt, 1e-3)
    _near(host(d), du, 1e-3)


@pytest.mark.parametrize("shape,T", [((16, 217, 181), 449), ((16, 217, 181), 513), ((5, 300, 500), 300),
                                     ((6, 40, 60, 70), 513), ((6, 40, 60, 70), 300)])
def test_fewer_layers_than_slots(shape, T):
    """Several hundred wave units: more than one layer and several groups of 64 thresholds in each, the last layer
    shorter."""
    nd = len(shape) - 1
    X = synth.grf_batch(shape[0], shape[1:], 2.0, T)
    u = np.array([0.6, 0.8] if nd == 2 else [0.48, 0.6, 0.64], dtype=np.float32)
    tau = np.linspace(float(X.min()), float(X.max()), T).astype(np.float32)
    alpha, lam = 0.01, 20.0
    g, ud, td = dev(X), dev(u), dev(tau)
    chi = O.soft_fwd_batch(X, u, alpha, tau, lam)
    gx, dt, du = O.soft_bwd_batch(X, u, alpha, tau, lam)
    _near(host(api.ecc_soft_fwd(g, nd, ud, alpha, td, lam)), chi, 1e-4)
    c, t, d, state = api.ecc_soft_fwd_save(g, nd, ud, alpha, td, lam)
    _near(host(c), chi, 1e-4)
    _near(host(t), dt, 1e-3)
    _near(host(d), du, 1e-3)
    _near(host(api.ecc_soft_bwd_saved(g, nd, ud, alpha, td, lam, state)), gx, 1e-3)


@pytest.mark.parametrize("shape,T", [((1100, 9, 13), 257), ((9000, 8, 9), 40), ((400, 9, 13), 300), ((1024, 31, 33), 300), ((600, 70, 50), 513),
                                     ((1024, 9, 10, 11), 290)])
def test_forward_of_a_large_batch_of_small_items(shape, T):
    """The forward pass alone and the one that saves: the same to the bit; a few items against the oracle."""
    nd = len(shape) - 1
    X = torch.randn(shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(T))
    un = np.array([0.6, 0.8] if nd == 2 else [0.48, 0.6, 0.64], dtype=np.float32)
    u, tau = dev(un), torch.linspace(-3.0, 3.0, T, device="cuda")
    for tilted in (False, True):
        a = api.ecc_soft_fwd(X, nd, u, 0.01, tau, 20.0, tilted_c=tilted)
        assert torch.equal(a, api.ecc_soft_fwd_save(X, nd, u, 0.01, tau, 20.0, tilted_c=tilted, want=())[0])
    a = api.ecc_soft_fwd(X, nd, u, 0.01, tau, 20.0)
    for i in (0, shape[0] // 2, shape[0] - 1):
        _near(host(a[i]), O.soft_fwd_batch(host(X[i:i + 1]), un, 0.01, host(tau), 20.0)[0], 1e-4)
