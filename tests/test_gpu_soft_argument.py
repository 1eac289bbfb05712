"""The argument of the sigmoid in the fused soft kernels: z = tau - X(p) - alpha <u, p>, with more than 256 thresholds
formed in float64 and rounded once, as the tile kernels form it.  A cone over the grid has one critical vertex (its tip, c = 1), so every sum is that
vertex's term alone and both kinds of kernels must agree to the bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2510_20271_amd import api
from tests.gpu_util import dev, host

pytestmark = pytest.mark.gpu

ALPHA, LAM = 0.013, 20.0


def _cone(shape, tip):
    axes = np.meshgrid(*[np.arange(n, dtype=np.float64) for n in shape], indexing="ij")
    r = np.sqrt(sum((a - t) ** 2 for a, t in zip(axes, tip)))
    return (0.731 + 0.1 * r).astype(np.float32)[None]


def _u(nd):
    return np.array([0.6, 0.8] if nd == 2 else [0.48, 0.6, 0.64], dtype=np.float32)


def _both(call):
    got = call()
    prev = api.ecc_debug_force(api.ECC_FORCE_SOFT_TILES)
    try:
        want = call()
    finally:
        api.ecc_debug_force(prev)
    return [(host(a), host(b)) for a, b in zip(got, want)]


@pytest.mark.parametrize("T", [257, 300, 1000])
@pytest.mark.parametrize("shape,tip", [((70, 90), (37, 53)), ((20, 300), (11, 271)), ((12, 30, 70), (7, 17, 41))])
def test_one_rounding_as_in_the_tile_kernels(shape, tip, T):
    nd = len(shape)
    X = dev(_cone(shape, tip))
    y = 0.731 + ALPHA * float(np.dot(_u(nd), tip[::-1]))
    tau = dev(np.linspace(y - 1.9, y + 2.3, T).astype(np.float32))  # (|lambda z| up to 66 bits: nothing is dropped)
    args = (X, nd, dev(_u(nd)), ALPHA, tau, LAM)
    for a, b in _both(lambda: (api.ecc_soft_fwd(*args), api.ecc_soft_bwd(*args)[1], *api.ecc_soft_fwd_save(*args)[:2])):
        np.testing.assert_array_equal(a, b)
    for j in (0, T // 3, T - 1):  # an upstream gradient for one threshold: one term in each entry of grad_X too
        g = torch.zeros(1, T, device="cuda")
        g[0, j] = 1.0

        def grad_x():
            state = api.ecc_soft_fwd_save(*args)[3]
            return api.ecc_soft_bwd(*args, grad_chi=g)[0], api.ecc_soft_bwd_saved(*args, state, grad_chi=g)
        for a, b in _both(grad_x):
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("side", [-1, 1])
@pytest.mark.parametrize("shape,tip", [((70, 90), (37, 53)), ((12, 30, 70), (7, 17, 41))])
def test_many_thresholds_drop_no_sigmoid_that_float32_holds(shape, tip, side):
    """All 300 sigmoids of the vertex between 2^-100 and 2^-70 (of 0 or of 1): their derivatives are kept."""
    nd = len(shape)
    X = dev(_cone(shape, tip))
    y = 0.731 + ALPHA * float(np.dot(_u(nd), tip[::-1]))
    bit = np.log(2.0) / LAM
    tau = dev((y + side * bit * np.linspace(70.0, 100.0, 300)).astype(np.float32))
    args = (X, nd, dev(_u(nd)), ALPHA, tau, LAM)
    pairs = _both(lambda: (api.ecc_soft_fwd(*args), api.ecc_soft_bwd(*args)[1], *api.ecc_soft_fwd_save(*args)[:2]))
    for a, b in pairs:
        np.testing.assert_array_equal(a, b)
    assert (pairs[1][0] > 0).all()

    def grad_x():
        state = api.ecc_soft_fwd_save(*args)[3]
        return api.ecc_soft_bwd(*args)[0], api.ecc_soft_bwd_saved(*args, state)
    for a, b in _both(grad_x):  # 300 positive terms in another order: 300 half ulps at the most
        assert np.max(np.abs(a - b)) <= 300 * 2.0 ** -24 * np.max(np.abs(b)) and np.max(np.abs(b)) > 0
