"""Strip sweep on rows that start anywhere: widths around a lane's four columns, a strip's 248 and a wave's 256, and
grids that begin in the middle of a dword.  Enough rows that the plain kernels of tiny inputs do not take them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import ecc_oracle as O
from oracle import ecc_oracle_c as OC
from paper_2510_20271_amd import api
from tests.gpu_util import host

pytestmark = pytest.mark.gpu

KINDS = {"u8": torch.uint8, "u16": torch.uint16, "i16": torch.int16, "f16": torch.float16, "bf16": torch.bfloat16,
         "f32": torch.float32}


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("W", [8, 9, 31, 63, 250, 255, 256, 257, 258, 259, 260, 497, 502, 505])
def test_odd_rows(kind, W):
    rng = np.random.default_rng(W)
    H = 65536 // (2 * W) + 3
    n = 2 * H * W
    for start in (0, 1, 2, 3):  # elements before the grid
        a = rng.integers(5, 45, size=start + n).astype(np.int16)
        t = torch.from_numpy(a).cuda()
        t = t.view(torch.uint16) if kind == "u16" else t.to(KINDS[kind])
        g = t[start:].view(2, H, W)
        Y = a[start:].reshape(2, H, W).astype(np.float32)
        levels = kind in ("u8", "u16")
        th = O.thresholds_levels(50) if levels else O.thresholds_equal_width(8.0, 40.0, 50)
        rng_arg = None if levels else (8.0, 40.0)
        np.testing.assert_array_equal(host(api.ecc_hard(g, 2, 50, range=rng_arg)), OC.ecc_hard_batch(Y, th))
        if kind in ("f16", "bf16", "f32") and start < 2:  # lists, the range tracked on the way
            want = OC.ecc_hard_batch(Y, O.thresholds_equal_width(Y.min(), Y.max(), 50))
            prev = api.ecc_debug_force(api.ECC_FORCE_NO_SMALL)
            try:
                np.testing.assert_array_equal(host(api.ecc_hard(g, 2, 50)), want)
            finally:
                api.ecc_debug_force(prev)
            np.testing.assert_array_equal(host(api.ecc_hard(g, 2, 50)), want)
