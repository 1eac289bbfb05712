"""Rows per wave of the strip sweep, over what the launch plan chooses: the same integer curves as the plain
one-thread-per-vertex kernels (whole numbers: equal)."""
import pytest

torch = pytest.importorskip("torch")

from paper_2510_20271_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,dtype,bins,known", [
    ((9000, 64, 64), torch.uint8, 256, True),     # histogram sweeps: 16 rows, a block an image
    ((1100, 100, 310), torch.uint8, 256, True),   # 8, two strips wide
    ((1030, 190, 200), torch.float32, 100, True),  # 24
    ((600, 256, 256), torch.float32, 100, True),  # 32
    ((3, 2048, 2048), torch.uint8, 256, True),    # 8, blocks that share rows of the histogram
    ((1, 2050, 2047), torch.float32, 64, True),   # 8
    ((2780, 144, 112), torch.float32, 256, True),  # 40, a block an image
    ((300, 384, 384), torch.float32, 4096, True),  # 48
    ((200, 245, 627), torch.float32, 4096, True),  # 64
    ((3000, 270, 143), torch.float16, 1024, True),  # 72
    ((600, 300, 250), torch.float16, 4096, True),  # 80
    ((200, 500, 300), torch.float32, 4096, True),  # 88
    ((5000, 30, 41), torch.float32, 64, False),   # lists that blocks share, four units an image
    ((4200, 64, 50), torch.float32, 64, False),
    ((4200, 65, 50), torch.float32, 64, False),
    ((1, 30000, 30), torch.float32, 64, False),   # a list per block, narrow grids
    ((1, 500000, 9), torch.float32, 64, False),
    ((1024, 128, 128), torch.float32, 64, False),  # a list per block, a block an image: 32, 24 and 40 rows a wave
    ((1030, 69, 171), torch.float16, 64, False),
    ((1100, 142, 57), torch.float32, 64, False),
    ((33, 1024, 1024), torch.float64, 64, False),
])
def test_curves_equal_those_of_the_plain_kernels(shape, dtype, bins, known):
    gen = torch.Generator(device="cuda").manual_seed(sum(shape))
    if dtype == torch.uint8:
        x, rng = torch.randint(0, 256, shape, generator=gen, device="cuda", dtype=torch.int16).to(dtype), None
    else:
        x, rng = torch.randn(shape, generator=gen, device="cuda").to(dtype), (-3.0, 3.0) if known else None
    got = api.ecc_hard(x, 2, bins, range=rng)
    prev = api.ecc_debug_force(api.ECC_FORCE_GENERIC)
    try:
        want = api.ecc_hard(x, 2, bins, range=rng)
    finally:
        api.ecc_debug_force(prev)
    assert torch.equal(got, want)
