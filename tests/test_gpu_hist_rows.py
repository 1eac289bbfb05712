"""Histogram sweeps whose blocks leave their counters in rows of the workspace: a row for each block (one bin per level, few
blocks), rows that blocks share (many blocks on one item), and none (few blocks with a table, more bins than the scan of
rows takes, a workspace without room).  Sublevel and superlevel curves against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import ecc_oracle as O
from oracle import ecc_oracle_c as OC
from paper_2510_20271_amd import api, synth
from tests.gpu_util import dev, host

pytestmark = pytest.mark.gpu


# (batch, *item): 1, 2, 20, 63 and 64 blocks of the plain sweep; 7 blocks an item; 208 blocks; volumes with few and many
SHAPES = [(1, 3, 9), (1, 20, 21), (1, 64, 79), (1, 252, 256), (1, 256, 256), (3, 100, 300), (1, 1100, 1300),
          (2, 9, 40, 70), (1, 60, 190, 130)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("bins", [1, 3, 64, 100, 256, 257, 1000, 1024, 1025, 4096, 6000])
def test_rows_of_levels(shape, bins):
    rng = np.random.default_rng(bins + shape[-1])
    dtype = np.uint8 if bins <= 257 else np.uint16
    X = rng.integers(0, min(bins + bins // 4 + 2, np.iinfo(dtype).max), size=shape, endpoint=True).astype(dtype)
    nd = len(shape) - 1
    np.testing.assert_array_equal(host(api.ecc_hard(dev(X), nd, bins)), OC.ecc_hard_batch(X, O.thresholds_levels(bins)))
    np.testing.assert_array_equal(host(api.ecc_hard(dev(X), nd, bins, superlevel=True)),
                                  O.ecc_super_batch(X, O.thresholds_levels_super(bins)))


@pytest.mark.parametrize("shape", [(1, 3, 9), (1, 300, 301), (1, 1100, 1300), (2, 700, 1300), (1, 100, 190, 130)])
@pytest.mark.parametrize("bins", [1, 100, 256, 1024, 1025, 4096, 8193])
def test_rows_of_a_known_range(shape, bins):
    nd = len(shape) - 1
    if nd == 3 and bins > 8000:
        shape = (1, 30, 60, 60)  # (the plain sweep)
    X = np.stack([synth.grf(shape[1:], 2.0, 5 + i) for i in range(shape[0])])
    t = O.thresholds_equal_width(-1.5, 1.0, bins)
    np.testing.assert_array_equal(host(api.ecc_hard(dev(X), nd, bins, range=(-1.5, 1.0))), OC.ecc_hard_batch(X, t))
    np.testing.assert_array_equal(host(api.ecc_hard(dev(X), nd, bins, range=(-1.5, 1.0), superlevel=True)),
                                  O.ecc_super_batch(X, O.thresholds_lower(t, -1.5)))
