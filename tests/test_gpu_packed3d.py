"""The packed 3D sweep (volumes of one- and two-byte elements): curves of all four conventions and the coefficient map
against the oracle, where it can go wrong: chunks of eight planes and their remainders, rows that are no multiple of
four, strips of 62 columns, folded last strips, elements at the ends of their type's range (no key stands for "beyond
the grid"), signed zeros, and both ways through a chunk (vertex by vertex when it is dense, bit by bit when it is not)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import ecc_oracle as O
from oracle import ecc_oracle_c as OC
from paper_2510_20271_amd import api, synth
from tests.gpu_util import dev, host

pytestmark = pytest.mark.gpu

# (batch, D, H, W); every one large enough for the sweep with known thresholds
SHAPES = [(1, 2, 130, 260), (1, 8, 97, 126), (1, 9, 61, 193), (1, 17, 64, 70), (1, 31, 50, 63), (3, 16, 33, 62),
          (1, 41, 39, 64), (1, 70, 8, 186), (600, 3, 5, 9)]


def _tensor(kind, values):
    if kind == "bf16":
        return torch.from_numpy(values.astype(np.float32)).to(torch.bfloat16).cuda()
    return dev(values.astype({"u8": np.uint8, "u16": np.uint16, "i16": np.int16, "f16": np.float16}[kind]))


def _values(kind, fill, shape, rng):
    if kind in ("f16", "bf16"):
        if fill == "ends":  # the largest finite values of float16, its smallest denormal, both zeros
            return rng.choice([65504.0, -65504.0, 6e-8, -6e-8, 0.0, -0.0, 1.0], size=shape)
        x = np.stack([synth.grf(shape[1:], 2.0, 7 + i) for i in range(min(shape[0], 3))])
        return np.concatenate([x] * (-(-shape[0] // len(x))))[: shape[0]]
    lo, hi = {"u8": (0, 255), "u16": (0, 65535), "i16": (-32768, 32767)}[kind]
    if fill == "ends":
        return rng.choice([lo, lo + 1, hi - 1, hi], size=shape)
    if fill == "noise":
        return rng.integers(lo, lo + 300, size=shape, endpoint=True) if kind != "u8" else rng.integers(0, 256, size=shape)
    return rng.integers(0, 2, size=shape).cumsum(-1) // 3 % 200  # long runs of equal values


@pytest.mark.parametrize("kind", ["u8", "u16", "i16", "f16", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_packed_sweep_against_the_oracle(kind, shape, flow):
    rng = np.random.default_rng(sum(shape))
    for fill in ("ends", "noise", "runs"):
        x = _values(kind, fill, shape, rng)
        g = _tensor(kind, x)
        Y = g.float().cpu().numpy() if kind in ("f16", "bf16") else x.astype(np.float32)
        bins = 100
        cases = [((-200.0, 150.0), O.thresholds_equal_width(-200.0, 150.0, bins))]
        if kind in ("u8", "u16"):
            cases.append((None, O.thresholds_levels(bins)))
        elif kind in ("f16", "bf16"):
            cases.append((None, O.thresholds_equal_width(float(Y.min()), float(Y.max()), bins)))
        for rng_, t in cases:
            lower = O.thresholds_levels_super(bins) if rng_ is None and kind in ("u8", "u16") else \
                O.thresholds_lower(t, rng_[0] if rng_ else float(Y.min()))
            some = slice(0, 4)  # (the numpy oracle on a few items of a large batch)
            np.testing.assert_array_equal(host(api.ecc_hard(g, 3, bins, range=rng_)), OC.ecc_hard_batch(Y, t))
            np.testing.assert_array_equal(host(api.ecc_hard(g, 3, bins, range=rng_, top=True))[some],
                                          O.ecc_top_batch(Y[some], t))
            for top in (False, True):
                got = host(api.ecc_hard(g, 3, bins, range=rng_, top=top, superlevel=True))
                np.testing.assert_array_equal(got[some], O.ecc_super_batch(Y[some], lower, top))
        if kind in ("u8", "u16"):
            c = host(api.ecc_coeff(g, 3))
            for i in range(min(shape[0], 4)):
                np.testing.assert_array_equal(c[i], O.coeff(Y[i]))


@pytest.mark.parametrize("kind", ["f16", "bf16"])
@pytest.mark.parametrize("shape", [(7, 73, 94, 93), (36, 75, 46, 42), (6, 51, 70, 63)])
def test_lists_keep_to_the_room_of_float32(kind, shape, flow):
    """A list for each block whose segments of eight planes would need more room than the workspace has: longer ones."""
    x = np.stack([np.roll(synth.grf(shape[1:], 2.0, 5), 3 * i, axis=2) for i in range(shape[0])])
    g = _tensor(kind, x)
    Y = g.float().cpu().numpy()
    t = O.thresholds_equal_width(float(Y.min()), float(Y.max()), 200)
    np.testing.assert_array_equal(host(api.ecc_hard(g, 3, 200)), OC.ecc_hard_batch(Y, t))


def test_shared_lists_of_a_large_volume():
    """More vertices than a list for each block is kept for: lists that blocks share, and their sweep in reserve."""
    x = synth.grf((330, 320, 322), 2.0, 9)  # (beyond 2^25)
    for y in (x, np.random.default_rng(1).standard_normal(x.shape).astype(np.float32)):  # (noise: the lists run over)
        g = _tensor("f16", y[None])
        Y = g.float().cpu().numpy()
        t = O.thresholds_equal_width(float(Y.min()), float(Y.max()), 200)
        np.testing.assert_array_equal(host(api.ecc_hard(g, 3, 200)), OC.ecc_hard_batch(Y, t))
