"""The operands of the piece-product tests do what they are for: at every size of those tests, an entropy from which one of the
six products of the bf16 pieces is left out, or taken twice, is off by at least twice the tests' bar."""
import numpy as np
import pytest

from helpers import piece_operands
from test_gpu_fp32_pieces import CASES

PRODUCTS = ((2, 0), (1, 1), (0, 2), (1, 0), (0, 1), (0, 0))  # pieces of (W_lm, hidden)


def _pieces(a):
    out = []
    for _ in range(3):
        piece = (a.view(np.uint32) & 0xffff0000).view(np.float32)
        out.append(piece.astype(np.float64))
        a = a - piece
    assert not a.any()
    return out


def _entropy(z):
    z = z - z.max(axis=1, keepdims=True)
    e = np.exp(z)
    return np.log(e.sum(axis=1)) - (e * z).sum(axis=1) / e.sum(axis=1)


@pytest.mark.parametrize("d,V,T", sorted({c[:3] for c in CASES}))
def test_every_piece_product_shows(d, V, T):
    worst = np.zeros((len(PRODUCTS), 2))
    for hidden, w_lm in piece_operands(np.random.default_rng(9600 + T), T, V, d):
        some = hidden[:24]
        h, w = _pieces(some), _pieces(w_lm)
        z = some.astype(np.float64) @ w_lm.astype(np.float64).T
        want = _entropy(z)
        # sums of magnitudes below 2^24 of the smallest unit: exact in fp32 in any order
        unit = lambda a: np.gcd.reduce((a[a != 0][:5000].astype(np.float64) * 2.0 ** 40).astype(np.int64)) * 2.0 ** -40
        assert (np.abs(some).astype(np.float64) @ np.abs(w_lm).astype(np.float64).T).max() < 2.0 ** 24 * unit(some) * unit(w_lm)
        for i, (a, b) in enumerate(PRODUCTS):
            part = h[b] @ w[a].T
            for k, sign in enumerate((-1.0, 1.0)):
                worst[i, k] = max(worst[i, k], np.abs(_entropy(z + sign * part) - want).max())
    assert worst.min() >= 2 * 2e-5, worst / 2e-5
