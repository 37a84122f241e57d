"""The sampled interval's weight from its keys in FP64: for W < 2^61 the
rounded product (U_{i+1} - U_i) (W 2^-64) is w_i exactly, also where the upper
key is the all-ones end."""
import numpy as np
import pytest


def weight_fp64(lo, hi, W):
    """The sampling kernels' operations in IEEE double: each conversion of a
    64-bit word adds its halves with one rounding."""
    def conv(v):
        return np.float64(v >> 32) * np.float64(2.0 ** 32) + np.float64(v & 0xFFFFFFFF)
    return int(np.rint(conv(hi - lo) * (conv(W) * np.float64(2.0 ** -64))))


@pytest.mark.parametrize("wmax", [1, 2, 3, 2 ** 31, 2 ** 32 - 2, 2 ** 32 - 1])
@pytest.mark.parametrize("bits", [1, 20, 33, 52, 53, 54, 60, 61])
def test_weight_from_keys(wmax, bits):
    rng = np.random.default_rng(bits * 7 + wmax % 1000)
    for trial in range(400):
        top = (1 << bits) - 1  # the largest total of the size
        W = top - int(rng.integers(0, min(top, 1 << 40))) if trial % 2 else top
        w = min(W, wmax - int(rng.integers(0, min(wmax, 50))))
        C = int(rng.integers(0, 2 ** 63)) % (W - w + 1)
        C = (0, W - w, C)[trial % 3]
        key = lambda c: -((-(c << 64)) // W)  # noqa: E731
        lo = key(C)
        hi = key(C + w) if C + w < W else 2 ** 64 - 1
        assert weight_fp64(lo, hi, W) == w, (W, C, w)
