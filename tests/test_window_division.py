"""The row kernels divide by the window length L with a multiplication by ceil(2^32 / L); the launcher allows it where the
largest dividend times L stays below 2^32.  Every L, at the multiples of L around which a quotient could slip."""
import numpy as np


def test_reciprocal_of_the_window_length_is_exact():
    rng = np.random.default_rng(1)
    for L in range(2, 257):
        recip = -(-2 ** 32 // L)
        assert recip < 2 ** 32
        most = (2 ** 32 - 1) // L                       # the largest dividend allowed
        q = np.concatenate([np.arange(300), rng.integers(0, most // L, 2000), [most // L]]).astype(np.uint64)
        v = np.concatenate([q * L, q * L + (L - 1), np.maximum(q * L, 1) - 1, [most]]).astype(np.uint64)
        v = v[v <= most]
        assert ((v * np.uint64(recip)) >> np.uint64(32) == v // np.uint64(L)).all(), L
