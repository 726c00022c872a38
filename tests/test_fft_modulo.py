"""The convolution's modulo by a transform length, checked on the CPU over the arguments the kernels form.

The z spectra take roots at (k z) mod M with k <= M / 2 and z < (M + 1) / 2 (products below 2^23 for M <= 4608): the
quotient is the high half of a * magic, magic = floor(2^32 / M) + 1, exact or one too large, and the unsigned minimum
of t and t + M takes back the step where it is."""
import numpy as np
import pytest


def mod_by(a, M):
    magic = np.uint64((1 << 32) // M + 1)
    q = (a.astype(np.uint64) * magic) >> np.uint64(32)
    t = (a - (q * np.uint64(M)).astype(np.uint32)).astype(np.uint32)
    return np.minimum(t, (t + np.uint32(M)).astype(np.uint32))


@pytest.mark.parametrize("M", [9, 15, 16, 64, 135, 375, 450, 480, 512, 1024, 2048, 2592, 4096, 4500, 4608])
def test_mod_by_is_exact(M):
    top = (M // 2 + 1) * ((M + 1) // 2)
    a = np.arange(0, top + 1, dtype=np.uint32)
    assert top < 1 << 23
    assert np.array_equal(mod_by(a, M), a % np.uint32(M))
