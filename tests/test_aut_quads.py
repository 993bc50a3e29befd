"""Host check of the automorphism's grouped gather (no GPU): in the
bit-reversed evaluation order the sources of an aligned group of four
positions are one aligned group, in the order the kernels take it, for
rotations and for conjugation at every ring degree."""
import numpy as np
import pytest


def brev(x, bits):
    r = np.zeros_like(x)
    for _ in range(bits):
        r = (r << 1) | (x & 1)
        x = x >> 1
    return r


def sources(log_n, g):
    """Position of every position's source, from the definition 2k'+1 = g(2k+1) mod 2N."""
    n = 1 << log_n
    k = brev(np.arange(n, dtype=np.int64), log_n)
    return brev(((g * (2 * k + 1)) % (2 * n) - 1) >> 1, log_n)


def quads(log_n, g):
    """The kernels' steps: one group offset, then the arrangement of its four entries."""
    n = 1 << log_n
    pos = np.arange(0, n, 4, dtype=np.int64)
    k = brev(pos >> 2, log_n - 2)
    kp = (g * k + (g >> 1)) & (n - 1)
    off = brev(kp & ((n >> 2) - 1), log_n - 2) << 2
    rot, neg = kp >> (log_n - 2), bool(g & 2)
    v = [off + i for i in range(4)]
    w = [v[0], v[3] if neg else v[2], v[1], v[2] if neg else v[3]]
    r = (4 - rot) if neg else rot
    odd, half = (r & 1) == 1, (r & 2) == 2
    w = [np.where(odd, w[(i + 1) & 3], w[i]) for i in range(4)]
    x = [None] * 4
    x[0], x[2] = np.where(half, w[2], w[0]), np.where(half, w[3], w[1])
    x[1], x[3] = np.where(half, w[0], w[2]), np.where(half, w[1], w[3])
    return np.stack(x, axis=1).reshape(-1)


@pytest.mark.parametrize("log_n", [12, 13, 14, 15, 16])
def test_groups_of_four_sources(log_n):
    n = 1 << log_n
    for k in (0, 1, 2, 3, 5, 77, n // 4, n // 2 - 1):
        g = pow(5, k, 2 * n)
        assert np.array_equal(quads(log_n, g), sources(log_n, g))
    assert np.array_equal(quads(log_n, 2 * n - 1), sources(log_n, 2 * n - 1))
