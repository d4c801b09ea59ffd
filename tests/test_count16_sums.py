"""The sums that the int16 count of values forms from its counts (no GPU): n,
mean and M2 against Python integers, where a sum that leaves its 64 bits would
show (every value 786431 times is the most that all values' low parts hold)."""
import ctypes
from fractions import Fraction

import numpy as np
import pytest

import paper_1211_4896_amd as tsa

VALUES = np.arange(-32768, 32768, dtype=np.int64)


def _moments(counts):
    f = ctypes.CDLL(tsa.LIB_PATH).tsa_internal_moments16
    f.restype = None
    f.argtypes = [ctypes.c_void_p] * 4
    c = np.ascontiguousarray(counts, np.uint64)
    n, mean, m2 = ctypes.c_uint64(), ctypes.c_double(), ctypes.c_double()
    f(c.ctypes.data, ctypes.byref(n), ctypes.byref(mean), ctypes.byref(m2))
    return n.value, mean.value, m2.value


def _even(c):
    return np.full(65536, c, np.uint64)


def _only(values, c):
    x = np.zeros(65536, np.uint64)
    for v in values:
        x[v + 32768] = c
    return x


def _outer(k, c):
    """the k values at either end, c times each"""
    x = np.zeros(65536, np.uint64)
    x[:k] = x[-k:] = c
    return x


CASES = {f"even {c}": _even(c) for c in (1, 786431, 786432, 819200, 900000, (1 << 20) - 1, 1 << 20, (1 << 30) - 1)}
CASES.update({f"extremes {c}": _only((-32768, 32767), c) for c in (1, (1 << 20) - 1, 1 << 20, (1 << 45) - 1)})
CASES["lowest 2^46"] = _only((-32768,), 1 << 46)
CASES["one value 2^46 - 1"] = _only((7,), (1 << 46) - 1)
CASES["outer 12200, 2^20 - 1 each (25.6 G voxels)"] = _outer(12200, (1 << 20) - 1)
CASES["drawn"] = np.random.default_rng(8).integers(0, 1 << 30, 65536).astype(np.uint64)


@pytest.mark.parametrize("name", sorted(CASES))
def test_moments_from_counts(name):
    c = CASES[name]
    ints = [int(x) for x in c]
    n = sum(ints)
    s = sum(v * x for v, x in zip(VALUES.tolist(), ints))
    q = sum(v * v * x for v, x in zip(VALUES.tolist(), ints))
    mean, m2 = Fraction(s, n), Fraction(n * q - s * s, n)
    gn, gmean, gm2 = _moments(c)
    assert gn == n
    # two roundings each: the integer to double, then the division
    assert abs(Fraction(gmean) - mean) <= abs(mean) / 2 ** 51, (name, gmean, float(mean))
    assert abs(Fraction(gm2) - m2) <= m2 / 2 ** 51, (name, gm2, float(m2))
