"""The kernels' division by a divisor the launch knows (one high product): exact for every 0 <= n < 2^31."""
import ctypes
import random

import pytest

from paper_2405_16256_amd import binding as hh

TOP = 2**31 - 1


def quotient(n, d):
    f = hh.lib.hh_internal_quotient
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_int, ctypes.c_int]
    return f(n, d)


@pytest.mark.parametrize("d", [1, 2, 3, 4, 5, 6, 7, 8, 9, 63, 64, 65, 129, 641, 1000, 3300, 4095, 4096, 4097, 65535, 65537, 2**30 - 1, 2**30, 2**30 + 1, TOP])
def test_edges(d):
    multiples = [m * d for m in (0, 1, 2, 3, 7, TOP // d // 2, TOP // d - 1, TOP // d) if m >= 0]
    for n in {max(0, min(TOP, m + e)) for m in multiples + [TOP] for e in (-2, -1, 0, 1, 2)}:
        assert quotient(n, d) == n // d, (n, d)


def test_random():
    rng = random.Random(3)
    for _ in range(100000):
        d, n = rng.randint(1, 2 ** rng.randint(1, 31) - 1), rng.randint(0, 2 ** rng.randint(1, 31) - 1)
        assert quotient(n, d) == n // d, (n, d)
