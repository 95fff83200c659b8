"""The multipliers that the kernels divide by launch constants with, in the forms the kernels use them.  Needs no GPU."""
import ctypes as C
import random

import pytest

from paper_2011_06295_amd import binding as B


class FastDiv(C.Structure):
    _fields_ = [("mul", C.c_uint32), ("shift", C.c_uint32)]


_make = B.raw_library()["_ZN2sc12make_fastdivEi"]   # sc::make_fastdiv(int)
_make.restype, _make.argtypes = FastDiv, [C.c_int]

LARGEST = 2**31 - 1
DIVISORS = sorted({1, 3, 7, 10, 641, 12345, 46341, 2**30 + 12345} | {2**s + off for s in range(1, 31) for off in (-1, 0, 1)} | {LARGEST - 1, LARGEST})


@pytest.mark.parametrize("d", DIVISORS)
def test_quotients_are_exact(d):
    """Around multiples of the divisor from 0 to the largest number, and at random ones: the upper half of 2 n * mul shifted, and (unless
    d = 1) that of n * mul shifted a bit less."""
    f = _make(d)
    rng = random.Random(d)
    most = LARGEST // d
    of = {0, 1, 2, most // 2, most - 1, most} | {rng.randint(0, most) for _ in range(300)}
    numbers = {q * d + off for q in of for off in (-1, 0, 1)} | {rng.randint(0, LARGEST) for _ in range(300)} | {LARGEST - 1, LARGEST}
    for n in numbers:
        if not 0 <= n <= LARGEST:
            continue
        assert (2 * n % 2**32 * f.mul >> 32) >> f.shift == n // d, n
        assert (f.shift == 0) == (d == 1)
        if f.shift:
            assert (n * f.mul >> 32) >> (f.shift - 1) == n // d, n
