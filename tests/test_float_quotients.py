"""Quotients of small numbers without a division.  Block counts of the
adjusted-occupancy simulation (Sec. 3.2): floor(left / x) as the truncated
float32 product (left + 1/2) * (1/x), with 1/x the correctly rounded float32
reciprocal, for 0 <= left <= 2^22 - 2.  The exact product is at least 1/(2x)
from every integer and the two roundings shift it by less than
2^-23 (left + 1/2) / x, so the floor is exact; checked here against integer
division around the multiples of every divisor class, where it could fail
first.  Shares and slowdown factors: a / b as the product with the correctly
rounded fp64 reciprocal and one correction step, for all integers up to 255."""
from fractions import Fraction

import numpy as np
import pytest

TOP = (1 << 22) - 2


def floors(left, x):
    inv = np.float32(1.0) / x.astype(np.float32)
    return ((left.astype(np.float32) + np.float32(0.5)) * inv).astype(np.int64)


def check(left, x):
    left, x = np.broadcast_arrays(np.asarray(left, np.int64), np.asarray(x, np.int64))
    got = floors(left, x)
    bad = np.nonzero(got != left // x)[0]
    assert bad.size == 0, (x[bad][:4], left[bad][:4], got[bad][:4])


@pytest.mark.parametrize("first", range(1, 4097, 512))
def test_multiples_of_every_divisor_up_to_4096(first):
    for x in range(first, first + 512):
        last = TOP // x
        m = np.unique(np.concatenate([np.arange(min(last, 300) + 1),
                                      np.arange(max(0, last - 300), last + 1)])) * x
        n = np.concatenate([m, m - 1, m + 1, [TOP]])
        n = n[(n >= 0) & (n <= TOP)]
        check(n, np.full(n.shape, x))


def test_every_divisor_at_its_last_multiples():
    x = np.arange(1, TOP + 1, dtype=np.int64)
    for back in range(3):
        m = (TOP // x - back) * x
        for d in (-1, 0, 1):
            n = m + d
            ok = (n >= 0) & (n <= TOP)
            check(n[ok], x[ok])
    check(np.full(x.shape, TOP), x)


def test_warps_as_half_integers():
    # left <= 127 warps are held as 2 left + 1 and divided by 2 W_b
    left, wb = np.meshgrid(np.arange(128), np.arange(1, 128))
    inv = np.float32(1.0) / (2 * wb).astype(np.float32)
    got = ((2 * left + 1).astype(np.float32) * inv).astype(np.int64)
    assert np.array_equal(got, left // wb)


def test_zero_demand_sets_no_limit():
    assert (np.float32(0.5) * np.float32(np.inf)) == np.inf


def test_quotients_up_to_255_are_correctly_rounded():
    # float(Fraction) rounds once, as a fused multiply-add does
    for b in range(1, 256):
        y = 1.0 / b
        for a in range(256):
            q0 = a * y
            r = float(a - Fraction(q0) * b)
            assert float(Fraction(r) * Fraction(y) + Fraction(q0)) == a / b, (a, b)
