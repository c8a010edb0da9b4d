"""Products in the Montgomery domain of 2^32 (csrc/field_fp.h fp_mul32, fp_pow32)
and what is built on them, replayed with exact integers: operand ranges, the
batched propagator inversion of both reduction schedules, and the largest
values its results meet in the finish of a current."""
import random

import pytest

R = 1 << 64
GENERAL = [3, 5, 7, 65537, 998244353, 1073741789, 2147483647, 2147483629, 2147483587]
SMALL_FOLD = [p for p in GENERAL if min((1 << 32) % p, p - (1 << 32) % p) <= 1 << 22]


def bal(x, p):
    x %= p
    return x - p if x > (p - 1) // 2 else x


def s32(x):
    x &= 0xFFFFFFFF
    return x - (1 << 32) if x >> 31 else x


def redc1(T, p):
    """One 32-bit REDC step as the kernel forms it."""
    assert -(1 << 63) <= T < 1 << 63
    t1 = s32(T * pow(p, -1, 1 << 32))
    U = T - t1 * p
    assert -(1 << 63) <= U < 1 << 63 and U % (1 << 32) == 0
    return U >> 32


def fold(T, p):
    c32 = bal(1 << 32, p)
    return (T >> 32) * c32 + (T & 0xFFFFFFFF)


def mul32(a, b, p):
    r = redc1(a * b, p)
    assert -(1 << 31) <= r < 1 << 31
    return r


@pytest.mark.parametrize("p", GENERAL)
def test_ranges(p):
    rng = random.Random(p)
    top = (1 << 31) - 1
    vals = [top, -top, -(1 << 31), 0, 1, -1] + [rng.randint(-top, top) for _ in range(40)]
    for a in vals:
        for b in vals:
            assert (mul32(a, b, p) - a * b * pow(1 << 32, -1, p)) % p == 0
        assert abs(redc1(a, p)) <= (p - 1) // 2             # one REDC of an int32 is balanced
    ends = [p - 1, 1 - p, p // 2, -(p // 2), 1]
    for a in ends + [rng.randint(1 - p, p - 1) for _ in range(40)]:
        for b in ends + [rng.randint(1 - p, p - 1) for _ in range(40)]:
            assert abs(mul32(a, b, p)) < p


def pow32(a, e, p):
    r = a
    for b in range(e.bit_length() - 2, -1, -1):
        r = mul32(r, r, p)
        if e >> b & 1:
            r = mul32(r, a, p)
    return r


@pytest.mark.parametrize("p", GENERAL)
@pytest.mark.parametrize("count", [1, 2, 9, 20])
def test_batched_inversion(p, count):
    """y -> 2 R / y (general) and 2 R / y 2^-32 (small fold constant), in
    (-p, p); the wide kernel's factor -2 R 2^-32 likewise."""
    rng = random.Random(count + p)
    y = [bal(rng.randrange(1, p), p) for _ in range(count)]
    for factor, scale in ((bal(1 << 33, p), 2 * R), (2, 2 * R * pow(1 << 32, -1, p)), (-bal(2 * R, p), -2 * R * (1 << 32))):
        pre = [y[0]]
        for v in y[1:]:
            pre.append(mul32(pre[-1], v, p))
        t = mul32(pow32(pre[-1], p - 2, p), factor, p)
        for s in range(count - 1, -1, -1):
            inv = mul32(t, pre[s - 1], p) if s else t
            assert abs(inv) < p or p == 3
            assert (inv * y[s] - scale) % p == 0
            t = mul32(t, y[s], p)


@pytest.mark.parametrize("p", GENERAL)
def test_finish_takes_unbalanced_inverses(p):
    """fp_redc2 of (one REDC step of a folded accumulator) x inverse: below 2^62;
    small fold constant: a fold takes any int64."""
    c32 = abs(bal(1 << 32, p))
    folded = (1 << 31) * c32 + (1 << 32)
    step = folded // (1 << 32) + 1 + (p + 1) // 2
    assert step < 1 << 31 and step * (p - 1) < 1 << 62
    if p in SMALL_FOLD:
        assert folded < 1 << 54
        # a sum of squares of unreduced differences: one product beside a folded one
        assert (p - 1) ** 2 + (1 << 54) < 257 * (1 << 54) <= 511 * (1 << 54)
