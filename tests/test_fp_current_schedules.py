"""Worst-case int64 bounds and exact replays of Z_p arithmetic as the kernels
do it where test_fp_bounds.py and test_fp_products32.py describe other
schedules: the register kernels' propagators from unreduced differences and
their inverses in (-p, p), the state sum, Garner's digits, the end of a
contraction, the lane-group kernels' inverse factor."""
import random

import pytest

from test_fp_bounds import (PRIMES, Bounds, FieldModelSC, TrackedVec, Vec, _c32_extreme_prime, _register_variants,
                            _sc_extreme_prime)
from test_fp_products32 import GENERAL, R, bal, mul32, pow32

SMALL_FOLD_PRIMES = [2**31 - 1, 2147483629, _sc_extreme_prime(+1), _sc_extreme_prime(-1), 65537, 13]


class SmallFold(FieldModelSC):
    @staticmethod
    def ux_units(UX):
        return {6: 256, 4: 129, 2: 66}[UX]


def mul32_bound(B, a, b):
    """fp_mul32: any int32 operands, an int32 result."""
    assert a <= 2**31 and b <= 2**31
    r = (a * b + 2**31 * B.p) >> 32
    assert r < 2**31
    return r


def inverse_bound(B, y):
    """Batched inversion of values below y: every product stays in (-p, p)."""
    assert y < B.p and mul32_bound(B, B.p - 1, B.p - 1) < B.p
    return B.p - 1


def replay_small_fold(p, N, DL, L):
    B = Bounds(p)
    F = SmallFold(B, DL, L)
    h = B.h
    nb, lazyP = h + 2**23, 2 * h
    nc = F.ndot(h, h, lazy=True)                           # legs
    y = F.ndot(lazyP, lazyP, UX=6)                         # -P.P from unreduced differences
    assert y <= h
    inv = inverse_bound(B, y)
    for j in range(1, N):
        for i in range(j - 1, -1, -1):
            K, nD, uD = TrackedVec(B), 0, 0
            for t in range(i, j):
                nDm = F.ndot(nb, nb, lazy=True)
                dot = lambda rides: (F.ndot_sub2(lazyP, nb, nc, h, UX=4, UZ=3, lazy=True) if rides else
                                     F.ndot_sub(lazyP, nb, nc, UX=4, UZ=3, lazy=True))
                nc2, nc3 = dot(t > i), dot(t + 1 < j)
                assert max(nDm, nc2, nc3) <= nb
                K.kaxpy(66, nDm, h)                        # times Q_{t+1}
                K.kaxpy(66, nc2, nb)
                K.kaxpy(66, nc3, nb)
                if uD + 66 > F.MAXU:
                    nD, uD = B.fold(nD), F.FOLDU
                uD += 66
                nD = B.chk(nD + nDm * h, "nDacc")
            K.kaxpy(128, B.redc2(B.fold(nD)), 2 * h)       # times Q_i + Q_{j+1}
            for _q in range((j - i) * (j - i - 1) // 2):   # four-gluon splits
                K.kaxpy(66, F.ndot(nb, nb, lazy=True), nb)
            if i == 0 and j == N - 1:
                B.redc2(B.fold(K.b))
                F.ndot(h, h)                               # eps_n . K
            else:
                J = B.redc1(B.fold(B.chk(B.redc1(B.fold(K.b)) * inv, "finish product")))
                nc = max(nc, F.ndot(lazyP, nb, UX=4, lazy=True))
                assert max(J, nc) <= nb


@pytest.mark.parametrize("p", SMALL_FOLD_PRIMES)
def test_register_small_fold(p):
    for N, DL, L in _register_variants():
        replay_small_fold(p, N, DL, L)


def test_register_small_fold_needs_its_units():
    """The replay is able to fail: counted as products of normalised values
    (66 units), the propagators' products pass int64."""
    B = Bounds(2**31 - 1)
    F = FieldModelSC(B, 6, 1)
    with pytest.raises(AssertionError):
        F.ndot(2 * B.h, 2 * B.h, UX=5)


@pytest.mark.parametrize("p", PRIMES)
def test_general_finish_takes_the_inverses(p):
    """Any folded accumulator, one 32-bit REDC step, times an inverse in (-p, p)."""
    B = Bounds(p)
    inv = inverse_bound(B, B.h)
    assert B.redc2(B.chk(B.redc1(B.fold(2**63 - 1)) * inv, "finish_mul32")) <= B.h


def test_state_sum():
    """csrc/bg_states.hip: a state's component as it was read (any int32) times
    a balanced current, a fold after every two, one REDC step; the products of
    two such folded into the sum; one product with 2^128 at the end."""
    for p in PRIMES:
        B = Bounds(p)
        for D in range(4, 11):
            acc = 0
            for _s in range(D - 2):
                t = Vec(B)
                for mu in range(D):
                    t.axpy(2**31, B.h)
                    if mu & 1:
                        t.fold()
                if D & 1:
                    t.fold()
                dot = B.redc1(t.b)
                acc = B.fold(B.chk(acc + dot * dot, "state sum"))
            assert mul32_bound(B, B.redc1(acc), B.h) < p


def test_garner_digits():
    """csrc/bg_rational.hip: the residue plus earlier digits (canonical modulo
    primes of any size below 2^31) times balanced weights, a fold after every
    two; one REDC step and one product with the balanced inverse."""
    for p in PRIMES:
        B = Bounds(p)
        for i in range(32):
            T = p - 1
            for j in range(i):
                T = B.chk(T + (2**31 - 2) * B.h, "digit")
                if j & 1:
                    T = B.fold(T)
            assert mul32_bound(B, B.redc1(B.fold(T)), B.h) < p


def test_contraction():
    """csrc/bg_ffops.hip: four products of balanced values between folds, two
    values of j at a time; one REDC step and one product with 2^64 mod p."""
    for p in PRIMES:
        B = Bounds(p)
        acc = Vec(B)
        for j0 in range(0, 4096, 2):
            acc.axpy(B.h, B.h)
            acc.axpy(B.h, B.h)
            if j0 & 2:
                acc.fold()
            assert mul32_bound(B, B.redc1(B.fold(acc.b)), B.h) < p


@pytest.mark.parametrize("p", GENERAL + [_c32_extreme_prime(+1), _c32_extreme_prime(-1)])
@pytest.mark.parametrize("count", [1, 2, 9, 20])
def test_lane_group_inverse_factor(p, count):
    """2 R / y 2^32 (general) and 2 R / y 2^-32 (small fold constant), in (-p, p)."""
    rng = random.Random(3 * count + p)
    y = [bal(rng.randrange(1, p), p) for _ in range(count)]
    for factor, scale in ((bal(2 * R, p), 2 * R << 32), (2, 2 * R * pow(1 << 32, -1, p))):
        pre = [y[0]]
        for v in y[1:]:
            pre.append(mul32(pre[-1], v, p))
        t = mul32(pow32(pre[-1], p - 2, p), factor, p)
        for s in range(count - 1, -1, -1):
            inv = mul32(t, pre[s - 1], p) if s else t
            assert abs(inv) < p and (inv * y[s] - scale) % p == 0
            t = mul32(t, y[s], p)
