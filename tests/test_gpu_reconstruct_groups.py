"""Rational reconstruction with quotients taken in groups on the leading bits:
one prime count per limb count and its edges, with inputs whose Euclidean
quotients are small, huge, at the bound and absent, against oracle/rational.py
(exact)."""
import random
from math import gcd, prod

import numpy as np
import pytest

from oracle import rational as R

from test_gpu_parity import torch_dev  # noqa: F401
from test_gpu_rational import check_against_oracle
from test_oracle_rational import primes_below

pytestmark = pytest.mark.gpu
BIG = primes_below(2 ** 31, 32)
SMALL = [3, 5, 7, 11, 101, 65537, 1048583, 536870923]


@pytest.mark.parametrize("primes", [BIG[:k] for k in (4, 6, 7, 10, 11, 12, 14, 15, 20, 21, 28, 29)] +
                         [SMALL[:3], SMALL, SMALL[::-1] + BIG[:5]], ids=lambda p: f"{len(p)}p{p[0]}")
def test_reconstruct_groups(torch_dev, primes):
    M = prod(primes)
    B = R.bound(M)
    rng = random.Random(len(primes))
    xs = [0, 1, 2, M - 1, M - 2, M // 2, B, B + 1, M - B, M - B - 1, (M - 1) // 2]
    f0, f1 = 1, 1                       # M / x near the golden ratio: quotients all 1 at first
    while f1 < M:
        f0, f1 = f1, f0 + f1
    xs += [M * f0 // f1, M * f0 // (f0 + f1)]
    for e in range(1, M.bit_length(), 7):   # one quotient of e bits, then ordinary ones
        xs += [M >> e, (M >> e) + rng.randrange(1 << 20), rng.randrange((M >> e) + 1)]
    for _ in range(150):
        hb = rng.randint(0, B.bit_length())
        a, b = rng.randint(-B, B) >> rng.randint(0, B.bit_length()), rng.randint(1, max(1, B >> hb))
        if gcd(b, M) == 1:
            xs.append(a * pow(b, -1, M) % M)
    xs += [rng.randrange(M) for _ in range(80)]
    res = np.array([[x % p for x in xs] for p in primes], dtype=np.int64)
    check_against_oracle(torch_dev, primes, res)
