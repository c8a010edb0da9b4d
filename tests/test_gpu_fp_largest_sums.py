"""The largest sums that the standalone Z_p kernels can meet, of one sign and of
both: balanced operands of (p - 1) / 2 and (p + 1) / 2 = -(p - 1) / 2 for the
contraction, currents of these and states of p - 1 for the state sum, whose
states enter as they were read.  A fold too few overflows here; random residues
cancel.  Every output against Python integers."""
import numpy as np
import pytest

from paper_2502_07060_amd import bg

from test_gpu_parity import torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu
PRIMES = [2147483647, 998244353, 1717986917, 1717986953]   # the last two: 2^32 mod p is nearly -p / 2 and p / 2


def up(torch_dev, a):
    torch, dev = torch_dev
    return torch.from_numpy(np.ascontiguousarray(a.astype(np.uint32)).view(np.int32)).to(dev)


def u32(t):
    return t.cpu().numpy().view(np.uint32).astype(np.int64)


@pytest.mark.parametrize("p", PRIMES)
@pytest.mark.parametrize("batched", [True, False])
@pytest.mark.parametrize("Id,J,K", [(1, 3, 1), (2, 5, 8), (6, 37, 6), (8, 64, 3), (9, 130, 5), (1, 4095, 2)])
def test_contract(torch_dev, p, batched, Id, J, K):
    h, n = (p - 1) // 2, 70
    rng = np.random.default_rng(J)
    x = np.where(rng.random((Id, J, n)) < 0.5, h, h + 1)
    y = np.where(rng.random((J, K, n)) < 0.5, h, h + 1)
    for q, (a, b) in enumerate(((h, h), (h + 1, h + 1), (h, h + 1), (h + 1, h))):   # +, +, -, -
        x[:, :, q], y[:, :, q] = a, b
    x[:, ::4, 5], y[::4, :, 5] = h, h                                   # four at a time
    if not batched:
        y = np.full((J, K), h)
    z, st = bg.bg_fp_contract(p, up(torch_dev, x), up(torch_dev, y), y_batched=batched)
    yy = y if batched else y[:, :, None]
    want = np.zeros((Id, K, n), np.int64)
    for j in range(J):
        want = (want + x[:, j, None] * yy[j][None] % p) % p
    assert int(st.sum()) == 0 and np.array_equal(u32(z), want)


@pytest.mark.parametrize("p", PRIMES)
@pytest.mark.parametrize("d", range(4, 11))
def test_state_sum(torch_dev, p, d):
    h, n = (p - 1) // 2, 70
    rng = np.random.default_rng(d)
    pick = lambda *s: np.where(rng.random(s) < 0.5, h, h + 1)
    kl, kr = pick(d, n), pick(d, n)
    eps, epst = np.full((d - 2, d, n), p - 1), np.full((d - 2, d, n), p - 1)
    eps[:, :, 40:], epst[:, :, 40:] = h, h + 1
    for q, (a, b) in enumerate(((h, h), (h + 1, h + 1), (h, h + 1), (h + 1, h))):
        kl[:, q], kr[:, q] = a, b
        if q < 2:                                                       # component 0 enters with the other sign
            kl[0, q], kr[0, q] = p - a, p - b
    s, st = bg.bg_state_sum(up(torch_dev, kl), up(torch_dev, kr), up(torch_dev, eps), up(torch_dev, epst), p=p)
    want = []
    for q in range(n):
        t = 0
        for i in range(d - 2):
            dots = [sum((1 if m == 0 else -1) * int(e[i, m, q]) * int(k[m, q]) for m in range(d)) for e, k in ((eps, kl), (epst, kr))]
            t += dots[0] * dots[1]
        want.append(t % p)
    assert int(st.sum()) == 0 and u32(s).tolist() == want
