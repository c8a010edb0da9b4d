"""Edges of the layouts of the standalone Z_p kernels: counts around a
block's 4096 values, pointers that are not aligned to the wide accesses, and
small primes, value by value against Python integers."""
import numpy as np
import pytest

from oracle import fields
from oracle import states as S
from paper_2502_07060_amd import bg
from paper_2502_07060_amd import inputs as I

from test_gpu_parity import torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu
P = I.DEFAULT_PRIME
SENTINEL = 0xFFFFFFFF


def u32(t):
    return t.cpu().numpy().view(np.uint32).astype(np.int64)


@pytest.mark.parametrize("p", [3, 5, 1009, 1073741827, P, 2147483647])
@pytest.mark.parametrize("count,skip", [(1, 0), (4095, 0), (4096, 0), (4097, 0), (4096, 1), (9001, 1), (9001, 2)])
def test_from_rational_layout(torch_dev, p, count, skip):
    torch, dev = torch_dev
    rng = np.random.default_rng(count + skip + p % 97)
    num = rng.integers(-2 ** 63, 2 ** 63 - 1, size=count + skip, endpoint=True)
    den = rng.integers(-2 ** 63, 2 ** 63 - 1, size=count + skip, endpoint=True)
    num[-1], den[-1] = -2 ** 63, 2 ** 63 - 1
    den[skip + count // 2] = 0
    den[skip + count // 3] = -3 * p
    tn, td = torch.from_numpy(num).to(dev)[skip:], torch.from_numpy(den).to(dev)[skip:]
    out = torch.full((count + 2,), 7, dtype=torch.int32, device=dev)
    st = torch.full((count + 2,), 7, dtype=torch.uint8, device=dev)
    bg.bg_fp_from_rational(p, tn, td, out=out[1:-1] if skip == 2 else out[:-2],
                           status=st[1:-1] if skip else st[:-2])
    torch.cuda.synchronize()
    o, s = out.cpu().numpy().view(np.uint32), st.cpu().numpy()
    o0, s0 = 1 if skip == 2 else 0, 1 if skip else 0
    for e in range(count):
        b = int(den[skip + e]) % p
        assert s[s0 + e] == (1 if b == 0 else 0), e
        want = SENTINEL if b == 0 else int(num[skip + e]) % p * pow(b, -1, p) % p
        assert int(o[o0 + e]) == want, e
    assert (o[:o0] == 7).all() and (o[o0 + count:] == 7).all()   # nothing past the ends
    assert (s[:s0] == 7).all() and (s[s0 + count:] == 7).all()


@pytest.mark.parametrize("batched", [True, False])
@pytest.mark.parametrize("Id,J,K,n", [(8, 4, 8, 63), (9, 5, 7, 64), (7, 2, 9, 65), (16, 3, 17, 70), (17, 1, 16, 5), (6, 36, 6, 129),
                                      (1, 37, 8, 66), (8, 6, 1, 1), (2, 3, 2, 65535), (3, 2, 1, 65537)])
def test_contract_tiles(torch_dev, Id, J, K, n, batched):
    torch, dev = torch_dev
    p = 998244353 if (Id + J) % 2 else 2147483647
    rng = np.random.default_rng(Id * 100 + J * 10 + K)
    ld = n + 3
    x = rng.integers(0, p, size=(Id, J, ld))
    y = rng.integers(0, p, size=(J, K, ld) if batched else (J, K))
    x[:, :, 0] = p - 1                     # the largest sums of one sign
    bad = np.zeros(n, bool)
    if n > 4:
        x[Id - 1, J - 1, n - 1] = 0xFFFFFFFF   # in the last tile: outputs of the first ones are replaced too
        bad[n - 1] = True
        if batched:
            y[J - 1, K - 1, 2] = p
            bad[2] = True
    if batched:
        y[:, :, 0] = p - 1
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a.astype(np.uint32)).view(np.int32)).to(dev)
    z, st = bg.bg_fp_contract(p, up(x), up(y), y_batched=batched, npts=n)
    torch.cuda.synchronize()
    want = np.zeros((Id, K, n), np.int64)
    for j in range(J):                     # products below 2^62, reduced one by one
        yj = y[j][:, :n] if batched else y[j][:, None]
        want = (want + x[:, j, None, :n] % p * (yj[None] % p) % p) % p
    want[:, :, bad] = SENTINEL
    assert np.array_equal(u32(z)[:, :, :n], want)
    assert np.array_equal(st.cpu().numpy(), np.where(bad, 2, 0))


@pytest.mark.parametrize("p", [3, 1009, 1073741827, 2147483647])
@pytest.mark.parametrize("count,skip", [(1, 0), (1023, 0), (1025, 0), (4095, 0), (4096, 0), (4097, 0), (4096, 1), (9001, 3)])
def test_divide_layout(torch_dev, p, count, skip):
    torch, dev = torch_dev
    rng = np.random.default_rng(count + skip + p % 89)
    x, y = rng.integers(0, p, size=count), rng.integers(1, p, size=count)
    x[-1], y[-1] = p - 1, p - 1
    y[count // 2] = 0
    if count > 8:
        x[count // 3], y[count // 4] = p, 0xFFFFFFFF
        x[count // 5], y[count // 5] = p + 1, 0     # a bad residue wins over the zero divisor
    shift = lambda a: torch.from_numpy(np.concatenate([np.zeros(skip, np.uint32), a.astype(np.uint32)]).view(np.int32)).to(dev)[skip:]
    bad, zero = (x >= p) | (y >= p), y == 0
    table = {}
    inv = np.array([table.setdefault(int(b), pow(int(b), -1, p)) if not (s or t) else 0 for b, s, t in zip(y, bad, zero)])
    want = np.where(bad | zero, SENTINEL, x % p * inv % p)
    z, st = bg.bg_fp_divide(p, shift(x), shift(y))
    torch.cuda.synchronize()
    assert np.array_equal(u32(z), want)
    assert np.array_equal(st.cpu().numpy(), np.where(bad, 2, np.where(zero, 1, 0)))
    d = p - 1 if count % 2 else p // 2
    z, st = bg.bg_fp_divide(p, shift(x), d)
    torch.cuda.synchronize()
    assert np.array_equal(u32(z), np.where(x >= p, SENTINEL, x % p * pow(d, -1, p) % p))
    assert np.array_equal(st.cpu().numpy(), np.where(x >= p, 2, 0))


@pytest.mark.parametrize("d", [4, 5, 6, 7, 8, 9, 10])
@pytest.mark.parametrize("p", [5, 13, 1009, 998244353, P])
def test_states_small_fields(torch_dev, d, p):
    """Small primes, where every denominator vanishes at some points and both
    spinor charts occur, against the oracle (statuses and residues)."""
    torch, dev = torch_dev
    n, ld = 300 if p < 1000 else 70, 301
    rng = np.random.default_rng(d * 10 + p % 7)
    k = I.fp_null(rng, p, (ld,), d) if p > 5 else rng.integers(0, p, size=(ld, d))   # not massless: the formulas hold
    chi = I.fp_null(rng, p, (ld,), 4)
    k[1, 3] = (p - k[1, 0]) % p            # k+ = 0
    chi[2] = [p - 1, 0, 0, 1]              # chi+ = 0
    k[3, 0] = p                            # not canonical
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a.T.astype(np.uint32)).view(np.int32)).to(dev)
    e, t, st = bg.bg_states_fp(up(k), up(chi), p, npts=n)
    torch.cuda.synchronize()
    e, t, st = u32(e), u32(t), st.cpu().numpy()
    F, ip = fields.Fp(p), I.fp_sqrt_minus_one(p)
    for q in range(n):
        if (k[q] >= p).any():
            assert st[q] == 2 and (e[:, :, q] == SENTINEL).all() and (t[:, :, q] == SENTINEL).all()
            continue
        s, E, T = S.states(F, [int(x) for x in k[q]], [int(x) for x in chi[q]], ip)
        assert st[q] == s, q
        if s == 0:
            assert np.array_equal(e[:, :, q], np.array(E)) and np.array_equal(t[:, :, q], np.array(T)), q
        else:
            assert (e[:, :, q] == SENTINEL).all() and (t[:, :, q] == SENTINEL).all()
