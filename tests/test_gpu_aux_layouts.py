"""Edges of the layouts of the standalone Z_p kernels: counts around a
block's 4096 values, pointers that are not aligned to the wide accesses, and
small primes, value by value against Python integers."""
import numpy as np
import pytest

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
