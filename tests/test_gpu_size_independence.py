"""Over C a point's result has the same bits in any call: one kernel serves a
(n, d) at every size.  A call is compared with the same points in chunks on both
sides of every size where a launch changes its form (blocks of one point, the
streaming form of the register kernels, sizes where the choice over Z_p
changes), amplitudes and root currents, and requests that are merged beyond
the streaming form's first size with single calls of their own."""
import pytest

from paper_2502_07060_amd import bg

from test_gpu_parity import torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu
SHAPES = ([(n, d) for n in range(4, 9) for d in (4, 6, 8, 10)] + [(9, 5), (9, 10), (10, 4), (10, 8), (11, 6), (12, 4)] +
          [(12, 6), (12, 8), (13, 4), (13, 8), (13, 10), (14, 4), (14, 6), (14, 8)])
CHUNKS = (1, 2, 62, 959, 1026, 2049, 4097, 9000, 17001)


def points(torch_dev, n, d, m):
    torch, dev = torch_dev
    g = torch.Generator(device=dev)
    g.manual_seed(100 * n + d)
    make = lambda: torch.view_as_complex(torch.randn(n, d, m, 2, generator=g, device=dev, dtype=torch.float64))
    return make(), make()


def bits(torch, t):
    return torch.view_as_real(t.contiguous()).view(torch.int64)


@pytest.mark.parametrize("n,d", SHAPES)
def test_chunks(torch_dev, n, d):
    torch, dev = torch_dev
    blocks = torch.cuda.get_device_properties(dev).multi_processor_count
    m = 2 * blocks * 128 + 300 if n <= 8 else sum(CHUNKS if n <= 12 else CHUNKS[:-1])
    k, e = points(torch_dev, n, d, m)
    amp, st = bg.bg_amplitudes_c128(k, e)
    cur, _ = bg.bg_currents_c128(k, e)
    assert int((st != 0).sum()) == 0
    q = 0
    for c in CHUNKS + (m,):
        c = min(c, m - q)
        if c == 0:
            break
        part = [t[:, :, q:q + c].contiguous() for t in (k, e)]
        assert torch.equal(bits(torch, bg.bg_amplitudes_c128(*part)[0]), bits(torch, amp[q:q + c])), (q, c)
        assert torch.equal(bits(torch, bg.bg_currents_c128(*part)[0]), bits(torch, cur[:, q:q + c])), ("current", q, c)
        q += c


@pytest.mark.parametrize("n,d", [(8, 4), (7, 8)])
def test_merged_requests(torch_dev, n, d):
    """Requests of 20000 points: alone below the streaming form's first size
    (65536 points with two lanes, 32768 with four), three or four of them above."""
    torch, dev = torch_dev
    sizes = [20000, 19999, 1, 20000, 500, 18000] * 3
    with bg.Server(1 << 31) as srv:
        reqs = []
        for i, m in enumerate(sizes):
            k, e = (t[:, :, i:i + m].cpu().contiguous().pin_memory() for t in points(torch_dev, n, d, 20100))
            out = torch.empty(m, dtype=torch.complex128).pin_memory()
            st = torch.empty(m, dtype=torch.uint8).pin_memory()
            reqs.append((k, e, out, st))
        ids = [srv.submit(k, e, out, st) for k, e, out, st in reqs]
        for rid in ids:
            srv.wait(rid, 60.0)
    for k, e, out, st in reqs:
        o, s = bg.bg_amplitudes_c128(k.to(dev), e.to(dev))
        assert torch.equal(bits(torch, out), bits(torch, o.cpu())) and torch.equal(st, s.cpu())
