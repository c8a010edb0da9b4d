"""The kernel chosen without a pin depends on the number of points: around every
size where the choice changes, results equal those of one fixed kernel (Z_p bit
for bit; complex within twice the 1e-11 that each kernel keeps to the exact
value, over the norm of all points), for amplitudes, root currents and both
metrics, with ld > npts and without a status array; served requests equal
single calls of their own size whatever they are merged with."""
import numpy as np
import pytest

from paper_2502_07060_amd import bg
from paper_2502_07060_amd import inputs as I

from test_gpu_parity import torch_dev  # noqa: F401
from test_gpu_server import same_bits

pytestmark = pytest.mark.gpu
P = I.DEFAULT_PRIME
POOL = 97
SIZES = [1, 2, 1023, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193, 16384, 16385, 32769, 65535, 65536, 131073]


def tiled(torch_dev, field, n, d, m, metric=bg.BG_METRIC_MOSTLY_MINUS):
    """m points in a row of ld = m + 3, tiled from POOL physical ones."""
    torch, dev = torch_dev
    if field == "fp":
        k, e = I.generic_fp(11 * n + d, n, d, POOL, P)
        if metric == bg.BG_METRIC_ALTERNATING:
            ip = pow(I.fp_sqrt_minus_one(P), -1, P)
            k, e = (np.where((np.arange(d) >= 2) & (np.arange(d) % 2 == 0), a.astype(np.int64) * ip % P, a) for a in (k, e))
        k, e = (I.to_soa(a.astype(np.uint32)).view(np.int32) for a in (k, e))
    else:
        k, e = I.generic_c128(11 * n + d, n, d, POOL)
        k, e = I.to_soa(k.astype(np.complex128)), I.to_soa(e.astype(np.complex128))
    at = torch.arange(m + 3, device=dev) % POOL
    return [torch.from_numpy(np.ascontiguousarray(a)).to(dev)[:, :, at].contiguous() for a in (k, e)]


@pytest.mark.parametrize("field,n,d", [("fp", 4, 6), ("fp", 5, 10), ("fp", 6, 4), ("fp", 7, 8), ("fp", 8, 6), ("fp", 9, 9),
                                       ("fp", 10, 7), ("fp", 11, 4), ("fp", 11, 6), ("fp", 11, 8), ("fp", 12, 10), ("fp", 13, 5),
                                       ("fp", 14, 8), ("c128", 4, 10), ("c128", 5, 8), ("c128", 6, 4), ("c128", 7, 6), ("c128", 8, 9),
                                       ("c128", 9, 5), ("c128", 10, 4), ("c128", 11, 8), ("c128", 12, 6), ("c128", 13, 8),
                                       ("c128", 13, 10), ("c128", 14, 4), ("c128", 14, 7)])
def test_sizes(torch_dev, field, n, d):
    torch, _ = torch_dev
    tag = bg.BG_FIELD_FP if field == "fp" else bg.BG_FIELD_C128
    fixed = [v for v in bg.bg_variants(tag, n, d) if v["generic"] and v["lanes"] >= 16][-1]["index"]
    amp = (lambda k, e, **kw: bg.bg_amplitudes_fp(k, e, P, **kw)) if field == "fp" else bg.bg_amplitudes_c128
    cur = (lambda k, e, **kw: bg.bg_currents_fp(k, e, P, **kw)) if field == "fp" else bg.bg_currents_c128
    big = tiled(torch_dev, field, n, d, POOL)
    bg.bg_select_variant(tag, n, d, fixed)
    try:
        want, wst = amp(*big, npts=POOL)
        wcur, _ = cur(*big, npts=POOL)
    finally:
        bg.bg_select_variant(tag, n, d, -1)

    def check(got, ref, what):
        ref = ref[..., torch.arange(got.shape[-1], device=ref.device) % POOL]
        if field == "fp":
            assert torch.equal(got, ref), what
        else:
            assert bool(torch.isfinite(torch.view_as_real(got)).all()), what
            err = float(torch.linalg.vector_norm(got - ref) / torch.linalg.vector_norm(ref))
            assert err <= 2e-11, (what, err)

    assert int((wst != 0).sum()) == 0
    for m in SIZES if n < 13 else [s for s in SIZES if s <= 65536]:
        k, e = tiled(torch_dev, field, n, d, m)
        out, st = amp(k, e, npts=m)
        check(out, want, m)
        assert int((st != 0).sum()) == 0
        c, st = cur(k, e, npts=m)
        check(c[:, :m], wcur, ("current", m))
        # no status array: the same values
        out2 = torch.zeros_like(out)
        args = (n, d, m, m + 3) + ((bg.ctypes.c_uint32(P),) if field == "fp" else ())
        fn = bg.lib().bg_amplitudes_fp if field == "fp" else bg.lib().bg_amplitudes_c128
        assert fn(*args, bg._ptr(k), bg._ptr(e), bg._ptr(out2), bg._ptr(None), bg._stream_ptr(None)) == bg.BG_OK
        assert torch.equal(torch.view_as_real(out2) if field == "c128" else out2,
                           torch.view_as_real(out) if field == "c128" else out), m
        if field == "fp" and m in (1025, 65536):
            ka, ea = tiled(torch_dev, field, n, d, m, bg.BG_METRIC_ALTERNATING)
            out, st = amp(ka, ea, npts=m, metric=bg.BG_METRIC_ALTERNATING)
            check(out, want, ("alternating", m))


@pytest.mark.parametrize("n,d,sizes", [(8, 4, (1000, 1024, 1025, 60, 17000)), (9, 6, (4096, 4097, 5, 2000)), (13, 8, (64, 2049, 3))])
def test_served_requests_of_unlike_sizes(torch_dev, n, d, sizes):
    torch, dev = torch_dev
    for plain in (False, True):
        with bg.Server(1 << 28, plain=plain) as srv:
            reqs = []
            for m in sizes * 2:
                k, e = (t.cpu().pin_memory() for t in tiled(torch_dev, "c128", n, d, m))
                out = torch.empty(m, dtype=torch.complex128).pin_memory()
                st = torch.empty(m, dtype=torch.uint8).pin_memory()
                reqs.append((m, k, e, out, st, srv.submit(k, e, out, st, npts=m)))
            for m, k, e, out, st, rid in reqs:
                srv.wait(rid, 60.0)
                o, s = bg.bg_amplitudes_c128(k.to(dev), e.to(dev), npts=m)
                torch.cuda.synchronize()
                assert same_bits(out.numpy(), o.cpu().numpy()) and np.array_equal(st.numpy(), s.cpu().numpy()), m
