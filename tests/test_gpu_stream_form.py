"""Complex register kernels that stay on the card and read each point's inputs
one point ahead (launches of more than two rounds of resident blocks): around the
size where they start, at whole and ragged numbers of rounds, amplitudes, root
currents and status equal those of the same kernel on one small batch, within
twice the 1e-11 that each launch keeps to the exact value, over the norm of all
points; singular points stay where they are."""
import numpy as np
import pytest

from paper_2502_07060_amd import bg
from paper_2502_07060_amd import inputs as I

from test_gpu_parity import torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu
POOL = 67
SINGULAR = 5  # this point of the pool has two equal and opposite momenta


@pytest.mark.parametrize("metric", [bg.BG_METRIC_MOSTLY_MINUS, bg.BG_METRIC_ALTERNATING])
@pytest.mark.parametrize("n,d,lanes,comps", [(5, 8, 2, 4), (6, 6, 2, 3), (6, 9, 4, 3), (7, 4, 2, 2), (7, 7, 4, 2),
                                             (8, 4, 2, 2), (8, 5, 4, 2)])
def test_rounds(torch_dev, n, d, lanes, comps, metric):
    torch, dev = torch_dev
    tag = bg.BG_FIELD_C128
    v = [v for v in bg.bg_variants(tag, n, d) if not v["generic"] and v["lanes"] == lanes and v["comps_per_lane"] == comps]
    assert len(v) == 1
    k, e = I.generic_c128(31 * n + d, n, d, POOL)
    k = np.array(k, dtype=np.complex128)
    k[SINGULAR, 1] = -k[SINGULAR, 0]  # P_{1,2} = 0
    k, e = (I.to_soa(np.asarray(a, dtype=np.complex128)) for a in (k, e))
    per_round = torch.cuda.get_device_properties(dev).multi_processor_count * (256 // lanes)

    def tiled(m):
        at = torch.arange(m + 3, device=dev) % POOL
        return [torch.from_numpy(np.ascontiguousarray(a)).to(dev)[:, :, at].contiguous() for a in (k, e)]

    bg.bg_select_variant(tag, n, d, v[0]["index"], metric)
    try:
        small = tiled(POOL)
        want, wst = bg.bg_amplitudes_c128(*small, npts=POOL, metric=metric)
        wcur = bg.bg_currents_c128(*small, npts=POOL)[0][:, :POOL]
        assert wst[SINGULAR] != 0 and int((wst != 0).sum()) == 1
        for m in (2 * per_round, 2 * per_round + 1, 3 * per_round - 1, 3 * per_round, 4 * per_round + 129):
            at = torch.arange(m, device=dev) % POOL
            ke = tiled(m)
            calls = [(bg.bg_amplitudes_c128(*ke, npts=m, metric=metric), want)]
            if metric == bg.BG_METRIC_MOSTLY_MINUS:  # root currents have no other
                calls.append((bg.bg_currents_c128(*ke, npts=m), wcur))
            for got, ref in calls:
                assert torch.equal(got[1], wst[at])
                x, y = got[0][..., :m], ref[..., at]
                bad = torch.isnan(y.real)
                assert torch.equal(torch.isnan(x.real), bad)
                err = torch.linalg.vector_norm(torch.where(bad, 0, x - y)) / torch.linalg.vector_norm(torch.where(bad, 0, y))
                assert float(err) <= 2e-11, (m, float(err))
    finally:
        bg.bg_select_variant(tag, n, d, -1, metric)
