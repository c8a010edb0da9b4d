"""Z_p, n = 13 and 14: around the sizes where the card's LDS is full of points of
one kernel and the choice without a pin changes, residues and statuses equal
those of one fixed kernel, with a prime of small and one of large 2^32 mod p."""
import pytest

from paper_2502_07060_amd import bg

from test_gpu_parity import torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [2147483629, 998244353])
@pytest.mark.parametrize("n,d,sizes", [(13, 9, (6144, 6145, 8192, 8193)), (14, 7, (3072, 3073)), (14, 8, (3072, 3073)),
                                       (14, 9, (4097, 12288, 12289))])
def test_choice(torch_dev, n, d, sizes, p):
    torch, dev = torch_dev
    g = torch.Generator(device=dev)
    g.manual_seed(100 * n + d)
    pool = [torch.randint(0, p, (n, d, 61), generator=g, device=dev, dtype=torch.int32) for _ in range(2)]
    fixed = [v for v in bg.bg_variants(bg.BG_FIELD_FP, n, d) if v["lanes"] == 64][-1]["index"]
    bg.bg_select_variant(bg.BG_FIELD_FP, n, d, fixed)
    try:
        want, wst = bg.bg_amplitudes_fp(*pool, p)
    finally:
        bg.bg_select_variant(bg.BG_FIELD_FP, n, d, -1)
    for m in sizes:
        at = torch.arange(m, device=dev) % 61
        out, st = bg.bg_amplitudes_fp(*[t[:, :, at].contiguous() for t in pool], p)
        assert torch.equal(out, want[at]) and torch.equal(st, wst[at]), m
