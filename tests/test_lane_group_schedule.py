"""The order in which the items of a complex lane group take the propagators
(csrc/bg_wide.h: propagators): every range of length 2 .. N-1 once, whatever N
and the number of items, with the division by N done as a product and a shift."""
import pytest


@pytest.mark.parametrize("G", [16, 32, 64])
@pytest.mark.parametrize("N", range(2, 14))
def test_every_range_once(N, G):
    rec = 65536 // N + 1
    seen = []
    for g in range(G):
        for e in range(g, N * (N // 2), G):
            row = (e * rec) >> 16
            t = e - row * N
            assert row == e // N
            n1 = N - 1 - row
            m, i = (row + 2, t) if t < n1 else (N - row, t - n1)
            if (t >= n1 and m <= row + 2) or m >= N:
                continue
            assert 0 <= i <= N - m
            seen.append((i, i + m - 1))
    assert len(seen) == len(set(seen))
    assert set(seen) == {(i, j) for i in range(N) for j in range(i + 1, N) if j - i + 1 < N}
