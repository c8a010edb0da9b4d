"""Worst-case int64 bounds of the Z_p lane-group kernels' small-fold-constant
schedule (csrc/bg_wide.h, FpField<DL, LC, true>), replayed with the largest
magnitude each operand can have, as test_fp_bounds does for the other kernels:
the fold decisions mirror the kernel's own unit counters, every partial sum is
bounded exactly.  And the general schedule's finish, which folds a current's
accumulator once, after the prefix sums joined it."""
import pytest

from test_fp_bounds import Bounds, FieldModel, FieldModelSC, Vec, _c32_extreme_prime, _sc_extreme_prime


def replay_small_fold(p, N, DL, LC):
    B = Bounds(p)
    F = FieldModelSC(B, DL, LC)
    h = B.h
    nb = h + 2**23                                # currents and lazy scalars
    lazyP = 2 * h
    inv = p - 1                                   # products of the 2^32 domain lie in (-p, p)
    nc = F.ndot(lazyP, h, UX=4, lazy=True)        # legs
    for m in range(2, N + 1):
        pairs = m // 2
        per = 1
        while per < pairs:
            per *= 2
        Kp, nDs = Vec(B), 0
        for _cut in range(2):
            nDm = F.ndot(nb, nb, lazy=True)
            nc2 = F.ndot_sub2(lazyP, nb, nc, h, UX=4, UZ=3, lazy=True)
            nc3 = F.ndot_sub2(lazyP, nb, nc, h, UX=4, UZ=3, lazy=True)
            assert max(nDm, nc2, nc3, nc) <= nb
            Kp.axpy(nDm, h)                       # times Q_{c+1} (balanced)
            Kp.axpy(nc2, nb)
            Kp.axpy(nc3, nb)
            nDs = B.chk(nDs + nDm * h, "nDs")     # not folded between the cuts
        Kp.fold()
        cnt = 0
        for _q in range(max(0, m - 2)):
            Kp.axpy(F.ndot(nb, nb, lazy=True), nb)
            cnt += 1
            if cnt == 7:
                Kp.fold()
                cnt = 0
        Kp.fold()
        nDs = B.fold(nDs)
        # sums over the item slots: no folds
        acc = B.chk(per * Kp.b, "sum of K")
        nd = B.chk(per * nDs, "sum of nDs")
        assert B.redc2(nd) <= h
        K = Vec(B)
        K.b = acc
        K.axpy(h, 2 * h)                          # Dh(S) (Q_i + Q_{j+1})
        if m == N:
            K.fold()
            assert B.redc2(B.fold(K.b)) <= h      # finish
            continue
        J = B.redc1(B.fold(B.chk(B.redc1(B.fold(K.b)) * inv, "finish product")))
        assert J <= nb
        t, u = 0, 0                               # P_S . J_S over a slot's components
        for _c in range(DL):
            if u + 129 > 511:
                t, u = B.fold(t), 1
            t = B.chk(t + lazyP * J, "P.J")
            u += 129
        t = B.chk(per * B.fold(t), "P.J over slots")
        nc = max(nc, F.finish_dot(t, 32, lazy=True))


@pytest.mark.parametrize("p", [2**31 - 1, 2147483629, _sc_extreme_prime(+1), _sc_extreme_prime(-1), 65537, 13])
def test_small_fold_schedule(p):
    from paper_2502_07060_amd import build as b
    for f, dm, G, _pad, LC in b.WIDE_VARIANTS:
        if f == "fp":
            for N in range(2, 14):
                replay_small_fold(p, N, dm // LC, LC)


@pytest.mark.parametrize("p", [2**31 - 1, _c32_extreme_prime(+1), _c32_extreme_prime(-1)])
def test_general_finish(p):
    B = Bounds(p)
    folded = 2**31 * B.h + 2**32                  # a folded sum of any items
    K = B.chk(folded + B.h * 2 * B.h, "Dh(S) (Q_i + Q_{j+1})")
    B.redc2(B.chk(B.redc1(B.fold(K)) * (p - 1), "finish_mul32"))
