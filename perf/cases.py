"""Workloads that stand for what programs built on this library ask of it,
through its public entry points (paper_2502_07060_amd.bg), with the kernels
that the library selects by itself:

  amp       one bg_amplitudes_* call on points resident in GPU memory;
  plan      one launch of a recorded batch of mixed (field, n, d) groups;
  cut       a one-leg cut: states of the cut leg, both trees' root currents,
            the sum over states;
  rational  exact rational amplitudes: residues of rational kinematics and
            Z_p amplitudes for each prime, then reconstruction;
  contract, divide  the Z_p operations on their own;
  served    a stream of requests in pinned host memory through the server.

Inputs are physical points made on the GPU from the seed: massless momenta
that add up to zero, transverse polarisations.
"""
import math
import random

import torch

from paper_2502_07060_amd import bg
from paper_2502_07060_amd import inputs as I

P31 = I.DEFAULT_PRIME     # 2^31 - 19, the library's default prime
P30 = 998244353           # a prime whose 2^32 mod p is not small
MM, ALT = bg.BG_METRIC_MOSTLY_MINUS, bg.BG_METRIC_ALTERNATING
SERVED_COLUMNS = 16384    # largest served request

# the largest primes below 2^31, as a multi-prime reconstruction takes them
PRIMES = [2147483647, 2147483629, 2147483587, 2147483579, 2147483563, 2147483549, 2147483543, 2147483497,
          2147483489, 2147483477, 2147483423, 2147483399, 2147483353, 2147483323, 2147483269, 2147483249,
          2147483237, 2147483179, 2147483171, 2147483137]


def listed():
    return [
        # five gluons, 10^4 points: a small call, where latency counts
        dict(name="amp_c128_n5_d4_10k", kind="amp", field="c128", n=5, d=4, p=0, npts=10_000, metric=MM),
        # the headline workload: 2^20 complex eight-gluon points in d = 4
        dict(name="amp_c128_n8_d4_1M", kind="amp", field="c128", n=8, d=4, p=0, npts=1 << 20, metric=MM),
        # the largest complex group of the mixed batch: many legs, a ragged count
        dict(name="amp_c128_n14_d6_163k", kind="amp", field="c128", n=14, d=6, p=0, npts=163_016, metric=MM),
        # the finite-field headline: eight gluons in d = 6
        dict(name="amp_fp_n8_d6_1M", kind="amp", field="fp", n=8, d=6, p=P31, npts=1 << 20, metric=MM),
        # finite field with many legs in d = 8, a ragged count
        dict(name="amp_fp_n12_d8_93k", kind="amp", field="fp", n=12, d=8, p=P31, npts=92_609, metric=MM),
        # the mixed batch: 88 groups, n 4..14, d 4..10, both fields, 4*10^6 points
        dict(name="plan_88groups_4M", kind="plan", total=4_000_000, sizes=4),
        # a one-leg cut of two six-point trees in d = 6 over Z_p
        dict(name="cut_fp_n6_d6_1M", kind="cut", field="fp", n=6, d=6, p=P31, npts=1 << 20),
        # rational five-gluon amplitudes with fourteen primes
        dict(name="rational_n5_d4_14p_262k", kind="rational", n=5, d=4, nprimes=14, npts=1 << 18),
        # z_ik = x_ij y_jk for every event
        dict(name="contract_6x6x6_1M", kind="contract", I=6, J=6, K=6, p=P31, npts=1 << 20, batched=True),
        # z_ik = x_ijl y_jlk for every event: two indices summed, a ragged count
        dict(name="contract_6x36x6_150k", kind="contract", I=6, J=36, K=6, p=P31, npts=150_001, batched=True),
        # elementwise quotients
        dict(name="divide_16M", kind="divide", count=1 << 24, p=P31, scalar=False),
        # a burst of mixed host requests, 1 to 16384 points each
        dict(name="served_96req", kind="served", count=96, trace=5),
    ]


def _log_uniform(rng, lo, hi):
    return int(min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["amp"] * 8 + ["plan", "cut", "cut", "rational", "contract", "contract", "divide", "served"])
    if kind == "amp":
        field = rng.choice(["c128", "fp"])
        n, d = rng.randint(4, 14), rng.choice([4, 4, 5, 6, 6, 7, 8, 9, 10])
        # no more work than the largest listed amplitude call
        cap = int(min(1 << 20, 163_016 * macs(14, 6) / macs(n, d)))
        return dict(kind="amp", field=field, n=n, d=d, p=0 if field == "c128" else rng.choice([P31, P31, P31, P30]),
                    npts=_log_uniform(rng, 1000, cap), metric=rng.choice([MM, MM, MM, MM, ALT]))
    if kind == "plan":
        return dict(kind="plan", total=_log_uniform(rng, 100_000, 4_000_000), sizes=rng.randint(5, 1000))
    if kind == "cut":
        field = rng.choice(["fp", "c128"])
        n, d = rng.randint(4, 7), rng.randint(4, 8)
        return dict(kind="cut", field=field, n=n, d=d, p=P31 if field == "fp" else 0,
                    npts=_log_uniform(rng, 1000, 1 << (20 if field == "fp" else 18)))
    if kind == "rational":
        n = rng.choice([4, 5])
        return dict(kind="rational", n=n, d=4, nprimes=rng.randint(6, 10) if n == 4 else rng.randint(13, 18),
                    npts=_log_uniform(rng, 2000, 1 << 18))
    if kind == "contract":
        J = rng.choice([rng.randint(1, 10), rng.randint(1, 10) * rng.randint(1, 6)])
        c = dict(kind="contract", I=rng.randint(1, 10), J=J, K=rng.randint(1, 10), p=rng.choice([P31, P31, P30]),
                 npts=1, batched=rng.random() < 0.7)
        cap = int(min(1 << 20, (1 << 20) * 108 / (c["I"] * J + J * c["K"] + c["I"] * c["K"])))
        c["npts"] = _log_uniform(rng, 1000, cap)
        return c
    if kind == "divide":
        return dict(kind="divide", count=_log_uniform(rng, 4096, 1 << 24), p=rng.choice([P31, P30]),
                    scalar=rng.random() < 0.3)
    return dict(kind="served", count=rng.randint(16, 96), trace=rng.randint(6, 1000))


# ---------------------------------------------------------------------------
# inputs, on the GPU
# ---------------------------------------------------------------------------
def _gen(seed, salt=0):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1_000_003 + salt) & 0x7FFFFFFF)
    return g


def _signs(d, metric=MM):
    return [1 if mu == 0 or (metric == ALT and mu % 2 == 0) else -1 for mu in range(d)]


def _cdot(x, y, sg):
    """Minkowski product over component axis 0."""
    s = x[0] * y[0]
    for mu in range(1, x.shape[0]):
        s = s + sg[mu] * (x[mu] * y[mu])
    return s


def _c128_points(g, n, d, m, metric=MM):
    """[n][d][m]: flat massless 2 -> n-2 phase space (all outgoing) and
    transverse random polarisations; in the alternating metric the components
    2, 4, ... carry the factor i that maps its products onto the others."""
    f = dict(generator=g, device="cuda", dtype=torch.float64)
    out = n - 2
    e = -torch.log(torch.rand(d - 2, out, m, **f)).sum(0)
    u = torch.randn(out, d - 1, m, **f)
    u /= u.norm(dim=1, keepdim=True)
    v = e[:, None] * u
    Q0, Q = e.sum(0), v.sum(0)
    M = (Q0 * Q0 - (Q * Q).sum(0)).sqrt()
    b, x, gam = -Q / M, 1000.0 / M, Q0 / M
    bq = (b[None] * v).sum(1)
    k = torch.zeros(n, d, m, device="cuda", dtype=torch.float64)
    k[0, 0] = k[1, 0] = k[0, d - 1] = -500.0
    k[1, d - 1] = 500.0
    k[2:, 0] = x * (gam * e + bq)
    k[2:, 1:] = x * (v + b[None] * e[:, None] + ((bq / (1 + gam))[:, None] * b[None]))
    q = torch.randn(d - 1, m, **f)
    q = torch.cat([q.norm(dim=0, keepdim=True), q])
    w = torch.complex(torch.randn(n, d, m, **f), torch.randn(n, d, m, **f))
    sg = _signs(d)
    eps = torch.empty_like(w)
    for l in range(n):
        eps[l] = w[l] - (_cdot(w[l], k[l], sg) / _cdot(q, k[l], sg)) * q
    k = k.to(torch.complex128)
    if metric == ALT:
        k[:, 2::2] *= 1j
        eps[:, 2::2] *= 1j
    return k.contiguous(), eps.contiguous()


def _fp_dot(x, y, sg, p):
    s = torch.zeros_like(x[0])
    for mu in range(x.shape[0]):
        s = (s + sg[mu] * (x[mu] * y[mu] % p)) % p
    return s


def _fp_null(g, d, m, p):
    """[d][m] null vectors mod p in light-cone form: k+ = a^2, k_T = a b, k- = |b|^2."""
    a = torch.randint(1, p, (m,), generator=g, device="cuda")
    b = torch.randint(0, p, (d - 2, m), generator=g, device="cuda")
    bb = torch.zeros_like(a)
    for r in b:
        bb = (bb + r * r % p) % p
    half = (p + 1) // 2
    kp = a * a % p
    v = torch.empty(d, m, device="cuda", dtype=torch.int64)
    v[0] = (kp + bb) % p * half % p
    v[d - 1] = (kp - bb) % p * half % p
    v[1:d - 1] = a * b % p
    return v


def _fp_pow(x, e, p):
    r = torch.ones_like(x)
    while e:
        if e & 1:
            r = r * x % p
        x = x * x % p
        e >>= 1
    return r


def _fp_points(g, n, d, m, p, metric=MM):
    """[n][d][m] residues (int32): null momenta closed by a pair, transverse
    polarisations (q.k) v - (v.k) q; alternating metric as for the complex points."""
    sg = _signs(d)
    k = torch.empty(n, d, m, device="cuda", dtype=torch.int64)
    for l in range(n - 2):
        k[l] = _fp_null(g, d, m, p)
    Q = (-k[:n - 2].sum(0)) % p
    r = _fp_null(g, d, m, p)
    t = _fp_dot(Q, Q, sg, p) * _fp_pow(2 * _fp_dot(Q, r, sg, p) % p, p - 2, p) % p
    k[n - 2] = t * r % p
    k[n - 1] = (Q - k[n - 2]) % p
    q = _fp_null(g, d, m, p)
    eps = torch.empty_like(k)
    for l in range(n):
        v = torch.randint(0, p, (d, m), generator=g, device="cuda")
        eps[l] = (_fp_dot(q, k[l], sg, p) * v % p - _fp_dot(v, k[l], sg, p) * q % p) % p
    if metric == ALT:
        ip = pow(I.fp_sqrt_minus_one(p), -1, p)
        k[:, 2::2] = k[:, 2::2] * ip % p
        eps[:, 2::2] = eps[:, 2::2] * ip % p
    return k.to(torch.int32), eps.to(torch.int32)


def _points(g, field, n, d, m, p, metric=MM):
    return _c128_points(g, n, d, m, metric) if field == "c128" else _fp_points(g, n, d, m, p, metric)


def _residues(g, shape, p, low=0):
    return torch.randint(low, p, shape, generator=g, device="cuda").to(torch.int32)


def _groups(c):
    return [g for g in I.batched_groups(total=c["total"], seed=c["sizes"]) if g["npts"] > 0]


def _requests(c):
    """Mixed requests: uniform field, n and d; sizes uniform in their logarithm."""
    r = random.Random(c["trace"])
    return [dict(field=r.choice(["c128", "fp"]), n=r.randint(4, 14), d=r.choice([4, 6, 10]),
                 npts=_log_uniform(r, 1, SERVED_COLUMNS)) for _ in range(c["count"])]


def _offsets(parts):
    """First output element of each part among those of its field, and the totals."""
    at, tot = [], {"c128": 0, "fp": 0}
    for q in parts:
        at.append(tot[q["field"]])
        tot[q["field"]] += q["npts"]
    return at, tot


def _cut_inputs(c, seed):
    """Legs of both trees; the cut leg l is the last one (l in the left, -l in the right tree)."""
    n, d, m, p = c["n"], c["d"], c["npts"], c["p"]
    g = _gen(seed)
    if c["field"] == "c128":
        v = torch.randn(d - 1, m, generator=g, device="cuda", dtype=torch.float64)
        l = torch.cat([v.norm(dim=0, keepdim=True), v]).to(torch.complex128)
        v = torch.randn(3, m, generator=g, device="cuda", dtype=torch.float64)
        chi = torch.cat([v.norm(dim=0, keepdim=True), v]).to(torch.complex128)
        (kL, eL), (kR, eR) = _c128_points(g, n, d, m), _c128_points(g, n, d, m)
        kL[n - 1], kR[n - 1] = l, -l
    else:
        l, chi = _fp_null(g, d, m, p).to(torch.int32), _fp_null(g, 4, m, p).to(torch.int32)
        (kL, eL), (kR, eR) = _fp_points(g, n, d, m, p), _fp_points(g, n, d, m, p)
        kL[n - 1], kR[n - 1] = l, ((p - l.to(torch.int64)) % p).to(torch.int32)
    return dict(l=l, chi=chi, kL=kL, eL=eL, kR=kR, eR=eR)


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def prepare(case, seed):
    c, g = case, _gen(seed)
    s = dict(case=case)
    if c["kind"] == "amp":
        s["k"], s["e"] = _points(g, c["field"], c["n"], c["d"], c["npts"], c["p"], c["metric"])
    elif c["kind"] == "plan":
        parts = _groups(c)
        at, tot = _offsets(parts)
        s["out_c"] = torch.empty(tot["c128"], dtype=torch.complex128, device="cuda")
        s["out_f"] = torch.empty(tot["fp"], dtype=torch.int32, device="cuda")
        s["st_c"] = torch.empty(tot["c128"], dtype=torch.uint8, device="cuda")
        s["st_f"] = torch.empty(tot["fp"], dtype=torch.uint8, device="cuda")
        s["in"], groups = [], []
        for i, (q, o) in enumerate(zip(parts, at)):
            f = "c" if q["field"] == "c128" else "f"
            ke = _points(_gen(seed, i + 1), q["field"], q["n"], q["d"], q["npts"], P31)
            s["in"].append(ke)
            groups.append(bg.make_group(*ke, s["out_" + f][o:o + q["npts"]], s["st_" + f][o:o + q["npts"]], p=P31))
        s["plan"] = bg.BatchPlan(groups)
    elif c["kind"] == "cut":
        s.update(_cut_inputs(c, seed))
    elif c["kind"] == "rational":
        pool = 128
        rep = -(-c["npts"] // pool)
        arrays = I.rational_points(seed, c["n"], c["d"], pool)
        s["kn"], s["kd"], s["en"], s["ed"] = [
            torch.from_numpy(a).cuda().permute(1, 2, 0).repeat(1, 1, rep)[:, :, :c["npts"]].contiguous() for a in arrays]
        shape = s["kn"].shape
        s["km"], s["em"] = (torch.empty(shape, dtype=torch.int32, device="cuda") for _ in range(2))
        s["kst"], s["est"] = (torch.empty(shape, dtype=torch.uint8, device="cuda") for _ in range(2))
        s["res"] = torch.empty((c["nprimes"], c["npts"]), dtype=torch.int32, device="cuda")
        s["ast"] = torch.empty((c["nprimes"], c["npts"]), dtype=torch.uint8, device="cuda")
    elif c["kind"] == "contract":
        s["x"] = _residues(g, (c["I"], c["J"], c["npts"]), c["p"])
        s["y"] = _residues(g, (c["J"], c["K"], c["npts"]) if c["batched"] else (c["J"], c["K"]), c["p"])
    elif c["kind"] == "divide":
        s["x"] = _residues(g, (c["count"],), c["p"])
        s["y"] = int(_residues(g, (1,), c["p"], 1)) if c["scalar"] else _residues(g, (c["count"],), c["p"], 1)
    else:
        parts = _requests(c)
        at, tot = _offsets(parts)
        pinned = lambda k, dt: torch.empty(k, dtype=dt, pin_memory=True)
        s["out_c"], s["out_f"] = pinned(tot["c128"], torch.complex128), pinned(tot["fp"], torch.int32)
        s["st_c"], s["st_f"] = pinned(tot["c128"], torch.uint8), pinned(tot["fp"], torch.uint8)
        s["requests"] = []
        for i, (q, o) in enumerate(zip(parts, at)):
            f = "c" if q["field"] == "c128" else "f"
            k, e = (pinned(t.shape, t.dtype).copy_(t) for t in
                    _points(_gen(seed, i + 1), q["field"], q["n"], q["d"], q["npts"], P31))
            s["requests"].append((k, e, s["out_" + f][o:o + q["npts"]], s["st_" + f][o:o + q["npts"]]))
        s["server"] = bg.Server(1 << 30)
    return s


def run(s):
    c = s["case"]
    if c["kind"] == "amp":
        metric = None if c["metric"] == MM else c["metric"]
        if c["field"] == "c128":
            out, st = bg.bg_amplitudes_c128(s["k"], s["e"], metric=metric)
        else:
            out, st = bg.bg_amplitudes_fp(s["k"], s["e"], c["p"], metric=metric)
        return {"out": out, "status": st}
    if c["kind"] == "plan":
        s["plan"].launch()
        return {k: s[k] for k in ("out_c", "out_f", "st_c", "st_f")}
    if c["kind"] == "cut":
        if c["field"] == "c128":
            eps, epst, st = bg.bg_states_c128(s["l"], s["chi"])
            KL, stL = bg.bg_currents_c128(s["kL"], s["eL"])
            KR, stR = bg.bg_currents_c128(s["kR"], s["eR"])
            S, stS = bg.bg_state_sum(KL, KR, eps, epst)
        else:
            eps, epst, st = bg.bg_states_fp(s["l"], s["chi"], c["p"])
            KL, stL = bg.bg_currents_fp(s["kL"], s["eL"], c["p"])
            KR, stR = bg.bg_currents_fp(s["kR"], s["eR"], c["p"])
            S, stS = bg.bg_state_sum(KL, KR, eps, epst, p=c["p"])
        return {"S": S, "KL": KL, "KR": KR, "eps": eps, "epst": epst, "status": [st, stL, stR, stS]}
    if c["kind"] == "rational":
        primes = PRIMES[:c["nprimes"]]
        for i, p in enumerate(primes):
            bg.bg_fp_from_rational(p, s["kn"], s["kd"], out=s["km"], status=s["kst"])
            bg.bg_fp_from_rational(p, s["en"], s["ed"], out=s["em"], status=s["est"])
            bg.bg_amplitudes_fp(s["km"], s["em"], p, out=s["res"][i], status=s["ast"][i])
        num, den, st = bg.bg_rational_reconstruct(primes, s["res"])
        return {"num": num, "den": den, "status": st, "residues": s["res"], "amp_status": s["ast"]}
    if c["kind"] == "contract":
        z, st = bg.bg_fp_contract(c["p"], s["x"], s["y"], y_batched=c["batched"])
        return {"z": z, "status": st}
    if c["kind"] == "divide":
        z, st = bg.bg_fp_divide(c["p"], s["x"], s["y"])
        return {"z": z, "status": st}
    ids = [s["server"].submit(k, e, out, st, p=0 if k.is_complex() else P31) for k, e, out, st in s["requests"]]
    for i in ids:
        s["server"].wait(i)
    return {k: s[k] for k in ("out_c", "out_f", "st_c", "st_f")}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def macs(n, d):
    """Field multiply-adds of one amplitude: three dot products and three axpys
    per three-gluon split, one of each per four-gluon split, propagators, root."""
    return d * (6 * math.comb(n, 3) + 4 * math.comb(n, 4) + (n - 1) * (n - 2) - 1)


def _amp_work(field, n, d, m):
    """Bytes (k_1..k_{n-1}, eps_1..eps_n, the result and its status) and
    operations (8 per complex, 2 per Z_p multiply-add)."""
    size = 16 if field == "c128" else 4
    return m * ((2 * n - 1) * d * size + size + 1), m * macs(n, d) * (8 if field == "c128" else 2)


def work(case):
    c = case
    if c["kind"] == "amp":
        b, f = _amp_work(c["field"], c["n"], c["d"], c["npts"])
    elif c["kind"] in ("plan", "served"):
        parts = _groups(c) if c["kind"] == "plan" else _requests(c)
        each = [_amp_work(q["field"], q["n"], q["d"], q["npts"]) for q in parts]
        b, f = sum(x for x, _ in each), sum(x for _, x in each)
    elif c["kind"] == "cut":
        size, ops = (16, 8) if c["field"] == "c128" else (4, 2)
        n, d, m = c["n"], c["d"], c["npts"]
        states = (d - 2) * d
        tree = (2 * n - 2) * d + d
        b = m * (size * (d + 4 + 2 * states + 2 * tree + 1) + 4)   # states and currents written, S from what is in hand
        f = m * ops * (2 * macs(n, d) + 4 * states)
    elif c["kind"] == "rational":
        n, d, m, k = c["n"], c["d"], c["npts"], c["nprimes"]
        L = bg.bg_rr_limbs(k)
        b = m * (2 * n * d * 16 + k * 5 + 8 * L + 1)
        f = m * (k * 2 * (macs(n, d) + 2 * n * d * 4) + 2 * 3 * k * k + 2 * 32 * k * L)
    elif c["kind"] == "contract":
        a = c["I"] * c["J"] + c["I"] * c["K"] + (c["J"] * c["K"] if c["batched"] else 0)
        b, f = c["npts"] * (4 * a + 1), 2 * c["npts"] * c["I"] * c["J"] * c["K"]
    else:
        b, f = c["count"] * (9 if c["scalar"] else 13), 2 * c["count"] * (1 if c["scalar"] else 5)
    return {"bytes": float(b), "flops": float(f)}


# ---------------------------------------------------------------------------
# the same numbers in plain torch (complex field; Z_p results are exact)
# ---------------------------------------------------------------------------
def _exact_current(k, e, sg):
    """K([1..n-1]) by the recursion of the paper's Sec. 2.2 as it stands; k, e: [n][d][m]."""
    N = k.shape[0] - 1
    dot = lambda x, y: _cdot(x, y, sg)
    J, Pm, D = {}, {}, {}
    for i in range(N):
        J[i, i], Pm[i, i] = e[i], k[i]
        for j in range(i + 1, N):
            Pm[i, j] = Pm[i, j - 1] + k[j]
    for length in range(2, N + 1):
        for i in range(N - length + 1):
            j = i + length - 1
            K = torch.zeros_like(k[0])
            D[i, j] = 0
            for t in range(i, j):
                A, B, PA, PB = J[i, t], J[t + 1, j], Pm[i, t], Pm[t + 1, j]
                ab = dot(A, B)
                K += ab * (PA - PB) + (2 * dot(PB, A)) * B - (2 * dot(PA, B)) * A
                D[i, j] = D[i, j] + ab
                if t > i:
                    K -= D[i, t] * B
                if t + 1 < j:
                    K -= D[t + 1, j] * A
                for u in range(t + 1, j):
                    K += (2 * dot(A, J[u + 1, j])) * J[t + 1, u]
            if length == N:
                return K
            J[i, j] = K / dot(Pm[i, j], Pm[i, j])


def _exact_amp(k, e, metric=MM):
    sg = _signs(k.shape[1], metric)
    return _cdot(e[-1], _exact_current(k, e, sg), sg)


def _exact_states(k, chi):
    """States and duals of the paper's Sec. 2.3, [d-2][d][m] each."""
    d, m = k.shape
    sg = _signs(4)
    k4 = k[:4]
    mu2, c2 = _cdot(k4, k4, sg), 2 * _cdot(chi, k4, sg)
    kb = k4 - (mu2 / c2) * chi

    def spinors(v):
        vp, vm = v[0] + v[3], v[0] - v[3]
        vt, vb = v[1] + 1j * v[2], v[1] - 1j * v[2]
        plus = vp.abs().square() >= vm.abs().square()
        one = torch.ones_like(vp)
        lam = torch.stack([torch.where(plus, one, vb / torch.where(plus, one, vm)),
                           torch.where(plus, vt / torch.where(plus, vp, one), one)])
        return lam, torch.stack([torch.where(plus, vp, vt), torch.where(plus, vb, vm)])

    def vec(u, w):
        a, b, cc, dd = u[0] * w[0], u[0] * w[1], u[1] * w[0], u[1] * w[1]
        return torch.stack([a + dd, b + cc, 1j * (b - cc), a - dd]) / 2

    cross = lambda a, b: a[0] * b[1] - a[1] * b[0]
    (lk, tk), (lc, tc) = spinors(kb), spinors(chi)
    E = torch.zeros(d - 2, d, m, dtype=k.dtype, device=k.device)
    T = torch.zeros_like(E)
    E[0, :4] = T[1, :4] = vec(lk, tc) / cross(tk, tc)
    E[1, :4] = T[0, :4] = 2 * vec(lc, tk) / cross(lk, lc)
    mu = lambda y: (k[4:y] * k[4:y]).sum(0)
    if d >= 5:
        E[2, :4] = kb - (mu2 / c2) * chi
        T[2] = E[2] / mu2
    if d >= 6:
        E[3, 4], E[3, 5] = k[5], -k[4]
        T[3] = E[3] / mu(6)
    for x in range(5, d - 1):
        E[x - 1, 4:x + 1] = k[4:x + 1] * k[x + 1]
        E[x - 1, x + 1] = -mu(x + 1)
        T[x - 1] = E[x - 1] / (mu(x + 1) * mu(x + 2))
    return E, T


def exact(case, seed):
    c = case
    if c["kind"] == "amp" and c["field"] == "c128":
        k, e = _points(_gen(seed), "c128", c["n"], c["d"], c["npts"], 0, c["metric"])
        return {"out": _exact_amp(k, e, c["metric"]), "status": None}
    if c["kind"] in ("plan", "served"):
        parts = _groups(c) if c["kind"] == "plan" else _requests(c)
        outs = [_exact_amp(*_points(_gen(seed, i + 1), "c128", q["n"], q["d"], q["npts"], 0))
                for i, q in enumerate(parts) if q["field"] == "c128"]
        return {"out_c": torch.cat(outs), "out_f": None, "st_c": None, "st_f": None} if outs else None
    if c["kind"] == "cut" and c["field"] == "c128":
        v = _cut_inputs(c, seed)
        sg = _signs(c["d"])
        E, T = _exact_states(v["l"], v["chi"])
        KL, KR = _exact_current(v["kL"], v["eL"], sg), _exact_current(v["kR"], v["eR"], sg)
        S = sum(_cdot(a, KL, sg) * _cdot(b, KR, sg) for a, b in zip(E, T))
        return {"S": S, "KL": KL, "KR": KR, "eps": E, "epst": T, "status": None}
    return None
