// From F_p samples back to rational numbers (paper Sec. 1 and Sec. 3: the
// finite-field values at rational kinematic points are reconstructed as
// rationals, as in the comparison with Caravel):
//
//   bg_fp_from_rational      residues n/d mod p of int64 fractions, for
//                            feeding rational kinematics to bg_amplitudes_fp;
//   bg_rational_reconstruct  Chinese remaindering of one residue per prime
//                            followed by rational reconstruction, one point
//                            per lane.
//
// Reconstruction (Wang; von zur Gathen and Gerhard, Modern Computer Algebra,
// Sec. 5.10).  With M = p_1 ... p_k and B = floor(sqrt((M - 1) / 2)):
// the residues give 0 <= x < M (Garner's mixed-radix form, then Horner in
// 32-bit limbs); the extended Euclidean algorithm runs on r_0 = M, r_1 = x,
// t_0 = 0, t_1 = 1 (every r_j = s_j M + t_j x) until the first r_j <= B; the
// result is sign(t_j) r_j / |t_j| when 0 < |t_j| <= B and gcd(t_j, M) = 1
// (which equals gcd(r_j, t_j) = 1, since gcd(s_j, t_j) = 1), else there is
// none.  A fraction with |a| <= B, 0 < b <= B, gcd(a, b) = 1 and a = b x
// (mod M) is unique (2 B^2 < M) and is what this returns.
//
// Limb arithmetic.  The remainders are K 32-bit limbs (K >= number of primes,
// so M < 2^(31 K)).  The cofactors alternate in sign, so their magnitudes are
// kept, with the sign of t_j aside; |t_j| <= M / r_{j-1} < M / B, so
// K / 2 + 1 limbs hold them.  Every limb loop is unrolled over K (no run-time
// register indexing).
#include <hip/hip_runtime.h>

#include <stdint.h>
#include <string.h>

#include <vector>

#include "bg.h"
#include "bg_registry.h"
#include "field_fp.h"

namespace bg {
namespace {

// ---------------------------------------------------------------------------
// residues of fractions
// ---------------------------------------------------------------------------
constexpr int kResidueChunk = 16;  // values per lane: one Fermat power per chunk
constexpr int kResidueVec = 4;     // adjacent values of a lane (32 bytes of num and of den)

struct ResidueArgs {
  const int64_t* num;
  const int64_t* den;
  uint32_t* out;
  uint8_t* status;
  int64_t count;
  FpConst fp;
};

// Bound by HBM traffic (21 bytes a value).  A block of 256 lanes takes 4096
// consecutive values; lane t holds those at 1024 g + 4 t + 0..3 (g < 4), so a
// wave's loads and stores cover whole contiguous pieces (num and den 16 bytes
// a lane and load, out 16 bytes, status 4).  With 16 consecutive values per
// lane every load of a wave touched 64 lines 128 bytes apart and used 8 bytes
// of each: 170 us for 5.2 10^6 values (0.65 TB/s); this layout and the
// three-instruction products take 20.3 us (5.4 TB/s).  VEC = false: single
// values 256 apart, for pointers that are not aligned to the wide accesses.
//
// Products are taken in the Montgomery domain of 2^32 (fp_mul32).  With a_u =
// d_u 2^-64 (balanced, so that d_u = 0 mod p shows as 0), n'_u = n_u 2^-32 and
// P_u = a_0 ... a_u 2^(-32 u), the power gives 2^64 / P_u, taken times 2^-32;
// then n'_u P_{u-1} 2^-32 times that times 2^-32 is n_u / d_u 2^32, and one
// more REDC step leaves n_u / d_u, balanced.
template <bool VEC>
__global__ __launch_bounds__(256) void residue_kernel(ResidueArgs a) {
  const int64_t base = (int64_t)blockIdx.x * (256 * kResidueChunk);
  const FpConst& F = a.fp;
  const bool full = base + 256 * kResidueChunk <= a.count;  // the same in the whole block
  const auto at = [&](int u) {
    return base + (VEC ? (int64_t)(u / kResidueVec) * (256 * kResidueVec) + threadIdx.x * kResidueVec + u % kResidueVec
                       : (int64_t)u * 256 + threadIdx.x);
  };
  int64_t nr[kResidueChunk], dr[kResidueChunk];
  if (VEC && full) {
#pragma unroll
    for (int u = 0; u < kResidueChunk; u += 2) {
      const longlong2 n2 = *reinterpret_cast<const longlong2*>(a.num + at(u));
      const longlong2 d2 = *reinterpret_cast<const longlong2*>(a.den + at(u));
      nr[u] = n2.x;
      nr[u + 1] = n2.y;
      dr[u] = d2.x;
      dr[u + 1] = d2.y;
    }
  } else {
#pragma unroll
    for (int u = 0; u < kResidueChunk; ++u) {
      const int64_t e = at(u);
      nr[u] = e < a.count ? a.num[e] : 0;
      dr[u] = e < a.count ? a.den[e] : 1;
    }
  }
  int32_t nm[kResidueChunk], dm[kResidueChunk];
  uint32_t zero = 0;
  int32_t acc = 0;
  // Montgomery batch inversion of the denominators (Montgomery 1987); a zero
  // denominator is replaced by 1 and its value flagged.
#pragma unroll
  for (int u = 0; u < kResidueChunk; ++u) {
    nm[u] = fp_redc1(fp_fold(nr[u], F), F);
    dm[u] = fp_redc2(fp_fold(dr[u], F), F);
    if (dm[u] == 0) {
      zero |= 1u << u;
      dm[u] = 1;
    }
    if (u > 0) nm[u] = fp_mul32(nm[u], acc, F);
    acc = u > 0 ? fp_mul32(acc, dm[u], F) : dm[0];
  }
  int32_t inv = fp_redc1((int64_t)fp_pow32(acc, (uint32_t)(F.p - 2), F), F);
  uint32_t v[kResidueChunk];
#pragma unroll
  for (int u = kResidueChunk - 1; u >= 0; --u) {
    const int32_t q = fp_mul32(nm[u], inv, F);
    inv = fp_mul32(inv, dm[u], F);
    v[u] = ((zero >> u) & 1u) ? 0xFFFFFFFFu : fp_to_canonical(fp_redc1((int64_t)q, F), F);
  }
  if (VEC && full) {
#pragma unroll
    for (int u = 0; u < kResidueChunk; u += kResidueVec) {
      *reinterpret_cast<uint4*>(a.out + at(u)) = make_uint4(v[u], v[u + 1], v[u + 2], v[u + 3]);
      if (a.status) {
        const uint32_t z = zero >> u;
        *reinterpret_cast<uint32_t*>(a.status + at(u)) =
            (z & 1u) | ((z & 2u) << 7) | ((z & 4u) << 14) | ((z & 8u) << 21);
      }
    }
  } else {
#pragma unroll
    for (int u = 0; u < kResidueChunk; ++u) {
      const int64_t e = at(u);
      if (e < a.count) {
        a.out[e] = v[u];
        if (a.status) a.status[e] = (uint8_t)((zero >> u) & 1u);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Chinese remaindering and rational reconstruction
// ---------------------------------------------------------------------------
constexpr int kPairs = BG_RR_MAX_PRIMES * (BG_RR_MAX_PRIMES - 1) / 2;

struct PrimeConst {
  int32_t p, c32, minv;  // minv = (p_0 ... p_{i-1})^-1 2^64 mod p_i, balanced
  uint32_t pinv;
};

struct RRArgs {
  const uint32_t* residues;  // [nprimes][ld]
  int32_t* num;              // [L][ld] two's complement limbs
  uint32_t* den;             // [L][ld]
  uint8_t* status;
  int64_t npts, ld;
  int nprimes, L;
  double B_double;
  PrimeConst pc[BG_RR_MAX_PRIMES];
  int32_t w[kPairs];  // w[i (i - 1) / 2 + j] = -(p_0 ... p_{j-1}) mod p_i, balanced (j < i)
  uint32_t M[BG_RR_MAX_PRIMES];
  uint32_t B[BG_RR_MAX_PRIMES / 2 + 1];
};

__device__ __forceinline__ FpConst fpc(const PrimeConst& c) {
  FpConst F{};
  F.p = c.p;
  F.pinv = c.pinv;
  F.negp = -c.p;
  F.c32 = c.c32;
  return F;
}

// x <= B, for B of KT limbs
template <int K, int KT>
__device__ __forceinline__ bool not_above(const uint32_t (&x)[K], const uint32_t* B) {
  uint32_t high = 0;
#pragma unroll
  for (int k = KT; k < K; ++k) high |= x[k];
  int64_t borrow = 0;
#pragma unroll
  for (int k = 0; k < (KT < K ? KT : K); ++k) borrow = ((int64_t)B[k] - (int64_t)x[k] + borrow) >> 32;
  return high == 0 && borrow == 0;
}

template <int K>
__device__ __forceinline__ bool below(const uint32_t (&x)[K], const uint32_t (&y)[K]) {
  int64_t borrow = 0;
#pragma unroll
  for (int k = 0; k < K; ++k) borrow = ((int64_t)x[k] - (int64_t)y[k] + borrow) >> 32;
  return borrow != 0;
}

// relative error below K 2^-53 (one rounding a limb)
template <int K>
__device__ __forceinline__ double to_double(const uint32_t (&x)[K]) {
  double v = (double)x[K - 1];
#pragma unroll
  for (int k = K - 2; k >= 0; --k) v = __builtin_fma(v, 4294967296.0, (double)x[k]);
  return v;
}

// x -= c y (mod 2^(32K)); returns the borrow out of the top limb as a signed
// count (negative iff x < c y when both are read as unsigned)
template <int K>
__device__ __forceinline__ int64_t submul(uint32_t (&x)[K], const uint32_t (&y)[K], uint32_t c) {
  uint64_t carry = 0;
  int64_t borrow = 0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const uint64_t prod = (uint64_t)c * y[k] + carry;
    carry = prod >> 32;
    const int64_t diff = (int64_t)x[k] - (int64_t)(uint32_t)prod + borrow;
    x[k] = (uint32_t)diff;
    borrow = diff >> 32;
  }
  return borrow - (int64_t)carry;
}

// x += c y (mod 2^(32K))
template <int K>
__device__ __forceinline__ void addmul(uint32_t (&x)[K], const uint32_t (&y)[K], uint32_t c) {
  uint64_t carry = 0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const uint64_t s = (uint64_t)c * y[k] + ((uint64_t)x[k] + carry);  // < 2^64
    x[k] = (uint32_t)s;
    carry = s >> 32;
  }
}

template <int K>
__device__ __forceinline__ void sub_from(uint32_t (&x)[K], const uint32_t (&y)[K]) {
  int64_t borrow = 0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int64_t d = (int64_t)x[k] - (int64_t)y[k] + borrow;
    x[k] = (uint32_t)d;
    borrow = d >> 32;
  }
}

// y << 32 s (limbs), s in [0, K): a barrel shifter of static moves
template <int K>
__device__ __forceinline__ void shift_limbs(const uint32_t (&y)[K], int s, uint32_t (&out)[K]) {
#pragma unroll
  for (int k = 0; k < K; ++k) out[k] = y[k];
#pragma unroll
  for (int b = 1; b < K; b <<= 1) {
    const bool on = (s & b) != 0;
#pragma unroll
    for (int k = K - 1; k >= 0; --k) out[k] = on ? (k >= b ? out[k - b] : 0u) : out[k];
  }
}

// (x, y) <- (a x - b y, d y - c x), both results in [0, 2^(32K)); a, b, c, d < 2^26
template <int K>
__device__ __forceinline__ void mix_sub(uint32_t (&x)[K], uint32_t (&y)[K], uint32_t a, uint32_t b, uint32_t c,
                                        uint32_t d) {
  int64_t cx = 0, cy = 0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const uint64_t X = (uint64_t)a * x[k] + (uint64_t)cx - (uint64_t)b * y[k];
    const uint64_t Y = (uint64_t)d * y[k] + (uint64_t)cy - (uint64_t)c * x[k];
    x[k] = (uint32_t)X;
    y[k] = (uint32_t)Y;
    cx = (int64_t)X >> 32;
    cy = (int64_t)Y >> 32;
  }
}

// (x, y) <- (a x + b y, d y + c x)
template <int K>
__device__ __forceinline__ void mix_add(uint32_t (&x)[K], uint32_t (&y)[K], uint32_t a, uint32_t b, uint32_t c,
                                        uint32_t d) {
  uint64_t cx = 0, cy = 0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const uint64_t X = (uint64_t)a * x[k] + cx + (uint64_t)b * y[k];
    const uint64_t Y = (uint64_t)d * y[k] + cy + (uint64_t)c * x[k];
    x[k] = (uint32_t)X;
    y[k] = (uint32_t)Y;
    cx = X >> 32;
    cy = Y >> 32;
  }
}

template <int K>
__device__ __forceinline__ void negate(uint32_t (&x)[K]) {
  uint64_t carry = 1;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const uint64_t s = (uint64_t)(~x[k]) + carry;
    x[k] = (uint32_t)s;
    carry = s >> 32;
  }
}

// whether p divides x: the limbs from the lowest up, each step a REDC of the
// sum so far (a division by 2^32 mod p); |sum| < 2^33, the last REDC balanced
template <int K>
__device__ __forceinline__ bool divisible(const uint32_t (&x)[K], const FpConst& F) {
  int64_t s = (int64_t)x[0];
#pragma unroll
  for (int k = 1; k < K; ++k) s = (int64_t)fp_redc1(s, F) + (int64_t)x[k];
  return fp_redc1((int64_t)fp_redc1(s, F), F) == 0;
}

// One Euclidean step on the whole numbers, for a quotient that the leading
// bits do not settle: (r0, r1) <- (r1, r0 mod r1), the cofactors likewise;
// a quotient of 2^31 or more is only begun (r0 less a multiple of r1).
template <int K, int KT>
__device__ __forceinline__ void full_step(uint32_t (&r0)[K], uint32_t (&r1)[K], uint32_t (&t0)[KT],
                                          uint32_t (&t1)[KT], bool& neg, double qe) {
  if (qe < 2147483648.0) {
    uint32_t qq = (uint32_t)qe;
    int64_t bo = submul(r0, r1, qq);
    while (bo < 0) {  // over-estimate: add r1 back
      uint64_t carry = 0;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const uint64_t s = (uint64_t)r0[k] + r1[k] + carry;
        r0[k] = (uint32_t)s;
        carry = s >> 32;
      }
      bo += (int64_t)carry;
      --qq;
    }
    while (!below(r0, r1)) {  // under-estimate
      sub_from(r0, r1);
      ++qq;
    }
    addmul(t0, t1, qq);
    neg = !neg;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const uint32_t a0 = r0[k];
      r0[k] = r1[k];
      r1[k] = a0;
    }
#pragma unroll
    for (int k = 0; k < KT; ++k) {
      const uint32_t b0 = t0[k];
      t0[k] = t1[k];
      t1[k] = b0;
    }
  } else {
    // take c 2^(32 s) out of the quotient, c < 2^64 an under-estimate
    int e = 0;
    (void)frexp(qe, &e);  // qe in [2^(e-1), 2^e)
    const int s = e > 64 ? (e - 64 + 31) / 32 : 0;
    const double scaled = ldexp(qe, -32 * s) * (1.0 - 0x1p-40);
    uint64_t c = scaled >= 18446744073709551616.0 ? ~0ull : (uint64_t)scaled;
    if (c > 0) c -= 1;
    uint32_t ys[K], ts[KT];
    // low 32 bits of c at limb offset s, high 32 bits at s + 1
    shift_limbs(r1, s, ys);
    (void)submul(r0, ys, (uint32_t)c);
    shift_limbs(t1, s, ts);
    addmul(t0, ts, (uint32_t)c);
    if (c >> 32) {
      shift_limbs(r1, s + 1, ys);
      (void)submul(r0, ys, (uint32_t)(c >> 32));
      shift_limbs(t1, s + 1, ts);
      addmul(t0, ts, (uint32_t)(c >> 32));
    }
  }
}

// One point per lane, bound by integer and FP64 instructions.  Euclid's steps
// are taken in groups on the leading bits (Lehmer): with u, v the two
// remainders scaled to 48 bits, pairs of quotients come from u, v alone and
// their product, a 2 x 2 matrix of factors below 2^26, is applied to the whole
// numbers once.  A group's last pair must satisfy, for the factors y of r_1,
//   w >= 4 y1,  v - w >= 4 (y1 + y0),  w - z >= 4 (y2 + y1),  z >= 4 y2 + B / 2^s + 4
// (u, v, w, z successive remainders).  u and v are within 2 of the scaled
// remainders (one truncation, and K 2^-53 of a value below 2^48), and a factor
// of r_0 is no larger than that of r_1, so a remainder formed from them is
// within 4 y of the scaled true one: the conditions make the true remainders
// fall strictly in turn and stay above B, so the quotients are Euclid's own
// (Collins' condition with room for the rounding) and the loop stops at the
// same step.  What they do not settle takes a full_step.
// A step on whole numbers at a time cost 2 K multiply-adds and two
// conversions of K limbs per quotient: 468 us for 2^18 points with 14 primes;
// the groups, limb counts that follow the number of primes, half-length
// cofactors and Garner's digits from a table of weights take 89 us.
template <int K>
__global__ __launch_bounds__(256) void rr_kernel(RRArgs a) {
  constexpr int KT = K / 2 + 1;
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= a.npts) return;
  const int P = a.nprimes;
  uint8_t st = 0;
  // ---- residues and Garner's mixed-radix digits v_i (x = v_0 + p_0 (v_1 + p_1 (...))):
  // v_i = (r_i - sum_{j<i} v_j p_0 ... p_{j-1}) (p_0 ... p_{i-1})^-1 mod p_i
  uint32_t v[K];
#pragma unroll
  for (int i = 0; i < K; ++i) v[i] = i < P ? a.residues[(int64_t)i * a.ld + q] : 0u;
#pragma unroll
  for (int i = 0; i < K; ++i) {
    if (i < P) {
      const FpConst F = fpc(a.pc[i]);
      if (v[i] >= (uint32_t)F.p) {
        st = 2;
        v[i] = 0;
      }
      int64_t T = (int64_t)v[i];
#pragma unroll
      for (int j = 0; j < i; ++j) {
        T = mad64((int32_t)v[j], a.w[i * (i - 1) / 2 + j], T);  // below 2^61 each
        if (j & 1) T = fp_fold(T, F);
      }
      const int32_t d = fp_mul32(fp_redc1(fp_fold(T, F), F), a.pc[i].minv, F);  // in (-p, p)
      v[i] = fp_to_canonical(d, F);
    }
  }
  // ---- r_1 = x: x = v_{P-1}; x = x p_i + v_i for i = P-2 .. 0
  uint32_t r0[K], r1[K], t0[KT], t1[KT];
#pragma unroll
  for (int k = 0; k < K; ++k) r1[k] = 0;
#pragma unroll
  for (int i = K - 1; i >= 0; --i) {
    if (i < P) {
      uint64_t carry = v[i];
      const uint32_t p = (uint32_t)a.pc[i].p;
#pragma unroll
      for (int k = 0; k < K - i; ++k) {  // the product so far fills P - i limbs
        const uint64_t s = (uint64_t)r1[k] * p + carry;
        r1[k] = (uint32_t)s;
        carry = s >> 32;
      }
    }
  }
  // ---- extended Euclid on (M, x) until the remainder is <= B
#pragma unroll
  for (int k = 0; k < K; ++k) r0[k] = a.M[k];
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    t0[k] = 0;
    t1[k] = k == 0 ? 1u : 0u;
  }
  bool neg = false;  // the sign of t_1
  // every step shrinks the remainders: a quotient at least halves r_j two
  // steps on, a large-quotient piece removes 32 bits or more; the cap only
  // guarantees that every lane leaves the loop
  const int cap = 96 * K + 64;
  int it = 0;
  for (; it < cap; ++it) {
    const double r0d = to_double(r0), r1d = to_double(r1);
    // clearly above B, else compare the limbs
    if (!(r1d > a.B_double * (1.0 + 0x1p-40)) && not_above<K, KT>(r1, a.B)) break;
    int e = __builtin_amdgcn_frexp_exp(r0d) - 48;
    e = e > 0 ? e : 0;
    double u = __builtin_trunc(__builtin_amdgcn_ldexp(r0d, -e)), v1 = __builtin_trunc(__builtin_amdgcn_ldexp(r1d, -e));
    const double stop = __builtin_amdgcn_ldexp(a.B_double, -e) + 4.0;
    double ma = 1.0, mb = 0.0, mc = 0.0, md = 1.0;  // u = ma r_0 - mb r_1, v1 = md r_1 - mc r_0
    bool some = false;
    for (;;) {
      // the estimates may be off by one for a large quotient: the conditions
      // then fail, as they do for v1 = 0 or w = 0 (a NaN compares false)
      const double q1 = __builtin_trunc(u * __builtin_amdgcn_rcp(v1));
      const double w = __builtin_fma(-q1, v1, u);
      const double q2 = __builtin_trunc(v1 * __builtin_amdgcn_rcp(w));
      const double z = __builtin_fma(-q2, w, v1);
      const double y1 = __builtin_fma(q1, md, mb), y2 = __builtin_fma(q2, y1, md);
      const bool ok = (w >= 4.0 * y1) & (v1 - w >= 4.0 * (y1 + md)) & (w - z >= 4.0 * (y2 + y1)) &
                      (z >= __builtin_fma(4.0, y2, stop));
      if (!ok) break;
      const double x1 = __builtin_fma(q1, mc, ma);
      mc = __builtin_fma(q2, x1, mc);
      ma = x1;
      mb = y1;
      md = y2;
      u = w;
      v1 = z;
      some = true;
    }
    if (some) {
      const uint32_t A = (uint32_t)ma, Bm = (uint32_t)mb, C = (uint32_t)mc, D = (uint32_t)md;
      mix_sub(r0, r1, A, Bm, C, D);
      mix_add(t0, t1, A, Bm, C, D);
    } else {
      full_step<K, KT>(r0, r1, t0, t1, neg, r0d / r1d);
    }
  }
  // ---- checks and output: a = sign(t) r, b = |t|
  uint32_t any = 0;
#pragma unroll
  for (int k = 0; k < KT; ++k) any |= t1[k];
  bool ok = st == 0 && it < cap && any != 0 && not_above<KT, KT>(t1, a.B);
#pragma unroll
  for (int i = 0; i < K; ++i)
    if (i < P && divisible(t1, fpc(a.pc[i]))) ok = false;  // gcd(t, M) != 1
  if (ok && neg) negate(r1);
  const int L = a.L;
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    if (k < L) {
      a.num[(int64_t)k * a.ld + q] = ok ? (int32_t)(k < K ? r1[k] : 0u) : 0;
      a.den[(int64_t)k * a.ld + q] = ok ? t1[k] : 0u;
    }
  }
  if (a.status) a.status[q] = st ? st : (ok ? 0 : 1);
}

// ---------------------------------------------------------------------------
// host side: limb integers
// ---------------------------------------------------------------------------
using Big = std::vector<uint32_t>;  // little-endian limbs

void big_mul_small(Big& x, uint32_t m) {
  uint64_t carry = 0;
  for (auto& w : x) {
    const uint64_t s = (uint64_t)w * m + carry;
    w = (uint32_t)s;
    carry = s >> 32;
  }
  if (carry) x.push_back((uint32_t)carry);
}

int big_cmp(const Big& x, const Big& y) {
  const size_t n = x.size() > y.size() ? x.size() : y.size();
  for (size_t k = n; k-- > 0;) {
    const uint32_t a = k < x.size() ? x[k] : 0, b = k < y.size() ? y[k] : 0;
    if (a != b) return a > b ? 1 : -1;
  }
  return 0;
}

Big big_sq(const Big& x) {
  Big r(2 * x.size() + 1, 0);
  for (size_t i = 0; i < x.size(); ++i) {
    uint64_t carry = 0;
    for (size_t j = 0; j < x.size(); ++j) {
      const uint64_t s = (uint64_t)x[i] * x[j] + r[i + j] + carry;
      r[i + j] = (uint32_t)s;
      carry = s >> 32;
    }
    size_t k = i + x.size();
    while (carry) {
      const uint64_t s = (uint64_t)r[k] + carry;
      r[k++] = (uint32_t)s;
      carry = s >> 32;
    }
  }
  return r;
}

// floor(sqrt(N)), bit by bit from the top
Big big_isqrt(const Big& N) {
  size_t bits = N.size() * 32;
  Big root((N.size() + 1) / 2 + 1, 0);
  for (size_t b = bits / 2 + 1; b-- > 0;) {
    Big cand = root;
    cand[b / 32] |= 1u << (b % 32);
    if (big_cmp(big_sq(cand), N) <= 0) root = cand;
  }
  return root;
}

uint64_t powmod64(uint64_t a, uint64_t e, uint64_t m) {
  uint64_t r = 1 % m;
  a %= m;
  while (e) {
    if (e & 1) r = (unsigned __int128)r * a % m;
    a = (unsigned __int128)a * a % m;
    e >>= 1;
  }
  return r;
}

int32_t bal(uint64_t x, uint64_t p) {
  x %= p;
  return x > (p - 1) / 2 ? (int32_t)((int64_t)x - (int64_t)p) : (int32_t)x;
}

}  // namespace
}  // namespace bg

extern "C" {

int bg_fp_from_rational(uint32_t p, int64_t count, const int64_t* num, const int64_t* den, uint32_t* out,
                        uint8_t* status, void* hip_stream) {
  if (p < 3 || p >= 0x80000000u || !bg::is_prime_u32(p)) return BG_ENOTPRIME;
  if (count < 0) return BG_EINVAL;
  if (count == 0) return BG_OK;
  if (!num || !den || !out) return BG_EINVAL;
  bg::ResidueArgs a{};
  a.num = num;
  a.den = den;
  a.out = out;
  a.status = status;
  a.count = count;
  a.fp = bg::make_fp_const(p);
  const int64_t per = 256 * bg::kResidueChunk;
  const int64_t blocks = (count + per - 1) / per;
  if (blocks > 0x7FFFFFFF) return BG_EINVAL;
  // wide accesses need their alignment (torch tensors and hipMalloc have it;
  // a view may not)
  const bool vec = (((uintptr_t)num | (uintptr_t)den | (uintptr_t)out) & 15) == 0 && ((uintptr_t)status & 3) == 0;
  const void* fn = vec ? reinterpret_cast<const void*>(&bg::residue_kernel<true>)
                       : reinterpret_cast<const void*>(&bg::residue_kernel<false>);
  void* args[] = {&a};
  return hipLaunchKernel(fn, dim3((unsigned)blocks), dim3(256), args, 0, static_cast<hipStream_t>(hip_stream)) ==
                 hipSuccess
             ? BG_OK
             : BG_EHIP;
}

int bg_rational_reconstruct(int nprimes, const uint32_t* primes, int64_t npts, int64_t ld,
                            const uint32_t* residues, int32_t* num, uint32_t* den, uint8_t* status,
                            void* hip_stream) {
  if (nprimes < 1 || nprimes > BG_RR_MAX_PRIMES || !primes) return BG_EINVAL;
  for (int i = 0; i < nprimes; ++i) {
    if (primes[i] < 3 || primes[i] >= 0x80000000u || !bg::is_prime_u32(primes[i])) return BG_ENOTPRIME;
    for (int j = 0; j < i; ++j)
      if (primes[j] == primes[i]) return BG_EINVAL;
  }
  if (npts < 0) return BG_EINVAL;
  if (npts == 0) return BG_OK;
  if (ld < npts || !residues || !num || !den) return BG_EINVAL;
  bg::RRArgs a{};
  memset(&a, 0, sizeof(a));
  a.residues = residues;
  a.num = num;
  a.den = den;
  a.status = status;
  a.npts = npts;
  a.ld = ld;
  a.nprimes = nprimes;
  a.L = BG_RR_LIMBS(nprimes);
  bg::Big M{1};
  for (int i = 0; i < nprimes; ++i) {
    const uint64_t p = primes[i];
    const bg::FpConst k = bg::make_fp_const((uint32_t)p);
    bg::PrimeConst& c = a.pc[i];
    c.p = k.p;
    c.c32 = k.c32;
    c.pinv = k.pinv;
    uint64_t prod = 1;  // p_0 ... p_{j-1} mod p_i
    for (int j = 0; j < i; ++j) {
      a.w[i * (i - 1) / 2 + j] = -bg::bal(prod, p);
      prod = (unsigned __int128)prod * (primes[j] % p) % p;
    }
    const uint64_t inv = bg::powmod64(prod, p - 2, p);
    c.minv = bg::bal((unsigned __int128)inv * bg::powmod64(2, 64, p) % p, p);
    bg::big_mul_small(M, (uint32_t)p);
  }
  bg::Big Mm1 = M;  // (M - 1) / 2; M is odd, so M - 1 only clears bit 0
  Mm1[0] -= 1;
  for (size_t k = 0; k < Mm1.size(); ++k) Mm1[k] = (Mm1[k] >> 1) | (k + 1 < Mm1.size() ? (Mm1[k + 1] << 31) : 0u);
  const bg::Big Bv = bg::big_isqrt(Mm1);
  for (size_t k = 0; k < M.size() && k < (size_t)BG_RR_MAX_PRIMES; ++k) a.M[k] = M[k];
  for (size_t k = Bv.size(); k-- > 0;) {
    if (k < sizeof(a.B) / sizeof(a.B[0])) a.B[k] = Bv[k];
    a.B_double = a.B_double * 4294967296.0 + (double)Bv[k];
  }
  const int64_t blocks = (npts + 255) / 256;
  if (blocks > 0x7FFFFFFF) return BG_EINVAL;
  static const void* const kernels[] = {
      reinterpret_cast<const void*>(&bg::rr_kernel<2>),  reinterpret_cast<const void*>(&bg::rr_kernel<4>),
      reinterpret_cast<const void*>(&bg::rr_kernel<6>),  reinterpret_cast<const void*>(&bg::rr_kernel<8>),
      reinterpret_cast<const void*>(&bg::rr_kernel<10>), reinterpret_cast<const void*>(&bg::rr_kernel<12>),
      reinterpret_cast<const void*>(&bg::rr_kernel<14>), reinterpret_cast<const void*>(&bg::rr_kernel<16>),
      reinterpret_cast<const void*>(&bg::rr_kernel<20>), reinterpret_cast<const void*>(&bg::rr_kernel<24>),
      reinterpret_cast<const void*>(&bg::rr_kernel<28>), reinterpret_cast<const void*>(&bg::rr_kernel<32>)};
  const void* fn = kernels[nprimes <= 16 ? (nprimes - 1) / 2 : 8 + (nprimes - 17) / 4];
  void* args[] = {&a};
  return hipLaunchKernel(fn, dim3((unsigned)blocks), dim3(256), args, 0, static_cast<hipStream_t>(hip_stream)) ==
                 hipSuccess
             ? BG_OK
             : BG_EHIP;
}

}  // extern "C"
