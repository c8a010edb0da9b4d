// Polarisation states of massless d-dimensional gluons (paper Sec. 2.3), one
// point per lane: bg_states_c128 and bg_states_fp.
//
// For a massless d-vector k and a massless four-dimensional reference chi:
//   k4 = (k^0..k^3, 0, ...), mu^2 = k4.k4, c = mu^2 / (2 chi.k4),
//   kb = k4 - c chi (massless),
//   e1 = <kb|gamma|chi] / (2 [kb chi]),   e2 = [kb|gamma|chi> / <kb chi>,
//   e1~ = e2, e2~ = e1;
//   d >= 5:  e3 = kb - c chi,  e3~ = e3 / mu^2;
//   d >= 6:  e4 = (0,0,0,0, k^5, -k^4, 0..),  e4~ = e4 / mu_6^2;
//   5 <= x <= d-2:  ex^i = k^i k^{x+1} (4 <= i <= x), ex^{x+1} = -mu_{x+1}^2,
//                   ex~ = ex / (mu_{x+1}^2 mu_{x+2}^2),
// with mu_y^2 = sum_{i=4}^{y-1} (k^i)^2 (the reading of the printed d > 6
// formula in the design notes).  Spinors of a massless four-vector v use the
// chart lam = (1, (v^1 + i v^2)/v+), lamt = (v+, v^1 - i v^2) when v+ != 0
// (F_p) or |v+|^2 >= |v-|^2 (complex), else lam = ((v^1 - i v^2)/v-, 1),
// lamt = (v^1 + i v^2, v-); the four-vector of u w^T is
// ((M11+M22)/2, (M12+M21)/2, i(M12-M21)/2, (M11-M22)/2).
//
// F_p: Montgomery residues of 2^32 (field_fp.h); i is the square root of -1
// g^((p-1)/4) for the smallest quadratic non-residue g, so p = 1 (mod 4) is
// required.  Every quantity is kept as a numerator over products of 2 chi.k4,
// the chart components and the brackets, so that one batched inversion
// (Montgomery's trick, one Fermat power) serves the point (point_states_fp).
// Over C the inverses are taken where they occur.
#include <hip/hip_runtime.h>

#include "bg.h"
#include "bg_registry.h"

namespace bg {
namespace {

constexpr int SD = BG_MAX_D;  // components held per point (d <= SD)

struct StatesArgs {
  const void* momenta;  // [d][ld]
  const void* chi;      // [4][ld]
  void* eps;            // [d-2][d][ld]
  void* epst;           // [d-2][d][ld]
  uint8_t* status;
  int64_t npts, ld;
  int d;
  FpConst fp;
  int32_t i_rep;  // F_p: sqrt(-1) 2^32 mod p
};

// ---- complex field ----------------------------------------------------------
struct COps {
  using T = cplx;
  __device__ T add(T a, T b) const { return cadd(a, b); }
  __device__ T sub(T a, T b) const { return csub(a, b); }
  __device__ T mul(T a, T b) const { return cmul(a, b); }
  __device__ T neg(T a) const { return cneg(a); }
  __device__ T zero() const { return {0.0, 0.0}; }
  __device__ T one() const { return {1.0, 0.0}; }
  __device__ T half() const { return {0.5, 0.0}; }
  __device__ T two() const { return {2.0, 0.0}; }
  __device__ T iu() const { return {0.0, 1.0}; }
  __device__ bool is_zero(T a) const { return a.re == 0.0 && a.im == 0.0; }
  __device__ bool plus_chart(T vp, T vm) const {
    return vp.re * vp.re + vp.im * vp.im >= vm.re * vm.re + vm.im * vm.im;
  }
  template <int M>
  __device__ void inv_batch(T (&x)[M], int n) const {
#pragma unroll
    for (int s = 0; s < M; ++s)
      if (s < n) {
        const double den = x[s].re * x[s].re + x[s].im * x[s].im;
        x[s] = {x[s].re / den, -x[s].im / den};
      }
  }
};

template <class Ops, class T>
__device__ __forceinline__ T mdot4(const Ops& o, const T* x, const T* y) {
  T s = o.mul(x[0], y[0]);
#pragma unroll
  for (int m = 1; m < 4; ++m) s = o.sub(s, o.mul(x[m], y[m]));
  return s;
}

// the four-vector of u w^T
template <class Ops, class T>
__device__ __forceinline__ void vec_of(const Ops& o, const T* u, const T* w, T* out) {
  const T m11 = o.mul(u[0], w[0]), m12 = o.mul(u[0], w[1]);
  const T m21 = o.mul(u[1], w[0]), m22 = o.mul(u[1], w[1]);
  out[0] = o.mul(o.add(m11, m22), o.half());
  out[1] = o.mul(o.add(m12, m21), o.half());
  out[2] = o.mul(o.mul(o.iu(), o.sub(m12, m21)), o.half());
  out[3] = o.mul(o.sub(m11, m22), o.half());
}

// spinors of a massless four-vector given the inverse of its chart component
template <class Ops, class T>
__device__ __forceinline__ void spinors(const Ops& o, const T* v, bool plus, T inv_chart, T* lam, T* lamt) {
  const T vp = o.add(v[0], v[3]), vm = o.sub(v[0], v[3]);
  const T iv2 = o.mul(o.iu(), v[2]);
  const T vt = o.add(v[1], iv2), vtb = o.sub(v[1], iv2);
  if (plus) {
    lam[0] = o.one();
    lam[1] = o.mul(vt, inv_chart);
    lamt[0] = vp;
    lamt[1] = vtb;
  } else {
    lam[0] = o.mul(vtb, inv_chart);
    lam[1] = o.one();
    lamt[0] = vt;
    lamt[1] = vm;
  }
}

template <class Ops, class T>
__device__ __forceinline__ T bracket(const Ops& o, const T* a, const T* b) {
  return o.sub(o.mul(a[0], b[1]), o.mul(a[1], b[0]));
}

// sum_{i=4}^{y-1} (k^i)^2
template <class Ops, class T>
__device__ __forceinline__ T mu2y(const Ops& o, const T* k, int y) {
  T s = o.zero();
#pragma unroll
  for (int i = 4; i < SD; ++i)
    if (i < y) s = o.add(s, o.mul(k[i], k[i]));
  return s;
}

// all d - 2 states and their duals of one point, handed to emit(state,
// component, e, e~) in order (every component, zeros included); false (and
// nothing emitted) if a required denominator vanishes
template <class Ops, class T, class Emit>
__device__ bool point_states(const Ops& o, const T* k, const T* chi, int d, Emit&& emit) {
  T k4[4], ch[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    k4[m] = k[m];
    ch[m] = chi[m];
  }
  const T mu2 = mdot4(o, k4, k4);
  const T ck = mdot4(o, ch, k4);
  // batch 1: 2 chi.k4, the chart component of chi, mu^2 (d >= 5), mu_6^2
  // (d >= 6), mu_{x+1}^2 mu_{x+2}^2 (5 <= x <= d-2)
  const T vpc = o.add(ch[0], ch[3]), vmc = o.sub(ch[0], ch[3]);
  const bool plus_c = o.plus_chart(vpc, vmc);
  // fixed slots (unused ones hold 1): 0 2 chi.k4, 1 chi chart, 2 mu^2,
  // 3 mu_6^2, 4 + (x - 5) the product for the extra state x
  constexpr int NB1 = 4 + (SD - 6);
  T b1[NB1];
  b1[0] = o.add(ck, ck);
  b1[1] = plus_c ? vpc : vmc;
  b1[2] = d >= 5 ? mu2 : o.one();
  b1[3] = d >= 6 ? mu2y(o, k, 6) : o.one();
#pragma unroll
  for (int x = 5; x < SD - 1; ++x)
    b1[4 + x - 5] = x <= d - 2 ? o.mul(mu2y(o, k, x + 1), mu2y(o, k, x + 2)) : o.one();
  bool sing = false;
#pragma unroll
  for (int s = 0; s < NB1; ++s)
    if (o.is_zero(b1[s])) {
      sing = true;
      b1[s] = o.one();
    }
  o.inv_batch(b1, NB1);
  const T c = o.mul(mu2, b1[0]);
  T kb[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) kb[m] = o.sub(k4[m], o.mul(c, ch[m]));
  T lc[2], tc[2];
  spinors(o, ch, plus_c, b1[1], lc, tc);
  // batch 2: the chart component of kb
  const T vpk = o.add(kb[0], kb[3]), vmk = o.sub(kb[0], kb[3]);
  const bool plus_k = o.plus_chart(vpk, vmk);
  T b2[1] = {plus_k ? vpk : vmk};
  if (o.is_zero(b2[0])) {
    sing = true;
    b2[0] = o.one();
  }
  o.inv_batch(b2, 1);
  T lk[2], tk[2];
  spinors(o, kb, plus_k, b2[0], lk, tk);
  // batch 3: [kb chi], <kb chi>
  T b3[2] = {bracket(o, tk, tc), bracket(o, lk, lc)};
#pragma unroll
  for (int s = 0; s < 2; ++s)
    if (o.is_zero(b3[s])) {
      sing = true;
      b3[s] = o.one();
    }
  o.inv_batch(b3, 2);
  if (sing) return false;

  const T z = o.zero();
  T e1[4], e2[4], v[4];
  vec_of(o, lk, tc, v);
#pragma unroll
  for (int m = 0; m < 4; ++m) e1[m] = o.mul(v[m], b3[0]);
  vec_of(o, lc, tk, v);
  const T two_over_an = o.mul(o.two(), b3[1]);
#pragma unroll
  for (int m = 0; m < 4; ++m) e2[m] = o.mul(v[m], two_over_an);
#pragma unroll
  for (int m = 0; m < SD; ++m)
    if (m < d) {
      emit(0, m, m < 4 ? e1[m] : z, m < 4 ? e2[m] : z);
      emit(1, m, m < 4 ? e2[m] : z, m < 4 ? e1[m] : z);
    }
  if (d >= 5) {
#pragma unroll
    for (int m = 0; m < SD; ++m)
      if (m < d) {
        const T e3 = m < 4 ? o.sub(kb[m], o.mul(c, ch[m])) : z;
        emit(2, m, e3, o.mul(e3, b1[2]));
      }
  }
  if (d >= 6) {
#pragma unroll
    for (int m = 0; m < SD; ++m)
      if (m < d) {
        const T e4 = m == 4 ? k[5] : (m == 5 ? o.neg(k[4]) : z);
        emit(3, m, e4, o.mul(e4, b1[3]));
      }
  }
#pragma unroll
  for (int x = 5; x < SD - 1; ++x) {
    if (x <= d - 2) {
      const T kx1 = k[x + 1];
      const T top = o.neg(mu2y(o, k, x + 1));
#pragma unroll
      for (int m = 0; m < SD; ++m)
        if (m < d) {
          const T ex = (m >= 4 && m <= x) ? o.mul(k[m], kx1) : (m == x + 1 ? top : z);
          emit(x - 1, m, ex, o.mul(ex, b1[4 + x - 5]));  // e_x is state number x, slot x - 1
        }
    }
  }
  return true;
}

// ---- Z_p --------------------------------------------------------------------
// Values x stand for x 2^-32 ("Montgomery form") unless called plain, held
// canonical in [0, p) where they are added and in (-p, p) where they only
// enter products.
struct FpOps {
  const FpConst& k;
  __device__ uint32_t can(int32_t r) const { return min((uint32_t)r, (uint32_t)r + (uint32_t)k.p); }  // r in (-p, p)
  __device__ uint32_t add(uint32_t a, uint32_t b) const {
    const uint32_t s = a + b;
    return min(s, s - (uint32_t)k.p);
  }
  __device__ uint32_t sub(uint32_t a, uint32_t b) const { return can((int32_t)(a - b)); }
  __device__ int32_t muls(int32_t a, int32_t b) const { return fp_mul32(a, b, k); }
  __device__ uint32_t mul(int32_t a, int32_t b) const { return can(fp_mul32(a, b, k)); }
  __device__ uint32_t neg(uint32_t a) const { return a ? (uint32_t)k.p - a : 0u; }
};

// sum_{i=4}^{y-1} (k^i)^2
template <int D>
__device__ __forceinline__ uint32_t mu2y_fp(const FpOps& o, const uint32_t (&k)[D], int y) {
  uint32_t s = 0;
#pragma unroll
  for (int i = 4; i < D; ++i)
    if (i < y) s = o.add(s, o.mul(k[i], k[i]));
  return s;
}

// As point_states, over Z_p with every division put off to one batch.  With
// D2 = 2 chi.k4 and kb' = D2 k4 - mu^2 chi (= D2 kb), homogeneous spinors
// lam' = (v+, v^1 + i v^2), lamt' = (v+, v^1 - i v^2) (or with v-) of kb' and
// chi are lam and lamt times the chart component q; the brackets are
//   [kb chi] = Y / D2,  <kb chi> = X / (q_k q_c),
// with Y, X those of the primed spinors, so that
//   e1 = vec(lam'_k, lamt'_c) D2 / (q_k Y),  e2 = 2 vec(lam'_c, lamt'_k) q_k / (D2 X),
//   e3 = (D2 k4 - 2 mu^2 chi) / D2.
// A factor taken out of Montgomery form makes each product with it a plain
// residue, so the outputs need no conversion.  kp, k: plain and Montgomery
// momentum; emit gets plain canonical residues.
template <int D, class Emit>
__device__ __forceinline__ bool point_states_fp(const FpOps& o, const uint32_t (&kp)[D], const uint32_t (&k)[D],
                                                const uint32_t (&ch)[4], int32_t iu, Emit&& emit) {
  const auto dot4 = [&](const uint32_t* x, const uint32_t* y) {
    uint32_t s = o.mul(x[0], y[0]);
#pragma unroll
    for (int m = 1; m < 4; ++m) s = o.sub(s, o.mul(x[m], y[m]));
    return s;
  };
  const uint32_t mu2 = dot4(k, k);
  uint32_t D2 = dot4(ch, k);
  D2 = o.add(D2, D2);
  uint32_t kb[4], mch[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    mch[m] = o.mul(mu2, ch[m]);
    kb[m] = o.sub(o.mul(D2, k[m]), mch[m]);
  }
  // lam', lamt' and the chart component
  const auto spinors = [&](const uint32_t* v, uint32_t* lam, uint32_t* lamt) {
    const uint32_t vp = o.add(v[0], v[3]), vm = o.sub(v[0], v[3]);
    const uint32_t iv2 = o.mul(iu, v[2]);
    const uint32_t vt = o.add(v[1], iv2), vtb = o.sub(v[1], iv2);
    const bool plus = vp != 0;
    lam[0] = plus ? vp : vtb;
    lam[1] = plus ? vt : vm;
    lamt[0] = plus ? vp : vt;
    lamt[1] = plus ? vtb : vm;
    return plus ? vp : vm;
  };
  uint32_t lk[2], tk[2], lc[2], tc[2];
  const uint32_t qk = spinors(kb, lk, tk), qc = spinors(ch, lc, tc);
  const uint32_t Y = o.sub(o.mul(tk[0], tc[1]), o.mul(tk[1], tc[0]));
  const uint32_t X = o.sub(o.mul(lk[0], lc[1]), o.mul(lk[1], lc[0]));
  // the batch: q_k Y, D2 X, mu^2 (D >= 5), mu_6^2 (D >= 6), mu_{x+1}^2 mu_{x+2}^2 (5 <= x <= D-2)
  constexpr int NB = 2 + (D >= 5) + (D >= 6) + (D > 6 ? D - 6 : 0);
  uint32_t b[NB];
  b[0] = o.mul(qk, Y);
  b[1] = o.mul(D2, X);
  if constexpr (D >= 5) b[2] = mu2;
  if constexpr (D >= 6) b[3] = mu2y_fp<D>(o, k, 6);
#pragma unroll
  for (int x = 5; x < D - 1; ++x) b[4 + x - 5] = o.mul(mu2y_fp<D>(o, k, x + 1), mu2y_fp<D>(o, k, x + 2));
  bool sing = qc == 0;
#pragma unroll
  for (int s = 0; s < NB; ++s)
    if (b[s] == 0) {
      sing = true;
      b[s] = 1;
    }
  int32_t pre[NB], inv[NB];
  pre[0] = (int32_t)b[0];
#pragma unroll
  for (int s = 1; s < NB; ++s) pre[s] = o.muls(pre[s - 1], b[s]);
  // 1 / x in Montgomery form is x^(p-2) there
  int32_t t = fp_pow32(pre[NB - 1], (uint32_t)(o.k.p - 2), o.k);
#pragma unroll
  for (int s = NB - 1; s >= 0; --s) {
    inv[s] = s > 0 ? o.muls(t, pre[s - 1]) : t;
    if (s > 0) t = o.muls(t, b[s]);
  }
  if (sing) return false;

  const auto plain = [&](int32_t x) { return fp_redc1((int64_t)x, o.k); };
  // the four-vector of u w^T times 2
  const auto vec2 = [&](const uint32_t* u, const uint32_t* w, uint32_t* out) {
    const uint32_t m11 = o.mul(u[0], w[0]), m12 = o.mul(u[0], w[1]);
    const uint32_t m21 = o.mul(u[1], w[0]), m22 = o.mul(u[1], w[1]);
    out[0] = o.add(m11, m22);
    out[1] = o.add(m12, m21);
    out[2] = (uint32_t)o.muls(iu, o.sub(m12, m21));
    out[3] = o.sub(m11, m22);
  };
  const int32_t half = (int32_t)(((uint32_t)o.k.p + 1) / 2);  // plain 1/2
  const int32_t s1 = o.muls(o.muls(D2, inv[0]), half);
  const int32_t s2 = plain(o.muls(qk, inv[1]));
  uint32_t e1[4], e2[4], v[4];
  vec2(lk, tc, v);
#pragma unroll
  for (int m = 0; m < 4; ++m) e1[m] = o.mul(v[m], s1);
  vec2(lc, tk, v);
#pragma unroll
  for (int m = 0; m < 4; ++m) e2[m] = o.mul(v[m], s2);
#pragma unroll
  for (int m = 0; m < D; ++m) {
    emit(0, m, m < 4 ? e1[m] : 0u, m < 4 ? e2[m] : 0u);
    emit(1, m, m < 4 ? e2[m] : 0u, m < 4 ? e1[m] : 0u);
  }
  if constexpr (D >= 5) {
    const int32_t g = plain(o.muls(X, inv[1]));  // 1 / D2
#pragma unroll
    for (int m = 0; m < D; ++m) {
      const uint32_t e3 = m < 4 ? o.mul(o.sub(kb[m], mch[m]), g) : 0u;
      emit(2, m, e3, m < 4 ? o.mul(e3, inv[2]) : 0u);
    }
  }
  if constexpr (D >= 6) {
#pragma unroll
    for (int m = 0; m < D; ++m) {
      const uint32_t e4 = m == 4 ? kp[5] : (m == 5 ? o.neg(kp[4]) : 0u);
      emit(3, m, e4, m == 4 || m == 5 ? o.mul(e4, inv[3]) : 0u);
    }
  }
#pragma unroll
  for (int x = 5; x < D - 1; ++x) {
    const uint32_t top = o.can(plain((int32_t)o.neg(mu2y_fp<D>(o, k, x + 1))));
#pragma unroll
    for (int m = 0; m < D; ++m) {
      const uint32_t ex = (m >= 4 && m <= x) ? o.mul(k[m], kp[x + 1]) : (m == x + 1 ? top : 0u);
      emit(x - 1, m, ex, m >= 4 && m <= x + 1 ? o.mul(ex, inv[4 + x - 5]) : 0u);  // e_x is state number x, slot x - 1
    }
  }
  return true;
}

// Bound by HBM traffic (4 (2 D (D - 2) + D + 4) + 1 bytes a point).  With
// three Fermat powers a point, guards on the run-time d and a conversion of
// every output it was bound by its arithmetic: 2^20 points at D = 6 in 100 us
// (2.5 TB/s), 51 us (4.8 TB/s) now.
template <int D>
__global__ __launch_bounds__(256) void states_fp_kernel(StatesArgs a) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= a.npts) return;
  const FpOps o{a.fp};
  const uint32_t* km = static_cast<const uint32_t*>(a.momenta);
  const uint32_t* cm = static_cast<const uint32_t*>(a.chi);
  uint32_t kp[D], k[D], cp[4], chi[4];
#pragma unroll
  for (int m = 0; m < D; ++m) kp[m] = km[(int64_t)m * a.ld + q];
#pragma unroll
  for (int m = 0; m < 4; ++m) cp[m] = cm[(int64_t)m * a.ld + q];
  uint32_t maxraw = 0;
#pragma unroll
  for (int m = 0; m < D; ++m) {
    maxraw = max(maxraw, kp[m]);
    k[m] = o.mul((int32_t)kp[m], a.fp.c64);  // x 2^32
  }
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    maxraw = max(maxraw, cp[m]);
    chi[m] = o.mul((int32_t)cp[m], a.fp.c64);
  }
  const bool bad = maxraw >= (uint32_t)a.fp.p;
  uint32_t* eo = static_cast<uint32_t*>(a.eps);
  uint32_t* to = static_cast<uint32_t*>(a.epst);
  const auto emit = [&](int s, int m, uint32_t e, uint32_t et) {
    const int64_t off = ((int64_t)s * D + m) * a.ld + q;
    eo[off] = e;
    to[off] = et;
  };
  const bool ok = !bad && point_states_fp<D>(o, kp, k, chi, a.i_rep, emit);
  if (!ok) {
    for (int s = 0; s < D - 2; ++s)
      for (int m = 0; m < D; ++m) emit(s, m, 0xFFFFFFFFu, 0xFFFFFFFFu);
  }
  if (a.status) a.status[q] = bad ? PT_BADRESIDUE : (ok ? PT_OK : PT_SINGULAR);
}

__global__ __launch_bounds__(256) void states_c128_kernel(StatesArgs a) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= a.npts) return;
  const COps o{};
  const double2* km = static_cast<const double2*>(a.momenta);
  const double2* cm = static_cast<const double2*>(a.chi);
  cplx k[SD], chi[4];
#pragma unroll
  for (int m = 0; m < SD; ++m) {
    k[m] = {0.0, 0.0};
    if (m < a.d) {
      const double2 x = km[(int64_t)m * a.ld + q];
      k[m] = {x.x, x.y};
    }
  }
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const double2 x = cm[(int64_t)m * a.ld + q];
    chi[m] = {x.x, x.y};
  }
  double2* eo = static_cast<double2*>(a.eps);
  double2* to = static_cast<double2*>(a.epst);
  const auto emit = [&](int s, int m, cplx e, cplx et) {
    const int64_t off = ((int64_t)s * a.d + m) * a.ld + q;
    eo[off] = double2{e.re, e.im};
    to[off] = double2{et.re, et.im};
  };
  const bool ok = point_states(o, k, chi, a.d, emit);
  if (!ok) {
    const double nan = __builtin_nan("");
    for (int s = 0; s < a.d - 2; ++s)
      for (int m = 0; m < a.d; ++m) {
        const int64_t off = ((int64_t)s * a.d + m) * a.ld + q;
        eo[off] = double2{nan, nan};
        to[off] = double2{nan, nan};
      }
  }
  if (a.status) a.status[q] = ok ? PT_OK : PT_SINGULAR;
}

int64_t mulmod(int64_t a, int64_t b, int64_t p) { return (int64_t)((__int128)a * b % p); }

int64_t powmod64(int64_t a, int64_t e, int64_t p) {
  int64_t r = 1 % p;
  a %= p;
  while (e) {
    if (e & 1) r = mulmod(r, a, p);
    a = mulmod(a, a, p);
    e >>= 1;
  }
  return r;
}

int32_t balanced32(int64_t x, int64_t p) {
  x %= p;
  if (x < 0) x += p;
  return x > (p - 1) / 2 ? (int32_t)(x - p) : (int32_t)x;
}

int launch_states(bool fp, int d, int64_t npts, int64_t ld, uint32_t p, const void* momenta, const void* chi,
                  void* eps, void* epst, uint8_t* status, void* stream) {
  if (d < 4 || d > BG_MAX_D) return BG_EDOMAIN;
  if (npts < 0) return BG_EINVAL;
  if (fp && (p < 3 || p >= 0x80000000u || !is_prime_u32(p))) return BG_ENOTPRIME;
  if (fp && p % 4 != 1) return BG_EDOMAIN;  // no square root of -1 in F_p
  if (npts == 0) return BG_OK;
  if (ld < npts || !momenta || !chi || !eps || !epst) return BG_EINVAL;
  StatesArgs a{};
  a.momenta = momenta;
  a.chi = chi;
  a.eps = eps;
  a.epst = epst;
  a.status = status;
  a.npts = npts;
  a.ld = ld;
  a.d = d;
  if (fp) {
    a.fp = make_fp_const(p);
    // i 2^64 (balanced) times 2^-32, as i 2^32 = (i 2^64) (2^32)^(p-2) mod p
    const int64_t i64 = fp_sqrt_minus_one_mont(p);
    a.i_rep = balanced32(mulmod(i64 < 0 ? i64 + p : i64, powmod64(powmod64(2, 32, p), (int64_t)p - 2, p), p), p);
  }
  const int64_t blocks = (npts + 255) / 256;
  if (blocks > 0x7FFFFFFF) return BG_EINVAL;
  void* args[] = {&a};
  static const void* const fp_kernels[] = {
      reinterpret_cast<const void*>(&states_fp_kernel<4>), reinterpret_cast<const void*>(&states_fp_kernel<5>),
      reinterpret_cast<const void*>(&states_fp_kernel<6>), reinterpret_cast<const void*>(&states_fp_kernel<7>),
      reinterpret_cast<const void*>(&states_fp_kernel<8>), reinterpret_cast<const void*>(&states_fp_kernel<9>),
      reinterpret_cast<const void*>(&states_fp_kernel<10>)};
  static_assert(BG_MAX_D == 10, "one kernel per d from 4 to BG_MAX_D");
  const hipError_t e = hipLaunchKernel(fp ? fp_kernels[d - 4] : reinterpret_cast<const void*>(&states_c128_kernel),
                                       dim3((unsigned)blocks), dim3(256), args, 0, static_cast<hipStream_t>(stream));
  return e == hipSuccess ? BG_OK : BG_EHIP;
}

// ---------------------------------------------------------------------------
// sums over the states of one cut leg: S = sum_s (e_s . K_L)(e~_s . K_R)
// ---------------------------------------------------------------------------
// With K_L, K_R the root currents of two trees whose last leg is the cut leg
// (momentum l in one, -l in the other), M_L(e_s) = e_s . K_L and
// M_R(e~_s) = e~_s . K_R, so S is the state sum of their product (paper
// Sec. 2.1, the leading pole of the cut equation; Sec. 2.3 states).  One
// point per lane; mostly-minus products.
struct StateSumArgs {
  const void* kl;
  const void* kr;
  const void* eps;
  const void* epst;
  void* out;
  uint8_t* status;
  int64_t npts, ld;
  FpConst fp;
  int32_t r2;  // F_p: 2^128 mod p, balanced
};

// Bound by HBM traffic (4 (2 D + 2 (D - 2) D + 1) + 1 bytes a point): one
// kernel per d, so that no load sits behind a guard and a state's rows are
// loaded together.  Products take the currents balanced and the states as
// they are (canonical), below 2^61 each: two beside a folded accumulator.
// 2^20 points at D = 6: 76 us with guards on the run-time d, 50 us (5.0 TB/s) now.
template <int D>
__global__ __launch_bounds__(256) void state_sum_fp_kernel(StateSumArgs a) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= a.npts) return;
  const FpConst& F = a.fp;
  const uint32_t* kl = static_cast<const uint32_t*>(a.kl) + q;
  const uint32_t* kr = static_cast<const uint32_t*>(a.kr) + q;
  const uint32_t* ep = static_cast<const uint32_t*>(a.eps) + q;
  const uint32_t* et = static_cast<const uint32_t*>(a.epst) + q;
  uint32_t maxraw = 0;
  // a value >= p is taken as it is: the point's output is replaced below
  int32_t L[D], Rv[D];
#pragma unroll
  for (int mu = 0; mu < D; ++mu) {
    const uint32_t l = kl[mu * a.ld], r = kr[mu * a.ld];
    maxraw = max(maxraw, max(l, r));
    L[mu] = fp_from_canonical(l, F);
    Rv[mu] = fp_from_canonical(r, F);
  }
  L[0] = sub32(0, L[0]);  // primed: sum_mu L'_mu x_mu = -(L . x)
  Rv[0] = sub32(0, Rv[0]);
  // (e.K_L)(e~.K_R) = (-(e.K_L))(-(e~.K_R)); each dot is reduced to t 2^-32
  // (below 1.5 2^30), the products of two such are summed in int64 (2^-64) and
  // reduced once more (2^-96), and one product with 2^128 restores S
  int64_t acc = 0;
#pragma unroll 2
  for (int s = 0; s < D - 2; ++s) {
    uint32_t e[D], f[D];
#pragma unroll
    for (int mu = 0; mu < D; ++mu) {
      e[mu] = ep[((int64_t)s * D + mu) * a.ld];
      f[mu] = et[((int64_t)s * D + mu) * a.ld];
    }
    int64_t tl = 0, tr = 0;
#pragma unroll
    for (int mu = 0; mu < D; ++mu) {
      maxraw = max(maxraw, max(e[mu], f[mu]));
      tl = mad64((int32_t)e[mu], L[mu], tl);
      tr = mad64((int32_t)f[mu], Rv[mu], tr);
      if (mu & 1) {
        tl = fp_fold(tl, F);
        tr = fp_fold(tr, F);
      }
    }
    if constexpr (D & 1) {
      tl = fp_fold(tl, F);
      tr = fp_fold(tr, F);
    }
    acc = fp_fold(mad64(fp_redc1(tl, F), fp_redc1(tr, F), acc), F);
  }
  const bool bad = maxraw >= (uint32_t)F.p;
  const int32_t sum = fp_mul32(fp_redc1(acc, F), a.r2, F);  // in (-p, p)
  static_cast<uint32_t*>(a.out)[q] = bad ? 0xFFFFFFFFu : fp_to_canonical(sum, F);
  if (a.status) a.status[q] = bad ? PT_BADRESIDUE : PT_OK;
}

template <int D>
__global__ __launch_bounds__(256) void state_sum_c128_kernel(StateSumArgs a) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= a.npts) return;
  const double2* kl = static_cast<const double2*>(a.kl) + q;
  const double2* kr = static_cast<const double2*>(a.kr) + q;
  const double2* ep = static_cast<const double2*>(a.eps) + q;
  const double2* et = static_cast<const double2*>(a.epst) + q;
  double2 L[D], Rv[D];
#pragma unroll
  for (int mu = 0; mu < D; ++mu) {
    L[mu] = kl[mu * a.ld];
    Rv[mu] = kr[mu * a.ld];
  }
  double sre = 0.0, sim = 0.0;
  for (int s = 0; s < D - 2; ++s) {
    double lre = 0.0, lim = 0.0, rre = 0.0, rim = 0.0;
#pragma unroll
    for (int mu = 0; mu < D; ++mu) {
      const double g = mu == 0 ? 1.0 : -1.0;
      const double2 e = ep[((int64_t)s * D + mu) * a.ld];
      const double2 f = et[((int64_t)s * D + mu) * a.ld];
      lre = __builtin_fma(g * e.x, L[mu].x, __builtin_fma(-g * e.y, L[mu].y, lre));
      lim = __builtin_fma(g * e.x, L[mu].y, __builtin_fma(g * e.y, L[mu].x, lim));
      rre = __builtin_fma(g * f.x, Rv[mu].x, __builtin_fma(-g * f.y, Rv[mu].y, rre));
      rim = __builtin_fma(g * f.x, Rv[mu].y, __builtin_fma(g * f.y, Rv[mu].x, rim));
    }
    sre = __builtin_fma(lre, rre, __builtin_fma(-lim, rim, sre));
    sim = __builtin_fma(lre, rim, __builtin_fma(lim, rre, sim));
  }
  const bool nan = sre != sre || sim != sim;
  static_cast<double2*>(a.out)[q] = double2{sre, sim};
  if (a.status) a.status[q] = nan ? PT_SINGULAR : PT_OK;
}

int launch_state_sum(bool fp, int d, int64_t npts, int64_t ld, uint32_t p, const void* kl, const void* kr,
                     const void* eps, const void* epst, void* out, uint8_t* status, void* stream) {
  if (d < 4 || d > BG_MAX_D) return BG_EDOMAIN;
  if (fp && (p < 3 || p >= 0x80000000u || !is_prime_u32(p))) return BG_ENOTPRIME;
  if (npts < 0) return BG_EINVAL;
  if (npts == 0) return BG_OK;
  if (ld < npts || !kl || !kr || !eps || !epst || !out) return BG_EINVAL;
  StateSumArgs a{};
  a.kl = kl;
  a.kr = kr;
  a.eps = eps;
  a.epst = epst;
  a.out = out;
  a.status = status;
  a.npts = npts;
  a.ld = ld;
  if (fp) {
    a.fp = make_fp_const(p);
    const int64_t R = powmod64(2, 64, p);
    a.r2 = balanced32(mulmod(R, R, p), p);
  }
  const int64_t blocks = (npts + 255) / 256;
  if (blocks > 0x7FFFFFFF) return BG_EINVAL;
  void* args[] = {&a};
  static const void* const kernels[2][7] = {
      {reinterpret_cast<const void*>(&state_sum_c128_kernel<4>), reinterpret_cast<const void*>(&state_sum_c128_kernel<5>),
       reinterpret_cast<const void*>(&state_sum_c128_kernel<6>), reinterpret_cast<const void*>(&state_sum_c128_kernel<7>),
       reinterpret_cast<const void*>(&state_sum_c128_kernel<8>), reinterpret_cast<const void*>(&state_sum_c128_kernel<9>),
       reinterpret_cast<const void*>(&state_sum_c128_kernel<10>)},
      {reinterpret_cast<const void*>(&state_sum_fp_kernel<4>), reinterpret_cast<const void*>(&state_sum_fp_kernel<5>),
       reinterpret_cast<const void*>(&state_sum_fp_kernel<6>), reinterpret_cast<const void*>(&state_sum_fp_kernel<7>),
       reinterpret_cast<const void*>(&state_sum_fp_kernel<8>), reinterpret_cast<const void*>(&state_sum_fp_kernel<9>),
       reinterpret_cast<const void*>(&state_sum_fp_kernel<10>)}};
  const hipError_t e = hipLaunchKernel(kernels[fp ? 1 : 0][d - 4], dim3((unsigned)blocks), dim3(256), args, 0, static_cast<hipStream_t>(stream));
  return e == hipSuccess ? BG_OK : BG_EHIP;
}

}  // namespace
}  // namespace bg

extern "C" {

int bg_state_sum_c128(int d, int64_t npts, int64_t ld, const double* kl, const double* kr, const double* eps,
                      const double* epst, double* out, uint8_t* status, void* hip_stream) {
  return bg::launch_state_sum(false, d, npts, ld, 0, kl, kr, eps, epst, out, status, hip_stream);
}

int bg_state_sum_fp(int d, int64_t npts, int64_t ld, uint32_t p, const uint32_t* kl, const uint32_t* kr,
                    const uint32_t* eps, const uint32_t* epst, uint32_t* out, uint8_t* status, void* hip_stream) {
  return bg::launch_state_sum(true, d, npts, ld, p, kl, kr, eps, epst, out, status, hip_stream);
}

int bg_states_c128(int d, int64_t npts, int64_t ld, const double* momenta, const double* chi, double* eps,
                   double* epst, uint8_t* status, void* hip_stream) {
  return bg::launch_states(false, d, npts, ld, 0, momenta, chi, eps, epst, status, hip_stream);
}

int bg_states_fp(int d, int64_t npts, int64_t ld, uint32_t p, const uint32_t* momenta, const uint32_t* chi,
                 uint32_t* eps, uint32_t* epst, uint8_t* status, void* hip_stream) {
  return bg::launch_states(true, d, npts, ld, p, momenta, chi, eps, epst, status, hip_stream);
}

}  // extern "C"
