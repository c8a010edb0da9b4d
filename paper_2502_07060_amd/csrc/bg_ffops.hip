// Standalone batched Z_p operations (paper Sec. 3: the finite-field library
// that the recursion is built on, usable on its own): tensor contraction over
// any group of indices, with the second operand per event or shared, and
// division.  Residues are canonical uint32 in [0, p); the event index is the
// fastest one in every array (element e of event q at e * ld + q), as in the
// amplitude entry points, so the lanes of a wave read consecutive words.
//
// Contraction, one event per lane: z[i][k] = sum_j x[i][j] y[j][k] as a sum of
// outer products, a tile of TI x TK outputs in registers (below).  Values
// are taken as balanced representatives (|v| <= (p-1)/2), so a product is
// below 2^60 and four of them fit beside a folded accumulator (field_fp.h);
// each output is reduced once at the end.
//
// Division: Montgomery batch inversion over 16 values per lane (one Fermat
// power per 16 quotients).
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <utility>

#include "bg.h"
#include "bg_registry.h"
#include "field_fp.h"

namespace bg {
namespace {

constexpr int kTile = 8;  // largest tile side
constexpr int kDivChunk = 16;

struct ContractArgs {
  const uint32_t* x;
  const uint32_t* y;
  uint32_t* z;
  uint8_t* status;
  int64_t npts, ld;
  int I, J, K;
  FpConst fp;
};

// A tile of outputs per lane: TI x TK int64 accumulators; each step of j loads
// TI values of x and TK of y and adds their products, so an event's inputs are
// read once when I, K <= 8 (ceil(K / TK) and ceil(I / TI) times otherwise,
// mostly from cache).  Bound by HBM traffic: the loads of the next two j are
// issued before the products of the current two, without conditions on values,
// so a wave keeps 2 (TI + TK) loads in flight.  The tile sides are compile-time
// (no guards inside); they split I and K evenly into tiles of at most 8, the
// last tile repeating its last row or column where they do not divide.
// Before, y lay in an 8 x 8 array behind run-time guards for J, K <= 8 (each
// load waited for in a block of its own), and larger J or K read y once per
// row of x after a pass over all inputs for the status.  Events by I x J x K,
// before and now: 2^20 of 6x6x6 256 -> 100 us (4.5 TB/s, a large copy
// reaches 4.9); 150001 of 6x36x6 660 -> 72 us.
//
// YB: y per event; else one y for all events, read through scalar loads.
template <int TI, int TK, bool YB>
__global__ __launch_bounds__(256) void contract_kernel(ContractArgs a) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= a.npts) return;
  const FpConst& F = a.fp;
  const uint32_t* const xq = a.x + q;
  const uint32_t* const yq = YB ? a.y + q : a.y;
  const int64_t ys = YB ? a.ld : 1;  // element stride of y ([J][K][ld] or [J][K])
  const bool one_tile = a.I <= TI && a.K <= TK;
  uint32_t maxraw = 0;
  for (int i0 = 0; i0 < a.I; i0 += TI) {
    for (int k0 = 0; k0 < a.K; k0 += TK) {
      int64_t acc[TI][TK];
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int k = 0; k < TK; ++k) acc[i][k] = 0;
      uint32_t xn[2][TI], yn[2][TK];
      const auto load = [&](int j0) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          if (j0 + u < a.J) {
#pragma unroll
            for (int i = 0; i < TI; ++i) {
              const int ii = i0 + i < a.I ? i0 + i : a.I - 1;
              xn[u][i] = xq[((int64_t)ii * a.J + j0 + u) * a.ld];
            }
#pragma unroll
            for (int k = 0; k < TK; ++k) {
              const int kk = k0 + k < a.K ? k0 + k : a.K - 1;
              yn[u][k] = yq[((int64_t)(j0 + u) * a.K + kk) * ys];
            }
          } else {
#pragma unroll
            for (int i = 0; i < TI; ++i) xn[u][i] = 0;
#pragma unroll
            for (int k = 0; k < TK; ++k) yn[u][k] = 0;
          }
        }
      };
      load(0);
      for (int j0 = 0; j0 < a.J; j0 += 2) {
        uint32_t xc[2][TI], yc[2][TK];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
          for (int i = 0; i < TI; ++i) xc[u][i] = xn[u][i];
#pragma unroll
          for (int k = 0; k < TK; ++k) yc[u][k] = yn[u][k];
        }
        if (j0 + 2 < a.J) load(j0 + 2);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          // a value >= p is taken as it is (its event's outputs are replaced
          // by the sentinel, whatever its products were)
          int32_t yv[TK];
#pragma unroll
          for (int k = 0; k < TK; ++k) {
            maxraw = max(maxraw, yc[u][k]);
            yv[k] = fp_from_canonical(yc[u][k], F);
          }
#pragma unroll
          for (int i = 0; i < TI; ++i) {
            maxraw = max(maxraw, xc[u][i]);
            const int32_t xv = fp_from_canonical(xc[u][i], F);
#pragma unroll
            for (int k = 0; k < TK; ++k) acc[i][k] = mad64(xv, yv[k], acc[i][k]);
          }
        }
        if (j0 & 2) {  // four products of < 2^60 beside a folded accumulator
#pragma unroll
          for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int k = 0; k < TK; ++k) acc[i][k] = fp_fold(acc[i][k], F);
        }
      }
      // sum 2^-32 2^64 2^-32, in (-p, p); with more than one tile an event that
      // turns out to hold a non-canonical input is overwritten at the end
      const bool bad = one_tile && maxraw >= (uint32_t)F.p;
#pragma unroll
      for (int i = 0; i < TI; ++i) {
        if (i0 + i < a.I) {
#pragma unroll
          for (int k = 0; k < TK; ++k) {
            if (k0 + k < a.K) {
              const int32_t s = fp_mul32(fp_redc1(fp_fold(acc[i][k], F), F), F.c64, F);
              a.z[((int64_t)(i0 + i) * a.K + k0 + k) * a.ld + q] = bad ? 0xFFFFFFFFu : fp_to_canonical(s, F);
            }
          }
        }
      }
    }
  }
  const bool bad = maxraw >= (uint32_t)F.p;
  if (bad && !one_tile)
    for (int e = 0; e < a.I * a.K; ++e) a.z[(int64_t)e * a.ld + q] = 0xFFFFFFFFu;
  if (a.status) a.status[q] = bad ? PT_BADRESIDUE : PT_OK;
}

// the kernel of a tile shape: index ((TI - 1) kTile + TK - 1) 2 + YB
template <int... Is>
const void* contract_table(int at, std::integer_sequence<int, Is...>) {
  static const void* const fn[] = {
      reinterpret_cast<const void*>(&contract_kernel<Is / 2 / kTile + 1, Is / 2 % kTile + 1, (Is & 1) != 0>)...};
  return fn[at];
}

// side of the tiles that split n evenly into tiles of at most kTile
int tile_side(int n) {
  const int tiles = (n + kTile - 1) / kTile;
  return (n + tiles - 1) / tiles;
}

struct DivideArgs {
  const uint32_t* x;
  const uint32_t* y;  // null in divide_scalar_kernel
  uint32_t* z;
  uint8_t* status;
  int64_t count;
  int32_t yinv;  // divide_scalar_kernel: 2^32 / y mod p, balanced
  FpConst fp;
};

// Bound by HBM traffic (13 bytes a quotient), with about 40 instructions each
// beside it.  A block of 256 lanes takes 4096 consecutive values; lane t holds
// those at 1024 g + 4 t + 0..3 (g < 4), so that x, y and z move 16 bytes and
// the status 4 bytes a lane and access.  VEC = false: single values 256
// apart, for pointers that are not aligned to the wide accesses.
// Products are taken in the Montgomery domain of 2^32 (three instructions),
// and the residues enter as they are: with P_u = y_0 ... y_u 2^(-32 u) the
// power gives 2^64 / P_u, and x_u P_{u-1} 2^-32 times that times 2^-32 is
// 2^32 x_u / y_u, so one REDC step ends it.  2^24 quotients: 63.7 us with
// 4-byte accesses and five-instruction products, 42.6 us (5.1 TB/s) now.
template <bool VEC>
__global__ __launch_bounds__(256) void divide_kernel(DivideArgs a) {
  const int64_t base = (int64_t)blockIdx.x * (256 * kDivChunk);
  const FpConst& F = a.fp;
  const bool full = base + 256 * kDivChunk <= a.count;  // the same in the whole block
  const auto at = [&](int u) {
    return base + (VEC ? (int64_t)(u / 4) * 1024 + threadIdx.x * 4 + u % 4 : (int64_t)u * 256 + threadIdx.x);
  };
  uint32_t xr[kDivChunk], yr[kDivChunk];
  if (VEC && full) {
#pragma unroll
    for (int u = 0; u < kDivChunk; u += 4) {
      const uint4 x4 = *reinterpret_cast<const uint4*>(a.x + at(u));
      const uint4 y4 = *reinterpret_cast<const uint4*>(a.y + at(u));
      xr[u] = x4.x; xr[u + 1] = x4.y; xr[u + 2] = x4.z; xr[u + 3] = x4.w;
      yr[u] = y4.x; yr[u + 1] = y4.y; yr[u + 2] = y4.z; yr[u + 3] = y4.w;
    }
  } else {
#pragma unroll
    for (int u = 0; u < kDivChunk; ++u) {
      const int64_t e = at(u);
      xr[u] = e < a.count ? a.x[e] : 0u;
      yr[u] = e < a.count ? a.y[e] : 1u;
    }
  }
  const uint32_t p = (uint32_t)F.p;
  uint32_t bad = 0, zero = 0;
  int32_t xm[kDivChunk], ym[kDivChunk], acc = 0;
#pragma unroll
  for (int u = 0; u < kDivChunk; ++u) {
    const bool b = xr[u] >= p || yr[u] >= p, z = yr[u] == 0;
    bad |= b ? 1u << u : 0u;
    zero |= z ? 1u << u : 0u;
    xm[u] = (int32_t)xr[u];
    ym[u] = b || z ? 1 : (int32_t)yr[u];
    if (u > 0) xm[u] = fp_mul32(xm[u], acc, F);  // x_u P_{u-1} 2^-32 (x >= p: replaced below)
    acc = u > 0 ? fp_mul32(acc, ym[u], F) : ym[0];
  }
  int32_t inv = fp_pow32(acc, p - 2, F);
  uint32_t v[kDivChunk];
#pragma unroll
  for (int u = kDivChunk - 1; u >= 0; --u) {
    const int32_t q = fp_mul32(xm[u], inv, F);
    inv = fp_mul32(inv, ym[u], F);
    v[u] = (((bad | zero) >> u) & 1u) ? 0xFFFFFFFFu : fp_to_canonical(fp_redc1((int64_t)q, F), F);
  }
  // status of value u: bad residue, else zero divisor, else 0
  const auto st = [&](int u) -> uint32_t {
    return ((bad >> u) & 1u) ? PT_BADRESIDUE : (((zero >> u) & 1u) ? PT_SINGULAR : PT_OK);
  };
  if (VEC && full) {
#pragma unroll
    for (int u = 0; u < kDivChunk; u += 4) {
      *reinterpret_cast<uint4*>(a.z + at(u)) = make_uint4(v[u], v[u + 1], v[u + 2], v[u + 3]);
      if (a.status)
        *reinterpret_cast<uint32_t*>(a.status + at(u)) =
            st(u) | st(u + 1) << 8 | st(u + 2) << 16 | st(u + 3) << 24;
    }
  } else {
#pragma unroll
    for (int u = 0; u < kDivChunk; ++u) {
      const int64_t e = at(u);
      if (e < a.count) {
        a.z[e] = v[u];
        if (a.status) a.status[e] = (uint8_t)st(u);
      }
    }
  }
}

// One divisor for every value: a product each (9 bytes of HBM traffic), four
// values a lane.
template <bool VEC>
__global__ __launch_bounds__(256) void divide_scalar_kernel(DivideArgs a) {
  const FpConst& F = a.fp;
  const int64_t base = (int64_t)blockIdx.x * 1024;
  const bool full = base + 1024 <= a.count;
  const auto at = [&](int u) { return base + (VEC ? (int64_t)threadIdx.x * 4 + u : (int64_t)u * 256 + threadIdx.x); };
  uint32_t xr[4], v[4];
  if (VEC && full) {
    const uint4 x4 = *reinterpret_cast<const uint4*>(a.x + at(0));
    xr[0] = x4.x; xr[1] = x4.y; xr[2] = x4.z; xr[3] = x4.w;
  } else {
#pragma unroll
    for (int u = 0; u < 4; ++u) xr[u] = at(u) < a.count ? a.x[at(u)] : 0u;
  }
  uint32_t st = 0;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const bool b = xr[u] >= (uint32_t)F.p;
    st |= b ? (uint32_t)PT_BADRESIDUE << (8 * u) : 0u;
    v[u] = b ? 0xFFFFFFFFu : fp_to_canonical(fp_mul32((int32_t)xr[u], a.yinv, F), F);  // in (-p, p)
  }
  if (VEC && full) {
    *reinterpret_cast<uint4*>(a.z + at(0)) = make_uint4(v[0], v[1], v[2], v[3]);
    if (a.status) *reinterpret_cast<uint32_t*>(a.status + at(0)) = st;
  } else {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (at(u) < a.count) {
        a.z[at(u)] = v[u];
        if (a.status) a.status[at(u)] = (uint8_t)(st >> (8 * u));
      }
  }
}

uint64_t powmod_u64(uint64_t a, uint64_t e, uint64_t m) {
  uint64_t r = 1 % m;
  a %= m;
  while (e) {
    if (e & 1) r = (unsigned __int128)r * a % m;
    a = (unsigned __int128)a * a % m;
    e >>= 1;
  }
  return r;
}

int32_t balanced_of(uint64_t x, uint64_t p) {
  x %= p;
  return x > (p - 1) / 2 ? (int32_t)((int64_t)x - (int64_t)p) : (int32_t)x;
}

}  // namespace
}  // namespace bg

extern "C" {

int bg_fp_contract(uint32_t p, int I, int J, int K, int64_t npts, int64_t ld, const uint32_t* x,
                   const uint32_t* y, int y_batched, uint32_t* z, uint8_t* status, void* hip_stream) {
  if (p < 3 || p >= 0x80000000u || !bg::is_prime_u32(p)) return BG_ENOTPRIME;
  if (I < 1 || J < 1 || K < 1 || I > BG_FP_MAX_DIM || J > BG_FP_MAX_DIM || K > BG_FP_MAX_DIM) return BG_EDOMAIN;
  if (npts < 0) return BG_EINVAL;
  if (npts == 0) return BG_OK;
  if (ld < npts || !x || !y || !z) return BG_EINVAL;
  bg::ContractArgs a{};
  a.x = x;
  a.y = y;
  a.z = z;
  a.status = status;
  a.npts = npts;
  a.ld = ld;
  a.I = I;
  a.J = J;
  a.K = K;
  a.fp = bg::make_fp_const(p);
  // one wave a block: few events still reach every CU (blocks of 256 lanes are
  // no faster at 2^20 events: 100 us both)
  const int block = 64;
  const int64_t blocks = (npts + block - 1) / block;
  if (blocks > 0x7FFFFFFF) return BG_EINVAL;
  void* args[] = {&a};
  const int at = ((bg::tile_side(I) - 1) * bg::kTile + bg::tile_side(K) - 1) * 2 + (y_batched ? 1 : 0);
  const void* fn = bg::contract_table(at, std::make_integer_sequence<int, 2 * bg::kTile * bg::kTile>{});
  return hipLaunchKernel(fn, dim3((unsigned)blocks), dim3((unsigned)block), args, 0,
                         static_cast<hipStream_t>(hip_stream)) == hipSuccess
             ? BG_OK
             : BG_EHIP;
}

static int launch_divide(uint32_t p, int64_t count, const uint32_t* x, const uint32_t* y, uint32_t yscalar,
                         uint32_t* z, uint8_t* status, void* hip_stream) {
  bg::DivideArgs a{};
  a.x = x;
  a.y = y;
  a.z = z;
  a.status = status;
  a.count = count;
  a.fp = bg::make_fp_const(p);
  if (!y) {
    const uint64_t inv = bg::powmod_u64(yscalar, p - 2, p);
    a.yinv = bg::balanced_of(inv * (bg::powmod_u64(2, 32, p)), p);
  }
  const int64_t per = y ? 256 * bg::kDivChunk : 1024;
  const int64_t blocks = (count + per - 1) / per;
  if (blocks > 0x7FFFFFFF) return BG_EINVAL;
  // wide accesses need their alignment (a view of a tensor may not have it)
  const bool vec = (((uintptr_t)x | (uintptr_t)y | (uintptr_t)z) & 15) == 0 && ((uintptr_t)status & 3) == 0;
  const void* fn = y ? (vec ? reinterpret_cast<const void*>(&bg::divide_kernel<true>)
                            : reinterpret_cast<const void*>(&bg::divide_kernel<false>))
                     : (vec ? reinterpret_cast<const void*>(&bg::divide_scalar_kernel<true>)
                            : reinterpret_cast<const void*>(&bg::divide_scalar_kernel<false>));
  void* args[] = {&a};
  return hipLaunchKernel(fn, dim3((unsigned)blocks), dim3(256), args, 0, static_cast<hipStream_t>(hip_stream)) ==
                 hipSuccess
             ? BG_OK
             : BG_EHIP;
}

int bg_fp_divide(uint32_t p, int64_t count, const uint32_t* x, const uint32_t* y, uint32_t* z, uint8_t* status,
                 void* hip_stream) {
  if (p < 3 || p >= 0x80000000u || !bg::is_prime_u32(p)) return BG_ENOTPRIME;
  if (count < 0) return BG_EINVAL;
  if (count == 0) return BG_OK;
  if (!x || !y || !z) return BG_EINVAL;
  return launch_divide(p, count, x, y, 0, z, status, hip_stream);
}

int bg_fp_divide_scalar(uint32_t p, int64_t count, const uint32_t* x, uint32_t y, uint32_t* z, uint8_t* status,
                        void* hip_stream) {
  if (p < 3 || p >= 0x80000000u || !bg::is_prime_u32(p)) return BG_ENOTPRIME;
  if (y >= p) return BG_EINVAL;
  if (y == 0) return BG_EDOMAIN;  // no inverse
  if (count < 0) return BG_EINVAL;
  if (count == 0) return BG_OK;
  if (!x || !z) return BG_EINVAL;
  return launch_divide(p, count, x, nullptr, y, z, status, hip_stream);
}

}  // extern "C"
