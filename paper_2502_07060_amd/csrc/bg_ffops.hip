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
// before and now: 2^20 of 6x6x6 247 -> 100 us (4.5 TB/s, a large copy
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
  const uint32_t* y;
  uint32_t* z;
  uint8_t* status;
  int64_t count;
  uint32_t yscalar;  // used when y == nullptr: its inverse times R (Montgomery form)
  FpConst fp;
  int32_t r2;
};

// Lane t of block b takes the values b 4096 + u 256 + t, u < 16: each of the
// 16 loads of a wave reads 256 consecutive bytes.
__global__ __launch_bounds__(256) void divide_kernel(DivideArgs a) {
  const int64_t base = (int64_t)blockIdx.x * 256 * kDivChunk + threadIdx.x;
  const FpConst& F = a.fp;
  int32_t xm[kDivChunk], ym[kDivChunk];
  uint8_t st[kDivChunk];
  int32_t acc = F.one;
#pragma unroll
  for (int u = 0; u < kDivChunk; ++u) {
    const int64_t e = base + (int64_t)u * 256;
    if (e < a.count) {
      const uint32_t xr = a.x[e];
      const uint32_t yr = a.y ? a.y[e] : 1u;
      st[u] = (xr >= (uint32_t)F.p || yr >= (uint32_t)F.p) ? PT_BADRESIDUE : PT_OK;
      xm[u] = fp_mul(fp_from_canonical(xr < (uint32_t)F.p ? xr : 0u, F), a.r2, F);  // x R
      ym[u] = a.y ? fp_mul(fp_from_canonical(yr < (uint32_t)F.p ? yr : 0u, F), a.r2, F) : F.one;
      if (st[u] == PT_OK && ym[u] == 0) st[u] = PT_SINGULAR;
      if (ym[u] == 0) ym[u] = F.one;
      xm[u] = fp_mul(xm[u], acc, F);  // x_u (y_0 ... y_{u-1})
      acc = fp_mul(acc, ym[u], F);
    }
  }
  int32_t inv = a.y ? fp_pow(acc, (uint32_t)(F.p - 2), F) : (int32_t)a.yscalar;
#pragma unroll
  for (int u = kDivChunk - 1; u >= 0; --u) {
    const int64_t e = base + (int64_t)u * 256;
    if (e < a.count) {
      const int32_t qv = fp_mul(xm[u], inv, F);
      inv = fp_mul(inv, ym[u], F);
      const int32_t v = fp_redc2((int64_t)qv, F);
      a.z[e] = st[u] == PT_OK ? fp_to_canonical(v, F) : 0xFFFFFFFFu;
      if (a.status) a.status[e] = st[u];
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

int32_t r2_of(uint32_t p) {
  const uint64_t R = powmod_u64(2, 64, p);
  return balanced_of((unsigned __int128)R * R % p, p);
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
  a.r2 = bg::r2_of(p);
  if (!y) {  // (1 / y) R mod p, balanced
    const uint64_t inv = bg::powmod_u64(yscalar, p - 2, p);
    const uint64_t R = bg::powmod_u64(2, 64, p);
    a.yscalar = (uint32_t)bg::balanced_of((unsigned __int128)inv * R % p, p);
  }
  const int64_t blocks = (count + 256 * bg::kDivChunk - 1) / (256 * bg::kDivChunk);
  if (blocks > 0x7FFFFFFF) return BG_EINVAL;
  void* args[] = {&a};
  return hipLaunchKernel(reinterpret_cast<const void*>(&bg::divide_kernel), dim3((unsigned)blocks), dim3(256),
                         args, 0, static_cast<hipStream_t>(hip_stream)) == hipSuccess
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
