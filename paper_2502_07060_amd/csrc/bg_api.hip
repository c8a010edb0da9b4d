// C-ABI entry points of libbg_mi355x.so (declared in include/bg.h).
#include <hip/hip_runtime.h>
#include <string.h>

#include <algorithm>
#include <mutex>

#include "bg.h"
#include "bg_wide.h"
#include "bg_registry.h"

namespace bg {

std::vector<Variant>& registry() {
  static std::vector<Variant> r;
  return r;
}

// ---------------------------------------------------------------------------
// primes and Montgomery constants
// ---------------------------------------------------------------------------
static uint64_t powmod(uint64_t a, uint64_t e, uint64_t m) {
  uint64_t r = 1 % m;
  a %= m;
  while (e) {
    if (e & 1) r = (unsigned __int128)r * a % m;
    a = (unsigned __int128)a * a % m;
    e >>= 1;
  }
  return r;
}

// Deterministic Miller-Rabin for n < 4,759,123,141 with bases 2, 7, 61
// (Jaeschke 1993).
bool is_prime_u32(uint32_t n) {
  if (n < 2) return false;
  for (uint32_t sp : {2u, 3u, 5u, 7u, 11u, 13u, 61u})
    if (n % sp == 0) return n == sp;
  uint32_t dd = n - 1;
  int r = 0;
  while ((dd & 1) == 0) { dd >>= 1; ++r; }
  for (uint32_t base : {2u, 7u, 61u}) {
    uint64_t x = powmod(base, dd, n);
    if (x == 1 || x == n - 1) continue;
    bool comp = true;
    for (int i = 1; i < r; ++i) {
      x = (unsigned __int128)x * x % n;
      if (x == n - 1) { comp = false; break; }
    }
    if (comp) return false;
  }
  return true;
}

static int32_t balanced(uint64_t x, uint32_t p) {
  x %= p;
  return x > (p - 1) / 2 ? (int32_t)((int64_t)x - p) : (int32_t)x;
}

FpConst make_fp_const(uint32_t p) {
  FpConst k;
  k.p = (int32_t)p;
  k.h = (int32_t)((p - 1) / 2);
  uint32_t inv = p;  // Newton iteration for p^-1 mod 2^32 (p odd)
  for (int i = 0; i < 5; ++i) inv *= 2u - p * inv;
  k.pinv = inv;
  k.negp = -(int32_t)p;
  const uint64_t c32 = (uint64_t(1) << 32) % p;
  const uint64_t R = (unsigned __int128)c32 * c32 % p;  // 2^64 mod p
  k.c32 = balanced(c32, p);
  k.c64 = balanced(R, p);
  k.one = k.c64;
  k.two = balanced(2 * R, p);
  k.two32 = balanced(2 * c32, p);  // 2^33 mod p
  k.inv2 = balanced((unsigned __int128)R * ((p + 1) / 2) % p, p);
  const uint64_t R2 = (unsigned __int128)R * R % p;
  k.r4 = balanced((unsigned __int128)R2 * R2 % p, p);
  // 2^-32 mod p = (2^32 mod p)^(p-2)
  const uint64_t inv32 = powmod(c32, p - 2, p);
  k.r4s = balanced((unsigned __int128)((unsigned __int128)R2 * R2 % p) * inv32 % p, p);
  k.r3 = balanced((unsigned __int128)R2 * R % p, p);
  k.r3s = balanced((unsigned __int128)((unsigned __int128)R2 * R % p) * inv32 % p, p);
  return k;
}

// a square root of -1 mod p (p = 1 mod 4) in Montgomery form: g^((p-1)/4) R
// for the smallest quadratic non-residue g, balanced
int32_t fp_sqrt_minus_one_mont(uint32_t p) {
  uint64_t g = 2;
  while (powmod(g, (p - 1) / 2, p) != p - 1) ++g;
  const uint64_t i = powmod(g, (p - 1) / 4, p);
  const uint64_t c32 = (uint64_t(1) << 32) % p;
  const uint64_t R = (unsigned __int128)c32 * c32 % p;
  return balanced((unsigned __int128)i * R % p, p);
}

// ---------------------------------------------------------------------------
// variant choice
// ---------------------------------------------------------------------------
static bool fits(const Variant& v, int field, int n, int d) {
  if (v.field != field) return false;
  if (v.generic) return v.DL >= d;
  return v.N == n - 1 && v.DL * v.L >= d;
}

// selections, per metric: launches in the alternating metric have pins of
// their own (a kernel's two metric forms can compile to code of different
// speed), and fall back to the mostly-minus choice
struct Pin {
  int field, n, d, metric, index;
};
static std::mutex g_pin_mu;
static std::vector<Pin> g_pins;

static int pinned(int field, int n, int d, int metric) {
  std::lock_guard<std::mutex> lk(g_pin_mu);
  for (const Pin& p : g_pins)
    if (p.field == field && p.n == n && p.d == d && p.metric == metric) return p.index;
  return -1;
}

bool is_pinned(int field, int n, int d, int metric) { return pinned(field, n, d, metric) >= 0; }

int pinned_index(int field, int n, int d, int metric) { return pinned(field, n, d, metric); }

int select_variant(int metric, int field, int n, int d, int index) {
  if (field != BG_FIELD_C128 && field != BG_FIELD_FP) return BG_EINVAL;
  if (metric != BG_METRIC_MOSTLY_MINUS && metric != BG_METRIC_ALTERNATING) return BG_EINVAL;
  if (n < 3 || n > BG_MAX_N || d < 1 || d > BG_MAX_D) return BG_EDOMAIN;
  if (index >= 0 && (index >= (int)registry().size() || !fits(registry()[index], field, n, d)))
    return BG_EINVAL;
  std::lock_guard<std::mutex> lk(g_pin_mu);
  for (auto it = g_pins.begin(); it != g_pins.end(); ++it)
    if (it->field == field && it->n == n && it->d == d && it->metric == metric) {
      g_pins.erase(it);
      break;
    }
  if (index >= 0) g_pins.push_back({field, n, d, metric, index});
  return BG_OK;
}

// the register kernel of (field, n) with L lanes per point and the fewest
// components per lane that cover d (null if none is compiled)
static const Variant* register_variant(int field, int n, int d, int L) {
  const Variant* best = nullptr;
  for (const Variant& v : registry()) {
    if (v.generic || v.field != field || v.N != n - 1 || v.L != L || v.DL * L < d) continue;
    if (!best || v.DL < best->DL || (v.DL == best->DL && v.lds_tables && !best->lds_tables)) best = &v;
  }
  return best;
}

// the lane-group kernel of G work items on LC lanes each (null if not compiled)
static const Variant* lane_group_variant(int field, int dmax, int G, int LC, bool padded) {
  for (const Variant& v : registry())
    if (v.generic && v.field == field && v.DL == dmax && v.L == G * LC && v.L > 1 && v.split == LC && v.padded == padded)
      return &v;
  return nullptr;
}

// Kernel choice without a pin.  Over C it goes by (n, d) alone: two kernels sum
// in different orders, and a point has to come out with the same bits however
// many points share its launch (a job in chunks, a request merged with others).
// Over Z_p, where every kernel gives the same residues, it also goes by the
// number of points.
// Measured on gfx950 with every compiled kernel at n = 4..14, d = 4..10 and 100
// to 2^20 points; figures are us per launch, this choice against the next one.
//
// A launch takes the longer of one wave's latency and its share of the issue
// slots.  While the waves of all points fit the chip at once the latency
// decides, and more lanes per point shorten it: the lane-group kernels with the
// most lanes (they hold 3 to 4 waves per SIMD, so up to kGroupPts points run
// at once), then the register kernels with four lanes per point (one wave per
// SIMD, kFourLanePts points).  Past that the kernel with the fewest
// instructions per point wins.
constexpr int64_t kGroupPts = 4096;      // points whose lane-group waves run at once
constexpr int64_t kFourLanePts = 16384;  // points whose four-lane waves (16 points each) do, one per SIMD
constexpr int64_t kManyPts = 65536;      // several waves of any register kernel per SIMD

// Lane-group kernels over C (no register kernel is compiled for n >= 13, for
// n = 12 with d > 4, n >= 9 with d > 8): two lanes per work item (half the
// components each).  32 items per point at n >= 13, where the long ranges have
// the cuts for them, 16 below (n = 12, d = 6, 64000 points: 581 against 732,
// though 100 points take 30 against 26); d = 7, 8 with four lanes per item and 16
// items up to n = 13 (n = 12, 64000 points: 773 against 913 with two).  Padded
// rows at n = 14, d <= 4 (2000 points: 35 against 43 unpadded; 64000: 728 against
// 710), n = 14, d = 7, 8 (64000: 1374 against 1601) and n = 13, d = 9, 10 (64000:
// 1469 against 1582).
static const Variant* lane_group_c128(int n, int d) {
  if (d <= 4) return lane_group_variant(FIELD_C128, 4, 32, 2, n >= 14);
  if (d <= 6) return lane_group_variant(FIELD_C128, 6, n >= 13 ? 32 : 16, 2, false);
  if (d <= 8) return n >= 14 ? lane_group_variant(FIELD_C128, 8, 32, 2, true) : lane_group_variant(FIELD_C128, 8, 16, 4, false);
  return lane_group_variant(FIELD_C128, 10, n >= 13 ? 32 : 16, 2, n == 13);
}

// Lane-group kernels over Z_p: one lane per item and 16 items per point for
// many points (n = 12, d = 8, 10^5 points, unpadded rows: 417 against 501
// padded), 32 at n = 14 (d = 6: 676 against 731), where d = 7, 8 takes padded
// rows (2 10^4 points: 175 against 194); two lanes per item for few points
// (n = 11, d = 8, 1000 points: 22 against 29 with 16 lanes per point) and for
// d = 9, 10 from n = 12 on (n = 14, 10^5 points: 1039 against 1070), where the
// LDS holds 6144 points of n = 13 with two lanes and 8192 with one (7000 points: 77
// against 76, with a prime of large 2^32 mod p 87 against 79), and at n = 14 one
// lane and 32 items keep up to 12288 points (6000: 79 against 76, such a prime 88
// against 80; 12000: 162 against 158, 181 against 170).  At n = 14, d = 7, 8 the 64
// lanes of a point end at 3072 points, what the LDS of 256 CUs holds of them (3000
// points: 44 against 48 on 32 lanes, 4000: 54 against 48; such a prime 49 against 51
// and 60 against 51).
static const Variant* lane_group_fp(int n, int d, int64_t npts) {
  if (npts <= kGroupPts / 2) {
    if (d <= 4) return lane_group_variant(FIELD_FP, 4, 32, 1, false);
    return lane_group_variant(FIELD_FP, d <= 8 ? 8 : 10, 32, 2, false);
  }
  if (npts <= (n >= 14 && (d == 7 || d == 8) ? kGroupPts * 3 / 4 : kGroupPts)) {
    if (d <= 4) return lane_group_variant(FIELD_FP, 4, n >= 12 ? 32 : 16, 1, false);
    if (d > 8) return lane_group_variant(FIELD_FP, 10, n >= 13 ? 32 : 16, 2, false);
    if (d <= 6 && n >= 13) return lane_group_variant(FIELD_FP, 6, 32, 1, false);
    return lane_group_variant(FIELD_FP, 8, d > 6 && n >= 13 ? 32 : 16, 2, false);
  }
  if (d > 8) {
    if (n >= 14 && npts <= 3 * kGroupPts) return lane_group_variant(FIELD_FP, 10, 32, 1, false);
    const bool one = n < 12 || (n == 13 && npts > kGroupPts * 3 / 2 && npts <= 2 * kGroupPts);
    return lane_group_variant(FIELD_FP, 10, 16, one ? 1 : 2, false);
  }
  const int dmax = d <= 4 ? 4 : d <= 6 ? 6 : 8;
  const bool items32 = n >= 14 && (dmax > 4 || npts <= kManyPts / 2);
  return lane_group_variant(FIELD_FP, dmax, items32 ? 32 : 16, 1, items32 && dmax == 8);
}

// Register kernels over C.  Four lanes per point where two would hold too many
// components to keep the currents in registers: d = 9, 10 from n = 5 on (n = 7,
// 128000 points: 161 against 245), d = 7, 8 from n = 6 on (n = 8, 128000: 175
// against 294), d = 5, 6 from n = 9 on (n = 9, 128000: 275 against 277, 1000
// points 1.5 times faster), any d from n = 11 on; else two (n = 8, d = 4, 512000:
// 294 against 443).  Four lanes lose from 16385 to 32768 points, where their
// waves share a SIMD and those of two lanes still run one to a SIMD (n = 6, d = 8,
// 20000 points: 16.1 against 14.5, 48000: 22.4 against 28.6; n = 6, d = 9 up to
// 10^5 points, 64000: 48.5 against 45.6, 256000: 171 against 191).  n = 5, d = 7, 8
// stay on two: the gain beyond that window is small (256000: 67 against 70).
static const Variant* register_c128(int n, int d) {
  const Variant* four = register_variant(FIELD_C128, n, d, 4);
  const Variant* two = register_variant(FIELD_C128, n, d, 2);
  if (!four || !two) return four ? four : two;
  return n >= (d >= 9 ? 5 : d >= 7 ? 6 : d >= 5 ? 9 : 11) ? four : two;
}

// Register kernels over Z_p.  One lane per point (no sums over lanes, 30 %
// fewer instructions) for many points of d <= 6 (n = 6, d = 6, 5 10^5 points:
// 64 against 79), at n = 7, 8 with d = 5, 6 only up to two waves per SIMD
// (n = 8, d = 6, 10^5 points: 47 against 50; 2 10^5: 93 against 83).  Four for
// few points (n = 6, d = 10, 10^4 points: 10.0 against 11.6 with two), except
// at n = 4, d = 9, 10 (6.6 against 6.0).  Else two (n = 6, d = 10, 5 10^4
// points: 18 against 25 with four).
static const Variant* register_fp(int n, int d, int64_t npts) {
  const Variant* four = register_variant(FIELD_FP, n, d, 4);
  const Variant* one = register_variant(FIELD_FP, n, d, 1);
  const Variant* two = register_variant(FIELD_FP, n, d, 2);
  if (four && npts <= kFourLanePts && (d >= 9 ? n >= 5 : d >= 7 || (d >= 5 && n <= 6))) return four;
  if (one && npts >= kManyPts && (n <= 6 || d <= 4 || npts <= 2 * kManyPts)) return one;
  return two ? two : (one ? one : four);
}

const Variant* default_variant(int field, int n, int d, int64_t npts) {
  const Variant* v = nullptr;
  if (field == FIELD_C128) {
    v = register_c128(n, d);
    if (!v) v = lane_group_c128(n, d);
  } else {
    // lane-group from n = 8 (d > 4) for few points, at n = 11 up to
    // kFourLanePts (d = 6, 10^4 points: 44 against 49), and there for d > 6 at
    // any size (d = 8, 10^5 points: 337 against 599: the register kernel
    // spills) and for d <= 4 from kManyPts on (10^5 points: 201 against 211); at
    // n = 10, d <= 4 up to three times kGroupPts (12000 points: 29 against 34).  The
    // lines are those of 2^31 - 19; primes of large 2^32 mod p take them too, though
    // their register kernels spill at n = 10, d > 6 and n = 11, where a lane-group
    // kernel would be faster (64000 points: n = 10, d = 8 192 against 244, n = 11,
    // d = 4 152 against 266)
    const int64_t few = n == 11           ? (d > 6 ? INT64_MAX : kFourLanePts)
                        : n == 10         ? (d > 6 ? 2 * kGroupPts : d <= 4 ? 3 * kGroupPts : kGroupPts)
                        : n == 9          ? kGroupPts
                        : n == 8 && d > 4 ? kGroupPts / 4
                                          : 0;
    v = register_fp(n, d, npts);
    if (!v || npts <= few || (n == 11 && d <= 4 && npts >= kManyPts)) v = lane_group_fp(n, d, npts);
  }
  if (v) return v;
  for (const Variant& w : registry())  // whatever covers (field, n, d)
    if (fits(w, field, n, d)) return &w;
  return nullptr;
}

const Variant* choose_variant(int field, int n, int d, int64_t npts) {
  const int idx = pinned(field, n, d, BG_METRIC_MOSTLY_MINUS);
  if (idx >= 0 && idx < (int)registry().size() && fits(registry()[idx], field, n, d))
    return &registry()[idx];
  return default_variant(field, n, d, npts);
}

bool only_lane_groups(int field, int n, int d) {
  if (pinned(field, n, d, BG_METRIC_MOSTLY_MINUS) >= 0) return true;
  for (const Variant& v : registry())
    if (!v.generic && fits(v, field, n, d)) return false;
  return true;
}

int max_lds_per_block() {
  static std::once_flag once;
  static int v = 65536;
  std::call_once(once, [] {
    int dev = 0, val = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&val, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess &&
        val > 0)
      v = val;
  });
  return v;
}

static int cu_count() {
  static std::once_flag once;
  static int v = 256;
  std::call_once(once, [] {
    int dev = 0, val = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&val, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && val > 0)
      v = val;
  });
  return v;
}

int prepare(int field, int n, int d, int64_t npts, int64_t ld, const void* momenta, const void* pols,
            void* out, uint8_t* status, const FpConst& fp, LaunchSpec& spec, const Variant* force) {
  const Variant* v = force ? force : choose_variant(field, n, d, npts);
  if (!v) return BG_ENOTIMPL;
  LaunchArgs& a = spec.args;
  a.momenta = momenta;
  a.pols = pols;
  a.out = out;
  a.status = status;
  a.npts = npts;
  a.ld = ld;
  a.d = d;
  a.fp = fp;
  a.metric = BG_METRIC_MOSTLY_MINUS;
  a.ialt = fp.one;  // the mostly-minus factor; launch() sets i R for the alternating metric
  a.cur = nullptr;
  spec.variant = v;
  spec.fn = (field == FIELD_FP && v->fn_sc && fp_small_fold(fp)) ? v->fn_sc : v->fn;
  spec.generic = v->generic;
  spec.lanes = v->L;
  spec.N = n - 1;
  if (!v->generic) {
    const int64_t threads = npts * v->L;
    int64_t blocks = (threads + v->block - 1) / v->block;
    if (blocks > 0x7FFFFFFF) return BG_EINVAL;
    // more than two rounds of blocks (one per CU for the kernels that have a
    // streaming form): the blocks stay and read ahead.  Up to two rounds a block
    // has at most one point to read ahead for, and the read after the last one
    // costs more than that gains: n = 8, d = 4, 50000 points 37 -> 38 us, 70000
    // points 55 us either way, 100000 points 73 -> 72 us
    if (v->fn_stream && blocks > (int64_t)2 * cu_count()) {
      spec.fn = v->fn_stream;
      blocks = cu_count();
    }
    spec.grid = (unsigned)blocks;
    spec.block = (unsigned)v->block;
    spec.shmem = 0;
    return BG_OK;
  }
  const size_t per = v->lds_per_point ? v->lds_per_point(n - 1) : 0;
  const int maxlds = max_lds_per_block();
  if (per == 0 || per > (size_t)maxlds) return BG_ENOTIMPL;
  int P;  // points per block
  if (v->L == 1) {
    P = (int)std::min<size_t>(256, (size_t)maxlds / per);
    if (P >= 64) P = P / 64 * 64;
  } else {
    P = wide_points_per_block(*v, per);
    // up to one wave per SIMD: the smallest blocks of whole wavefronts, so that
    // the points spread evenly over the CUs (n = 13, d = 6, 1000 points: 40 us
    // in blocks of 4 points, 30 us in blocks of one; at 3000 points larger
    // blocks are faster again, n = 14, d = 6: 59 against 80 us)
    const int step = v->L < 64 ? 64 / v->L : 1;
    if (P > step && npts <= (int64_t)4 * cu_count() * step) P = step;
  }
  if (P < 1) return BG_ENOTIMPL;
  const size_t shmem = per * P;
  if (shmem > 65536) {
    static std::mutex mu;
    std::lock_guard<std::mutex> lk(mu);
    (void)hipFuncSetAttribute(spec.fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
  }
  const int64_t blocks = (npts + P - 1) / P;
  if (blocks > 0x7FFFFFFF) return BG_EINVAL;
  spec.grid = (unsigned)blocks;
  spec.block = (unsigned)(P * v->L);
  spec.shmem = (unsigned)shmem;
  return BG_OK;
}

int wide_points_per_block(const Variant& v, size_t per) {
  // G lanes per point: the block size whose blocks hold the most points per
  // CU (LDS and 32 wave slots per CU), among blocks of whole wavefronts when
  // one fits: a block of fewer lanes than a wave still takes a wave slot and
  // issues every instruction for 64 lanes, so half-full waves halve the work
  // done per instruction
  const int maxlds = max_lds_per_block();
  const int pmax = std::min<int>(256 / v.L, (int)((size_t)maxlds / per));
  const int step = v.L < 64 ? 64 / v.L : 1;  // points per whole wave
  const int first = step <= pmax ? step : 1;
  const int inc = step <= pmax ? step : 1;
  int P = 1;
  long bestres = 0;
  for (int c = first; c <= pmax; c += inc) {
    const long waves = ((long)c * v.L + 63) / 64;
    const long blocks = std::min<long>((long)maxlds / ((long)c * (long)per), 32 / waves);
    const long res = blocks * c;
    if (res > bestres || (res == bestres && c > P)) { bestres = res; P = c; }
  }
  return P;
}

int enqueue(LaunchSpec& spec, hipStream_t stream) {
  void* args_reg[] = {&spec.args};
  void* args_gen[] = {&spec.args, &spec.N};
  hipError_t e = hipLaunchKernel(spec.fn, dim3(spec.grid), dim3(spec.block),
                                 spec.generic ? args_gen : args_reg, spec.shmem, stream);
  return e == hipSuccess ? BG_OK : BG_EHIP;
}

// Without a pin of their own, alternating-metric launches take the
// mostly-minus choice, except that a one-lane F_p register kernel is replaced
// by the two-lane one of the same (n, d): the one-lane kernels' alternating
// body runs about twice as long as their mostly-minus body (the compiler waits
// for each of its loads before issuing the next; n = 8, d = 6: 0.97 against
// 0.47 ms per 2^20 points), the two-lane kernel's within a few percent of its
// own.
static const Variant* alternating_variant(const Variant* v, int field, int n, int d) {
  if (!v || field != FIELD_FP || v->generic || v->L != 1) return v;
  const Variant* best = nullptr;
  for (const Variant& w : registry()) {
    if (w.generic || w.field != field || w.N != n - 1 || w.L != 2 || w.DL * 2 < d) continue;
    if (!best || w.DL < best->DL || (w.DL == best->DL && w.lds_tables && !best->lds_tables)) best = &w;
  }
  return best ? best : v;
}

int launch(int field, int n, int d, int64_t npts, int64_t ld, const void* momenta, const void* pols,
           void* out, uint8_t* status, const FpConst& fp, hipStream_t stream, int metric = BG_METRIC_MOSTLY_MINUS) {
  LaunchSpec spec;
  const Variant* force = nullptr;
  if (metric == BG_METRIC_ALTERNATING) {
    const int idx = pinned(field, n, d, BG_METRIC_ALTERNATING);
    force = idx >= 0 ? &registry()[idx] : alternating_variant(choose_variant(field, n, d, npts), field, n, d);
  }
  const int rc = prepare(field, n, d, npts, ld, momenta, pols, out, status, fp, spec, force);
  if (rc != BG_OK) return rc;
  spec.args.metric = metric;
  if (metric == BG_METRIC_ALTERNATING && field == FIELD_FP) spec.args.ialt = fp_sqrt_minus_one_mont((uint32_t)fp.p);
  return enqueue(spec, stream);
}

static int check_common(int n, int d, int64_t npts, int64_t ld) {
  if (n < 3 || n > BG_MAX_N || d < 1 || d > BG_MAX_D) return BG_EDOMAIN;
  if (npts < 0) return BG_EINVAL;
  (void)ld;
  return BG_OK;
}

static int check_buffers(int64_t npts, int64_t ld, const void* m, const void* e, const void* o) {
  if (ld < npts || !m || !e || !o) return BG_EINVAL;
  return BG_OK;
}

}  // namespace bg

extern "C" {

int bg_amplitudes_c128_metric(int metric, int n, int d, int64_t npts, int64_t ld, const double* momenta,
                              const double* pols, double* out, uint8_t* status, void* hip_stream) {
  if (metric != BG_METRIC_MOSTLY_MINUS && metric != BG_METRIC_ALTERNATING) return BG_EINVAL;
  int rc = bg::check_common(n, d, npts, ld);
  if (rc != BG_OK) return rc;
  if (npts == 0) return BG_OK;
  rc = bg::check_buffers(npts, ld, momenta, pols, out);
  if (rc != BG_OK) return rc;
  bg::FpConst none;
  memset(&none, 0, sizeof(none));
  return bg::launch(bg::FIELD_C128, n, d, npts, ld, momenta, pols, out, status, none,
                    static_cast<hipStream_t>(hip_stream), metric);
}

int bg_amplitudes_c128(int n, int d, int64_t npts, int64_t ld, const double* momenta,
                       const double* pols, double* out, uint8_t* status, void* hip_stream) {
  return bg_amplitudes_c128_metric(BG_METRIC_MOSTLY_MINUS, n, d, npts, ld, momenta, pols, out, status,
                                   hip_stream);
}

int bg_amplitudes_fp_metric(int metric, int n, int d, int64_t npts, int64_t ld, uint32_t p,
                            const uint32_t* momenta, const uint32_t* pols, uint32_t* out, uint8_t* status,
                            void* hip_stream) {
  if (metric != BG_METRIC_MOSTLY_MINUS && metric != BG_METRIC_ALTERNATING) return BG_EINVAL;
  int rc = bg::check_common(n, d, npts, ld);
  if (rc != BG_OK) return rc;
  if (p < 3 || p >= 0x80000000u || !bg::is_prime_u32(p)) return BG_ENOTPRIME;
  if (metric == BG_METRIC_ALTERNATING && p % 4 != 1) return BG_EDOMAIN;  // needs a square root of -1
  if (npts == 0) return BG_OK;
  rc = bg::check_buffers(npts, ld, momenta, pols, out);
  if (rc != BG_OK) return rc;
  const bg::FpConst k = bg::make_fp_const(p);
  return bg::launch(bg::FIELD_FP, n, d, npts, ld, momenta, pols, out, status, k,
                    static_cast<hipStream_t>(hip_stream), metric);
}

int bg_amplitudes_fp(int n, int d, int64_t npts, int64_t ld, uint32_t p, const uint32_t* momenta,
                     const uint32_t* pols, uint32_t* out, uint8_t* status, void* hip_stream) {
  return bg_amplitudes_fp_metric(BG_METRIC_MOSTLY_MINUS, n, d, npts, ld, p, momenta, pols, out, status,
                                 hip_stream);
}

// root current K([1..n-1]) instead of M: same preparation, `cur` in place of `out`
static int launch_currents(int field, int n, int d, int64_t npts, int64_t ld, const void* momenta,
                           const void* pols, void* cur, uint8_t* status, const bg::FpConst& fp,
                           hipStream_t stream) {
  bg::LaunchSpec spec;
  const int rc = bg::prepare(field, n, d, npts, ld, momenta, pols, nullptr, status, fp, spec);
  if (rc != BG_OK) return rc;
  spec.args.cur = cur;
  return bg::enqueue(spec, stream);
}

int bg_currents_c128(int n, int d, int64_t npts, int64_t ld, const double* momenta, const double* pols,
                     double* cur, uint8_t* status, void* hip_stream) {
  int rc = bg::check_common(n, d, npts, ld);
  if (rc != BG_OK) return rc;
  if (npts == 0) return BG_OK;
  rc = bg::check_buffers(npts, ld, momenta, pols, cur);
  if (rc != BG_OK) return rc;
  bg::FpConst none;
  memset(&none, 0, sizeof(none));
  return launch_currents(bg::FIELD_C128, n, d, npts, ld, momenta, pols, cur, status, none,
                         static_cast<hipStream_t>(hip_stream));
}

int bg_currents_fp(int n, int d, int64_t npts, int64_t ld, uint32_t p, const uint32_t* momenta,
                   const uint32_t* pols, uint32_t* cur, uint8_t* status, void* hip_stream) {
  int rc = bg::check_common(n, d, npts, ld);
  if (rc != BG_OK) return rc;
  if (p < 3 || p >= 0x80000000u || !bg::is_prime_u32(p)) return BG_ENOTPRIME;
  if (npts == 0) return BG_OK;
  rc = bg::check_buffers(npts, ld, momenta, pols, cur);
  if (rc != BG_OK) return rc;
  const bg::FpConst k = bg::make_fp_const(p);
  return launch_currents(bg::FIELD_FP, n, d, npts, ld, momenta, pols, cur, status, k,
                         static_cast<hipStream_t>(hip_stream));
}

int bg_variants(int field, int n, int d, bg_variant_info* out, int cap) {
  if (field != BG_FIELD_C128 && field != BG_FIELD_FP) return BG_EINVAL;
  if (n < 3 || n > BG_MAX_N || d < 1 || d > BG_MAX_D) return BG_EDOMAIN;
  const bg::Variant* cur = bg::choose_variant(field, n, d, INT64_MAX);
  int count = 0;
  const auto& reg = bg::registry();
  for (int i = 0; i < (int)reg.size(); ++i) {
    if (!bg::fits(reg[i], field, n, d)) continue;
    if (out && count < cap) {
      bg_variant_info& o = out[count];
      o.index = i;
      o.lanes = reg[i].L;
      o.comps_per_lane = reg[i].DL / reg[i].split;
      o.lds_tables = reg[i].lds_tables ? 1 : 0;
      o.generic = reg[i].generic ? 1 : 0;
      o.padded = reg[i].padded ? 1 : 0;
      o.max_d = reg[i].generic ? reg[i].DL : reg[i].DL * reg[i].L;
      o.selected = (&reg[i] == cur) ? 1 : 0;
    }
    ++count;
  }
  return count;
}

int bg_select_variant(int field, int n, int d, int index) {
  return bg::select_variant(BG_METRIC_MOSTLY_MINUS, field, n, d, index);
}

int bg_select_variant_metric(int metric, int field, int n, int d, int index) {
  return bg::select_variant(metric, field, n, d, index);
}

const char* bg_strerror(int code) {
  switch (code) {
    case BG_OK: return "success";
    case BG_EINVAL: return "invalid argument (null pointer, npts < 0 or ld < npts)";
    case BG_EDOMAIN: return "n or d outside the supported range";
    case BG_ENOTPRIME: return "p is not an odd prime below 2^31";
    case BG_EHIP: return "HIP runtime error or kernel launch failure";
    case BG_ENOTIMPL: return "no kernel for this (field, n, d)";
    case BG_ENOMEM: return "request does not fit the memory budget";
    case BG_EBUSY: return "queue full";
    default: return "unknown error code";
  }
}

int bg_version(void) { return 100; }

}  // extern "C"
