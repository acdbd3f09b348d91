// dcs_device.hpp -- device primitives of the divide-and-conquer sampler
// (gfx950, HIP).  Everything here is part of the sample's definition: the
// same operations, in the same order and precision, give the same bits on
// every launch geometry.  Compile with -ffp-contract=off (no fused
// multiply-add is formed from the separate multiplies and adds written here).
//
// Contents:
//   * Philox-4x32-10 (Salmon et al., SC'11): the hash h of a subproblem's
//     identity that drives every random decision (paper Sec. 3.2).
//   * exact uniform conversions and the multiply-shift range map;
//   * logarithms by the atanh series (fixed polynomial, fixed order);
//   * ln(a!) - ln(b!) without cancellation;
//   * the hypergeometric split deviate (paper Sec. 3; Stadlober's
//     ratio-of-uniforms method) and the binomial one (Sec. 4.6).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lnfact_dev.inc"

namespace dcs {

// ---------------------------------------------------------------------------
// Stream purposes: the third component of the identity (j, k, t) hashed in
// Algorithm P (Sec. 3.2) -- which decision of a node a stream feeds.
// ---------------------------------------------------------------------------
enum Purpose : uint32_t {
  kSplit = 1,    // hypergeometric split of a without-replacement node
  kLeaf = 2,     // sparse leaf: uniform offsets (Algorithm H)
  kBern = 3,     // dense leaf: geometric skips (Algorithm B)
  kRepair = 4,   // dense leaf: hits removed by the repair step
  kBChunk = 5,   // Bernoulli sampling: geometric skips of one chunk
  kWrSplit = 6,  // binomial split of a with-replacement node
  kWrLeaf = 7,   // with-replacement leaf: uniform offsets
  kSegSplit = 8, // uneven universe: split of a subtree of segments
  kSegSeed = 9,  // uneven universe: seed of one segment's own tree
  kWChunk = 10,  // whole-range Algorithm B: skips of one chunk
  kWRepair = 11, // whole-range Algorithm B: hits removed by the repair
};

constexpr uint64_t kLeafMaxRange = 1ull << 32;

// ---------------------------------------------------------------------------
// Philox-4x32-10
// ---------------------------------------------------------------------------
struct Stream {
  uint32_t k0, k1;  // key = seed
  uint32_t c1;      // purpose << 24 | attempt
  uint32_t c2, c3;  // node id (low, high)
};

__device__ __forceinline__ Stream make_stream(uint64_t seed, uint64_t node, uint32_t purpose,
                                              uint32_t attempt) {
  Stream s;
  s.k0 = static_cast<uint32_t>(seed);
  s.k1 = static_cast<uint32_t>(seed >> 32);
  s.c1 = (purpose << 24) | (attempt & 0xFFFFFFu);
  s.c2 = static_cast<uint32_t>(node);
  s.c3 = static_cast<uint32_t>(node >> 32);
  return s;
}

// One 128-bit block: counter (block, c1, c2, c3), key (k0, k1), ten rounds.
__device__ __forceinline__ uint4 philox_block(const Stream& s, uint32_t block) {
  uint32_t x0 = block, x1 = s.c1, x2 = s.c2, x3 = s.c3;
  uint32_t k0 = s.k0, k1 = s.k1;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    // one 32x32->64 multiply-add each (v_mad_u64_u32) gives both halves
    const uint64_t pa = static_cast<uint64_t>(0xD2511F53u) * x0;
    const uint64_t pb = static_cast<uint64_t>(0xCD9E8D57u) * x2;
    // three-input XOR in one instruction (truth table 0x96 = a ^ b ^ c)
    const uint32_t n0 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(pb >> 32), x1, k0, 0x96);
    const uint32_t n2 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(pa >> 32), x3, k1, 0x96);
    x1 = static_cast<uint32_t>(pb);
    x3 = static_cast<uint32_t>(pa);
    x0 = n0;
    x2 = n2;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return make_uint4(x0, x1, x2, x3);
}

__device__ __forceinline__ uint32_t pick(const uint4& v, unsigned j) {
  return j == 0 ? v.x : (j == 1 ? v.y : (j == 2 ? v.z : v.w));
}

// Sequential reader of 64-bit draws: draw t = words 2(t&1) | 2(t&1)+1 << 32
// of block t/2.
struct Draws64 {
  Stream s;
  uint64_t t;
  uint32_t gbits = 6;  // wave mode: groups of 2^gbits lanes share a deviate
  __device__ __forceinline__ uint64_t next() {
    const uint4 b = philox_block(s, static_cast<uint32_t>(t >> 1));
    const uint64_t v = (t & 1) ? (static_cast<uint64_t>(b.z) | (static_cast<uint64_t>(b.w) << 32))
                               : (static_cast<uint64_t>(b.x) | (static_cast<uint64_t>(b.y) << 32));
    ++t;
    return v;
  }
};

// ---------------------------------------------------------------------------
// Uniform conversions
// ---------------------------------------------------------------------------
// (0,1]: ((x >> 11) + 1) 2^-53 and [0,1): (x >> 11) 2^-53 -- both exact.
__device__ __forceinline__ double unit_open0(uint64_t x) {
  return static_cast<double>((x >> 11) + 1) * 0x1p-53;
}
__device__ __forceinline__ double unit_closed0(uint64_t x) {
  return static_cast<double>(x >> 11) * 0x1p-53;
}

// Geometric uniform in [2^-32, 1]: the integer w+1 rounded to nearest float,
// times 2^-32.
__device__ __forceinline__ float geom_unit(uint32_t w) {
  const float x = (w == 0xFFFFFFFFu) ? 4294967296.0f : static_cast<float>(w + 1u);
  return x * 0x1p-32f;
}

// Range map for s in [1, 2^32]: value (w*s) >> 32, void when the low half of
// w*s is below 2^32 mod s (that threshold is passed in, precomputed per
// range).  Returns false for a void draw.
__device__ __forceinline__ bool range_map(uint32_t w, uint64_t s, uint32_t threshold,
                                          uint32_t* v) {
  const uint64_t m = static_cast<uint64_t>(w) * s;
  *v = static_cast<uint32_t>(m >> 32);
  return static_cast<uint32_t>(m) >= threshold;
}

__host__ __device__ __forceinline__ uint32_t range_threshold(uint64_t s) {
  return static_cast<uint32_t>((1ull << 32) % s);
}

// ---------------------------------------------------------------------------
// Logarithms (atanh series after reduction to [sqrt(1/2), sqrt(2))).
// ---------------------------------------------------------------------------
// ln 2 = kLn2Hi + kLn2Lo with kLn2Hi holding 32 significant bits.
constexpr double kLn2Hi = 0x1.62e42feep-1;
constexpr double kLn2Lo = 0x1.a39ef35793c76p-33;
constexpr double kSqrt2 = 0x1.6a09e667f3bcdp+0;
constexpr float kLn2HiF = 0x1.62e4p-1f;      // 16 significant bits
constexpr float kLn2LoF = 0x1.7f7d1cp-20f;
constexpr float kSqrt2F = 0x1.6a09e6p+0f;

// sum_{j=0}^{10} z^j / (2j+3), Horner from the innermost coefficient 1/23.
__device__ __forceinline__ double series64(double z) {
  double p = 1.0 / 23.0;
  p = 1.0 / 21.0 + z * p;
  p = 1.0 / 19.0 + z * p;
  p = 1.0 / 17.0 + z * p;
  p = 1.0 / 15.0 + z * p;
  p = 1.0 / 13.0 + z * p;
  p = 1.0 / 11.0 + z * p;
  p = 1.0 / 9.0 + z * p;
  p = 1.0 / 7.0 + z * p;
  p = 1.0 / 5.0 + z * p;
  return 1.0 / 3.0 + z * p;
}

// 2 atanh(s) for s = f/(2+f).
__device__ __forceinline__ double atanh2_64(double f) {
  const double s = f / (2.0 + f);
  const double z = s * s;
  const double t = s + s;
  return t + t * (z * series64(z));
}

__device__ __forceinline__ double log64(double x) {
  const uint64_t bits = static_cast<uint64_t>(__double_as_longlong(x));
  int e = static_cast<int>((bits >> 52) & 0x7FF) - 1023;
  double m = __longlong_as_double(
      static_cast<long long>((bits & 0x000FFFFFFFFFFFFFull) | 0x3FF0000000000000ull));
  if (m >= kSqrt2) {
    m = m * 0.5;
    e += 1;
  }
  const double r = atanh2_64(m - 1.0);
  const double de = static_cast<double>(e);
  return de * kLn2Hi + (de * kLn2Lo + r);
}

__device__ __forceinline__ double log1p64(double x) {
  if (x > -0.25 && x < 0.25) return atanh2_64(x);
  return log64(1.0 + x);
}

__device__ __forceinline__ float series32(float z) {
  float p = 1.0f / 11.0f;
  p = 1.0f / 9.0f + z * p;
  p = 1.0f / 7.0f + z * p;
  p = 1.0f / 5.0f + z * p;
  return 1.0f / 3.0f + z * p;
}

// f / d for |f| < 1/2 and d in [3/2, 5/2] (the logarithm's reduced
// argument): no operand scaling or special case can arise, so a hardware
// reciprocal refined by one Newton step, the product, and one correction
// from the exact (fused) residual give the correctly rounded quotient -- for
// every f the reduction can produce, which a test checks against the
// correctly rounded division.
__device__ __forceinline__ float div_reduced(float f, float d) {
  float y = __builtin_amdgcn_rcpf(d);
  y = __builtin_fmaf(__builtin_fmaf(-d, y, 1.0f), y, y);
  const float q = f * y;
  return __builtin_fmaf(__builtin_fmaf(-q, d, f), y, q);
}

__device__ __forceinline__ float log32(float x) {
  const uint32_t bits = __float_as_uint(x);
  int e = static_cast<int>((bits >> 23) & 0xFF) - 127;
  float m = __uint_as_float((bits & 0x007FFFFFu) | 0x3F800000u);
  if (m >= kSqrt2F) {
    m = m * 0.5f;
    e += 1;
  }
  const float f = m - 1.0f;
  const float s = div_reduced(f, 2.0f + f);
  const float z = s * s;
  const float t = s + s;
  const float r = t + t * (z * series32(z));
  const float fe = static_cast<float>(e);
  return fe * kLn2HiF + (fe * kLn2LoF + r);
}

// Geometric skip floor(ln(U) * c) for U from one 32-bit word.
__device__ __forceinline__ int geom_skip32(uint32_t w, float c) {
  return static_cast<int>(floorf(log32(geom_unit(w)) * c));
}

// The skips of four words, by every lane of a wave.  The defined skip is the
// floor of x = log32(U) c; nearly always it can be read off a cheaper x':
// the hardware's base-2 logarithm times c ln 2.  Over all 2^32 words that
// logarithm times ln 2 lies within 2.1405e-7 of log32(U), relative (a test
// evaluates every word); the roundings of c ln 2, of x' and of x add 3 2^-24, so |x' - x|
// <= 4.0e-7 x', and where no integer lies within 5e-7 x' + 2^-22 of x' the two
// floors are equal.  Otherwise (a word of all ones too: x' is infinite) the
// wave takes the defined skip of that word.  About 13 issue slots a draw
// instead of 45; at p = 0.01 one group of four words in about 30 needs a
// second look.
__device__ __forceinline__ void geom_skips32(const uint4& w, float c, uint32_t (&skip)[4]) {
  const float c2 = c * 0x1.62e43p-1f;
  bool unsure[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float u = static_cast<float>(pick(w, j) + 1u) * 0x1p-32f;
    const float x = __builtin_amdgcn_logf(u) * c2;
    const float off = __builtin_amdgcn_fractf(x) - 0.5f;
    unsure[j] = !(__builtin_fabsf(off) <= __builtin_fmaf(x, -5e-7f, 0.5f - 0x1p-22f));
    skip[j] = static_cast<uint32_t>(x);
  }
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(unsure[0] || unsure[1] || unsure[2] ||
                                                   unsure[3]) != 0, 0)) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (__builtin_amdgcn_ballot_w64(unsure[j]) != 0)
        skip[j] = static_cast<uint32_t>(geom_skip32(pick(w, j), c));
  }
}

// Double-precision skips.  The defined skip is the floor of x = log64(U) c
// (at most 2^33); nearly always it can be read off x' = ln'(U) c with
//   ln'(U) = e ln 2 + T_i + (r - r^2/2 + r^3/3 - r^4/4 + r^5/5),
// U = 2^e m, i the leading 7 bits of m, r = m / c_i - 1 (|r| <= 2^-8) and
// T_i = ln c_i from a table of 128 entries.  Both logarithms lie within 2^-46
// of ln U (|ln U| < 37), so |x' - x| < 2^-45 |c| + x 2^-52 < 2^-44 |c|, and
// where no integer lies within 2^-43 |c| of x' the floors are equal;
// otherwise the defined skip is taken.
struct LogEntry {
  double inv, ln;  // 1/c_i, -ln of it
};
constexpr uint32_t kLogEntries = 128;
__device__ __forceinline__ LogEntry log_entry(uint32_t i) {
  LogEntry t;
  t.inv = 1.0 / (1.0 + (static_cast<double>(i) + 0.5) * (1.0 / kLogEntries));
  t.ln = -log64(t.inv);
  return t;
}

// x' of one 64-bit draw.
__device__ __forceinline__ double geom_quick64(uint32_t dlo, uint32_t dhi, double c,
                                               const LogEntry* tab) {
  // 2^64 U = the draw's leading 53 bits plus one, exact
  const double lo = static_cast<double>(dlo & 0xFFFFF800u) + 2048.0;
  const double x64 = __builtin_fma(static_cast<double>(dhi), 0x1p32, lo);
  const uint64_t bits = static_cast<uint64_t>(__double_as_longlong(x64));
  const uint32_t hi = static_cast<uint32_t>(bits >> 32);
  const LogEntry t = tab[(hi >> 13) & (kLogEntries - 1)];
  const double m = __longlong_as_double(static_cast<long long>(
      (bits & 0xFFFFFFFFull) |
      (static_cast<uint64_t>((hi & 0x000FFFFFu) | 0x3FF00000u) << 32)));
  const double e = static_cast<double>(static_cast<int>(hi >> 20) - (1023 + 64));
  const double r = __builtin_fma(m, t.inv, -1.0);
  double p = __builtin_fma(r, 1.0 / 5.0, -1.0 / 4.0);
  p = __builtin_fma(r, p, 1.0 / 3.0);
  p = __builtin_fma(r, p, -1.0 / 2.0);
  p = __builtin_fma(r * r, p, r);
  return __builtin_fma(e, 0x1.62e42fefa39efp-1, t.ln + p) * c;
}

// The skips of a Philox block's two 64-bit draws as doubles, not yet cut at
// 2^33 (every lane of a wave); half = 1/2 - 2^-43 |c|.
__device__ __forceinline__ void geom_skips64(const uint4& w, double c, double half,
                                             const LogEntry* tab, double g[2]) {
  const double x0 = geom_quick64(w.x, w.y, c, tab), x1 = geom_quick64(w.z, w.w, c, tab);
  const double f0 = __builtin_amdgcn_fract(x0), f1 = __builtin_amdgcn_fract(x1);
  g[0] = x0 - f0;
  g[1] = x1 - f1;
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(__builtin_fabs(f0 - 0.5) <= half) ||
                                                   !(__builtin_fabs(f1 - 0.5) <= half)) != 0,
                       0)) {
#pragma unroll 1
    for (int j = 0; j < 2; ++j) {
      const uint64_t d = static_cast<uint64_t>(j ? w.z : w.x) |
                         (static_cast<uint64_t>(j ? w.w : w.y) << 32);
      const double x = __builtin_floor(log64(unit_open0(d)) * c);
      (j ? g[1] : g[0]) = x;
    }
  }
}

// ---------------------------------------------------------------------------
// ln(a!) - ln(b!)
// ---------------------------------------------------------------------------
constexpr double kHalfLn2Pi = 0x1.d67f1c864beb5p-1;
constexpr uint64_t kStirlingDiffMin = 64;

__device__ __forceinline__ double lnfact_table(uint64_t k) {
  return __longlong_as_double(static_cast<long long>(dcs_lnfact_bits[k]));
}

// 1/(12 z) - 1/(360 z^3) + 1/(1260 z^5)
__device__ __forceinline__ double stirling_tail(double z) {
  const double r = 1.0 / z;
  const double r2 = r * r;
  return r * (1.0 / 12.0 - r2 * (1.0 / 360.0 - r2 * (1.0 / 1260.0)));
}

__device__ __forceinline__ double lnfact(uint64_t x) {
  if (x < DCS_LNFACT_ENTRIES) return lnfact_table(x);
  const double z = static_cast<double>(x) + 1.0;
  return (z - 0.5) * log64(z) - z + kHalfLn2Pi + stirling_tail(z);
}

__device__ __forceinline__ double lnfact_diff(uint64_t a, uint64_t b) {
  if (a == b) return 0.0;
  if (a >= kStirlingDiffMin && b >= kStirlingDiffMin) {
    const double za = static_cast<double>(a) + 1.0;
    const double zb = static_cast<double>(b) + 1.0;
    const double d = static_cast<double>(static_cast<int64_t>(a) - static_cast<int64_t>(b));
    const double t1 = (zb - 0.5) * log1p64(d / zb);
    const double t2 = d * (log64(za) - 1.0);
    const double t3 = stirling_tail(za) - stirling_tail(zb);
    return (t1 + t2) + t3;
  }
  return lnfact(a) - lnfact(b);
}

// ---------------------------------------------------------------------------
// Exact floor(x*y/z) for x, y, z < 2^53 and a quotient below 2^53 (the
// splits' modes): the FP64 quotient is within 2 of it, and 128-bit products
// correct it (a 128-bit integer division would run bit by bit).
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t floor_muldiv(uint64_t x, uint64_t y, uint64_t z) {
  const unsigned __int128 p = static_cast<unsigned __int128>(x) * y;
  const double e = (static_cast<double>(x) * static_cast<double>(y)) / static_cast<double>(z);
  uint64_t q = e < 0x1p63 ? static_cast<uint64_t>(e) : (1ull << 63);
  unsigned __int128 qz = static_cast<unsigned __int128>(q) * z;
  while (qz > p) {
    --q;
    qz -= z;
  }
  while (p - qz >= z) {
    ++q;
    qz += z;
  }
  return q;
}

// ---------------------------------------------------------------------------
// Ratio-of-uniforms deviates (Stadlober 1990).
// ---------------------------------------------------------------------------
constexpr double kD1 = 0x1.b72cd3f331398p+0;  // 2 sqrt(2/e)
constexpr double kD2 = 0x1.cc3ebd3bc711ap-1;  // 3 - 2 sqrt(3/e)
constexpr uint64_t kInversionMax = 16;

// Accept/reject for 2 ln U <= T with the two squeezes; lu2 = 2 ln U.
__device__ __forceinline__ bool rou_accept(double u, double T, double lu2) {
  if (u * (4.0 - u) - 3.0 <= T) return true;
  if (u * (u - T) >= 1.0) return false;
  return lu2 <= T;
}

// An attempt's outcome as a cheaper evaluation sees it.
enum RouOutcome : int { kRouReject = 0, kRouAccept = 1, kRouUnsure = 2 };

// The ratio-of-uniforms loop: attempt a takes draws 2a (U) and 2a+1 (V),
// i.e. Philox block a, and the deviate is the first accepted attempt.
// quick(u, v, &k) decides an attempt (nearly always), exact(u, v, &k) decides
// the ones it leaves open.  kWave: the lanes of a wave form aligned groups of
// G = 2^d.gbits lanes (the whole wave when gbits = 6), each group sampling one
// deviate: lane r of a group tries attempt G j + r in round j, and the group
// takes its lowest accepted attempt (the same deviate, found in one round
// instead of one attempt after another).
template <bool kWave, class Quick, class Exact>
__device__ __forceinline__ uint64_t rou_first_accepted(Draws64& d, Quick quick, Exact exact) {
  uint32_t r = 0, base = 0, step = 1;
  unsigned long long gmask = 0;
  if constexpr (kWave) {
    uint32_t lane = threadIdx.x & 63u;
    asm volatile("" : "+v"(lane));
    step = 1u << d.gbits;
    r = lane & (step - 1u);
    base = lane - r;
    gmask = d.gbits >= 6 ? ~0ull : (1ull << step) - 1ull;
  }
  for (uint32_t a = r;; a += step) {
    const uint4 b = philox_block(d.s, a);
    const double u = unit_open0(static_cast<uint64_t>(b.x) | (static_cast<uint64_t>(b.y) << 32));
    const double v = unit_closed0(static_cast<uint64_t>(b.z) | (static_cast<uint64_t>(b.w) << 32));
    uint64_t k = 0;
    int got = quick(u, v, &k);
    if constexpr (kWave) {
      unsigned long long m = (__builtin_amdgcn_ballot_w64(got == kRouAccept) >> base) & gmask;
      // an open attempt matters only ahead of the group's first accepted one
      if (got == kRouUnsure && (m & ((1ull << r) - 1ull)) == 0)
        got = exact(u, v, &k) ? kRouAccept : kRouReject;
      m = (__builtin_amdgcn_ballot_w64(got == kRouAccept) >> base) & gmask;
      if (m != 0) {
        const uint32_t f = static_cast<uint32_t>(__ffsll(static_cast<long long>(m)) - 1);
        uint32_t lo, hi;
        if (d.gbits >= 6) {
          lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(k), f);
          hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(k >> 32), f);
        } else {
          lo = static_cast<uint32_t>(__shfl(static_cast<int>(k), static_cast<int>(base + f)));
          hi = static_cast<uint32_t>(__shfl(static_cast<int>(k >> 32), static_cast<int>(base + f)));
        }
        return static_cast<uint64_t>(lo) | (static_cast<uint64_t>(hi) << 32);
      }
    } else {
      if (got == kRouUnsure) got = exact(u, v, &k) ? kRouAccept : kRouReject;
      if (got == kRouAccept) return k;
    }
  }
}

// ---------------------------------------------------------------------------
// Quick evaluation of an attempt.  The defined steps (about 1000 dependent
// double-precision instructions: four ln-factorial differences with two
// logarithms and five correctly rounded divisions each) decide two things: the
// integer k = floor(x) and the sign of T - 2 ln U.  Both are read off cheaper
// values with proven error bounds; where a bound does not decide, the defined
// steps do.
//
// With delta = k - mode every ln-factorial difference is a sum of ln z over
// |delta| consecutive z, centred at z_i; over a centred run
//   sum ln(z + j) = delta ln z - sum j^2/(2 z^2) - sum j^4/(4 z^4) - ...
// so T = delta ln(z2 z3 / (z1 z4)) + the runs' corrections: one logarithm of a
// ratio near 1 instead of eight, and single-precision corrections.
// ---------------------------------------------------------------------------
// 1/d to 2^-45 and sqrt(x) to 2^-47, relative (2^-48.7 and 2^-47.7 measured).
__device__ __forceinline__ double quick_rcp(double d) {
  const double y = __builtin_amdgcn_rcp(d);
  return __builtin_fma(__builtin_fma(-d, y, 1.0), y, y);
}
__device__ __forceinline__ double quick_sqrt(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double g = x * y, h = 0.5 * y;
  return __builtin_fma(g, __builtin_fma(-h, g, 0.5), g);
}

// ---------------------------------------------------------------------------
// Edges of a graph (Sec. 7): pair (u, v), v < u, of edge index k < 2^62, u the
// integer with u(u-1)/2 <= k < u(u+1)/2, i.e. the floor of (1 + sqrt(8k+1))/2,
// as one word (u at the lower address).  The index is base + v (base, -1 or
// more, usually
// the same for a whole row); 8k + 1 is formed in double and its quick root is
// within 2^-47 of itself, so (1 + root)/2, less 2^-14, never exceeds the exact
// value and misses it by less than one: the floor is u or u - 1, and one
// comparison with the triangular number says which.
// ---------------------------------------------------------------------------
template <class V>
__device__ __forceinline__ uint64_t edge_pair(uint64_t base, V v) {
  const double x = __builtin_fma(static_cast<double>(v), 8.0,
                                 __builtin_fma(static_cast<double>(static_cast<int64_t>(base)), 8.0, 1.0));
  uint32_t u = static_cast<uint32_t>(__builtin_fma(quick_sqrt(x), 0.5, 0.5 - 0x1p-14));
  const uint64_t d = base + v - ((static_cast<uint64_t>(u) * (u - 1u)) >> 1);  // 0 if u is 0
  const bool next = d >= u;
  uint32_t r = static_cast<uint32_t>(d);
  r -= next ? u : 0u;
  u += next ? 1u : 0u;
  return static_cast<uint64_t>(u) | (static_cast<uint64_t>(r) << 32);
}

// What a sample's value lo + 1 + v is written as: itself, or with kEdges the
// pair of edge index lo + v (b1 = lo + 1).
template <bool kEdges, class V>
__device__ __forceinline__ uint64_t out_value(uint64_t b1, V v) {
  return kEdges ? edge_pair(b1 - 1, v) : b1 + v;
}

// floor(x y / z) for a quotient below 2^41 and z at most 2^63 + 1: the quick
// quotient is within 2^-3, so the integer nearest to it is the floor or one
// above, and the remainder (at most 0.63 z in size, so its low 64 bits hold
// it) says which.
__device__ __forceinline__ uint64_t quick_muldiv(uint64_t x, uint64_t y, uint64_t z) {
  const double e = (static_cast<double>(x) * static_cast<double>(y)) *
                   quick_rcp(static_cast<double>(z));
  const uint64_t q = static_cast<uint64_t>(e + 0.5);
  return static_cast<int64_t>(x * y - q * z) < 0 ? q - 1 : q;
}

// One centred run's correction divided by delta (d2 = delta^2), with h =
// delta^2 / z^2 and R = 1/z^2:
//   (h - R)/24 + (h - R)(3h - 7R)/960 + (h - R)(3h^2 - 18hR + 31R^2)/8064;
// the next term is about h^4 / 18432.
__device__ __forceinline__ float run_correction(float d2, float z) {
  const float r = __builtin_amdgcn_rcpf(z);
  const float R = r * r, h = d2 * R;
  const float e = __builtin_fmaf(h, __builtin_fmaf(h, 3.0f, -18.0f * R), 31.0f * R * R);
  const float f = __builtin_fmaf(h, 3.0f / 960.0f, __builtin_fmaf(R, -7.0f / 960.0f, 1.0f / 24.0f));
  return (h - R) * __builtin_fmaf(e, 1.0f / 8064.0f, f);
}

// What the quick evaluation keeps of a deviate: x = a + s (V - 1/2) / U, its
// mode, the largest outcome q, and kcap ~ a + 16 sqrt(var + 1/2).
struct RouQuick {
  double a, s, kcap, q, mode;
  bool on;  // within the bounds' range
};

// The attempt's outcome; z1 .. z4 (at delta) from zs(delta, z), runs 2 and 4
// without corrections for a binomial (kRuns = 2: constants).
template <int kRuns, class Zs>
__device__ __forceinline__ int rou_quick(const RouQuick& g, double u, double v, uint64_t* out,
                                         Zs zs) {
  if (!g.on) return kRouUnsure;
  const double off = (g.s * (v - 0.5)) * quick_rcp(u);
  const double x = g.a + off;
  // |x - the defined x| <= eps: a and s differ by less than 2^-44 of
  // themselves from the defined ones, the quotient by 2^-44 more
  const double eps = g.a * 0x1p-43 + __builtin_fabs(off) * 0x1p-42;
  const double k = __builtin_floor(x);
  const double fr = x - k;
  if (x < -eps) return kRouReject;
  if (!(fr > eps && fr < 1.0 - eps)) return kRouUnsure;
  if (k > g.q || k > g.kcap + 2.0) return kRouReject;
  if (k < 0.0 || k > g.kcap - 2.0) return kRouUnsure;
  *out = static_cast<uint64_t>(k);
  const double delta = k - g.mode;
  double z[4];
  zs(delta, z);
  const double Q = z[0] * z[3];
  const double num = __builtin_fma(z[1], z[2], -Q), den = __builtin_fma(z[1], z[2], Q);
  const double t = num * quick_rcp(den);  // ln(z2 z3 / (z1 z4)) = 2 atanh t
  const double t2 = t * t;
  double p = __builtin_fma(t2, 2.0 / 9.0, 2.0 / 7.0);
  p = __builtin_fma(t2, p, 2.0 / 5.0);
  p = __builtin_fma(t2, p, 2.0 / 3.0);
  p = __builtin_fma(t2, p, 2.0) * t;
  const float df = static_cast<float>(delta), d2 = df * df;
  const float z1 = static_cast<float>(z[0]), z3 = static_cast<float>(z[2]);
  float zmin = fminf(z1, z3);
  float corr = run_correction(d2, z1) - run_correction(d2, z3);
  if (kRuns == 4) {
    const float z2 = static_cast<float>(z[1]), z4 = static_cast<float>(z[3]);
    zmin = fminf(zmin, fminf(z2, z4));
    corr += run_correction(d2, z4) - run_correction(d2, z2);
  }
  const float lu2 = __builtin_amdgcn_logf(static_cast<float>(u)) * 0x1.62e43p+0f;  // 2 ln U
  if (!(zmin >= 8.0f && 4.0f * d2 <= zmin * zmin && t2 <= 1.0 / 9.0)) {
    // Far from the mode.  Each step away from it multiplies the mass by at
    // most the factors by which two of the four counts fall below their
    // value at the mode, so T <= -D (D - 1)/2 (1/A + 1/B), D = |delta|, A and
    // B those counts at the mode.
    const float D = __builtin_fabsf(df);
    const float up = static_cast<float>(0.5 * (delta + 1.0)), down = up - 1.0f;
    const float A = df > 0 ? z3 + down : z1 - up;
    float inv = __builtin_amdgcn_rcpf(A);
    if (kRuns == 4)
      inv += __builtin_amdgcn_rcpf(df > 0 ? static_cast<float>(z[1]) + down
                                          : static_cast<float>(z[3]) - up);
    return D * (D - 1.0f) * inv * -0.499f < lu2 * 1.001f - 1e-3f ? kRouReject : kRouUnsure;
  }
  const double T = delta * (p + static_cast<double>(corr));
  // Errors: for |delta| <= z/8 and |t| <= 1/8, T's corrections 2.7e-9 |delta|
  // (single precision; they are below 2.6e-3 |delta|) and its series 2.2e-11
  // |delta|; up to |delta| = z/2 and |t| = 1/3 the terms left out, 2.5e-6
  // |delta|; the defined T's own roundings 1e-13 |delta|; 2 ln U from single
  // precision 5.2e-7 of itself and 1.2e-7.  (Both squeezes of the defined
  // test follow the comparison wherever it is decided by more than rounding:
  // u(4-u) - 3 >= 2 ln u >= u - 1/u on (0, 1].)
  const double margin = T - static_cast<double>(lu2);
  const bool near = 64.0f * d2 <= zmin * zmin && t2 <= 1.0 / 64.0;
  const double err = __builtin_fabs(delta) * (near ? 4e-9 : 1e-5) +
                     static_cast<double>(lu2 * -1e-6f) + 5e-7;
  if (margin > err) return kRouAccept;
  if (margin < -err) return kRouReject;
  return kRouUnsure;
}

// The defined steps of an attempt (rou_first_accepted's `exact`): the accepted
// integer, or kRouNone.  Out of line where lanes share a deviate: there they
// are rare, and inlined their registers cost those kernels a wave per SIMD
// (k_segments with 300000 segments 412 us inlined, 323 so).  A lane alone
// takes them inlined: some lane of its wave needs them in most splits with
// means of a few tens (200001 values in leaves of 15, k_tree: 97 us, 102 by
// call).
constexpr uint64_t kRouNone = ~0ull;
__device__ __forceinline__ uint64_t hyp_exact_steps(uint64_t n, uint64_t M, uint64_t N,
                                                         double u, double v) {
  const uint64_t q = n < M ? n : M;
  const uint64_t rest = N - M - n;
  const double pm = static_cast<double>(M) / static_cast<double>(N);
  const double mu = static_cast<double>(n) * pm;
  const double var =
      (mu * (1.0 - pm)) * (static_cast<double>(N - n) / static_cast<double>(N - 1));
  const double a = mu + 0.5;
  const double w = __builtin_sqrt(var + 0.5);
  const double s = kD1 * w + kD2;
  const double x = a + (s * (v - 0.5)) / u;
  const double kcap = floor(a + 16.0 * w);
  uint64_t kmax = q + 1;
  if (kcap < static_cast<double>(kmax)) kmax = static_cast<uint64_t>(kcap);
  if (x < 0.0 || x >= static_cast<double>(kmax)) return kRouNone;
  const uint64_t k = static_cast<uint64_t>(floor(x));
  const uint64_t mode = floor_muldiv(n + 1, M + 1, N + 2);
  double T = 0.0;
#pragma nounroll
  for (int i = 0; i < 4; ++i) {
    uint64_t ta = mode, tb = k;
    if (i == 1) {
      ta = M - mode;
      tb = M - k;
    } else if (i == 2) {
      ta = n - mode;
      tb = n - k;
    } else if (i == 3) {
      ta = rest + mode;
      tb = rest + k;
    }
    T = T + lnfact_diff(ta, tb);  // 0.0 + the first term is that term
  }
  return rou_accept(u, T, 2.0 * log64(u)) ? k : kRouNone;
}
__device__ __attribute__((noinline)) uint64_t hyp_exact(uint64_t n, uint64_t M, uint64_t N, double u, double v) {
  return hyp_exact_steps(n, M, N, u, v);
}

// Hypergeometric core for 1 <= n, M <= N/2.
template <bool kWave>
__device__ __forceinline__ uint64_t hyp_core(uint64_t n, uint64_t M, uint64_t N, Draws64& d) {
  const uint64_t q = n < M ? n : M;
  const uint64_t big = n < M ? M : n;
  if (q <= kInversionMax) {
    double p0 = 1.0;
    for (uint64_t i = 0; i < q; ++i)
      p0 = p0 * (static_cast<double>(N - big - i) / static_cast<double>(N - i));
    for (;;) {
      double u = unit_open0(d.next());
      double p = p0;
      for (uint64_t k = 0;; ++k) {
        if (u <= p) return k;
        u = u - p;
        if (k == q) break;
        const double r = (static_cast<double>(M - k) / static_cast<double>(k + 1)) *
                         (static_cast<double>(n - k) / static_cast<double>(N - M - n + k + 1));
        p = p * r;
      }
    }
  }
  RouQuick g;
  const uint64_t rest = N - M - n;
  const double nd = static_cast<double>(n), Md = static_cast<double>(M);
  const double Nd = static_cast<double>(N), rd = static_cast<double>(rest);
  {
    const double pm = Md * quick_rcp(Nd);
    const double mu = nd * pm;
    const double var = (mu * (1.0 - pm)) *
                       (static_cast<double>(N - n) * quick_rcp(static_cast<double>(N - 1)));
    const double w = quick_sqrt(var + 0.5);
    g.a = mu + 0.5;
    g.s = __builtin_fma(kD1, w, kD2);
    g.kcap = __builtin_fma(16.0, w, g.a);
    g.q = static_cast<double>(q);
    g.on = N < (1ull << 63) && mu < 0x1p40;
    g.mode = g.on ? static_cast<double>(quick_muldiv(n + 1, M + 1, N + 2)) : 0.0;
  }
  return rou_first_accepted<kWave>(
      d,
      [&](double u, double v, uint64_t* out) {
        return rou_quick<4>(g, u, v, out, [&](double delta, double (&z)[4]) {
          const double up = g.mode + 0.5 * (delta + 1.0), down = g.mode + 0.5 * (delta - 1.0);
          z[0] = up;
          z[1] = Md - down;
          z[2] = nd - down;
          z[3] = rd + up;
        });
      },
      [&](double u, double v, uint64_t* out) {
        *out = kWave ? hyp_exact(n, M, N, u, v) : hyp_exact_steps(n, M, N, u, v);
        return *out != kRouNone;
      });
}

// Hyp(n, M, N): successes among n draws without replacement from N items, M
// of them successes; stream (seed, node, purpose, 0), purpose SPLIT for the
// recursion tree.  kWave: called by every lane of the wave, each aligned
// group of 2^gbits lanes with the same arguments.
template <bool kWave = false>
__device__ __forceinline__ uint64_t hypergeometric(uint64_t n, uint64_t M, uint64_t N, uint64_t seed,
                                   uint64_t node, uint32_t purpose = kSplit,
                                   uint32_t gbits = 6) {
  if (n == 0 || M == 0) return 0;
  if (M == N) return n;
  if (n == N) return M;
  Draws64 d{make_stream(seed, node, purpose, 0), 0, gbits};
  const bool flip_n = n > N - n;
  const uint64_t n1 = flip_n ? N - n : n;
  const bool flip_m = M > N - M;
  const uint64_t M1 = flip_m ? N - M : M;
  uint64_t k = hyp_core<kWave>(n1, M1, N, d);
  if (flip_m) k = n1 - k;
  if (flip_n) k = M - k;
  return k;
}

__device__ __forceinline__ uint64_t binom_exact_steps(uint64_t n, uint64_t l, uint64_t Nv,
                                                           double u, double v) {
  const uint64_t r = Nv - l;
  const double pp = static_cast<double>(l) / static_cast<double>(Nv);
  const double mu = static_cast<double>(n) * pp;
  const double var = mu * (1.0 - pp);
  const double a = mu + 0.5;
  const double w = __builtin_sqrt(var + 0.5);
  const double s = kD1 * w + kD2;
  const double x = a + (s * (v - 0.5)) / u;
  const double kcap = floor(a + 16.0 * w);
  uint64_t kmax = n + 1;
  if (kcap < static_cast<double>(kmax)) kmax = static_cast<uint64_t>(kcap);
  if (x < 0.0 || x >= static_cast<double>(kmax)) return kRouNone;
  const uint64_t k = static_cast<uint64_t>(floor(x));
  const uint64_t mode = floor_muldiv(n + 1, l, Nv);
  const double lodds = log1p64(
      static_cast<double>(static_cast<int64_t>(2 * l) - static_cast<int64_t>(Nv)) /
      static_cast<double>(r));
  double T = static_cast<double>(static_cast<int64_t>(k) - static_cast<int64_t>(mode)) * lodds;
  T = T + lnfact_diff(mode, k);
  T = T + lnfact_diff(n - mode, n - k);
  return rou_accept(u, T, 2.0 * log64(u)) ? k : kRouNone;
}
__device__ __attribute__((noinline)) uint64_t binom_exact(uint64_t n, uint64_t l, uint64_t Nv, double u, double v) {
  return binom_exact_steps(n, l, Nv, u, v);
}

// Binomial core for 1 <= l <= Nv - l.
template <bool kWave>
__device__ __forceinline__ uint64_t binom_core(uint64_t n, uint64_t l, uint64_t Nv, Draws64& d) {
  const uint64_t r = Nv - l;
  if (n <= kInversionMax) {
    const double qv = static_cast<double>(r) / static_cast<double>(Nv);
    double p0 = 1.0;
    for (uint64_t i = 0; i < n; ++i) p0 = p0 * qv;
    const double odds = static_cast<double>(l) / static_cast<double>(r);
    for (;;) {
      double u = unit_open0(d.next());
      double p = p0;
      for (uint64_t k = 0;; ++k) {
        if (u <= p) return k;
        u = u - p;
        if (k == n) break;
        p = p * ((static_cast<double>(n - k) / static_cast<double>(k + 1)) * odds);
      }
    }
  }
  RouQuick g;
  const double nd = static_cast<double>(n), ld = static_cast<double>(l);
  const double rd = static_cast<double>(r);
  {
    const double pp = ld * quick_rcp(static_cast<double>(Nv));
    const double mu = nd * pp;
    const double w = quick_sqrt(mu * (1.0 - pp) + 0.5);
    g.a = mu + 0.5;
    g.s = __builtin_fma(kD1, w, kD2);
    g.kcap = __builtin_fma(16.0, w, g.a);
    g.q = nd;
    g.on = Nv < (1ull << 63) && mu < 0x1p40;
    g.mode = g.on ? static_cast<double>(quick_muldiv(n + 1, l, Nv)) : 0.0;
  }
  return rou_first_accepted<kWave>(
      d,
      [&](double u, double v, uint64_t* out) {
        return rou_quick<2>(g, u, v, out, [&](double delta, double (&z)[4]) {
          z[0] = g.mode + 0.5 * (delta + 1.0);
          z[1] = ld;
          z[2] = nd - (g.mode + 0.5 * (delta - 1.0));
          z[3] = rd;
        });
      },
      [&](double u, double v, uint64_t* out) {
        *out = kWave ? binom_exact(n, l, Nv, u, v) : binom_exact_steps(n, l, Nv, u, v);
        return *out != kRouNone;
      });
}

// Bin(n, l/Nv) from stream (seed, node, WRSPLIT, 0).  kWave: called by
// every lane of the wave, each aligned group of 2^gbits lanes with the same
// arguments.
template <bool kWave = false>
__device__ __forceinline__ uint64_t binomial(uint64_t n, uint64_t l, uint64_t Nv, uint64_t seed,
                                             uint64_t node, uint32_t gbits = 6) {
  if (n == 0 || l == 0) return 0;
  if (l == Nv) return n;
  Draws64 d{make_stream(seed, node, kWrSplit, 0), 0, gbits};
  if (l > Nv - l) return n - binom_core<kWave>(n, Nv - l, Nv, d);
  return binom_core<kWave>(n, l, Nv, d);
}

__host__ __device__ __forceinline__ uint64_t isqrt64(uint64_t x) {
  // Integer square root by bitwise restoring method (exact).
  uint64_t r = 0;
  uint64_t bit = 1ull << 62;
  while (bit > x) bit >>= 2;
  while (bit != 0) {
    if (x >= r + bit) {
      x -= r + bit;
      r = (r >> 1) + bit;
    } else {
      r >>= 1;
    }
    bit >>= 2;
  }
  return r;
}

}  // namespace dcs
