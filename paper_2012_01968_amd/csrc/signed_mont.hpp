// Modular products of signed lazy values for primes q < 2^60 (Montgomery's reduction in radix
// 2^31 on signed 32-bit digits).  Plain C++ on both sides: the kernels and the host checks compile
// this file.
//
// A fixed multiplicand w is stored as two residues, A = w 2^31 mod q and B = w 2^63 mod q, each
// centred in [-q/2, q/2] and split into signed digits A = A1 2^31 + A0 with A0 in [-2^30, 2^30).
// For a signed 64-bit value b = b1 2^32 + b0 with b0 in [-2^31, 2^31),
//   P = b0 A0 + b1 B0,   m = -P q^-1 mod 2^31 in [-2^30, 2^30),   P + m q0 = 0 mod 2^31,
//   r = ((P + m q0) >> 31) + b0 A1 + b1 B1 + m q1 = (b0 A + b1 B + m q) / 2^31 = b w mod q,
// exactly: the shift drops zeros.  Every product is one signed 32 x 32 + 64 bit multiply-add, and a
// product takes 11 instructions (47 SIMD cycles a wave on gfx950) where Shoup's product with an
// estimated quotient took 13 to 14 (58 cycles).
//
// Ranges.  |P| <= 2^61 + |b1| 2^30 + 2^60 < 2^63 for any b the bounds below allow, and
//   |r| <= q/2 (b0) + |b| q / 2^64 (b1) + q/2 (m) <= q + |b| / 16,
// so a product is near q whatever it multiplied, and, being signed, X + r and X - r need no offset.
// Bounds are kept at compile time in sixteenths of q; the largest is kMontLimit (7.75 q < 2^63).
// A Cooley-Tukey stage adds about q + q/16 per q of its inputs, so X is reduced every fourth or
// fifth stage (it was every other stage with unsigned values below 16 q).
//
// Measured on the kernels (VALU instructions of a wave, before and after): 256-point forward row
// 1019 and 764, 512-point two-operand product row 3057 and 2404 (740 and 2117 since the rows are one
// basic block); product of 2 polynomials at N = 2^17, 60 primes 362 and 308 us (301 with that), forward and inverse of 2 polynomials at N = 2^16, 45 primes
// with the tables cached 103 and 91 us.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define NTTK_HD __host__ __device__ __forceinline__
#else
#define NTTK_HD inline
#endif

namespace nttk {

struct MontMod {
  uint64_t q;
  int32_t q0, q1;      // signed digits of q
  uint32_t qi2;        // 2 (-q^-1 mod 2^31): a product's low word is 2 m
  int32_t nl, nh;      // -q = nh 2^32 + nl
  uint32_t qm, qsh;    // quotient estimate: floor(2^(s+6) / q) and s - 3, s = bitlen(q)
};

constexpr int kMontLimit = 124;     // sixteenths of q
constexpr int kMontCanon = 16;      // inputs in [0, q)
constexpr int kMontReduced = 14;    // after mont_reduce: [-5/8 q, 7/8 q)
constexpr int mont_product_bound(int b) { return 16 + b / 16 + 1; }

// The two digit pairs of A and B of a fixed multiplicand, as stored: w = {A0, A1}, wb = {B0, B1}.
NTTK_HD int32_t lo32(uint64_t v) { return (int32_t)(uint32_t)v; }
NTTK_HD int32_t hi32(uint64_t v) { return (int32_t)(uint32_t)(v >> 32); }

// Keeps the compiler from regrouping a sum around v (it would split the multiply-add chains and
// spend a 64-bit add on joining them).
template <typename T>
NTTK_HD void keep(T& v) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm("" : "+v"(v));
#else
  (void)v;
#endif
}

NTTK_HD int64_t mont_mul(int64_t b, uint64_t A, uint64_t B, const MontMod& m) {
  const int32_t b0 = lo32((uint64_t)b);
  const int32_t b1 = hi32((uint64_t)b) + (int32_t)((uint32_t)b >> 31);
  int64_t P = (int64_t)b0 * lo32(A);
  P += (int64_t)b1 * lo32(B);
  const int32_t t = (int32_t)((uint32_t)P * m.qi2) >> 1;
  P += (int64_t)t * m.q0;
  int64_t r = P >> 31;
  keep(r);
  r += (int64_t)b0 * hi32(A);
  keep(r);
  r += (int64_t)b1 * hi32(B);
  keep(r);
  r += (int64_t)t * m.q1;
  return r;
}

// x - k q for the estimate k = floor((t qm + bias) / 512) of x / q, t = floor(x / 2^(s-3)).  For
// |x| <= 7.75 q: |t| <= 64, and e = t qm / 512 lies in (x/q - 3/8, x/q + 1/8] (t drops less than
// q/4 of x, qm less than |t| / 512 <= 1/8 of e, toward zero).
NTTK_HD int64_t mont_sub_estimate(int64_t x, const MontMod& m, int32_t bias) {
  const int32_t t = (int32_t)(x >> m.qsh);
#if defined(__HIP_DEVICE_COMPILE__)
  const int32_t k = (__mul24(t, (int32_t)m.qm) + bias) >> 9;
#else
  const int32_t k = (t * (int32_t)m.qm + bias) >> 9;
#endif
  const uint64_t y = (uint64_t)(x + (int64_t)k * m.nl);
  uint32_t kh = (uint32_t)k * (uint32_t)m.nh;
  keep(kh);
  return (int64_t)((uint32_t)y | (uint64_t)((uint32_t)(y >> 32) + kh) << 32);
}
NTTK_HD int64_t mont_reduce(int64_t x, const MontMod& m) { return mont_sub_estimate(x, m, 256); }

NTTK_HD uint64_t masked(uint64_t v, uint64_t sign_of) {   // v where sign_of is negative, else 0
  const uint32_t s = (uint32_t)(hi32(sign_of) >> 31);
  return ((uint32_t)v & s) | (uint64_t)((uint32_t)(v >> 32) & s) << 32;
}

// [-q, q) -> [0, q) and, for |x| <= 7.75 q, x -> [0, q): with bias -1/8 the estimate is never above
// x / q and less than 3/2 below it.
NTTK_HD uint64_t add_if_negative(uint64_t x, uint64_t v) { return x + masked(v, x); }
NTTK_HD uint64_t mont_canonical(int64_t x, const MontMod& m) {
  const uint64_t r = (uint64_t)mont_sub_estimate(x, m, -64);
  return add_if_negative(r - m.q, m.q);
}
// |x| < 2q -> [0, q)
NTTK_HD uint64_t mont_canonical_2q(int64_t x, const MontMod& m) {
  const uint64_t r = add_if_negative((uint64_t)x, m.q + m.q);
  return add_if_negative(r - m.q, m.q);
}

// x y 2^-62 mod q for |x|, |y| <= q: two digits of x in turn.  |result| <= |x y| / 2^62 + q/2 + 2 < q.
NTTK_HD int64_t mont_product(int64_t x, int64_t y, const MontMod& m) {
  int32_t x0 = (int32_t)((uint32_t)x << 1) >> 1, x1 = (int32_t)((x + (1 << 30)) >> 31);
  int32_t y0 = (int32_t)((uint32_t)y << 1) >> 1, y1 = (int32_t)((y + (1 << 30)) >> 31);
  keep(x0);   // as 32-bit values: seen through, the upper digits would make 64-bit products
  keep(x1);
  keep(y0);
  keep(y1);
  int64_t P = (int64_t)x0 * y0;
  const int32_t t0 = (int32_t)((uint32_t)P * m.qi2) >> 1;
  P += (int64_t)t0 * m.q0;
  int64_t T = P >> 31;
  keep(T);
  T += (int64_t)x0 * y1;
  keep(T);
  T += (int64_t)t0 * m.q1;
  keep(T);
  T += (int64_t)x1 * y0;
  const int32_t t1 = (int32_t)((uint32_t)T * m.qi2) >> 1;
  T += (int64_t)t1 * m.q0;
  int64_t r = T >> 31;
  keep(r);
  r += (int64_t)x1 * y1;
  keep(r);
  r += (int64_t)t1 * m.q1;
  return r;
}

// Value bounds of the fast Cooley-Tukey stages, in sixteenths of q: IN before local stage 0 of a
// sub-transform, the same for all values of a stage.  A stage turns X, Y into X + r, X - r with r
// near q; X is reduced first where the outputs would pass the limit otherwise.
constexpr int kCtCanon = kMontCanon;   // sub-transforms that read the caller's input
constexpr int kCtLazy = kMontLimit;    // those that read what an earlier pass left
template <int IN>
struct CtRange {
  static constexpr bool reduce_at(int b) { return b + mont_product_bound(b) > kMontLimit; }
  static constexpr int before(int s) {
    int b = IN;
    for (int j = 0; j < s; ++j) b = (reduce_at(b) ? kMontReduced : b) + mont_product_bound(b);
    return b;
  }
  static constexpr bool reduce(int s) { return reduce_at(before(s)); }
};

// Value bounds of the fast Gentleman-Sande stages, in sixteenths of q.  In the local stage i of a
// step, register u (bit i clear) pairs with u | 2^i; both played the same part in the stage
// before (bit i-1 of u), so they share a bound.  A difference is multiplied at once, so it may
// reach the limit: values stay within half of it.  A sum doubles the bound and is reduced only
// when it would pass that half.
constexpr int kGsCanon = kMontCanon;      // inputs in [0, q)
constexpr int kGsLazy = kMontLimit / 2;   // what any stage leaves
template <int IN>
struct GsRange {
  static_assert(IN >= 1 && IN <= kGsLazy, "Gentleman-Sande inputs must lie within half the limit");
  // bound of register u before local stage i
  static constexpr int before(int i, int u) {
    int b = IN;
    for (int j = 0; j < i; ++j)
      b = (u >> j) & 1 ? mont_product_bound(2 * b) : (2 * b > kGsLazy ? kMontReduced : 2 * b);
    return b;
  }
  static constexpr bool reduce(int i, int u) { return 2 * before(i, u) > kGsLazy; }
};

}  // namespace nttk
