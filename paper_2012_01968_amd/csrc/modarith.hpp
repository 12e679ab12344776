// Device modular arithmetic for 64-bit NTT-friendly primes on gfx950.
//
// Shoup's modular multiplication (Algorithm 4 of the paper): with the companion
// wb = floor(w * 2^64 / q) precomputed for a fixed operand w < q, the quotient
// estimate qh = floor(b * wb / 2^64) is within one of floor(b * w / q) for any
// b < 2^64, so r = b*w - qh*q lies in [0, 2q) and only the low 64 bits of the two
// products are needed.  The paper's listing writes the quotient step with a garbled
// shift and tests `r > p`; the reading here is the high half of the 128-bit product
// and a lazy result (the final reduction to [0, q) happens once, at the end of a
// transform).  Butterflies keep their values in lazy ranges in the manner of Harvey,
// whom the paper cites for Algorithm 2's [0, 4p) input bound.
//
// Two arithmetic policies, chosen per plan from the largest prime:
//
//  Arith<false>  any q < 2^62.  Shoup's product with the exact quotient; Cooley-Tukey values in
//                [0, 4q), Gentleman-Sande values in [0, 2q) (Harvey's bounds).
//  Arith<true>   q < 2^60.  Signed values and Montgomery products of signed digits
//                (signed_mont.hpp), with the bounds of every value tracked at compile time
//                (CtRange, GsRange).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "signed_mont.hpp"

namespace nttk {

// A fixed multiplicand, stored as one 16-byte entry: the factor and its Shoup companion for
// Arith<false>, the signed digits of its two Montgomery forms for Arith<true>.
struct Tw {
  uint64_t w, wb;
};

struct Mod {  // per-prime constants
  uint64_t q, q2;   // q, 2q
  MontMod mm;       // Arith<true>
  Mod() = default;
  // From a per-prime constant row {q, 2q, q0 | q1 << 32, nl | nh << 32, qi2, qm | qsh << 32}.
  template <typename Ptr>
  static __device__ __forceinline__ Mod load(Ptr c) {
    Mod m;
    m.q = m.mm.q = c[0];
    m.q2 = c[1];
    const uint64_t d = c[2], n = c[3], f = c[5];
    m.mm.q0 = lo32(d);
    m.mm.q1 = hi32(d);
    m.mm.nl = lo32(n);
    m.mm.nh = hi32(n);
    m.mm.qi2 = (uint32_t)c[4];
    m.mm.qm = (uint32_t)f;
    m.mm.qsh = (uint32_t)(f >> 32);
    return m;
  }
};

__device__ __forceinline__ uint64_t mulhi64(uint64_t a, uint64_t b) { return __umul64hi(a, b); }

__device__ __forceinline__ uint64_t csub(uint64_t x, uint64_t m) { return x >= m ? x - m : x; }

__device__ __forceinline__ uint64_t make_u64(uint32_t lo, uint32_t hi) {
  return __builtin_bit_cast(uint64_t, (uint2{lo, hi}));
}

template <bool FAST>
struct Arith;

template <>
struct Arith<false> {
  // b * w mod q in [0, 2q), any b < 2^64.
  static __device__ __forceinline__ uint64_t mul(uint64_t b, const Tw& t, const Mod& m) {
    const uint64_t qh = mulhi64(b, t.wb);
    return b * t.w - qh * m.q;
  }
  // Cooley-Tukey: X, Y in [0, 4q) -> X + WY, X - WY in [0, 4q).
  static __device__ __forceinline__ void ct(uint64_t& X, uint64_t& Y, const Tw& t, const Mod& m) {
    const uint64_t x = csub(X, m.q2);
    const uint64_t v = mul(Y, t, m);
    X = x + v;
    Y = x - v + m.q2;
  }
  // Same with the twiddle applied as two factors (on-the-fly twiddling, Section VII).
  static __device__ __forceinline__ void ct2(uint64_t& X, uint64_t& Y, const Tw& a, const Tw& b, const Mod& m) {
    const uint64_t x = csub(X, m.q2);
    const uint64_t v = mul(mul(Y, a, m), b, m);
    X = x + v;
    Y = x - v + m.q2;
  }
  // Gentleman-Sande: X, Y in [0, 2q) -> X + Y, (X - Y) W in [0, 2q).
  static __device__ __forceinline__ void gs(uint64_t& X, uint64_t& Y, const Tw& t, const Mod& m) {
    const uint64_t s = csub(X + Y, m.q2);
    const uint64_t d = X - Y + m.q2;
    X = s;
    Y = mul(d, t, m);
  }
  static __device__ __forceinline__ void gs2(uint64_t& X, uint64_t& Y, const Tw& a, const Tw& b, const Mod& m) {
    const uint64_t s = csub(X + Y, m.q2);
    const uint64_t d = X - Y + m.q2;
    X = s;
    Y = mul(mul(d, a, m), b, m);
  }
  // Last inverse stage with the 1/N scale: X' = (X + Y)/N, Y' = (X - Y) W/N, in [0, 2q).
  static __device__ __forceinline__ void gs_scaled(uint64_t& X, uint64_t& Y, const Tw& wn, const Tw& n,
                                                   const Mod& m) {
    const uint64_t s = X + Y;
    const uint64_t d = X - Y + m.q2;
    X = mul(s, n, m);
    Y = mul(d, wn, m);
  }
  static __device__ __forceinline__ uint64_t fwd_final(uint64_t x, const Mod& m) { return csub(csub(x, m.q2), m.q); }
  static __device__ __forceinline__ uint64_t inv_final(uint64_t x, const Mod& m) { return csub(x, m.q); }
  template <int NB>
  static __device__ __forceinline__ void mul_n(uint64_t (&r)[NB], const uint64_t (&b)[NB], const Tw (&t)[NB],
                                               const Mod& m) {
#pragma unroll
    for (int k = 0; k < NB; ++k) r[k] = mul(b[k], t[k], m);
  }
};

template <>
struct Arith<true> {
  static __device__ __forceinline__ uint64_t mul(uint64_t b, const Tw& t, const Mod& m) {
    return (uint64_t)mont_mul((int64_t)b, t.w, t.wb, m.mm);
  }
  template <int NB>
  static __device__ __forceinline__ void mul_n(uint64_t (&r)[NB], const uint64_t (&b)[NB], const Tw (&t)[NB],
                                               const Mod& m) {
#pragma unroll
    for (int k = 0; k < NB; ++k) r[k] = mul(b[k], t[k], m);
  }
  static __device__ __forceinline__ uint64_t reduce(uint64_t x, const Mod& m) {
    return (uint64_t)mont_reduce((int64_t)x, m.mm);
  }
  // Stage 0 of the whole inverse, with the 1/N scale: products below 3/2 q.
  static __device__ __forceinline__ void gs_scaled(uint64_t& X, uint64_t& Y, const Tw& wn, const Tw& n,
                                                   const Mod& m) {
    const uint64_t s = X + Y, d = X - Y;
    X = mul(s, n, m);
    Y = mul(d, wn, m);
  }
  static __device__ __forceinline__ uint64_t fwd_final(uint64_t x, const Mod& m) {
    return mont_canonical((int64_t)x, m.mm);
  }
  static __device__ __forceinline__ uint64_t inv_final(uint64_t x, const Mod& m) {
    return mont_canonical_2q((int64_t)x, m.mm);
  }
};

// General a * b mod q for a, b < q < 2^62 (no precomputed companion): Barrett
// reduction with s = bitlen(q), mu = floor(2^(2s) / q) < 2^(s+1).
// x = a*b < 2^(2s); x1 = floor(x / 2^(s-1)); qh = floor(x1 * mu / 2^(s+1)) undershoots
// floor(x / q) by at most 2, so r = x - qh*q < 3q and two conditional subtractions
// finish the reduction.
__device__ __forceinline__ uint64_t mulmod_barrett(uint64_t a, uint64_t b, uint64_t q, uint64_t mu, uint32_t s) {
  const uint64_t lo = a * b;
  const uint64_t hi = mulhi64(a, b);
  const uint64_t x1 = (lo >> (s - 1)) | (hi << (65 - s));   // s >= 2; s - 1 >= 1 so both shifts are < 64
  const uint64_t plo = x1 * mu;
  const uint64_t phi = mulhi64(x1, mu);
  const uint64_t qh = (plo >> (s + 1)) | (phi << (63 - s));  // s <= 62: 63 - s >= 1
  uint64_t r = lo - qh * q;
  r = csub(r, q);
  r = csub(r, q);
  return r;
}

// The element-wise product between the forward and the inverse row stages: x as the forward stages
// leave it, f a canonical key value (PAIR = false) or the second operand as they leave it.
// Arith<true> leaves x f 2^-62 mod q within q of 0 (the scale of the products' inverse passes
// carries 2^62), Arith<false> the canonical product.
template <bool FAST, bool PAIR>
__device__ __forceinline__ uint64_t ntt_domain_product(uint64_t x, uint64_t f, const Mod& m, uint64_t mu, uint32_t bits) {
  using A = Arith<FAST>;
  if constexpr (FAST)
    return (uint64_t)mont_product(mont_reduce((int64_t)x, m.mm), PAIR ? mont_reduce((int64_t)f, m.mm) : (int64_t)f, m.mm);
  else
    return mulmod_barrett(A::fwd_final(x, m), PAIR ? A::fwd_final(f, m) : f, m.q, mu, bits);
}

}  // namespace nttk
