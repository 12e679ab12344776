// Host-side number theory for building a plan: primality, the root convention and the
// twiddle tables with their companions.  Written independently of any test code.
#pragma once
#include <stdint.h>
#include <vector>

namespace nttp {

using u128 = unsigned __int128;

inline uint64_t mulmod(uint64_t a, uint64_t b, uint64_t q) { return (uint64_t)(((u128)a * b) % q); }

inline uint64_t powmod(uint64_t b, uint64_t e, uint64_t q) {
  uint64_t r = 1 % q;
  b %= q;
  while (e) {
    if (e & 1) r = mulmod(r, b, q);
    b = mulmod(b, b, q);
    e >>= 1;
  }
  return r;
}

// Deterministic Miller-Rabin for 64-bit n: the first twelve primes as bases decide
// primality for all n < 3.3e24 (Sorenson and Webster, 2015).
inline bool is_prime(uint64_t n) {
  static const uint64_t bases[] = {2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37};
  if (n < 2) return false;
  for (uint64_t p : bases)
    if (n % p == 0) return n == p;
  uint64_t d = n - 1;
  int s = 0;
  while ((d & 1) == 0) {
    d >>= 1;
    ++s;
  }
  for (uint64_t a : bases) {
    uint64_t x = powmod(a, d, n);
    if (x == 1 || x == n - 1) continue;
    bool witness = true;
    for (int r = 1; r < s; ++r) {
      x = mulmod(x, x, n);
      if (x == n - 1) {
        witness = false;
        break;
      }
    }
    if (witness) return false;
  }
  return true;
}

// Shoup companion floor(w * 2^64 / q) of a fixed multiplicand w < q (Algorithm 4).
inline uint64_t shoup_companion(uint64_t w, uint64_t q) { return (uint64_t)(((u128)w << 64) / q); }

// v where c holds, else 0, without a branch: branches on residues go wrong every other time.  The tables
// of 60 primes at N = 2^17 take 8 to 11 ms on 16 threads with this and the gathers of build_plan, 16 to 20
// with branches and entry by entry.  (The empty statement keeps the compiler from making a branch.)
inline uint64_t where(bool c, uint64_t v) {
  uint64_t mask = 0 - (uint64_t)c;
  asm("" : "+r"(mask));
  return v & mask;
}

// a * w mod q with the companion wb of w, any a < 2^64.
inline uint64_t mul_shoup(uint64_t a, uint64_t w, uint64_t wb, uint64_t q) {
  const uint64_t r = a * w - (uint64_t)(((u128)a * wb) >> 64) * q;
  return r - where(r >= q, q);
}

// Signed digits of v, low one in [-2^30, 2^30): d0 | d1 << 32 with v = d1 2^31 + d0.
inline uint64_t digits31(int64_t v) {
  const int32_t d0 = (int32_t)((uint32_t)v << 1) >> 1;
  return (uint32_t)d0 | (uint64_t)(uint32_t)(int32_t)((v - d0) >> 31) << 32;
}

// What the kernels keep of one fixed multiplicand w < q (nttk::Tw): w and its Shoup companion, or,
// for primes below 2^60, the digits of w 2^31 and w 2^63 mod q, centred (signed_mont.hpp).
struct Multiplicand {
  uint64_t q;
  bool mont;
  uint64_t c31, c31b, c63, c63b;
  Multiplicand(uint64_t q_, bool mont_) : q(q_), mont(mont_) {
    c31 = ((uint64_t)1 << 31) % q;
    c63 = ((uint64_t)1 << 63) % q;
    c31b = shoup_companion(c31, q);
    c63b = shoup_companion(c63, q);
  }
  uint64_t centred(uint64_t v) const { return digits31((int64_t)(v - where(v > q / 2, q))); }
  void put(uint64_t w, uint64_t& a, uint64_t& b) const {
    if (mont) {
      a = centred(mul_shoup(w, c31, c31b, q));
      b = centred(mul_shoup(w, c63, c63b, q));
    } else {
      a = w;
      b = shoup_companion(w, q);
    }
  }
};

inline uint32_t bitrev(uint32_t x, int bits) {   // x < 2^bits
  x = (x >> 1 & 0x55555555u) | (x & 0x55555555u) << 1;
  x = (x >> 2 & 0x33333333u) | (x & 0x33333333u) << 2;
  x = (x >> 4 & 0x0F0F0F0Fu) | (x & 0x0F0F0F0Fu) << 4;
  x = (x >> 8 & 0x00FF00FFu) | (x & 0x00FF00FFu) << 8;
  x = x >> 16 | x << 16;
  return bits ? x >> (32 - bits) : 0;
}

// Smallest primitive 2N-th root of unity mod q (q prime, q = 1 mod 2N).  A generator
// g of the multiplicative group gives one primitive root g^((q-1)/2N); its odd powers
// are all of them.  Returns 0 if no generator candidate below 2^20 works (cannot
// happen for a prime q = 1 mod 2N, but keeps the search bounded).
inline uint64_t smallest_primitive_root(uint64_t q, uint64_t N) {
  const uint64_t e = (q - 1) / (2 * N);
  uint64_t r0 = 0;
  for (uint64_t g = 2; g < (1u << 20); ++g) {
    const uint64_t y = powmod(g, e, q);
    if (powmod(y, N, q) == q - 1) {
      r0 = y;
      break;
    }
  }
  if (!r0) return 0;
  const uint64_t r2 = mulmod(r0, r0, q), r2b = shoup_companion(r2, q);
  uint64_t best = r0, cur = r0;
  for (uint64_t k = 1; k < N; ++k) {
    cur = mul_shoup(cur, r2, r2b, q);
    if (cur < best) best = cur;
  }
  return best;
}

}  // namespace nttp
