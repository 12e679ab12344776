// Host check of the signed Montgomery arithmetic (csrc/signed_mont.hpp, the code the kernels
// compile) against __int128, for odd moduli of 3 to 60 bits, the widest and narrowest of each size
// among them:
//   * products are exact and within their bound for every |b| <= 7.75 q, digit edges included;
//   * the quotient estimates leave [-5/8 q, 7/8 q) and the canonical residue;
//   * products of two values carry 2^-62 and stay within q;
//   * random Cooley-Tukey and Gentleman-Sande stages keep every value within the bound that CtRange
//     and GsRange give, and congruent.
// PLANT=1..4 plants a mistake in what is expected (the check must then fail).
#include <cstdio>
#include <random>

#include "plan_math.hpp"
#include "signed_mont.hpp"

#ifndef PLANT
#define PLANT 0
#endif

using namespace nttk;
typedef __int128 i128;

static long failures = 0;
static void check(bool ok, const char* what) {
  if (!ok && failures++ < 20) std::printf("FAIL %s\n", what);
}
static std::mt19937_64 rng(2012);

static MontMod constants(uint64_t q) {
  MontMod m;
  const int64_t neg = -(int64_t)q;
  uint32_t inv = 1;
  for (int k = 0; k < 5; ++k) inv *= 2 - (uint32_t)q * inv;
  int s = 0;
  while (q >> s) ++s;
  const uint64_t d = nttp::digits31((int64_t)q);
  m.q = q;
  m.q0 = lo32(d);
  m.q1 = hi32(d);
  m.qi2 = (uint32_t)(0u - inv) << 1;
  m.nl = (int32_t)(uint32_t)(uint64_t)neg;
  m.nh = (int32_t)((neg - m.nl) >> 32);
  m.qm = (uint32_t)(((nttp::u128)1 << (s + 6)) / q);
  m.qsh = (uint32_t)(s - 3);
  return m;
}

static int64_t residue(i128 x, uint64_t q) {
  const int64_t r = (int64_t)(x % (i128)q);
  return r < 0 ? r + (int64_t)q : r;
}
static bool within(i128 x, int bound, uint64_t q) { return (x < 0 ? -x : x) * 16 <= (i128)bound * q; }

// A value of |x| <= bound q / 16 congruent to nothing in particular.
static int64_t draw(int bound, uint64_t q) {
  const i128 lim = (i128)bound * q / 16;
  switch (rng() % 8) {
    case 0: return (int64_t)lim;
    case 1: return (int64_t)-lim;
    default: return (int64_t)((i128)((((nttp::u128)rng() << 64) | rng()) % (nttp::u128)(2 * lim + 1)) - lim);
  }
}

template <int IN>
static void cooley_tukey(uint64_t q, const MontMod& m, const nttp::Multiplicand& f) {
  int64_t X = draw(IN, q), Y = draw(IN, q);
  int64_t x = residue(X, q), y = residue(Y, q);
  for (int s = 0; s < 20; ++s) {
    const uint64_t w = rng() % q;
    uint64_t a, b;
    f.put(w, a, b);
    const int64_t v = mont_mul(Y, a, b, m);
    const int64_t xr = CtRange<IN>::reduce_at(CtRange<IN>::before(s)) ? mont_reduce(X, m) : X;
    const int64_t vy = (int64_t)((nttp::u128)y * w % q);
    X = xr + v;
    Y = xr - v;
    const int64_t x2 = residue((i128)x + vy, q), y2 = residue((i128)x - vy, q);
    x = x2;
    y = y2;
    const int bound = CtRange<IN>::before(s + 1) - (PLANT == 1 ? 24 : 0);
    check(within(X, bound, q) && within(Y, bound, q), "Cooley-Tukey bound");
    check(residue(X, q) == x && residue(Y, q) == y, "Cooley-Tukey value");
    if (rng() & 1) std::swap(X, Y), std::swap(x, y);   // either output may play either part next
  }
  check(CtRange<IN>::before(20) <= kMontLimit, "Cooley-Tukey limit");
  check((int64_t)mont_canonical(X, m) == x, "forward result");
}

template <int IN>
static void gentleman_sande(uint64_t q, const MontMod& m, const nttp::Multiplicand& f) {
  int64_t v[8];
  int64_t r[8];
  for (int u = 0; u < 8; ++u) v[u] = draw(IN, q), r[u] = residue(v[u], q);
  for (int i = 0; i < 3; ++i)
    for (int u = 0; u < 8; ++u) {
      if (u & (1 << i)) continue;
      const int o = u | (1 << i);
      const uint64_t w = rng() % q;
      uint64_t a, b;
      f.put(w, a, b);
      const int bound = GsRange<IN>::before(i, u);
      check(within(v[u], bound, q) && within(v[o], bound, q), "Gentleman-Sande bound");
      const int64_t s = v[u] + v[o], d = v[u] - v[o];
      v[u] = GsRange<IN>::reduce(i, u) ? mont_reduce(s, m) : s;
      v[o] = mont_mul(d, a, b, m);
      const int64_t rs = residue((i128)r[u] + r[o], q), rd = residue((i128)residue((i128)r[u] - r[o], q) * (i128)w, q);
      r[u] = rs;
      r[o] = rd;
    }
  for (int u = 0; u < 8; ++u) {
    check(within(v[u], kGsLazy - (PLANT == 2 ? 36 : 0), q), "Gentleman-Sande output bound");
    check(residue(v[u], q) == r[u], "Gentleman-Sande value");
  }
}

int main() {
  for (int trial = 0; trial < 120000; ++trial) {
    const int bits = trial % 3 ? 60 : 3 + (int)(rng() % 58);
    uint64_t q = (rng() >> (64 - bits)) | (1ull << (bits - 1)) | 1;
    if (trial % 16 == 5) q = (1ull << bits) - 1 - 2 * (rng() % 2);
    if (trial % 16 == 7) q = (1ull << (bits - 1)) + 1 + 2 * (rng() % 2);
    if (q < 5) q = 5;
    const MontMod m = constants(q);
    const nttp::Multiplicand f(q, true);
    const uint64_t w = trial % 5 == 0 ? q - 1 : trial % 5 == 1 ? q / 2 + rng() % 2 : rng() % q;
    uint64_t a, b;
    f.put(w, a, b);
    int64_t x = draw(kMontLimit, q);
    if (trial % 7 == 3) {   // digit edges: the low word at either end of its range
      const int64_t e = (int64_t)(((uint64_t)x & ~0xffffffffull) | (trial & 8 ? 0x80000000ull : 0x7fffffffull));
      if (within(e, kMontLimit, q)) x = e;
    }
    const int64_t r = mont_mul(x, a, b, m);
    const i128 ax = x < 0 ? -(i128)x : x;
    check(residue(r, q) == residue((i128)residue(x, q) * (i128)w, q), "product value");
    check(within(r, mont_product_bound((int)(ax * 16 / q + 1)) - (PLANT == 3 ? 9 : 0), q), "product bound");
    const int64_t z = mont_reduce(x, m);
    check(residue(z, q) == residue(x, q) && (i128)z * 8 >= -5 * (i128)q && (i128)z * 8 < 7 * (i128)q, "reduction");
    check((int64_t)mont_canonical(x, m) == residue(x, q), "canonical");
    const int64_t x2 = draw(31, q);
    check((int64_t)mont_canonical_2q(x2, m) == residue(x2, q), "canonical below 2q");
    const int64_t y = trial & 1 ? (int64_t)(rng() % q) : mont_reduce(draw(kMontLimit, q), m);
    const int64_t p = mont_product(z, y, m);
    const int64_t c62 = residue((i128)1 << (PLANT == 4 ? 61 : 62), q);
    check(residue((i128)residue(p, q) * c62, q) == residue((i128)residue(z, q) * residue(y, q), q), "two-value product");
    check(within(p, 16, q), "two-value product bound");
    if (trial % 8 == 0) {
      cooley_tukey<kCtCanon>(q, m, f);
      cooley_tukey<kCtLazy>(q, m, f);
      gentleman_sande<kGsCanon>(q, m, f);
      gentleman_sande<kGsLazy>(q, m, f);
    }
  }
  std::printf("%ld failures\n", failures);
  return failures != 0;
}
