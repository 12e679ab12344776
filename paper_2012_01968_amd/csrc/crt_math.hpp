// Tables of the RNS <-> integer conversion (Section III-B), computed on the host with plain
// multi-precision arithmetic over little-endian 64-bit words.  Host only: no device code,
// so the host test suite compiles it with g++.
//
// For primes q_0 .. q_{L-1} with product Q (W words):
//   inv[l]     = (Q / q_l)^-1 mod q_l
//   M[l]       = Q / q_l, W words
// Reconstruction forms x' = sum_l y_l M_l with y_l = r_l inv[l] mod q_l (so x' < L Q and
// x' = x mod Q) and subtracts the multiple k Q, k = floor(x' / Q).
//
// Both conversions run as products with a constant matrix of base-256 digits (digit_matrix_*
// below), which the kernels take as int8 matrix-instruction operands.
#pragma once
#include <algorithm>
#include <cstdint>
#include <cstring>
#include <vector>

namespace nttc {

typedef unsigned __int128 u128;
constexpr uint32_t kCrtMaxInWords = 64;   // widest integer ntt_rns_decompose accepts

// a *= m (a grows by a word when needed)
inline void mp_mul_small(std::vector<uint64_t>& a, uint64_t m) {
  uint64_t carry = 0;
  for (uint64_t& w : a) {
    const u128 t = (u128)w * m + carry;
    w = (uint64_t)t;
    carry = (uint64_t)(t >> 64);
  }
  if (carry) a.push_back(carry);
}

// quotient of a / d (same length as a), remainder returned
inline uint64_t mp_divmod_small(const std::vector<uint64_t>& a, uint64_t d, std::vector<uint64_t>& quot) {
  quot.assign(a.size(), 0);
  u128 rem = 0;
  for (size_t i = a.size(); i-- > 0;) {
    const u128 cur = (rem << 64) | a[i];
    quot[i] = (uint64_t)(cur / d);
    rem = cur % d;
  }
  return (uint64_t)rem;
}

inline uint64_t mulmod_u128(uint64_t a, uint64_t b, uint64_t q) { return (uint64_t)((u128)a * b % q); }

inline uint64_t powmod_u128(uint64_t b, uint64_t e, uint64_t q) {
  uint64_t r = 1 % q;
  b %= q;
  while (e) {
    if (e & 1) r = mulmod_u128(r, b, q);
    b = mulmod_u128(b, b, q);
    e >>= 1;
  }
  return r;
}

struct CrtBase {
  uint32_t L = 0, W = 0;                 // primes, words of Q
  std::vector<uint64_t> Q;               // W words
  std::vector<uint64_t> inv;             // [L]
  std::vector<uint64_t> M;               // [L][W]
};

inline CrtBase crt_base(const std::vector<uint64_t>& primes) {
  CrtBase t;
  t.L = (uint32_t)primes.size();
  t.Q = {1};
  for (uint64_t q : primes) mp_mul_small(t.Q, q);
  while (t.Q.size() > 1 && t.Q.back() == 0) t.Q.pop_back();
  t.W = (uint32_t)t.Q.size();
  t.inv.assign(t.L, 0);
  t.M.assign((size_t)t.L * t.W, 0);
  std::vector<uint64_t> quot;
  for (uint32_t l = 0; l < t.L; ++l) {
    const uint64_t q = primes[l];
    const uint64_t rem = mp_divmod_small(t.Q, q, quot);
    (void)rem;   // zero: q divides Q
    for (uint32_t w = 0; w < t.W; ++w) t.M[(size_t)l * t.W + w] = quot[w];
    std::vector<uint64_t> tmp;
    const uint64_t m_mod_q = mp_divmod_small(quot, q, tmp);
    t.inv[l] = powmod_u128(m_mod_q, q - 2, q);
  }
  return t;
}

// The same with the word-wise tables of the definitions, which the host check compares it with:
//   pow2[l][w] = 2^(64 w) mod q_l   (w < kCrtMaxInWords)
//   kQ[k]      = k * Q, W + 1 words, k = 0 .. L
struct CrtTables : CrtBase {
  std::vector<uint64_t> pow2;            // [L][kCrtMaxInWords]
  std::vector<uint64_t> kQ;              // [L + 1][W + 1]
};

inline CrtTables crt_tables(const std::vector<uint64_t>& primes) {
  CrtTables t;
  static_cast<CrtBase&>(t) = crt_base(primes);
  t.pow2.assign((size_t)t.L * kCrtMaxInWords, 0);
  t.kQ.assign((size_t)(t.L + 1) * (t.W + 1), 0);
  for (uint32_t l = 0; l < t.L; ++l) {
    const uint64_t q = primes[l], two64 = (uint64_t)(((u128)1 << 64) % q);
    uint64_t c = 1 % q;
    for (uint32_t w = 0; w < kCrtMaxInWords; ++w) {
      t.pow2[(size_t)l * kCrtMaxInWords + w] = c;
      c = mulmod_u128(c, two64, q);
    }
  }
  for (uint32_t k = 0; k <= t.L; ++k) {
    std::vector<uint64_t> kq = t.Q;
    mp_mul_small(kq, k);
    for (uint32_t w = 0; w < t.W + 1 && w < kq.size(); ++w) t.kQ[(size_t)k * (t.W + 1) + w] = kq[w];
  }
  return t;
}

// ------------------------------------------------------------------- digit matrices
//
// A matrix instruction multiplies a 32 x 32 tile of int8 digits (32 rows of the constant matrix,
// a K slice of 32 digits) with 32 digits of 32 coefficients.  Lane (h, m) = (lane / 32, lane % 32)
// of a wave holds 16 digits of the K slice: slots 2h and 2h + 1 of 8 digits each, where slot z
// of slice s is limb (or word) 4 s + z.  The result of row m lands in lane half (m / 4) % 2,
// register (m % 4) + 4 (m / 8); rows are assigned so that half h of the result holds 16
// consecutive entries of the product.
constexpr uint32_t kDigitTile = 64 * 16;   // bytes of one operand tile
constexpr uint32_t tile_row(uint32_t m) { return 16 * ((m >> 2) & 1) + (m & 3) + 4 * (m >> 3); }

// A word's bytes plus kBias are its signed digits plus 128, the carry going on to the next word.
constexpr uint64_t kBias = 0x8080808080808080ull;

// Base-256 digits of an integer in [-128, 127], one digit longer than its bytes.
inline std::vector<int8_t> signed_digits(const uint64_t* a, size_t words) {
  std::vector<int8_t> d(8 * words + 1);
  u128 sum = 0;
  for (size_t w = 0; w < words; ++w) {
    sum = (sum >> 64) + a[w] + kBias;
    const uint64_t digits = (uint64_t)sum ^ kBias;
    std::memcpy(&d[8 * w], &digits, 8);
  }
  d[8 * words] = (int8_t)(sum >> 64);
  return d;
}

// Base-256 digits of the integer's negative, those of the integer then lying in [-127, 128].
inline std::vector<int8_t> negated_digits(const uint64_t* a, size_t words) {
  std::vector<int8_t> d(8 * words + 1);
  int carry = 0;
  for (size_t i = 0; i < d.size(); ++i) {
    int v = (i < 8 * words ? (int)((a[i / 8] >> (8 * (i % 8))) & 255) : 0) + carry;
    carry = v > 128;
    if (carry) v -= 256;
    d[i] = (int8_t)-v;
  }
  return d;
}

// Reconstruction: row b of the product is the base-256 column b of sum_l y_l M_l - k Q, where
// limb l's slot holds the digits of y_l and slot L the digit k.  [tiles][slices] operand tiles.
inline uint32_t reconstruct_tiles(uint32_t W) { return W / 4 + 1; }        // 32 columns each, sign included
inline uint32_t reconstruct_slices(uint32_t L) { return L / 4 + 1; }       // L limbs and k
inline std::vector<int8_t> digit_matrix_reconstruct(const CrtBase& t) {
  const uint32_t T = reconstruct_tiles(t.W), S = reconstruct_slices(t.L);
  std::vector<int8_t> f((size_t)T * S * kDigitTile, 0);
  std::vector<int8_t> d(8 + 32 * (size_t)T, 0);   // the digits above seven zeros and more: d[8 + b], b >= -8
  for (uint32_t l = 0; l <= t.L; ++l) {
    const std::vector<int8_t> v = l < t.L ? signed_digits(&t.M[(size_t)l * t.W], t.W) : negated_digits(t.Q.data(), t.W);
    std::copy(v.begin(), v.end(), d.begin() + 8);   // 8 W + 1 digits, at most 32 T
    const size_t lane0 = 32 * ((l % 4) / 2), slot = 8 * (l % 2);
    for (uint32_t tile = 0; tile < T; ++tile)
      for (uint32_t m = 0; m < 32; ++m) {
        const uint32_t b = 32 * tile + tile_row(m);
        int8_t* out = &f[((size_t)tile * S + l / 4) * kDigitTile + (lane0 + m) * 16 + slot];
        if (l == t.L) {
          *out = d[8 + b];
        } else {   // column b takes digit b - i of M_l at i = 0 .. 7
          uint64_t x;
          std::memcpy(&x, &d[1 + b], 8);
          x = __builtin_bswap64(x);
          std::memcpy(out, &x, 8);
        }
      }
  }
  return f;
}

// Decomposition: entry (l, i) of the product is sum_j u_j d_{j,i}, with d_{j,.} the digits of
// 256^j mod q_l and u_j the integer's bytes less 128.  `offsets` adds the 128s back: for an integer
// of s slices (32 s bytes), [s][l][z] is 128 sum_j d_{j,i} over i = 4 z .. 4 z + 3, weighted by
// 256^(i mod 4).
constexpr uint32_t kDecomposeSlices = kCrtMaxInWords / 4;
struct DecomposeMatrix {
  std::vector<int8_t> digits;      // [ceil(L / 4)][kDecomposeSlices] operand tiles
  std::vector<int64_t> offsets;    // [kDecomposeSlices + 1][L][2]
};
// 8 x 8 bytes: byte i of row j goes to byte j of row i.
inline void transpose_bytes(uint64_t (&x)[8]) {
  for (int s = 4; s; s /= 2) {
    const uint64_t m = s == 4 ? 0x00000000FFFFFFFFull : s == 2 ? 0x0000FFFF0000FFFFull : 0x00FF00FF00FF00FFull;
    for (int j = 0; j < 8; ++j) {
      if (j & s) continue;
      const uint64_t t = ((x[j] >> (8 * s)) ^ x[j + s]) & m;
      x[j + s] ^= t;
      x[j] ^= t << (8 * s);
    }
  }
}

inline DecomposeMatrix digit_matrix_decompose(const std::vector<uint64_t>& primes) {
  const uint32_t L = (uint32_t)primes.size(), T = (L + 3) / 4, S = kDecomposeSlices;
  DecomposeMatrix r;
  r.digits.assign((size_t)T * S * kDigitTile, 0);
  r.offsets.assign((size_t)(S + 1) * L * 2, 0);
  uint32_t row_of[32];   // operand row of each entry of a tile
  for (uint32_t m = 0; m < 32; ++m) row_of[tile_row(m)] = m;
  for (uint32_t l = 0; l < L; ++l) {
    const uint64_t q = primes[l];
    uint64_t k[8], kb[8], c = 1 % q;   // 256^(j + 1) mod q and its companion
    for (int j = 0; j < 8; ++j) {
      k[j] = (uint64_t)((u128)(j ? k[j - 1] : 1) * 256 % q);
      kb[j] = (uint64_t)(((u128)k[j] << 64) / q);
    }
    int64_t acc[2] = {0, 0};
    for (uint32_t w = 0; w < kCrtMaxInWords; ++w) {   // c = 2^(64 w) mod q
      uint64_t d[8], next = 0;   // row j: the digits of 256^(8 w + j) mod q, digit i in byte i
      for (int j = 0; j < 8; ++j) {
        const uint64_t biased = (j ? next : c) + kBias;   // below 2^62 + kBias: eight signed digits hold it
        d[j] = biased ^ kBias;
        acc[0] += 128 * ((int64_t)(uint32_t)biased - 0x80808080);
        acc[1] += 128 * ((int64_t)(biased >> 32) - 0x80808080);
        next = c * k[j] - (uint64_t)(((u128)c * kb[j]) >> 64) * q;
        if (next >= q) next -= q;
      }
      c = next;
      transpose_bytes(d);   // row i: digit i of the word's eight bytes
      int8_t* tile = &r.digits[((size_t)(l / 4) * S + w / 4) * kDigitTile];
      for (uint32_t i = 0; i < 8; ++i)
        std::memcpy(&tile[(32 * ((w % 4) / 2) + row_of[8 * (l % 4) + i]) * 16 + 8 * (w % 2)], &d[i], 8);
      if (w % 4 == 3)
        for (int z = 0; z < 2; ++z) r.offsets[((size_t)(w / 4 + 1) * L + l) * 2 + z] = acc[z];
    }
  }
  return r;
}

}  // namespace nttc
