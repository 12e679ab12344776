// 32-bit words (Section IV's word-size choice taken the other way): primes below 2^30, residues in
// 32-bit words.  The same modulus budget takes twice the limbs of the 64-bit path, at half the
// bytes per residue.
//
// Arithmetic: Montgomery products of signed values.  A fixed multiplicand w is stored as the single
// word A = w 2^32 mod q, centred in [-q/2, q/2]; with P = b A, m = -P q^-1 mod 2^32 (signed),
// (P + m q) / 2^32 = b w mod q exactly, and |b w| <= q/2 + |b| q / 2^33: below 3/4 q for any
// |b| <= 2 q < 2^31.  Two multiply-adds and a low product, as long as Shoup's product on 32-bit
// words, which needs a companion beside w: the tables are half its size, and every pass here is
// bound by its bytes.  Values are signed, so butterflies need no offset; X (Cooley-Tukey) and the
// sums (Gentleman-Sande) are brought back into [-q, q) when a stage's outputs would pass 2 q.
//
// Measured at N = 2^16, 90 primes, 2 polynomials, forward + inverse: 129 us before (one column per lane,
// tables of two words, vectorised neither way, rows not grouped by prime), 96 to 101 us now by box.  Under the
// profiler, which spaces the launches, column passes take 20-21 us (94 MB) and row passes 31 us
// (118 MB, of them 24 MB of twiddles where 47 MB were).  Between
// the byte and the instruction bound (16 us): 1.4 rounds of the chip's wave slots leave little
// overlap between waves.  Product at N = 2^14, 20 primes, 2 polynomials: 44 -> 20 us.
//
// Same two-pass structure as the 64-bit kernels (Section VI-C): a column pass over the first
// log2 N1 stages and a row pass over the rest, registers between LDS exchanges; N <= 2^12 runs in
// one row pass.  Data [n_vec][N] uint32, vector v reduced mod prime v mod L; tables [L][N].
#include "kernels.hpp"
#include "passes.hpp"

namespace nttk {

struct Args32 {
  uint32_t* data;
  const uint32_t* src;     // input of the first forward pass (data unless out of place)
  uint32_t* data2;         // forward column passes of two operands: the second one's output and input
  const uint32_t* src2;
  const uint32_t* other;   // product rows: the second operand
  const int32_t* tw;       // [L][N] of this direction (products: forward)
  const int32_t* twi;      // products: the inverse table
  const int32_t* scale;    // [L][2]: {1/N}, {Psi_inv[1]/N}
  const Prime32* primes;   // [L]
  uint64_t n_vec;
  uint32_t P, L, logN, logN1;
};

__device__ __forceinline__ int32_t mul32(int32_t b, int32_t A, const Prime32& p) {
  const int64_t P = (int64_t)b * A;
  const int32_t m = (int32_t)((uint32_t)P * p.nqi);
  return (int32_t)((uint64_t)(P + (int64_t)m * (int32_t)p.q) >> 32);
}
// [-2q, 2q) -> [-q, q)
__device__ __forceinline__ int32_t reduce32(int32_t x, const Prime32& p) {
  return x - (int32_t)p.q + ((int32_t)(2 * p.q) & (x >> 31));
}
// [-q, q) -> [0, q)
__device__ __forceinline__ int32_t canonical32(int32_t x, const Prime32& p) { return x + ((int32_t)p.q & (x >> 31)); }

typedef __attribute__((address_space(1))) uint32_t gu32;
typedef const __attribute__((address_space(4))) int32_t c32;   // tables: scalar loads where the index is uniform
template <int V>
struct Vec32;
template <> struct Vec32<1> { typedef int32_t type; };
template <> struct Vec32<2> { typedef int32_t type __attribute__((ext_vector_type(2))); };
template <> struct Vec32<4> { typedef int32_t type __attribute__((ext_vector_type(4))); };

// Register steps of an M-point sub-transform with 2^LR values per lane: the first step takes the
// NB0 = LOGM - LR (K - 1) top stages, every other one LR stages.  The first step's window holds the
// NB0 top index bits and the LR - NB0 low ones, so a lane's first loads (and an inverse pass's
// last stores) are vectors of 2^(LR - NB0) consecutive elements.
template <int LOGM, int LR_>
struct Steps32 {
  static constexpr int LR = LR_ < LOGM ? LR_ : LOGM;
  static constexpr int R = 1 << LR;
  static constexpr int K = (LOGM + LR - 1) / LR;
  static constexpr int NB0 = LOGM - LR * (K - 1);
  static constexpr int VEC = 1 << (LR - NB0);   // consecutive elements per lane in step 0
  static constexpr int nb(int k) { return k == 0 ? NB0 : LR; }
  static constexpr int top(int k) { return k == 0 ? LOGM : LOGM - NB0 - LR * (k - 1); }   // stages of bits below top
  static constexpr int lo(int k) { return top(k) - nb(k); }
  // register bit of index bit `bit` during step k
  static constexpr int reg_bit(int k, int bit) { return k == 0 ? bit - lo(0) + (LR - NB0) : bit - lo(k); }
  template <int k>
  __device__ static __forceinline__ uint32_t idx(uint32_t t, uint32_t u) {
    if constexpr (k == 0) {
      constexpr int vb = LR - NB0;
      return ((u >> vb) << lo(0)) | (t << vb) | (u & ((1u << vb) - 1u));
    } else {
      constexpr int l = lo(k);
      return ((t >> l) << (l + LR)) | (u << l) | (t & ((1u << l) - 1u));
    }
  }
};

// The twiddles of step K, one per butterfly block of each stage: stage of register bit i needs
// R >> (i + 1) of them when the step's window is contiguous; step 0 keeps its low window bits
// out of the index, so registers that differ there share one.
template <int LOGM, int LR, int K, int R>
__device__ __forceinline__ void load_twiddles32(int32_t (&w)[R], uint32_t t, uint32_t base, const c32* tab) {
  using S = Steps32<LOGM, LR>;
  constexpr int low = S::reg_bit(K, S::lo(K));   // register bits below the step's stages
  static_for<S::lo(K), S::top(K)>([&](auto bit_c) {
    constexpr int bit = decltype(bit_c)::value, s = LOGM - 1 - bit, i = S::reg_bit(K, bit);
    constexpr int n = R >> (i + 1), off = (R >> low) - (R >> i);
#pragma unroll
    for (int j = 0; j < n; ++j) w[off + j] = tab[(base << s) + (S::template idx<K>(t, (uint32_t)j << (i + 1)) >> (bit + 1))];
  });
}

// Cooley-Tukey step K.  CANON: the sub-transform's input is canonical (its first stage needs no
// reduction); otherwise values lie in [-2q, 2q).
template <int LOGM, int LR, int K, bool CANON, int R>
__device__ __forceinline__ void ct32_step(int32_t (&x)[R], const int32_t (&w)[R], const Prime32& p) {
  using S = Steps32<LOGM, LR>;
  constexpr int low = S::reg_bit(K, S::lo(K));
  static_for_down<S::top(K), S::lo(K)>([&](auto bit_c) {
    constexpr int bit = decltype(bit_c)::value, i = S::reg_bit(K, bit), off = (R >> low) - (R >> i);
#pragma unroll
    for (int u = 0; u < R; ++u) {
      if (u & (1 << i)) continue;
      const int32_t X = CANON && bit == LOGM - 1 ? x[u] : reduce32(x[u], p);
      const int32_t v = mul32(x[u | (1 << i)], w[off + (u >> (i + 1))], p);
      x[u] = X + v;
      x[u | (1 << i)] = X - v;
    }
  });
}

// Gentleman-Sande step K: values in [-q, q].  SCALE0: the step holds stage 0 of the whole
// transform, whose butterfly also applies 1/N.
template <int LOGM, int LR, int K, bool SCALE0, int R>
__device__ __forceinline__ void gs32_step(int32_t (&x)[R], const int32_t (&w)[R], const Prime32& p, int32_t sc0,
                                          int32_t sc1) {
  using S = Steps32<LOGM, LR>;
  constexpr int low = S::reg_bit(K, S::lo(K));
  static_for<S::lo(K), S::top(K)>([&](auto bit_c) {
    constexpr int bit = decltype(bit_c)::value, i = S::reg_bit(K, bit), off = (R >> low) - (R >> i);
#pragma unroll
    for (int u = 0; u < R; ++u) {
      if (u & (1 << i)) continue;
      const int32_t X = x[u], Y = x[u | (1 << i)];
      if constexpr (SCALE0 && bit == LOGM - 1) {
        x[u] = mul32(X + Y, sc0, p);
        x[u | (1 << i)] = mul32(X - Y, sc1, p);
      } else {
        x[u] = reduce32(X + Y, p);
        x[u | (1 << i)] = mul32(X - Y, w[off + (u >> (i + 1))], p);
      }
    }
  });
}

// ------------------------------------------------------------------------------ row pass

constexpr int kLR32 = 4;          // 16 values per lane: 16 VGPRs of data
constexpr int kRowThreads32 = 256;

template <int LOGM>
struct Row32 {
  using S = Steps32<LOGM, kLR32>;
  static constexpr int M = 1 << LOGM;
  static constexpr int T = M / S::R;     // a 1024-point row is one wave: no workgroup barrier
  static constexpr int V = T >= kRowThreads32 ? 1 : kRowThreads32 / T;
  static constexpr int NT = V * T;
  static constexpr int PITCH = M + M / 32;
  static __device__ __forceinline__ uint32_t at(uint32_t r) { return r + (r >> 5); }
};

template <int T>
__device__ __forceinline__ void row_sync32() {
  if constexpr (T <= 64) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// 2^LR elements of a row in step 0's positions, VEC consecutive ones per access.
template <typename C>
__device__ __forceinline__ void load_row32(int32_t (&x)[C::S::R], const uint32_t* row, uint32_t t) {
  typedef typename Vec32<(C::S::VEC > 4 ? 4 : C::S::VEC)>::type vec;
  constexpr int V = C::S::VEC > 4 ? 4 : C::S::VEC;
#pragma unroll
  for (int u = 0; u < C::S::R; u += V) {
    const vec v = *(const __attribute__((address_space(1))) vec*)(row + C::S::template idx<0>(t, u));
#pragma unroll
    for (int j = 0; j < V; ++j) {
      if constexpr (V == 1) x[u] = v;
      else x[u + j] = v[j];
    }
  }
}
template <typename C>
__device__ __forceinline__ void store_row32(const int32_t (&x)[C::S::R], uint32_t* row, uint32_t t) {
  typedef typename Vec32<(C::S::VEC > 4 ? 4 : C::S::VEC)>::type vec;
  constexpr int V = C::S::VEC > 4 ? 4 : C::S::VEC;
#pragma unroll
  for (int u = 0; u < C::S::R; u += V) {
    vec v;
#pragma unroll
    for (int j = 0; j < V; ++j) {
      if constexpr (V == 1) v = x[u];
      else v[j] = x[u + j];
    }
    *(__attribute__((address_space(1))) vec*)(row + C::S::template idx<0>(t, u)) = v;
  }
}

template <typename C, int FROM, int TO>
__device__ __forceinline__ void exchange32(int32_t (&x)[C::S::R], int32_t* l, uint32_t t) {
  using S = typename C::S;
#pragma unroll
  for (int u = 0; u < S::R; ++u) l[C::at(S::template idx<FROM>(t, u))] = x[u];
  row_sync32<C::T>();
#pragma unroll
  for (int u = 0; u < S::R; ++u) x[u] = l[C::at(S::template idx<TO>(t, u))];
  // the next exchange writes the slots that this lane just read
}

enum { kRow32Forward, kRow32Inverse, kRow32Product };

// Rows of M = N / N1 contiguous points, V rows per workgroup.  ONEP: single-pass transform (N1 = 1).
// A product takes the rows of both operands through the forward stages, multiplies them and
// runs the inverse stages (their factor 2^-32 is in the products' scale).
// Tiles are ordered (prime, row group, polynomial), each XCD taking a contiguous range, so a row's
// twiddles come from HBM once for all polynomials.
template <int LOGM, int MODE, bool ONEP>
__global__ __launch_bounds__(Row32<LOGM>::NT) void row32_kernel(Args32 a) {
  using C = Row32<LOGM>;
  using S = typename C::S;
  __shared__ int32_t lds[C::V * C::PITCH];
  const uint32_t tid = threadIdx.x, v = tid / C::T, t = tid % C::T;
  const uint64_t rows = a.n_vec << a.logN1;
  const uint32_t n_tiles = (uint32_t)((rows + C::V - 1) / C::V);
  const uint32_t per = (n_tiles + 7) / 8, tile = (blockIdx.x % 8) * per + blockIdx.x / 8;
  const uint32_t N1 = 1u << a.logN1;
  bool valid;
  uint32_t limb, row;
  uint64_t vec;
  if ((!ONEP && C::V <= 32) || (uint32_t)C::V <= N1) {   // the tile's rows lie in one vector (a split has N1 >= 32)
    valid = tile < n_tiles;
    const uint32_t tl = valid ? tile : 0, lg = a.logN1 - (uint32_t)__builtin_ctz((uint32_t)C::V);
    const uint32_t p = tl % a.P, rest = tl / a.P;
    limb = rest >> lg;
    row = (rest & ((1u << lg) - 1u)) * C::V + v;
    vec = (uint64_t)p * a.L + limb;
  } else {
    const uint64_t g = (uint64_t)tile * C::V + v;
    valid = tile < n_tiles && g < rows;
    vec = valid ? g >> a.logN1 : 0;
    row = (uint32_t)(g & (N1 - 1));
    limb = (uint32_t)vec % a.L;
  }
  // scalars where the lanes of a wave share them: the prime of one vector's rows, and the row itself
  // (its first step's twiddles then come through scalar loads)
  if constexpr ((!ONEP && C::V <= 32) || C::T >= 64) limb = __builtin_amdgcn_readfirstlane(limb);
  if constexpr (C::T >= 64) row = __builtin_amdgcn_readfirstlane(row);
  const Prime32 p = a.primes[limb];
  const c32* tab = (const c32*)a.tw + ((size_t)limb << a.logN);
  const uint32_t base = N1 + row;
  const size_t off = ((size_t)vec << a.logN) + (size_t)row * C::M;
  uint32_t* out = a.data + off;
  int32_t* l = lds + v * C::PITCH;
  int32_t x[S::R], w[S::R];
  if constexpr (MODE != kRow32Inverse) {
    auto forward = [&](const uint32_t* in) {
      load_row32<C>(x, in + off, t);   // padding rows read row 0 and store nothing
      static_for<0, S::K>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        load_twiddles32<LOGM, kLR32, k>(w, t, base, tab);   // before the exchange, which they overlap
        loads_issued();
        if constexpr (k > 0) exchange32<C, (k > 0 ? k - 1 : 0), k>(x, l, t);
        ct32_step<LOGM, kLR32, k, ONEP>(x, w, p);
      });
    };
    if constexpr (MODE == kRow32Forward) {
      forward(a.src);
#pragma unroll
      for (int u = 0; u < S::R; ++u) x[u] = canonical32(reduce32(x[u], p), p);
      if constexpr (S::K > 1) exchange32<C, S::K - 1, 0>(x, l, t);   // so that stores cover whole lines
      if (valid) store_row32<C>(x, out, t);
      return;
    } else {
      int32_t y[S::R];
      forward(a.other);
#pragma unroll
      for (int u = 0; u < S::R; ++u) y[u] = x[u];
      // the second operand's first exchange writes step 0's slots, which other lanes may still read
      if constexpr (S::K > 1) row_sync32<C::T>();
      forward(a.src);
#pragma unroll
      for (int u = 0; u < S::R; ++u) x[u] = mul32(reduce32(x[u], p), reduce32(y[u], p), p);
      tab = (const c32*)a.twi + ((size_t)limb << a.logN);
    }
  } else {
    const gu32* in = (const gu32*)(out) + S::template idx<S::K - 1>(t, 0);
    if constexpr (S::R % 4 == 0 && S::K > 1) {   // the last step's 2^LR elements are consecutive
      typedef Vec32<4>::type vec4;
#pragma unroll
      for (int u = 0; u < S::R; u += 4) {
        const vec4 q4 = *(const __attribute__((address_space(1))) vec4*)(in + u);
#pragma unroll
        for (int j = 0; j < 4; ++j) x[u + j] = q4[j];
      }
    } else {
      load_row32<C>(x, out, t);
    }
  }
  if constexpr (MODE != kRow32Forward) {
    int32_t sc0 = 0, sc1 = 0;
    if constexpr (ONEP) {
      sc0 = a.scale[2 * limb];
      sc1 = a.scale[2 * limb + 1];
    }
    static_for_down<S::K, 0>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      load_twiddles32<LOGM, kLR32, k>(w, t, base, tab);
      loads_issued();
      if constexpr (k < S::K - 1) exchange32<C, k + 1, k>(x, l, t);
      gs32_step<LOGM, kLR32, k, ONEP>(x, w, p, sc0, sc1);
    });
    if constexpr (ONEP) {
#pragma unroll
      for (int u = 0; u < S::R; ++u) x[u] = canonical32(x[u], p);
    }
    if (valid) store_row32<C>(x, out, t);
  }
}

// --------------------------------------------------------------------------- column pass
// W adjacent columns of one vector per workgroup, two adjacent columns and 8 rows per lane (8-byte
// accesses, row runs of 4 W bytes); the first N1 twiddles in LDS.

template <int LOGM, int WREQ>
struct Col32 {
  using S = Steps<LOGM, 3>;
  static constexpr int M = 1 << LOGM;
  static constexpr int T = M / S::R;
  // at most 512 lanes and 32 KB of exchange buffer
  static constexpr int W = WREQ * M > 8192 ? 8192 / M : WREQ;
  static constexpr int NT = W / 2 * T;
};
// The widest tile that N2 holds: 512 bytes and more per row run up to 64-point columns.
template <int LOGM>
constexpr int col32_wide() { return 8192 >> LOGM; }

typedef Vec32<2>::type i32x2;
typedef __attribute__((address_space(1))) i32x2 gi32x2;

template <int LOGM, bool INV, int WREQ>
__global__ __launch_bounds__((Col32<LOGM, WREQ>::NT)) void col32_kernel(Args32 a) {
  using C = Col32<LOGM, WREQ>;
  using S = typename C::S;
  __shared__ i32x2 lds[C::M * (C::W / 2)];
  __shared__ int32_t twl[C::M];
  const uint32_t tid = threadIdx.x, c = tid % (C::W / 2), t = tid / (C::W / 2);
  const uint32_t logN2 = a.logN - LOGM;
  const uint32_t groups = (1u << logN2) / C::W;
  const uint32_t n_tiles = (uint32_t)(a.n_vec * groups);
  const uint32_t per = (n_tiles + 7) / 8, tile = (blockIdx.x % 8) * per + blockIdx.x / 8;
  if (tile >= n_tiles) return;   // uniform per workgroup
  const uint32_t lp = tile / groups, cg = tile % groups;   // (prime, polynomial) order
  uint32_t poly = lp % a.P;
  const uint32_t limb = lp / a.P;
  uint32_t* data = a.data;
  const uint32_t* src = INV ? a.data : a.src;
  if (!INV && a.data2 && poly >= a.P / 2) {   // the second operand's polynomials follow the first's
    poly -= a.P / 2;
    data = a.data2;
    src = a.src2;
  }
  const Prime32 p = a.primes[limb];
  const int32_t* tab = a.tw + ((size_t)limb << a.logN);
  const size_t off = (((size_t)poly * a.L + limb) << a.logN) + (size_t)cg * C::W + 2 * c;
  const gi32x2* in = (const gi32x2*)(src + off);
  gi32x2* out = (gi32x2*)(data + off);
  const uint32_t step = logN2 - 1;   // log2 of a row's distance in pairs
  int32_t x[2][S::R];
  constexpr int first = INV ? S::K - 1 : 0, last = INV ? 0 : S::K - 1;
#pragma unroll
  for (int u = 0; u < S::R; ++u) {
    const i32x2 v = in[(size_t)S::template idx<first>(t, u) << step];
    x[0][u] = v.x;
    x[1][u] = v.y;
  }
  for (uint32_t i = tid; i < (uint32_t)C::M; i += C::NT) twl[i] = tab[i];
  __syncthreads();
  auto exchange = [&](auto from, auto to) {
#pragma unroll
    for (int u = 0; u < S::R; ++u)
      lds[S::template idx<decltype(from)::value>(t, u) * (C::W / 2) + c] = i32x2{x[0][u], x[1][u]};
    __syncthreads();
#pragma unroll
    for (int u = 0; u < S::R; ++u) {
      const i32x2 v = lds[S::template idx<decltype(to)::value>(t, u) * (C::W / 2) + c];
      x[0][u] = v.x;
      x[1][u] = v.y;
    }
  };
  // twiddle of register u's butterfly in the stage of index bit `bit`
  auto tw = [&](auto kc, uint32_t u, int bit) {
    const uint32_t r = S::template idx<decltype(kc)::value>(t, u);
    return twl[(1u << (LOGM - 1 - bit)) + (r >> (bit + 1))];
  };
  if constexpr (!INV) {
    static_for<0, S::K>([&](auto kc) {
      constexpr int k = decltype(kc)::value, lo = S::blo(k);
      if constexpr (k > 0) exchange(std::integral_constant<int, (k > 0 ? k - 1 : 0)>{}, kc);
      static_for_down<lo + S::nb(k), lo>([&](auto bit_c) {
        constexpr int bit = decltype(bit_c)::value, i = bit - lo;
#pragma unroll
        for (int u = 0; u < S::R; ++u) {
          if (u & (1 << i)) continue;
          const int32_t w = tw(kc, u, bit);
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int32_t X = bit == LOGM - 1 ? x[j][u] : reduce32(x[j][u], p);   // the first stage's input is canonical
            const int32_t v = mul32(x[j][u | (1 << i)], w, p);
            x[j][u] = X + v;
            x[j][u | (1 << i)] = X - v;
          }
        }
      });
    });
  } else {
    const int32_t sc0 = a.scale[2 * limb], sc1 = a.scale[2 * limb + 1];
    static_for_down<S::K, 0>([&](auto kc) {
      constexpr int k = decltype(kc)::value, lo = S::blo(k);
      if constexpr (k < S::K - 1) exchange(std::integral_constant<int, k + 1>{}, kc);
      static_for<lo, lo + S::nb(k)>([&](auto bit_c) {
        constexpr int bit = decltype(bit_c)::value, i = bit - lo;
#pragma unroll
        for (int u = 0; u < S::R; ++u) {
          if (u & (1 << i)) continue;
          int32_t w = 0;
          if constexpr (bit != LOGM - 1) w = tw(kc, u, bit);
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int32_t X = x[j][u], Y = x[j][u | (1 << i)];
            if constexpr (bit == LOGM - 1) {   // stage 0 of the whole transform
              x[j][u] = canonical32(mul32(X + Y, sc0, p), p);
              x[j][u | (1 << i)] = canonical32(mul32(X - Y, sc1, p), p);
            } else {
              x[j][u] = reduce32(X + Y, p);
              x[j][u | (1 << i)] = mul32(X - Y, w, p);
            }
          }
        }
      });
    });
  }
#pragma unroll
  for (int u = 0; u < S::R; ++u) out[(size_t)S::template idx<last>(t, u) << step] = i32x2{x[0][u], x[1][u]};
}

// ------------------------------------------------------------------------------ launchers

template <int LOGM, int MODE>
static hipError_t go_row32(const Args32& a, hipStream_t st) {
  using C = Row32<LOGM>;
  const uint64_t rows = a.n_vec << a.logN1;
  const dim3 grid((uint32_t)(((rows + C::V - 1) / C::V + 7) / 8 * 8));
  if (a.logN1 == 0) hipLaunchKernelGGL((row32_kernel<LOGM, MODE, true>), grid, dim3(C::NT), 0, st, a);
  else if constexpr (LOGM >= 5) hipLaunchKernelGGL((row32_kernel<LOGM, MODE, false>), grid, dim3(C::NT), 0, st, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

template <int LOGM, bool INV, int W>
static hipError_t launch_col32(const Args32& a, hipStream_t st) {
  using C = Col32<LOGM, W>;
  const uint64_t tiles = a.n_vec * ((1u << (a.logN - LOGM)) / C::W);
  hipLaunchKernelGGL((col32_kernel<LOGM, INV, W>), dim3((uint32_t)((tiles + 7) / 8 * 8)), dim3(C::NT), 0, st, a);
  return hipGetLastError();
}

// 32 columns where N2 holds no more, and up to 2^21 residues, where the wide tile leaves most CUs without
// a workgroup.
// Forward / inverse at 32 and at 8192 / N1 columns, us: 1 vector of 2^13 7.1 / 6.8 and 8.0 / 7.9, 6 of
// 2^14 7.5 / 7.3 and 8.3 / 8.5, 16 of 2^15 7.5 / 7.3 and 8.6 / 8.6, 16 of 2^17 12.4 / 12.3 and 13.1 / 12.8; but forward and
// inverse of 90 x 2 of 2^16, inputs from HBM, 98.8 and 96.0.
constexpr uint64_t kNarrowCols = 1u << 21;
template <int LOGM, bool INV>
static hipError_t go_col32(const Args32& a, hipStream_t st) {
  constexpr int wide = col32_wide<LOGM>();
  if constexpr (wide > 32)
    if ((1u << (a.logN - LOGM)) < (uint32_t)wide || (a.n_vec << a.logN) <= kNarrowCols)
      return launch_col32<LOGM, INV, 32>(a, st);
  return launch_col32<LOGM, INV, wide>(a, st);
}

template <int MODE>
static hipError_t row32(const Args32& a, hipStream_t st) {
  switch (a.logN - a.logN1) {
#define X(LM) \
  case LM:    \
    return go_row32<LM, MODE>(a, st);
    X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12)
#undef X
  }
  return hipErrorInvalidValue;
}

template <bool INV>
static hipError_t col32(const Args32& a, hipStream_t st) {
  switch (a.logN1) {
#define X(LM) \
  case LM:    \
    return go_col32<LM, INV>(a, st);
    X(5) X(6) X(7) X(8) X(9) X(10)
#undef X
  }
  return hipErrorInvalidValue;
}

// Split N = N1 x N2 with columns of 2^5 .. 2^10 points and rows of 2^5 .. 2^12 points (the
// column tile needs N2 >= 32), or one row pass (N1 = 1) for N <= 2^12.
bool shape32_supported(uint32_t logN, uint32_t logN1) {
  if (logN < 1 || logN > 17) return false;
  if (logN1 == 0) return logN <= 12;
  const uint32_t logN2 = logN - logN1;
  return logN1 >= 5 && logN1 <= 10 && logN2 >= 5 && logN2 <= 12;
}

static Args32 args32(const Plan32& p, uint32_t* data, const uint32_t* src, uint32_t n_polys, bool inverse) {
  Args32 a{};
  a.data = data;
  a.src = src;
  a.tw = inverse ? p.tw_inv : p.tw_fwd;
  a.twi = p.tw_inv;
  a.scale = p.scale;
  a.primes = p.primes;
  a.n_vec = (uint64_t)n_polys * p.L;
  a.P = n_polys;
  a.L = p.L;
  a.logN = p.logN;
  a.logN1 = p.logN1;
  return a;
}

hipError_t launch_transform32(const Plan32& p, uint32_t* data, uint32_t n_polys, bool inverse, hipStream_t st) {
  if (!shape32_supported(p.logN, p.logN1)) return hipErrorInvalidValue;
  const Args32 a = args32(p, data, data, n_polys, inverse);
  hipError_t e;
  if (!inverse) {
    if (p.logN1 && (e = col32<false>(a, st)) != hipSuccess) return e;
    return row32<kRow32Forward>(a, st);
  }
  if ((e = row32<kRow32Inverse>(a, st)) != hipSuccess) return e;
  return p.logN1 ? col32<true>(a, st) : hipSuccess;
}

hipError_t launch_product32(const Plan32& p, const uint32_t* a, const uint32_t* b, uint32_t* c, uint32_t n_polys,
                            uint32_t* tmp, hipStream_t st) {
  if (!shape32_supported(p.logN, p.logN1)) return hipErrorInvalidValue;
  hipError_t e;
  Args32 rows = args32(p, c, a, n_polys, false);
  rows.scale = p.scale_mul;
  rows.other = b;
  if (p.logN1) {
    Args32 cols = rows;
    cols.data2 = tmp;
    cols.src2 = b;
    cols.n_vec *= 2;
    cols.P *= 2;
    if ((e = col32<false>(cols, st)) != hipSuccess) return e;
    rows.src = c;
    rows.other = tmp;
  }
  if ((e = row32<kRow32Product>(rows, st)) != hipSuccess || !p.logN1) return e;
  Args32 inv = args32(p, c, c, n_polys, true);
  inv.scale = p.scale_mul;
  return col32<true>(inv, st);
}

// c = a * b mod q_l element-wise over [n_vec][N] uint32 (64-bit product, Barrett with
// mu = floor(2^64 / q): the estimate undershoots by at most 1).
__global__ __launch_bounds__(256) void pointwise32_kernel(const uint32_t* __restrict__ A, const uint32_t* __restrict__ B,
                                                          uint32_t* __restrict__ Cc, const uint32_t* __restrict__ qs,
                                                          const uint64_t* __restrict__ mus, uint64_t n,
                                                          uint32_t logN, uint32_t L) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t limb = (uint32_t)(i >> logN) % L;   // fewer than 2^31 vectors
    const uint32_t q = qs[limb];
    const uint64_t x = (uint64_t)A[i] * B[i];
    const uint64_t r = x - __umul64hi(x, mus[limb]) * q;
    const uint32_t r32 = (uint32_t)r;
    Cc[i] = r32 >= q ? r32 - q : r32;
  }
}

hipError_t launch_pointwise32(const uint32_t* A, const uint32_t* B, uint32_t* Cc, const uint32_t* qs,
                              const uint64_t* mus, uint64_t n, uint32_t logN, uint32_t L, hipStream_t st) {
  if (n == 0) return hipSuccess;
  uint64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(pointwise32_kernel, dim3((uint32_t)blocks), dim3(256), 0, st, A, B, Cc, qs, mus, n, logN, L);
  return hipGetLastError();
}

}  // namespace nttk
