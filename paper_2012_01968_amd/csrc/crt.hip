// RNS <-> integer conversion on either side of the transform (Section III-B): an integer
// coefficient below Q = q_0 ... q_{L-1} is held as its L residues.  Integers are stored as
// little-endian 64-bit words, word-major: word w of coefficient c of polynomial p sits at
// (p*W + w)*N + c, so the lanes of a wave (consecutive coefficients) read consecutive words.
//
// Both directions are products of a constant matrix with every coefficient's vector of base-256
// digits (decomposition: the digits of 256^j mod q_l; reconstruction: the digits of Q / q_l, one
// row per base-256 column of the result), so they run on the int8 matrix cores with exact int32
// sums: at most 513 digit products of at most 2^14, below 2^24.  The tables come from
// crt_math.hpp (host), laid out as the instruction's operands.
//
// A workgroup of four or eight waves takes 128 or 256 coefficients, 32 per wave (64 per wave need 172 VGPRs,
// two waves per SIMD, at 45 primes: decomposition 42 us instead of 38).  The
// coefficients' digits stay in registers for the whole kernel, their loads issued together, and the
// constant matrix streams through LDS one 32-row tile at a time, loaded while the previous tile
// is multiplied, so each workgroup reads the matrix (132 KB at 45 primes) once from L2.
#include "kernels.hpp"
#include "passes.hpp"

namespace nttk {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int cvt_coeffs(int nth) { return nth / 64 * 32; }   // coefficients per workgroup
constexpr uint64_t kDigitBias = 0x8080808080808080ull;

// b * w mod q in [0, 2q) for any b < 2^64, q < 2^62 (Shoup with the exact quotient).
__device__ __forceinline__ uint64_t shoup_exact(uint64_t b, uint64_t w, uint64_t wb, uint64_t q) {
  return b * w - __umul64hi(b, wb) * q;
}

__device__ __forceinline__ v4i digits16(uint64_t a, uint64_t b) {
  return v4i{(int)(uint32_t)a, (int)(uint32_t)(a >> 32), (int)(uint32_t)b, (int)(uint32_t)(b >> 32)};
}

// The values of the lanes (h, m) of the wave, h = lane / 32, seen from both halves.
struct Halves {
  uint32_t lo, hi;   // of lane (0, m) and of lane (1, m)
};
__device__ __forceinline__ Halves halves(uint32_t x) {
  const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return Halves{r[0], r[1]};
}

// Streams the matrix tiles [T][S][64 lanes][16 digits] through two LDS buffers: `body(t, lds)` runs
// with tile t's S slices in `lds`.  Every wave of the workgroup takes part in every tile.
template <int KS, int NTH, typename F>
__device__ __forceinline__ void for_matrix_tiles(const v4i* __restrict__ frag, uint32_t stride, uint32_t T, uint32_t S,
                                                 v4i (&lds)[2][KS * 64], F&& body) {
  constexpr int PER = (KS * 64 + NTH - 1) / NTH;
  const uint32_t tid = threadIdx.x, n = S * 64;
  v4i next[PER];
  auto fetch = [&](uint32_t t) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const uint32_t e = tid + i * NTH;
      if (e < n) next[i] = frag[(size_t)t * stride * 64 + e];
    }
  };
  auto put = [&](v4i* dst) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const uint32_t e = tid + i * NTH;
      if (e < n) dst[e] = next[i];
    }
  };
  fetch(0);
  put(lds[0]);
  __syncthreads();
  for (uint32_t t = 0; t < T; ++t) {
    if (t + 1 < T) fetch(t + 1);
    body(t, lds[t & 1]);
    if (t + 1 < T) put(lds[(t + 1) & 1]);   // last read before the previous barrier
    __syncthreads();
  }
}

// One tile's products: acc = tile (32 rows) x digits of the wave's 32 coefficients.
template <int KS>
__device__ __forceinline__ void tile_product(v16i& acc, const v4i* tile, const v4i (&b)[KS], uint32_t S, uint32_t lane) {
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0;
#pragma unroll
  for (int s = 0; s < KS; ++s)
    if ((uint32_t)s < S) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(tile[s * 64 + lane], b[s], acc, 0, 0, 0);
}

// c0 + 2^8 c1 + 2^16 c2 + 2^24 c3 + add over four int32 columns.
template <int R>
__device__ __forceinline__ int64_t columns4(const v16i& c, int64_t add) {
  return add + (int64_t)c[R] + (int64_t)c[R + 1] * (1 << 8) + (int64_t)c[R + 2] * (1 << 16) +
         (int64_t)c[R + 3] * (1 << 24);
}

// Integers of one word: a lane per residue and one exact product by floor(2^64 / q), which falls short of
// x / q by less than 2.  Bound by its bytes; the digit matrices take a whole K slice for the word and
// a fixed chain per tile (2^14 coefficients at 45 primes 3.7 us here, 12.0 there; 2^17 at 60 17.8 and 20.4).
__global__ __launch_bounds__(256) void rns_decompose_word_kernel(const uint64_t* __restrict__ words,
                                                                 uint64_t* __restrict__ res, uint64_t n_coeffs,
                                                                 uint32_t logN, uint32_t L,
                                                                 const DecomposePrime* __restrict__ primes) {
  const uint64_t j = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  const uint32_t l = blockIdx.y;
  if (j >= n_coeffs) return;
  const uint64_t q = primes[l].q, x = words[j];
  res[((((j >> logN) * L + l) << logN) | (j & ((1ull << logN) - 1)))] = csub(x - __umul64hi(x, primes[l].recip) * q, q);
}

// Residue l of an integer x: V = sum_j byte_j (256^j mod q_l), below 2^17 q_l, then one reduction.
// The bytes enter as signed digits less 128, `offsets` adds the 128s back.  With s = bitlen(q_l),
// t = floor(V / 2^(s-15)) < 2^32 and mu = floor(2^(s+31) / q_l) < 2^32, the estimate
// floor(t mu / 2^46) of V / q_l falls short by less than 1 + 2^-13, so V - est q_l < 2 q_l.
// 2 x 2^16 coefficients at 45 primes of 60 bits: 32 to 34 us by box (2.7 TB/s of words and residues; 132 matrix
// instructions per 32 coefficients are 7 us of it), against 201 us for one exact Shoup product per
// word and prime.  Bound by the loads of a wave's digits, which nothing of the same wave overlaps.
template <int KS, int NTH, bool PARTS>
__global__ __launch_bounds__(NTH) void rns_decompose_kernel(
    const uint64_t* __restrict__ words, uint32_t W, uint64_t* __restrict__ res, uint64_t n_coeffs, uint32_t logN,
    uint32_t L, const v4i* __restrict__ frag, uint32_t stride, const DecomposePrime* __restrict__ primes,
    const int64_t* __restrict__ offsets, uint32_t all_wide, uint32_t tiles_per) {
  __shared__ v4i lds[2][KS * 64];
  const uint32_t lane = threadIdx.x & 63, h = lane >> 5, S = (W + 3) / 4;
  const uint64_t N = 1ull << logN;
  const uint64_t j0 = (uint64_t)blockIdx.x * cvt_coeffs(NTH) + (threadIdx.x >> 6) * 32 + (lane & 31);
  const uint64_t j = j0 < n_coeffs ? j0 : n_coeffs - 1;   // past the end: read, never stored
  const uint64_t p = j >> logN, c = j & (N - 1);
  const uint64_t* x = words + p * W * N + c;
  uint64_t* out = res + p * L * N + c;
  v4i b[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    const uint32_t w = 4 * s + 2 * h;
    const uint64_t a0 = w < W ? x[(size_t)w * N] : 0, a1 = w + 1 < W ? x[(size_t)(w + 1) * N] : 0;
    b[s] = digits16(a0, a1);
  }
  loads_issued();
#pragma unroll
  for (int s = 0; s < KS; ++s) b[s] ^= (int)0x80808080;
  // the tiles of this workgroup (decompose_parts)
  const uint32_t T = (L + 3) / 4, t0 = PARTS ? blockIdx.y * tiles_per : 0;
  const uint32_t tiles = PARTS && T - t0 > tiles_per ? tiles_per : T - t0;
  for_matrix_tiles<KS, NTH>(frag + (size_t)t0 * stride * 64, stride, tiles, S, lds, [&](uint32_t t, const v4i* tile) {
    const uint32_t l0 = 4 * (t0 + t) + 2 * h;
    v16i acc;
    tile_product<KS>(acc, tile, b, S, lane);
    static_for<0, 2>([&](auto uc) {
      constexpr int u = decltype(uc)::value;
      const uint32_t l = l0 + u;
      if (l < L) {
        const DecomposePrime pr = primes[l];
        const int64_t o0 = offsets[2 * l], o1 = offsets[2 * l + 1];
        const int64_t v0 = columns4<8 * u>(acc, o0), v1 = columns4<8 * u + 4>(acc, o1);
        const uint64_t hi = (uint64_t)(v1 + (v0 >> 32));               // V >> 32 (V >= 0)
        const uint64_t low = (hi << 32) | (uint32_t)v0;                // V mod 2^64
        const int32_t high_shift = pr.shift - 32;
        uint32_t q15;
        if (all_wide) q15 = (uint32_t)(hi >> high_shift);
        else if (pr.shift >= 32) q15 = (uint32_t)(hi >> high_shift);
        else q15 = (uint32_t)(pr.shift >= 0 ? low >> pr.shift : low << -pr.shift);   // here V < 2^64
        const uint32_t k = __umulhi(q15, pr.mu) >> 14;
        const uint64_t r = csub(low - (uint64_t)k * pr.q, pr.q);
        if (j0 < n_coeffs) out[(size_t)l * N] = r;
      }
    });
  });
}

// x = sum_l y_l M_l - k Q with y_l = r_l inv_l mod q_l and k = floor(sum_l y_l / q_l).  k comes
// from 2^56-scaled reciprocals: each term falls short by less than 1.25 units, so the sum plus 2^10
// units gives k, or k + 1 when x lies within 2^-45 Q of Q; then x - Q < 0 shows in the sign of
// the result and Q is added back.  Each lane half holds 16 consecutive base-256 columns of a
// tile, carries them into four 32-bit words and passes its carry on (half 0 to half 1, half 1 to
// half 0 of the next tile).  2 x 2^16 coefficients at 45 primes of 60 bits: 35 to 38 us by box, against 576 us for
// 64-bit products with a carry chain per product (93.6 M products of 64 x 64 bits at one wave per
// SIMD) and a search for k; the same 132 matrix instructions as the decomposition.
template <int KS, int NTH>
__global__ __launch_bounds__(NTH) void crt_reconstruct_kernel(
    const uint64_t* __restrict__ res, uint64_t* __restrict__ out, uint64_t n_coeffs, uint32_t logN, uint32_t L,
    uint32_t W, const v4i* __restrict__ frag, const ReconstructPrime* __restrict__ primes,
    const uint64_t* __restrict__ Q) {
  __shared__ v4i lds[2][KS * 64];
  __shared__ ReconstructPrime pl[4 * KS];   // the primes' constants: a wave meets them one by one
  const uint32_t lane = threadIdx.x & 63, h = lane >> 5, S = L / 4 + 1, T = W / 4 + 1;
  const uint64_t N = 1ull << logN;
  const uint64_t j0 = (uint64_t)blockIdx.x * cvt_coeffs(NTH) + (threadIdx.x >> 6) * 32 + (lane & 31);
  const uint64_t j = j0 < n_coeffs ? j0 : n_coeffs - 1;   // past the end: read, never stored
  const uint64_t p = j >> logN, c = j & (N - 1);
  const uint64_t* in = res + p * L * N + c;
  uint64_t* o = out + p * W * N + c;
  uint64_t frac = 0, r[KS][2];
  v4i b[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const uint32_t l = 4 * s + 2 * h + u;
      r[s][u] = l < L ? in[(size_t)l * N] : 0;
    }
  loads_issued();
  if (threadIdx.x < L) pl[threadIdx.x] = primes[threadIdx.x];
  __syncthreads();
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    uint64_t y[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const uint32_t l = 4 * s + 2 * h + u;
      y[u] = 0;
      if (l < L) {
        const ReconstructPrime pr = pl[l];
        const uint32_t sh = __clzll(pr.q) - 2;
        y[u] = csub(shoup_exact(r[s][u], pr.inv, pr.inv_b, pr.q), pr.q);
        frac += __umul64hi(y[u] << sh, pr.rec);
      }
    }
    b[s] = digits16((y[0] + kDigitBias) ^ kDigitBias, (y[1] + kDigitBias) ^ kDigitBias);
  }
  {
    const Halves f0 = halves((uint32_t)frac), f1 = halves((uint32_t)(frac >> 32));
    const uint64_t f = make_u64(f0.lo, f1.lo) + make_u64(f0.hi, f1.hi) + 1024;
    const int k = (int)(f >> 56);   // at most L <= 64: one digit
#pragma unroll
    for (int s = 0; s < KS; ++s)
      if ((uint32_t)s == L / 4 && (L % 4) / 2 == h) b[s][L % 2 ? 2 : 0] = k;
  }
  uint32_t carry = 0, negative = 0;   // carry: out of the previous tile (signed)
  for_matrix_tiles<KS, NTH>(frag, S, T, S, lds, [&](uint32_t t, const v4i* tile) {
    v16i acc;
    tile_product<KS>(acc, tile, b, S, lane);
    const int64_t t0 = columns4<0>(acc, h ? 0 : (int32_t)carry);
    const int64_t t1 = columns4<4>(acc, t0 >> 32);
    const int64_t t2 = columns4<8>(acc, t1 >> 32);
    const int64_t t3 = columns4<12>(acc, t2 >> 32);
    int32_t over = (int32_t)(t3 >> 32);
    const uint64_t lo = make_u64((uint32_t)t0, (uint32_t)t1), hi = make_u64((uint32_t)t2, (uint32_t)t3);
    // half 1 takes half 0's carry: a sign-extended sum over both words and `over`
    const Halves below = halves((uint32_t)over);   // outside the conditional: both halves take part
    const int64_t cin = h ? (int32_t)below.lo : 0, sx = cin >> 63;
    const uint64_t lo2 = lo + (uint64_t)cin, c0 = lo2 < lo;
    const uint64_t hi1 = hi + (uint64_t)sx, hi2 = hi1 + c0;
    over += (int32_t)sx + (int32_t)(hi1 < hi) + (int32_t)(hi2 < c0);
    carry = halves((uint32_t)over).hi;
    negative = halves((uint32_t)(hi2 >> 32)).hi >> 31;
    const uint32_t w = 4 * t + 2 * h;
    if (j0 < n_coeffs) {
      if (w < W) o[(size_t)w * N] = lo2;
      if (w + 1 < W) o[(size_t)(w + 1) * N] = hi2;
    }
  });
  // x - Q came out for a lane of the wave: add Q back to the stored words, one lane per coefficient
  const bool fix = negative && j0 < n_coeffs;
  if (__any(fix)) {
    __threadfence_block();   // the words that the other half's lanes stored
    if (fix && h == 0) {
      uint64_t cy = 0;
      for (uint32_t w = 0; w < W; ++w) {
        const uint64_t a = o[(size_t)w * N], s = a + Q[w], r1 = s + cy;
        cy = (uint64_t)(s < a) | (uint64_t)(r1 < s);
        o[(size_t)w * N] = r1;
      }
    }
  }
}

// Slices of a launch rounded up to a built kernel: KS slices of digits stay in registers (4 VGPRs
// each), so a short chain does not pay for a long one's registers.
#define NTTK_CVT_CASES(X) X(2) X(4) X(8) X(12) X(17)

// f(lanes of a workgroup) for a launch over n coefficients: 512 where that still gives every CU one,
// since each workgroup reads the whole matrix.  256 / 512 lanes, us: 2^16 coefficients at 45 primes
// decomposition 25.0 / 24.0, reconstruction 26.9 / 25.3; 2^17 33.3 / 32.2 and 39.0 / 36.6; 2^18 at 30
// primes 48.6 / 47.9 and 50.5 / 47.9; but 2^15 at 24 primes (128 workgroups) 9.7 / 9.5 and
// 10.3 / 11.0.
constexpr uint64_t kWideCvt = 1u << 16;
template <typename F>
static hipError_t with_cvt_threads(uint64_t n, F&& f) {
  return n >= kWideCvt ? f(std::integral_constant<int, 512>{}) : f(std::integral_constant<int, 256>{});
}
static uint32_t cvt_blocks(uint64_t n, int nth) {
  return (uint32_t)((n + cvt_coeffs(nth) - 1) / cvt_coeffs(nth));
}

// Workgroups over the tiles of one decomposition launch of `blocks` workgroups over the coefficients: a
// wave takes its tiles one after the other, so a small launch waits for that chain, and parts of it in
// workgroups of their own cost only the digits read again.  Every part reads all digits, so wide
// integers (more than 3 slices, 12 words) take fewer.  us, one part and the parts taken here: 2^12
// coefficients of 42 words at 45 primes 17.6 / 5.5, of 4 words at 60 14.4 / 4.1; 2^14 of 56 words at 60 25.8 /
// 11.3, of 12 words 16.7 / 5.9; 2^16 of 42 words at 45 21.2 / 18.0, of 4 words 12.7 / 9.3; 2^17 of 42 words (one
// part) 31.6 against 37.2 with two.
static uint32_t decompose_parts(uint32_t blocks, uint32_t tiles, uint32_t slices) {
  const uint32_t parts = (slices <= 3 ? 1024u : 512u) / blocks;
  return parts < 1 ? 1 : parts < tiles ? parts : tiles;
}

hipError_t launch_rns_decompose(const uint64_t* words, uint32_t W, uint64_t* res, uint32_t n_polys, uint32_t logN,
                                uint32_t L, const void* frag, uint32_t frag_slices, const DecomposePrime* primes,
                                const int64_t* offsets, bool all_wide, hipStream_t st) {
  const uint64_t n = (uint64_t)n_polys << logN;
  const uint32_t S = (W + 3) / 4, T = (L + 3) / 4;
  if (W == 0 || S > frag_slices) return hipErrorInvalidValue;
  if (W == 1 && L <= 65535) {   // primes along the grid's second dimension
    hipLaunchKernelGGL(rns_decompose_word_kernel, dim3((uint32_t)((n + 255) / 256), L), dim3(256), 0, st, words, res, n,
                       logN, L, primes);
    return hipGetLastError();
  }
  return with_cvt_threads(n, [&](auto nth) {
    constexpr int NTH = decltype(nth)::value;
    const uint32_t blocks = cvt_blocks(n, NTH), parts = decompose_parts(blocks, T, S), per = (T + parts - 1) / parts;
    const dim3 grid(blocks, (T + per - 1) / per);
    auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, grid, dim3(NTH), 0, st, words, W, res, n, logN, L, static_cast<const v4i*>(frag),
                         frag_slices, primes, offsets + (size_t)S * L * 2, (uint32_t)all_wide, per);
      return hipGetLastError();
    };
#define X(KS) \
    if (S <= KS) return per < T ? launch(rns_decompose_kernel<KS, NTH, true>) : launch(rns_decompose_kernel<KS, NTH, false>);
    NTTK_CVT_CASES(X)
#undef X
    return hipErrorInvalidValue;
  });
}

hipError_t launch_crt_reconstruct(const uint64_t* res, uint64_t* out, uint32_t n_polys, uint32_t logN, uint32_t L,
                                  uint32_t W, const void* frag, const ReconstructPrime* primes, const uint64_t* Q,
                                  hipStream_t st) {
  const uint64_t n = (uint64_t)n_polys << logN;
  const uint32_t S = L / 4 + 1;
  if (L > 64) return hipErrorInvalidValue;   // k must fit one digit
  return with_cvt_threads(n, [&](auto nth) {
    constexpr int NTH = decltype(nth)::value;
#define X(KS)                                                                                                      \
    if (S <= KS) {                                                                                                 \
      hipLaunchKernelGGL((crt_reconstruct_kernel<KS, NTH>), dim3(cvt_blocks(n, NTH)), dim3(NTH), 0, st, res, out,  \
                         n, logN, L, W, static_cast<const v4i*>(frag), primes, Q);                                 \
      return hipGetLastError();                                                                                    \
    }
    NTTK_CVT_CASES(X)
#undef X
    return hipErrorInvalidValue;
  });
}

}  // namespace nttk
