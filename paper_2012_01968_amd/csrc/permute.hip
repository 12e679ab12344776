// Natural-order option (Section III-C): the forward transform leaves A_brv(i) in slot i
// (Algorithm 1's output order); a plan created with NTT_ORDER_NATURAL moves every slot i to
// slot brv(i) after the forward transform, and back before the inverse.  The bit-reversal
// permutation is an involution, so one kernel serves both directions.
//
// The permutation runs in place as swaps of tile pairs.  Write a slot index of log2 N bits as
// (h, m, l): h the top t bits, m the middle log2 N - 2t bits, l the low t bits.  Then
// brv(h, m, l) = (brv_t(l), brv(m), brv_t(h)), so the 2^t x 2^t tile of middle index m (rows
// h, each row 2^t consecutive slots) maps onto the tile of middle index brv(m), with row and
// column swapped and each bit-reversed.  A workgroup loads the tiles of m and brv(m) (one tile
// when they coincide) into LDS and writes each into the other's place, so global reads and
// writes go by rows of 2^t consecutive slots.
#include "kernels.hpp"
#include "passes.hpp"

namespace nttk {

constexpr int kPermThreads = 256;

// f(0), and f(1) where there is a second tile (uniform per workgroup)
template <typename F>
__device__ __forceinline__ void for_tiles(int n_tiles, F&& f) {
  f(std::integral_constant<int, 0>{});
  if (n_tiles > 1) f(std::integral_constant<int, 1>{});
}

// Bound by its bytes (one read, one write) and, where they stay in the Infinity Cache, by one memory
// round trip each way: a lane's loads, two adjacent slots each, go out together before the first
// LDS store (eight-byte accesses in two loops before).  24 x 2 vectors of 2^14 8.3 -> 6.1 us, 45 x 2 of
// 2^16 24.6 -> 22.3, 60 x 2 of 2^17 48.9 -> 38.3 (6.6 TB/s; what a natural-order forward takes above a
// bit-reversed one).
template <int TB>   // t = TB: tiles of 2^TB x 2^TB slots
__global__ __launch_bounds__(kPermThreads) void brv_permute_kernel(PassArgs a) {
  constexpr uint32_t T = 1u << TB, E = T * T, PITCH = T + 1;   // one pad slot per LDS row
  constexpr uint32_t V = TB ? 2 : 1, G = E / V;                // adjacent slots per access, accesses per tile
  constexpr uint32_t PER = (G + kPermThreads - 1) / kPermThreads;
  __shared__ uint64_t tile[2][T * PITCH];
  const uint32_t mb = a.logN - 2 * TB;                 // middle bits
  const uint64_t vec = blockIdx.x >> mb;
  const uint32_t m = blockIdx.x & ((1u << mb) - 1u);
  const uint32_t mr = mb ? __brev(m) >> (32 - mb) : 0u;
  if (vec >= a.n_vec || m > mr) return;                // each pair once (uniform per workgroup)
  gu64* base = vec_ref(a, vec).base;
  const uint32_t hs = a.logN - TB;                     // shift of h in a slot index
  typedef uint64_t word __attribute__((ext_vector_type(V)));
  typedef __attribute__((address_space(1))) word gword;
  auto at = [&](uint32_t mm, uint32_t g) {             // access g of the tile of middle index mm
    const uint32_t h = (g * V) >> TB, l = (g * V) & (T - 1);
    return (gword*)(base + (((size_t)h << hs) | ((size_t)mm << TB) | l));
  };
  const int n_tiles = m == mr ? 1 : 2;
  word x[2][PER];
  for_tiles(n_tiles, [&](auto k) {
#pragma unroll
    for (uint32_t i = 0; i < PER; ++i) {
      const uint32_t g = threadIdx.x + i * kPermThreads;
      if (G % kPermThreads == 0 || g < G) x[k][i] = *at(k ? mr : m, g);
    }
  });
  loads_issued();
  for_tiles(n_tiles, [&](auto k) {
#pragma unroll
    for (uint32_t i = 0; i < PER; ++i) {
      const uint32_t g = threadIdx.x + i * kPermThreads, h = (g * V) >> TB, l = (g * V) & (T - 1);
      if (G % kPermThreads == 0 || g < G)
#pragma unroll
        for (uint32_t v = 0; v < V; ++v) tile[k][h * PITCH + l + v] = x[k][i][v];
    }
  });
  __syncthreads();
  // the tile of m goes to brv(m) and the tile of brv(m) to m: destination row h', column l'
  // takes source row brv_t(l'), column brv_t(h')
  for_tiles(n_tiles, [&](auto k) {
#pragma unroll
    for (uint32_t i = 0; i < PER; ++i) {
      const uint32_t g = threadIdx.x + i * kPermThreads, h2 = (g * V) >> TB, l2 = (g * V) & (T - 1);
      if (G % kPermThreads != 0 && g >= G) continue;
      const uint32_t ls_ = TB ? __brev(h2) >> (32 - TB) : 0u;
      word y;
#pragma unroll
      for (uint32_t v = 0; v < V; ++v) {
        const uint32_t hs_ = TB ? __brev(l2 + v) >> (32 - TB) : 0u;
        y[v] = tile[k][hs_ * PITCH + ls_];
      }
      *at(k ? m : mr, g) = y;
    }
  });
}

template <int TB>
static hipError_t go_permute(const PassArgs& a, hipStream_t st) {
  const uint32_t mb = a.logN - 2 * TB;
  return for_vector_parts(a, (uint64_t)kPermThreads << mb, [&](const PassArgs& p) {
    hipLaunchKernelGGL(brv_permute_kernel<TB>, dim3((uint32_t)(p.n_vec << mb)), dim3(kPermThreads), 0, st, p);
    return hipGetLastError();
  });
}

hipError_t launch_brv_permute(const PassArgs& a, hipStream_t st) {
  if (a.logN < 1 || a.logN > 17) return hipErrorInvalidValue;
  const uint32_t t = a.logN / 2 < 5 ? a.logN / 2 : 5;   // 32 x 32 tiles from N = 2^10 up
  switch (t) {
    case 0: return go_permute<0>(a, st);
    case 1: return go_permute<1>(a, st);
    case 2: return go_permute<2>(a, st);
    case 3: return go_permute<3>(a, st);
    case 4: return go_permute<4>(a, st);
    default: return go_permute<5>(a, st);
  }
}

}  // namespace nttk
