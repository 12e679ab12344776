// Launch interface of the NTT kernels (host side).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nttk {

struct Tw;
struct PassArgs;
struct VecDesc;

// Whether a (log2 N, log2 N1, OT stages) combination has kernels built in.
bool shape_supported(uint32_t logN, uint32_t logN1, int ot_stages);

// Whether a tile shape of the split passes has kernels built in and fits the split: row pass
// log2 values per lane (0 = default, 2, 3) and workgroup lanes (0 = default, 64, 128, 256);
// column pass width (0 = automatic, 16, 32, 64, 128 or 256 adjacent columns, at most N2).
bool tiles_supported(uint32_t logN, uint32_t logN1, uint32_t row_lr, uint32_t row_nth, uint32_t col_w);

// Forward / inverse transform of every vector described by `a`, enqueued on `st`.
hipError_t launch_forward(const PassArgs& a, int ot_stages, hipStream_t st);
hipError_t launch_inverse(const PassArgs& a, int ot_stages, hipStream_t st);

// One kernel of a transform: pass 0 / 1 in execution order (see ntt_forward_pass).
hipError_t launch_forward_pass(const PassArgs& a, int ot_stages, int pass, hipStream_t st);
hipError_t launch_inverse_pass(const PassArgs& a, int ot_stages, int pass, hipStream_t st);

// Row passes of a product (forward row stages, element-wise product, inverse row stages in one
// launch) with an NTT-domain key (lists) or a second operand that goes through the forward stages
// too (dense); `af` holds the forward tables and the second factors, `ai` the inverse tables.  With logN1 = 0 this is the whole product; otherwise the forward column pass
// comes before it and the inverse column pass after it.
hipError_t launch_mul_rows(const PassArgs& af, const PassArgs& ai, int ot_stages, hipStream_t st);

// Fused single-launch transform (both passes, XCD-local queues); see fused.hpp.
struct FusedArgs;
bool fused_supported(uint32_t logN, uint32_t logN1, int ot_stages);
hipError_t launch_fused(const PassArgs& a, int ot_stages, bool inverse, uint32_t* ctr, uint32_t n_polys,
                        uint32_t lag, uint32_t max_grid, hipStream_t st);

// Transforms that keep the data in global memory between launches (stages.hip): one launch
// per group of log2_radix consecutive stages (1 = radix-2, one launch per stage).  Group g
// counts in execution order (the inverse runs the forward groups backwards).
uint32_t stage_group_count(uint32_t logN, int log2_radix);
hipError_t launch_stage_group(const PassArgs& a, int log2_radix, bool inverse, uint32_t g, hipStream_t st);
hipError_t launch_stage_groups(const PassArgs& a, int log2_radix, bool inverse, hipStream_t st);

// 32-bit words (kernels32.hip): primes below 2^30, tables of the centred words w 2^32 mod q.
struct Prime32 {
  uint32_t q, nqi;          // q and -q^-1 mod 2^32
};
struct Plan32 {
  const int32_t *tw_fwd, *tw_inv;        // [L][N]
  const int32_t *scale, *scale_mul;      // [L][2]: {1/N}, {Psi_inv[1]/N}; of products: times 2^32
  const Prime32* primes;                 // [L]
  uint32_t L, logN, logN1;
};
bool shape32_supported(uint32_t logN, uint32_t logN1);
hipError_t launch_transform32(const Plan32& p, uint32_t* data, uint32_t n_polys, bool inverse, hipStream_t st);
// c = a * b (negacyclic); `tmp` holds b's column pass (n_polys*L*N words; unused when logN1 = 0).
hipError_t launch_product32(const Plan32& p, const uint32_t* a, const uint32_t* b, uint32_t* c, uint32_t n_polys,
                            uint32_t* tmp, hipStream_t st);
hipError_t launch_pointwise32(const uint32_t* A, const uint32_t* B, uint32_t* C, const uint32_t* qs,
                              const uint64_t* mus, uint64_t n, uint32_t logN, uint32_t L, hipStream_t st);

// RNS <-> integer conversion (crt.hip): integers as [n_polys][W][N] little-endian words.  `frag`
// holds the digit matrices of crt_math.hpp.
struct DecomposePrime {
  uint64_t q;
  uint32_t mu;      // floor(2^(s+31) / q), s = bitlen(q)
  int32_t shift;    // s - 15
  uint64_t recip;   // floor(2^64 / q)
};
struct ReconstructPrime {
  uint64_t q, inv, inv_b;   // (Q/q)^-1 mod q and its Shoup companion
  uint64_t rec;             // floor(2^120 / (q << (62 - s)))
};
// `all_wide`: every prime has at least 47 bits (V >> (s - 15) comes from the high words alone).
hipError_t launch_rns_decompose(const uint64_t* words, uint32_t W, uint64_t* res, uint32_t n_polys, uint32_t logN,
                                uint32_t L, const void* frag, uint32_t frag_slices, const DecomposePrime* primes,
                                const int64_t* offsets, bool all_wide, hipStream_t st);
hipError_t launch_crt_reconstruct(const uint64_t* res, uint64_t* out, uint32_t n_polys, uint32_t logN, uint32_t L,
                                  uint32_t W, const void* frag, const ReconstructPrime* primes, const uint64_t* Q,
                                  hipStream_t st);

// In-place bit-reversal permutation of every vector described by `a` (slot i <-> slot
// brv(i)): turns the forward transform's bit-reversed output into natural order and back.
hipError_t launch_brv_permute(const PassArgs& a, hipStream_t st);

// Every vector of a list times its key vector, in place (Barrett products).
hipError_t launch_pointwise_list(const VecDesc* vecs, uint64_t n_vec, uint32_t logN, const uint64_t* qs,
                                 const uint64_t* mus, const uint32_t* bits, hipStream_t st);

// C = A * B mod q_l element-wise over n_elems elements of a [n_vec][N] batch.
hipError_t launch_pointwise(const uint64_t* A, const uint64_t* B, uint64_t* C, const uint64_t* qs,
                            const uint64_t* mus, const uint32_t* bits, uint64_t n_elems, uint32_t logN,
                            uint32_t L, hipStream_t st);

}  // namespace nttk
