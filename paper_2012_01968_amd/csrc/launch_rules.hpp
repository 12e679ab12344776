// Choices that automatic plans make for each launch, by the transform size and the vectors of the
// launch (the plan's tables serve every split).  Host only: no device code, so the host test suite
// compiles it with g++.
#pragma once
#include <algorithm>
#include <cstdint>

namespace nttr {

// N = 2^13 takes one pass (a workgroup of 1024 lanes and 68 KB of LDS per vector, one per CU) where
// the vectors fill the last round of the 256 CUs.  A round costs about the same however full it is,
// while the column and row passes cost as much as the vectors they have.  One pass / 32 x 256, us;
// forward, product, rows with a key:
//   vectors       160        200        288        384        448        520        600       1300
//   60 bits f  11.5/12.3  12.2/14.8  19.5/18.5  20.3/21.5  21.0/24.6  29.4/30.0  30.7/35.7  56.0/67.2
//           p  28.6/31.9  29.9/38.6  55.4/49.5  57.2/60.0  58.6/67.6  85.2/79.1  85.2/87.0   172/189
//           k  23.7/24.4  24.2/28.7  42.3/36.0  43.4/42.3  45.3/48.2  64.0/57.4  64.3/64.6   124/123
//   62 bits f  15.1/15.0  16.2/18.2  27.6/22.3  28.0/26.5  29.0/30.6  42.1/36.2  43.2/43.4  81.7/83.2
//           p  40.6/38.7  41.4/48.7  78.6/62.8  79.6/74.8  82.2/85.4   120/100    120/110    238/232
//           k  31.5/29.3  32.0/35.6  57.9/45.0  58.4/52.4  59.6/61.0  86.6/72.7  86.9/81.7   167/156
// Below 2^60 up to 176 of the last round's CUs may be idle, and any number from 1024 vectors on; above,
// where a round is longer, 112 or a sixteenth of the vectors.
inline bool one_pass_8192(uint64_t n_vec, bool fast) {
  constexpr uint64_t kCus = 256, kFirst = 192;
  const uint64_t idle = (kCus - n_vec % kCus) % kCus;
  return n_vec >= kFirst && (fast ? idle <= 176 || n_vec > 1024 : idle <= std::max<uint64_t>(112, n_vec / 16));
}

// log2 N1 of a launch over n_vec vectors, `log_n1` being the plan's.  N = 2^15 and 2^16 take columns of
// 2^7 points up to 2^21 residues, where the shorter rows' chain of stages counts: 39 vectors of 2^15
// 28.6 us against 29.3 with 2^6 (62-bit primes 33.4 against 35.2), 21 of 2^16 32.2 against 33.7 (37.5
// against 39.7); above, 90 vectors of 2^15 52.5 against 50.5.
constexpr uint64_t kSmallLaunch = 1u << 21;
inline uint32_t split(uint32_t log_n, uint32_t log_n1, uint64_t n_vec, bool fast) {
  if (log_n == 13 && one_pass_8192(n_vec, fast)) return 0;
  if ((log_n == 15 || log_n == 16) && (n_vec << log_n) <= kSmallLaunch) return 7;
  return log_n1;
}

// Whether the row pass of a split launch takes 4 values per lane and 64 lanes instead of 8 and 128: up to
// 2^21 residues, whose 8-value waves would not fill the SIMDs four deep, so that a wave's own chain of
// stages is what the launch waits for (rows of up to 2^12 points; a longer one needs more than 1024 lanes).
// Forward + inverse, us, 8 x 128 / 4 x 64: N = 2^13 x 7 vectors 14.5 / 13.1, 2^14 x 48 21.0 / 20.1, 2^16 x 21
// 34.0 / 32.2; 2^17 x 21 (2.75 M residues) 58.4 / 56.6, 2^15 x 90 (2.95 M) 51.3 / 51.9, 2^16 x 90 94 / 93.5.
inline bool small_rows(uint32_t log_n, uint32_t log_n1, uint64_t n_vec) {
  return log_n1 != 0 && log_n - log_n1 <= 12 && (n_vec << log_n) <= kSmallLaunch;
}

}  // namespace nttr
