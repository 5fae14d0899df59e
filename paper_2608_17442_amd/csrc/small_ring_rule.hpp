// Which batches take the fused kernels of N = 4096 (small_ring.hip).  Host
// arithmetic only, so that the limits can be tested without a GPU.
#pragma once

#include <cstddef>
#include <cstdint>

namespace fesc {

// Workgroups times digit primes up to which the repeated transforms cost less than
// the launches that they save (four workgroups of one prime's work on each CU), and
// the most digit primes that one of them transforms.  Rotations with either fusion
// alone, us, general -> fused, 50-bit primes:
//   ModUp   alpha 1, 8 rows: 45 -> 38 (72 workgroups), 69 -> 61 (576);
//           alpha 3, 15 rows: 46.7 -> 45.6 (90), 57 -> 63 (360), 78 -> 82 (720)
//   ModDown alpha 1, 15 rows: 52 -> 45 (30), 315 -> 300 (960);
//           alpha 3, 24 rows: 78 -> 73 (192), 110 -> 112 (384), 182 -> 185 (768)
// and one rotation with both 41 -> 27 (3 rows, alpha 1), 46 -> 42 (9 rows, alpha 3),
// 48 -> 37 (15 rows, alpha 2).  ModDown merged with the rescale, whose digit has
// one prime more:
//           alpha 1, 11 rows: 39.7 -> 35.0 (22), 289 -> 285 (704);
//           alpha 2, 15 rows: 44.9 -> 43.2 (30), 95 -> 93 (240);
//           alpha 3 (four primes), 11 rows: 46.3 -> 49.3 (22), 70.2 -> 72.3 (176),
//           23 rows: 52.9 -> 55.2 (46), 77.1 -> 79.4 (184).
// Rescale, one ciphertext of 2 .. 40 rows 18 -> 9.8; a matrix-vector product of 16
// outputs and 32 rows (1024) 128 -> 119.
constexpr uint32_t kSmallFill = 1024, kSmallPrimes = 3;

inline bool small_modup_pays(uint32_t log_n, uint32_t alpha, uint32_t nsrc, uint32_t level) {
  const uint64_t dnum = (level + alpha - 1) / alpha;
  return log_n == 12 && alpha <= kSmallPrimes &&
         alpha * nsrc * dnum * (level + alpha) <= kSmallFill;
}

// alpha special primes and, merged with the rescale, q_{l-1}.
inline bool small_moddown_pays(uint32_t log_n, uint32_t alpha, bool merged, uint32_t njobs,
                               uint32_t rows) {
  return log_n == 12 && alpha + merged <= kSmallPrimes &&
         (uint64_t)alpha * 2 * njobs * rows <= kSmallFill;
}

inline bool small_rescale_pays(uint32_t log_n, uint32_t count, uint32_t rows) {
  return log_n == 12 && (uint64_t)2 * count * rows <= kSmallFill;
}

// Words [a, a + na) and [b, b + nb) meet.
inline bool overlap(const uint64_t* a, size_t na, const uint64_t* b, size_t nb) {
  return a < b + nb && b < a + na;
}

}  // namespace fesc
