// Which form of the VALU basis conversion (k_bconv_outer, ntt.hip) a launch
// takes.  Host arithmetic only, so that the choice can be tested without a GPU.
#pragma once

#include <algorithm>
#include <cstdint>

namespace fesc {

// Workgroups that fill the chip at three waves per SIMD (256 CUs).
constexpr uint32_t kBconvFill = 768;

struct ValuConversion {
  uint32_t targets;  // target rows per workgroup, sharing a load of the digits: 1 or 3
  bool fuse;         // the digits' inverse columns finished by the conversion itself
};

// N = 4096 2^log_m; digits of at most `digit` primes, `targets` target rows for
// each of `groups` digits.  Whole calls in us, one rotation at a time unless a
// count is given, 50-bit primes.
//
// Fused, every workgroup that reads a digit finishes its columns again: log_m + 1
// steps (stages and a factor) on each of its primes for every target row.  It saves
// a launch and the digits' trip through memory (separate / fused in each pair):
//  - a chain of more than kFuseRepeat steps per column is waited for: digits of 1, 2, 3
//    primes, 12 to 24 rows (24 .. 216 steps): N = 2^13 61 / 54, 61 / 54, 67 / 62, N = 2^14
//    74 / 65, 72 / 65, 82 / 79, N = 2^16 with 4 to 6 rows 62 / 54, 78 / 72, 66 / 60; nine
//    primes and 9 rows: N = 2^13 (162) 60.4 / 58.1, N = 2^14 (243) 63.8 / 62.6, N = 2^15
//    (324) 65.5 / 70.4, N = 2^16 (405) 84.5 / 93.2; twelve and 24 rows: N = 2^13 (576) 69 /
//    72, N = 2^16 (1440) 153 / 186; sixteen: N = 2^16 175 / 217;
//  - the trip pays for 21 steps per column of a short digit, whatever the batch, the
//    launch for kFuseNet columns times the steps beyond (in brackets; from 960 calls
//    timed in both forms).  Three primes, ModDown of hoisted rotations of one input: N =
//    2^15, 3 rows, 24 rotations (0) 125.7 / 116.1, 9 rows, ten (7200) 155.1 / 150.3; N =
//    2^16, 9 rows, three (6912) 124.1 / 121.1; two primes, 6 rows, eight (4608) 163.2 /
//    158.7.  Rotations of an input each: N = 2^14, 24 rows, ten (12240) 461 / 467, N = 2^15, 12
//    rows, five (12960) 175.0 / 178.9, N = 2^16, 12 rows, two (14976) 147.6 / 153.7;
//  - of a longer digit it pays for 12, since the separate form shares its loads among
//    three rows sooner (below), and not in a launch of fewer than 128 column blocks,
//    where the chain of nine and more primes is waited for.  Nine primes, hoisted: N = 2^14,
//    4 rows, 16 rotations (0) 110.7 / 100.2, 6 rows, 24 (10368) 155.0 / 156.8, N = 2^15, 3
//    rows, 20 (0) 189.4 / 175.1, 6 rows, 12 (20736) 157.2 / 165.7; N = 2^16, 3 rows, three (96
//    blocks), twelve primes 104.5 / 109.6, sixteen 121.1 / 128.1.  Launches of less than
//    kFuseWork columns times steps are fused all the same.
//
// Three target rows per workgroup once such workgroups fill the chip, which takes
// fewer of them the longer the digits that they share (one / three rows, in brackets
// the launch's workgroups of three): three primes, N = 2^16, 12 rows, two (512) 140.2 /
// 134.1, N = 2^15, 12 rows, one (128) 69 / 73; nine, 24 rows: N = 2^15 one (216) 102.3 /
// 105.4, two (432) 153.7 / 146.3; twelve: N = 2^14 two (128) 96.2 / 105.1, four (256) 141.6 /
// 136.1, eight (512) 235.8 / 212.2; sixteen: N = 2^14 two (176) 107 / 117, four (352) 164 /
// 157.
constexpr uint32_t kFuseRepeat = 256, kFuseWork = 12288, kFuseShort = 3, kFuseNet = 9216;

inline ValuConversion valu_conversion(uint32_t log_m, uint32_t digit, uint32_t targets,
                                      uint32_t groups) {
  const uint64_t blocks = (uint64_t)groups << log_m, triples = (targets + 2) / 3 * blocks;
  const uint64_t steps = (uint64_t)targets * (log_m + 1);
  // the digits' columns times the steps on each, those that the trip pays for left out
  const auto net = [&](uint64_t paid) {
    return steps > paid ? digit * blocks * (steps - paid) : 0;
  };
  const bool pays = digit <= kFuseShort
                        ? net(21) <= kFuseNet
                        : net(0) <= kFuseWork || (blocks >= 128 && net(12) <= kFuseNet);
  // (N = 4096 has no column stages)
  if (log_m > 0 && triples < kBconvFill && digit * steps <= kFuseRepeat && pays) return {1, true};
  const uint32_t fill = std::max(kBconvFill / 3, std::min(kBconvFill, 2 * kBconvFill / digit));
  return {triples >= fill ? 3u : 1u, false};
}

}  // namespace fesc
