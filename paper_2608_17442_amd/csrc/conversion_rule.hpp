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
// Fused, every workgroup that reads a digit repeats log_m stages and a factor on
// each of its primes: `repeat` times per column of a group.  It saves a launch and a
// trip through memory, as long as
//  - the chain is short (kFuseRepeat; separate / fused): digits of 1, 2, 3 primes,
//    12 to 24 rows (repeat 24 .. 216): N = 2^13 61 / 54, 61 / 54, 67 / 62, N = 2^14
//    74 / 65, 72 / 65, 82 / 79, N = 2^16 with 4 to 6 rows 62 / 54, 78 / 72, 66 / 60;
//    nine primes and 9 rows: N = 2^13 (162) 60.4 / 58.1, N = 2^14 (243) 63.8 / 62.6, N =
//    2^15 (324) 65.5 / 70.4, N = 2^16 (405) 84.5 / 93.2; twelve and 24 rows: N = 2^13 (576)
//    69 / 72, N = 2^16 (1440) 153 / 186; sixteen: N = 2^16 175 / 217;
//  - the chip has room for the repeats (kFuseWork; work of the ModUp in brackets):
//    three primes, N = 2^13, 24 rows, four at a time (9216) 106.0 / 104.6, eight (18432)
//    162.4 / 163.5, N = 2^15, 12 rows, two (9216) 87.8 / 86.9, four (18432) 126.4 / 127.8,
//    N = 2^16, 12 rows, one (11520) 95.3 / 94.1, two (23040) 139.3 / 141.6.
//
// Three target rows per workgroup once such workgroups fill the chip, which takes
// fewer of them the longer the digits that they share (one / three rows, in brackets
// the launch's workgroups of three): three primes, N = 2^16, 12 rows, two (512) 140.2 /
// 134.1, N = 2^15, 12 rows, one (128) 69 / 73; nine, 24 rows: N = 2^15 one (216) 102.3 /
// 105.4, two (432) 153.7 / 146.3; twelve: N = 2^14 two (128) 96.2 / 105.1, four (256) 141.6 /
// 136.1, eight (512) 235.8 / 212.2; sixteen: N = 2^14 two (176) 107 / 117, four (352) 164 /
// 157.
constexpr uint32_t kFuseRepeat = 256, kFuseWork = 12288;

inline ValuConversion valu_conversion(uint32_t log_m, uint32_t digit, uint32_t targets,
                                      uint32_t groups) {
  const uint64_t triples = (uint64_t)((targets + 2) / 3) * groups << log_m;
  const uint64_t repeat = (uint64_t)digit * targets * (log_m + 1);
  // (N = 4096 has no column stages)
  if (log_m > 0 && triples < kBconvFill && repeat <= kFuseRepeat &&
      (repeat * groups << log_m) <= kFuseWork)
    return {1, true};
  const uint32_t fill = std::max(kBconvFill / 3, std::min(kBconvFill, 2 * kBconvFill / digit));
  return {triples >= fill ? 3u : 1u, false};
}

}  // namespace fesc
