// Radix-2 butterfly stages on 16-value register tiles, shared by the NTT
// kernels and the VALU calibration kernel, and the bounds of their lazy
// reduction.
#pragma once

#include "fesc_internal.hpp"

namespace fesc {

// Bounds in units of the prime q < 2^50.  A product mm_var(x, w) with |x| <= X q
// and |w| <= om q is off by at most three roundings of the quotient, 3 |x w / q|
// 2^-53 <= 0.375 om X, so it lands within (0.5 + 0.375 om X) q; sums and the
// product's parts are exact integers while |x| <= 8 q < 2^53.  Table twiddles
// are balanced (om = 0.5), generated ones are products of those (kTwGen).  The
// inner passes are bound by VALU issue (83% busy at N = 2^16 before this
// schedule), so values are reduced only where a bound would pass 8 q.
constexpr double kTwTable = 0.5;
constexpr double mul_bound(double x, double om) { return 0.5 + 0.375 * om * x; }
constexpr double kTwPow2 = mul_bound(0.5, 0.5);
constexpr double kTwPow4 = mul_bound(kTwPow2, kTwPow2);
constexpr double kTwPow8 = mul_bound(kTwPow4, kTwPow4);
constexpr double kTwGen = mul_bound(0.5, kTwPow8) > kTwPow8 ? mul_bound(0.5, kTwPow8) : kTwPow8;
constexpr double kRedBal = 0.5 + 1.0 / (1 << 20);  // |red_bal(x)|, |x| <= 8 q
constexpr double kTooLarge = 1e9;

// Forward (CT): u +- w v.  red: u is reduced first.
constexpr double ct_bound(double x, double om, bool red) {
  const double s = (red ? kRedBal : x) + mul_bound(x, om);
  return s <= 8.0 ? s : kTooLarge;
}

// Inverse (GS): u + v, w (u - v).  Bit r of m[k]: the sum that stage k (distance
// 2^k) leaves in register r is reduced.
struct GsPlan {
  uint32_t m[4];
};
constexpr double gs_bound(double x0, double om, const GsPlan& p, int stages = 4) {
  double x[16] = {};
  for (int r = 0; r < 16; ++r) x[r] = x0;
  for (int k = 0; k < stages; ++k)
    for (int r = 0; r < 16; ++r) {
      const int h = 1 << k;
      if (r & h) continue;
      const double s = x[r] + x[r + h];
      if (s > 8.0) return kTooLarge;
      x[r] = (p.m[k] >> r) & 1u ? kRedBal : s;
      x[r + h] = mul_bound(s, om);
    }
  double top = 0.0;
  for (int r = 0; r < 16; ++r) top = x[r] > top ? x[r] : top;
  return top;
}

// The forward schedule: the outer pass (up to four stages) reduces nothing, the
// inner pass stages 1, 6, 10 and 12 of its twelve.
constexpr double kCtOuter =
    ct_bound(ct_bound(ct_bound(ct_bound(1.0, kTwTable, false), kTwTable, false), kTwTable, false),
             kTwTable, false);
constexpr bool kCtRed[12] = {true,  false, false, false, false, true,
                             false, false, false, true,  false, true};
constexpr double ct_inner_bound() {
  double x = kCtOuter;
  for (int s = 0; s < 12; ++s) x = ct_bound(x, s < 8 ? kTwTable : kTwGen, kCtRed[s]);
  return x;
}
constexpr double kCtInner = ct_inner_bound();
static_assert(kCtInner < 1.9, "forward transforms end below 1.9 q");

// The inverse schedule, from canonical residues: bits 3..0, 7..4, 11..8 of the
// inner pass, then the outer pass (its first log M stages).
constexpr GsPlan kGs0{{0x0, 0x0, 0x101, 0x16}}, kGs1{{0x5555, 0x0, 0x202, 0x2d}},
    kGs2{{0x0, 0x1111, 0x202, 0x4}}, kGsOut{{0x5555, 0x0, 0x202, 0x0}};
constexpr double kGsB0 = gs_bound(1.0, kTwGen, kGs0), kGsB1 = gs_bound(kGsB0, kTwTable, kGs1),
                 kGsB2 = gs_bound(kGsB1, kTwTable, kGs2);
static_assert(kGsB2 < 5.0 && gs_bound(kGsB2, kTwTable, kGsOut, 1) < 5.0 &&
                  gs_bound(kGsB2, kTwTable, kGsOut, 2) < 5.0 &&
                  gs_bound(kGsB2, kTwTable, kGsOut, 3) < 5.0 &&
                  gs_bound(kGsB2, kTwTable, kGsOut, 4) < 5.0,
              "inverse transforms end below 5 q");

// Radix-2 stages on a 16-value register tile, pairs (r, r + H) with r & H == 0.
// tw(gi) gives the twiddle of group gi = r / 2H.
template <int H, bool RED, class TW>
__device__ __forceinline__ void ct_st(double (&x)[16], TW tw, double q, double qinv) {
#pragma unroll
  for (int g = 0; g < 16; g += 2 * H) {
    const double w = tw(g / (2 * H));
#pragma unroll
    for (int r = g; r < g + H; ++r) {
      const double u = RED ? red_bal(x[r], q, qinv) : x[r];
      const double v = mm_var(x[r + H], w, q, qinv);
      x[r] = u + v;
      x[r + H] = u - v;
    }
  }
}

template <int H, uint32_t RED, class TW>
__device__ __forceinline__ void gs_st(double (&x)[16], TW tw, double q, double qinv) {
#pragma unroll
  for (int g = 0; g < 16; g += 2 * H) {
    const double w = tw(g / (2 * H));
#pragma unroll
    for (int r = g; r < g + H; ++r) {
      const double u = x[r], v = x[r + H];
      x[r] = (RED >> r) & 1u ? red_bal(u + v, q, qinv) : u + v;
      x[r + H] = mm_var(u - v, w, q, qinv);
    }
  }
}

// The outer pass's stages on M-point columns, M = 2^LOGM: value m of column j in
// x[j M + m], tw the prime's power table; stage s uses psi_rev[2^s + m / 2^(LOGM - s)].
// Forward, from canonical residues or balanced values (below kCtOuter q).
template <int LOGM>
__device__ __forceinline__ void fwd_columns(double (&x)[16], const double* __restrict__ tw,
                                            double q, double qinv) {
  constexpr int M = 1 << LOGM, C = 16 / M;
#pragma unroll
  for (int s = 0; s < LOGM; ++s) {
    const int H = M >> (s + 1);
#pragma unroll
    for (int m = 0; m < M; ++m) {
      if (m & H) continue;
      const double w = tw[(1 << s) + (m >> (LOGM - s))];
#pragma unroll
      for (int j = 0; j < C; ++j) {
        const double u = x[j * M + m], v = mm_var(x[j * M + m + H], w, q, qinv);
        x[j * M + m] = u + v;
        x[j * M + m + H] = u - v;
      }
    }
  }
}

// Inverse: the same stages in reverse order (sums reduced as kGsOut says).
template <int LOGM>
__device__ __forceinline__ void inv_columns(double (&x)[16], const double* __restrict__ tw,
                                            double q, double qinv) {
  constexpr int M = 1 << LOGM, C = 16 / M;
#pragma unroll
  for (int s = LOGM - 1; s >= 0; --s) {
    const int H = M >> (s + 1);
#pragma unroll
    for (int m = 0; m < M; ++m) {
      if (m & H) continue;
      const double w = tw[(1 << s) + (m >> (LOGM - s))];
#pragma unroll
      for (int j = 0; j < C; ++j) {
        const double u = x[j * M + m], v = x[j * M + m + H];
        x[j * M + m] = (kGsOut.m[LOGM - 1 - s] >> m) & 1u ? red_bal(u + v, q, qinv) : u + v;
        x[j * M + m + H] = mm_var(u - v, w, q, qinv);
      }
    }
  }
}

}  // namespace fesc
