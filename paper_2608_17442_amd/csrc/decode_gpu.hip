// CKKS decoding on the device: evaluation-form plaintexts -> slot vectors, the
// inverse of the device encoder (encode_gpu.hip).
//
// Slot j of a plaintext with integer coefficients m is z_j = m(zeta^(e_j)) /
// Delta, zeta = exp(i pi / N), e_j = 5^j mod 2N.  With e_j = 2 p_j + 1,
//     m(zeta^(e_j)) = sum_k (m_k zeta^k) exp(2 pi i k p_j / N).
// The powers of 5 are the residues 1 mod 4, so every p_j is even, and with p_j =
// 2 p' the terms k and k + N/2 share their exponential:
//     sum_{k < N/2} (m_k zeta^k + m_{k+N/2} zeta^(k+N/2)) exp(2 pi i k p' / (N/2)),
// an inverse DFT of half the length.  Per plaintext:
//   1. inverse NTT of the limbs into scratch (canonical residues, coefficient
//      form);
//   2. k_dec_outer (past 32 limbs, or with primes more than a factor of two apart,
//      k_dec_crt before it, N > 4096): the centred integers m_k from their residues by a
//      mixed-radix CRT with balanced digits (Garner's method: v_0 = [y_0], v_i =
//      [(...((y_i - v_0) q_0^-1 - v_1) q_1^-1 ...) q_(i-1)^-1]_(q_i), each in
//      (-q_i/2, q_i/2]), so m_k = v_0 + q_0 (v_1 + q_1 (v_2 + ...)) exactly; the
//      Horner evaluation in fp64 rounds once per level; then the twist and the
//      R-point columns of the DFT (length R * 4096, k = 4096 n1 + n2, p' = k1 + R
//      k2) with the twiddle between the passes;
//   3. k_dec_rows: the 4096-point rows as decimation in frequency in three
//      radix-16 register steps with LDS transposes, and the store of z_j =
//      v[p_j] / Delta through the encoder's inverse slot table.
// For N = 4096 (N/2 = 2048) the full-length DFT is one row and half its outputs
// are dropped.  24 plaintexts at N = 2^16, 15 limbs: 220 us, of which, traced, 69 +
// 56 the inverse NTT, 74 k_dec_outer (VALU: 120 products per coefficient), 23 the rows;
// with a spilling CRT, sixteen radix-2 passes of full length and a copy before the
// inverse NTT it was 588 us.  The error against long doubles fell with it (2-norm
// 4.6e-16 from 6.3e-16: fewer roundings, smaller angles).
// Every twiddle is an entry of the encoder's table T[k] = exp(-i pi k / N), here
// conjugated.
#include <algorithm>

#include "fesc_internal.hpp"
#include "ops.hpp"

namespace fesc {

namespace {

constexpr int kThreads = 256;
constexpr uint32_t kRow = 4096;
constexpr int kLdsC = 4096 + 256;  // padded layout of the NTT's inner pass

// padded LDS address of element e = 256 a + 16 c + b: 272 a + 17 c + b
__device__ __forceinline__ uint32_t lds_e(uint32_t e) {
  return 272u * (e >> 8) + 17u * ((e >> 4) & 15u) + (e & 15u);
}

// a * conj(b), one rounding of the fused products
__device__ __forceinline__ double2 cmulc(double2 a, double2 b) {
  return double2{__builtin_fma(a.x, b.x, a.y * b.y), __builtin_fma(a.y, b.x, -(a.x * b.y))};
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) {
  return double2{a.x + b.x, a.y + b.y};
}
// a i^k
__device__ __forceinline__ double2 mul_i(double2 a, uint32_t k) {
  const double2 b = k & 1 ? double2{-a.y, a.x} : a;
  return k & 2 ? double2{-b.x, -b.y} : b;
}
// a conj(T[k]), k < 2N, through the table's first quarter turn: T[k + j N/2] =
// (-i)^j T[k], and entries of larger angles carry larger rounding errors.
__device__ __forceinline__ double2 mul_root(double2 a, const double2* __restrict__ T, uint32_t k,
                                            uint32_t n) {
  return mul_i(cmulc(a, T[k & (n / 2 - 1)]), 2 * k / n);
}

// Centred integers of NC coefficients, r[c * off + i * n] their residues at limb
// i, all digits in registers.  Limbs from `level` on (LMAX is the next multiple of
// 4) repeat the last limb; the Horner sum leaves them out.  Every prime is within a
// factor of two of the others: |t - v_j| < 2 q_i then, the product stays within
// 0.9 q_i and red_bal's quotient is exact.
template <int LMAX, int NC>
__device__ __forceinline__ void crt(const uint64_t* __restrict__ r, size_t off, uint32_t level,
                                    uint32_t L, uint32_t n, const PrimeK* __restrict__ pk,
                                    const double2* __restrict__ garner, double (&m)[NC]) {
  double t[NC][LMAX];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int i = 0; i < LMAX; ++i)
      t[c][i] = u2d(r[c * off + (size_t)min((uint32_t)i, level - 1) * n]);
#pragma unroll
  for (int j = 0; j < LMAX; ++j) {
    const uint32_t ju = min((uint32_t)j, level - 1);
    const double qj = pk[ju].q, qinvj = pk[ju].qinv;
#pragma unroll
    for (int c = 0; c < NC; ++c) t[c][j] = red_bal(t[c][j], qj, qinvj);
#pragma unroll
    for (int i = j + 1; i < LMAX; ++i) {
      const uint32_t iu = min((uint32_t)i, level - 1);
      const double w = garner[(size_t)iu * L + min((uint32_t)j, iu)].x;
      const double q = pk[iu].q, qinv = pk[iu].qinv;
#pragma unroll
      for (int c = 0; c < NC; ++c) t[c][i] = mm_var(t[c][i] - t[c][j], w, q, qinv);
    }
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) m[c] = 0.0;
#pragma unroll
  for (int i = LMAX - 1; i >= 0; --i) {
    const double q = pk[min((uint32_t)i, level - 1)].q;
#pragma unroll
    for (int c = 0; c < NC; ++c) m[c] = (uint32_t)i < level ? t[c][i] + q * m[c] : 0.0;
  }
}

// The same for any level and primes, one coefficient; its digits do not fit in
// registers.
__device__ __forceinline__ double crt_any(const uint64_t* r, uint32_t level, uint32_t L,
                                          uint32_t n, const PrimeK* __restrict__ pk,
                                          const double2* __restrict__ garner) {
  double v[FESC_MAX_PRIMES];
  for (uint32_t i = 0; i < level; ++i) {
    const PrimeK P = pk[i];
    double t = u2d(r[(size_t)i * n]);
    const double2* gi = garner + (size_t)i * L;
    for (uint32_t j = 0; j < i; ++j) {  // t = (t - v_j) q_j^-1 mod q_i
      const double2 w = gi[j];
      t = red_bal(mm_shoup(red_bal(t - v[j], P.q, P.qinv), w.x, w.y, P.q), P.q, P.qinv);
    }
    v[i] = center(red_full(t, P.q, P.qinv), P.q);
  }
  double m = v[level - 1];
  for (uint32_t i = level - 1; i-- > 0;) m = v[i] + pk[i].q * m;
  return m;
}

// crt_any of coefficient k of plaintext blockIdx.y, stored as fp64 over its residue
// at limb 0.  Bound by the chain through the digits, so every coefficient has a
// thread of its own: with both coefficients of an output in one thread of
// k_dec_outer a call of 36 limbs took, us, N = 2^13 210 (now 119; four plaintexts 228,
// now 140), N = 2^16 254 (154; four 434, 322; sixteen, where the chip is full, 1020, 1024).
__global__ __launch_bounds__(kThreads) void k_dec_crt(uint64_t* __restrict__ res, uint32_t level,
                                                      uint32_t L, uint32_t n,
                                                      const PrimeK* __restrict__ pk,
                                                      const double2* __restrict__ garner) {
  uint64_t* r = res + (size_t)blockIdx.y * level * n + blockIdx.x * kThreads + threadIdx.x;
  *reinterpret_cast<double*>(r) = crt_any(r, level, L, n, pk, garner);
}

// CRT, twist and R-point columns.  A workgroup takes 256 / R columns of
// plaintext blockIdx.y: thread (n1, column) forms the twisted input of index
// k = 4096 n1 + n2, thread (k1, column) the output X[k1][n2].  LMAX == 0, of
// the folded form: k_dec_crt has run, the coefficients stand at limb 0.
template <int LMAX, bool FOLD>
__global__ __launch_bounds__(kThreads) void k_dec_outer(const uint64_t* __restrict__ res,
                                                        uint32_t level, uint32_t L, uint32_t n,
                                                        uint32_t R, const PrimeK* __restrict__ pk,
                                                        const double2* __restrict__ garner,
                                                        const double2* __restrict__ T,
                                                        double2* __restrict__ X) {
  __shared__ double2 xs[kThreads];
  const uint32_t t = threadIdx.x, cols = kThreads / R, b = blockIdx.y;
  const uint32_t i1 = t / cols, col = t % cols;
  const uint32_t n2 = blockIdx.x * cols + col, k = kRow * i1 + n2;
  double m[FOLD ? 2 : 1];
  const uint64_t* r = res + (size_t)b * level * n + k;
  if constexpr (LMAX > 0) {
    crt<LMAX, FOLD ? 2 : 1>(r, n / 2, level, L, n, pk, garner, m);
  } else if constexpr (FOLD) {
    const double* rd = reinterpret_cast<const double*>(r);
    m[0] = rd[0];
    m[1] = rd[n / 2];
  } else {
    m[0] = crt_any(r, level, L, n, pk, garner);
  }
  const double2 w0 = T[k];
  double2 x{m[0] * w0.x, -m[0] * w0.y};
  if constexpr (FOLD) {  // zeta^(k + N/2) from the table as well, not as i zeta^k
    const double2 w1 = T[k + n / 2];
    x.x = __builtin_fma(m[1], w1.x, x.x);
    x.y = __builtin_fma(-m[1], w1.y, x.y);
  }
  double2* out = X + (size_t)b * R * kRow + k;  // i1 is k1 here
  if (R == 1) {
    *out = x;
    return;
  }
  xs[t] = x;
  __syncthreads();
  // output k1 = i1 of the R-point DFT, as the sum over n1 bit by bit: of the
  // factors exp(2 pi i n1 k1 / R) only those of odd n1 at R = 8 are no powers of i
  auto in = [&](uint32_t n1) { return xs[n1 * cols + col]; };
  auto two = [&](double2 a, double2 c) { return cadd(a, mul_i(c, 2 * i1)); };
  auto four = [&](double2 a, double2 p, double2 c, double2 q) {
    return cadd(two(a, c), mul_i(two(p, q), i1));
  };
  double2 y;
  if (R == 2) {
    y = two(in(0), in(1));
  } else if (R == 4) {
    y = four(in(0), in(1), in(2), in(3));
  } else {
    y = cadd(four(in(0), in(2), in(4), in(6)),
             mul_root(four(in(1), in(3), in(5), in(7)), T, (n / 4) * i1, n));
  }
  *out = mul_root(y, T, 4 * n2 * i1, n);  // exp(2 pi i n2 k1 / (N/2)), 4 n2 k1 < 2N
}

// One radix-2 DIF stage on register pairs (r, r + H): x_r <- x_r + x_{r+H},
// x_{r+H} <- (x_r - x_{r+H}) conj T[idx(r)].  The upper half of the H twiddles
// is i times the lower one (idx(r + H/2) = idx(r) + N/2).
template <int H, class IDX>
__device__ __forceinline__ void dif_st(double2 (&x)[16], const double2* __restrict__ T, IDX idx) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if (r & H) continue;
    const double2 u = x[r], v = x[r + H];
    x[r] = cadd(u, v);
    const bool upper = H > 1 && (r & (H / 2));
    x[r + H] = mul_i(cmulc(double2{u.x - v.x, u.y - v.y}, T[idx(upper ? r - H / 2 : r)]), upper);
  }
}

// Rows: row k1 = blockIdx.x of plaintext blockIdx.y (element e of the row starts
// at thread e % 256, register e / 256; a DIF stage of half size h multiplies the
// difference by exp(i pi (e mod h) / h) = conj T[(e mod h) N / h]), then the
// slots: position e of the row holds frequency p' = k1 + R bitrev12(e).
template <bool FOLD>
__global__ __launch_bounds__(kThreads) void k_dec_rows(const double2* __restrict__ X,
                                                       const double2* __restrict__ T,
                                                       const int32_t* __restrict__ inv,
                                                       double2* __restrict__ z, uint32_t n,
                                                       uint32_t R, double rdelta) {
  __shared__ double lre[kLdsC], lim[kLdsC];
  const uint32_t t = threadIdx.x, k1 = blockIdx.x, b = blockIdx.y;
  const double2* row = X + ((size_t)b * R + k1) * kRow;
  double2 x[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) x[r] = row[t + 256 * r];
  // the slots of positions 16 t + r, read ahead of the transform
  int32_t slot[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const uint32_t p = k1 + R * (__builtin_bitreverse32(16 * t + r) >> 20);
    slot[r] = inv[FOLD ? 2 * p : p];
  }
  // bits 11..8 in registers: h = 256 H, e mod h = t + 256 (r mod H)
  dif_st<8>(x, T, [&](int r) { return (size_t)(t + 256 * (r % 8)) * (n / 2048); });
  dif_st<4>(x, T, [&](int r) { return (size_t)(t + 256 * (r % 4)) * (n / 1024); });
  dif_st<2>(x, T, [&](int r) { return (size_t)(t + 256 * (r % 2)) * (n / 512); });
  dif_st<1>(x, T, [&](int) { return (size_t)t * (n / 256); });
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const uint32_t a = lds_e(t + 256 * r);
    lre[a] = x[r].x;
    lim[a] = x[r].y;
  }
  __syncthreads();
  // bits 7..4: thread t = 16 a + bb holds e = 256 a + 16 r + bb;
  // h = 16 H, e mod h = 16 (r mod H) + bb
  const uint32_t aa = t >> 4, bb = t & 15;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const uint32_t a = lds_e(256 * aa + 16 * r + bb);
    x[r] = double2{lre[a], lim[a]};
  }
  dif_st<8>(x, T, [&](int r) { return (size_t)(16 * (r % 8) + bb) * (n / 128); });
  dif_st<4>(x, T, [&](int r) { return (size_t)(16 * (r % 4) + bb) * (n / 64); });
  dif_st<2>(x, T, [&](int r) { return (size_t)(16 * (r % 2) + bb) * (n / 32); });
  dif_st<1>(x, T, [&](int) { return (size_t)bb * (n / 16); });
  // each thread overwrites the words it has read itself
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const uint32_t a = lds_e(256 * aa + 16 * r + bb);
    lre[a] = x[r].x;
    lim[a] = x[r].y;
  }
  __syncthreads();
  // bits 3..0: thread t holds e = 16 t + r; h = H, e mod h = r mod H
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const uint32_t a = lds_e(16 * t + r);
    x[r] = double2{lre[a], lim[a]};
  }
  dif_st<8>(x, T, [&](int r) { return (size_t)(r % 8) * (n / 8); });
  dif_st<4>(x, T, [&](int r) { return (size_t)(r % 4) * (n / 4); });
  dif_st<2>(x, T, [&](int r) { return (size_t)(r % 2) * (n / 2); });
  dif_st<1>(x, T, [&](int) { return (size_t)0; });
  double2* zb = z + (size_t)b * (n / 2);
#pragma unroll
  for (int r = 0; r < 16; ++r)
    if (FOLD || slot[r] >= 0)
      zb[(uint32_t)slot[r]] = double2{x[r].x * rdelta, x[r].y * rdelta};
}

template <int LMAX>
void launch_outer(const Context* c, const uint64_t* limbs, uint32_t level, uint32_t R, bool fold,
                  uint32_t m, double2* X, hipStream_t s) {
  const dim3 grid(kRow * R / kThreads, m);
  if (fold)
    k_dec_outer<LMAX, true><<<grid, kThreads, 0, s>>>(limbs, level, c->L, c->n, R, c->d_pk,
                                                      c->d_garner, c->d_enc_tw, X);
  else
    k_dec_outer<LMAX, false><<<grid, kThreads, 0, s>>>(limbs, level, c->L, c->n, R, c->d_pk,
                                                       c->d_garner, c->d_enc_tw, X);
}

}  // namespace

// Decodes `count` plaintexts pt[count][level][N] into z[count][N/2], as many
// per round as fit in the scratch ciphertext slots (limbs, then the complex
// transform input of each plaintext).
int op_decode_plain(Context* c, const uint64_t* pt, uint32_t count, uint32_t level, double scale,
                    double2* z, uint64_t* slots, uint32_t nslots, hipStream_t s) {
  const uint32_t n = c->n;
  const bool fold = n > kRow;
  const uint32_t len = fold ? n / 2 : n, R = len / kRow;
  const size_t per = (size_t)level * n + 2 * (size_t)len;
  const size_t room = (size_t)2 * c->L * n * nslots;
  const uint32_t cap = (uint32_t)std::min<size_t>(room / per, 65535);  // grid y limit
  if (cap == 0) return fail(FESC_ERR_ARG, "decode scratch too small");
  const double rdelta = 1.0 / scale;
  const auto [lo, hi] = std::minmax_element(c->primes.begin(), c->primes.begin() + level);
  // the digits of up to 32 limbs fit in registers
  const uint32_t bucket = *hi <= 2 * *lo && level <= 32 ? (level + 3) / 4 : 0;
  for (uint32_t b0 = 0; b0 < count; b0 += cap) {
    const uint32_t m = std::min(cap, count - b0);
    uint64_t* limbs = slots;                                                 // [m][level][N]
    double2* X = reinterpret_cast<double2*>(slots + (size_t)m * level * n);  // [m][R][4096]
    if (int rc = hip_check(launch_ntt_inv_from(c, pt + (size_t)b0 * level * n, limbs, m, level, s),
                           "decode iNTT"))
      return rc;
    switch (bucket) {
      case 1: launch_outer<4>(c, limbs, level, R, fold, m, X, s); break;
      case 2: launch_outer<8>(c, limbs, level, R, fold, m, X, s); break;
      case 3: launch_outer<12>(c, limbs, level, R, fold, m, X, s); break;
      case 4: launch_outer<16>(c, limbs, level, R, fold, m, X, s); break;
      case 5: launch_outer<20>(c, limbs, level, R, fold, m, X, s); break;
      case 6: launch_outer<24>(c, limbs, level, R, fold, m, X, s); break;
      case 7: launch_outer<28>(c, limbs, level, R, fold, m, X, s); break;
      case 8: launch_outer<32>(c, limbs, level, R, fold, m, X, s); break;
      default:
        if (fold) {
          k_dec_crt<<<dim3(n / kThreads, m), kThreads, 0, s>>>(limbs, level, c->L, n, c->d_pk,
                                                               c->d_garner);
          if (int rc = hip_check(hipGetLastError(), "k_dec_crt")) return rc;
        }
        launch_outer<0>(c, limbs, level, R, fold, m, X, s);
        break;
    }
    if (int rc = hip_check(hipGetLastError(), "k_dec_outer")) return rc;
    double2* zb = z + (size_t)b0 * (n / 2);
    if (fold)
      k_dec_rows<true><<<dim3(R, m), kThreads, 0, s>>>(X, c->d_enc_tw, c->d_enc_inv, zb, n, R,
                                                       rdelta);
    else
      k_dec_rows<false><<<dim3(R, m), kThreads, 0, s>>>(X, c->d_enc_tw, c->d_enc_inv, zb, n, R,
                                                        rdelta);
    if (int rc = hip_check(hipGetLastError(), "k_dec_rows")) return rc;
  }
  return FESC_OK;
}

}  // namespace fesc
