// CKKS encoding on the device: slot vectors -> evaluation-form plaintexts
// (offline plaintext preparation: the projection's diagonals, masks).
//
// Slot j is the evaluation at zeta^(5^j mod 2N), zeta = exp(i pi / N).  With
// y[(e_j - 1)/2] = z_j and y[N - 1 - (e_j - 1)/2] = conj(z_j), e_j = 5^j mod 2N,
// the real plaintext coefficients are
//     m_k = round(Delta / N * Re(zeta^-k Y_k)),   Y = DFT_N(y)   (e^{-2 pi i/N}),
// rounded half away from zero, as the host encoder computes them.  The DFT runs
// in fp64 in two passes over N = M * 4096 (n = 4096 n1 + n2, k = k1 + M k2):
//   pass 1 (columns n2): gather y through the inverse slot table, M-point DFT
//     over n1, twiddle w_N^(n2 k1) -> X[k1][n2];
//   pass 2 (rows k1): 4096-point decimation-in-frequency DFT over n2 in three
//     radix-16 register steps with padded-LDS transposes; the epilogue applies
//     the twist zeta^-k, scales and rounds, storing m in the transform's
//     digit-reversed order;
// then the lift to the RNS limbs inside the first forward NTT pass and the second
// pass of every limb (64 plaintexts at N = 2^16, 16 limbs: 432 us; with a lift of
// its own, gathering m once per limb, 815 us).  Every twiddle is an entry of one table
// T[k] = exp(-i pi k / N), k < 2N.
#include <algorithm>
#include <cmath>

#include "butterfly.hpp"
#include "fesc_internal.hpp"
#include "ops.hpp"

namespace fesc {

namespace {

constexpr int kThreads = 256;
constexpr int kRow = 4096;
constexpr int kLdsC = 4096 + 256;  // padded layout of the NTT's inner pass

// padded LDS address of element e = 256 a + 16 c + b: 272 a + 17 c + b
__device__ __forceinline__ uint32_t lds_e(uint32_t e) {
  return 272u * (e >> 8) + 17u * ((e >> 4) & 15u) + (e & 15u);
}

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return double2{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}

// Pass 1: 256 / S columns n2 of plaintext blockIdx.y.  The workgroup gathers
// their M inputs into LDS once; its S parts then form M / S outputs of every
// column each (whole wavefronts, so the DFT's factors are scalar): one plaintext
// alone then runs 64 workgroups at N = 2^16 instead of 16 (whole call 46 -> 37 us).
template <int M>
__global__ __launch_bounds__(kThreads) void k_enc_outer(const double2* __restrict__ z,
                                                        const int32_t* __restrict__ inv,
                                                        const double2* __restrict__ T,
                                                        double2* __restrict__ X, uint32_t n) {
  constexpr int S = M < 4 ? M : 4, kCols = kThreads / S, K = M / S;
  __shared__ double2 ys[M][kCols];
  const uint32_t part = __builtin_amdgcn_readfirstlane(threadIdx.x / kCols);
  const uint32_t col = threadIdx.x % kCols;
  const uint32_t n2 = blockIdx.x * kCols + col;
  const uint32_t b = blockIdx.y;
  const double2* zb = z + (size_t)b * (n / 2);
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const uint32_t n1 = part * K + i;
    const int32_t s = inv[n1 * kRow + n2];
    const double2 v = zb[s >= 0 ? s : ~s];
    ys[n1][col] = s >= 0 ? v : double2{v.x, -v.y};
  }
  __syncthreads();
  double2 y[M];
#pragma unroll
  for (int n1 = 0; n1 < M; ++n1) y[n1] = ys[n1][col];
  double2* Xb = X + (size_t)b * n;
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const uint32_t k1 = part * K + i;
    double2 acc{0.0, 0.0};
#pragma unroll
    for (int n1 = 0; n1 < M; ++n1) {
      // w_M^(n1 k1) = T[(2N / M) (n1 k1 mod M)]
      const double2 w = T[(size_t)(2 * n / M) * ((n1 * k1) % M)];
      const double2 p = cmul(y[n1], w);
      acc.x += p.x;
      acc.y += p.y;
    }
    // twiddle w_N^(n2 k1) = T[2 n2 k1 mod 2N]
    Xb[(size_t)k1 * kRow + n2] = cmul(acc, T[(2 * n2 * k1) & (2 * n - 1)]);
  }
}

// The 15 twiddles of a radix-16 step: entry H - 1 + r mod H is that of register r
// in the stage of half size H.  Read a step ahead from the table of the row DFT
// (Context::d_enc_row: the entries of T in the order of use, adjacent lanes
// adjacent; the rows of 32 plaintexts at N = 2^16 take 29 us so, 38 us with the
// strided entries of T), first = its first entry for this thread, stride = from
// one entry to the next.
struct Tw16 {
  double2 w[15];
  __device__ __forceinline__ Tw16(const double2* __restrict__ first, uint32_t stride) {
#pragma unroll
    for (int i = 0; i < 15; ++i) w[i] = first[i * stride];
  }
};

// One radix-2 DIF stage on register pairs (r, r + H): x_r <- x_r + x_{r+H},
// x_{r+H} <- (x_r - x_{r+H}) w_{2H}^(r mod H).
template <int H>
__device__ __forceinline__ void dif_st(double2 (&x)[16], const Tw16& tw) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if (r & H) continue;
    const double2 u = x[r], v = x[r + H];
    x[r] = double2{u.x + v.x, u.y + v.y};
    x[r + H] = cmul(double2{u.x - v.x, u.y - v.y}, tw.w[H - 1 + r % H]);
  }
}
__device__ __forceinline__ void dif16(double2 (&x)[16], const Tw16& tw) {
  dif_st<8>(x, tw);
  dif_st<4>(x, tw);
  dif_st<2>(x, tw);
  dif_st<1>(x, tw);
}

__device__ __forceinline__ int64_t round_half_away(double v) {
  return (int64_t)(v >= 0.0 ? floor(v + 0.5) : ceil(v - 0.5));
}

// Pass 2: row k1 = blockIdx.x of plaintext blockIdx.y.  Element e of the row
// (its n2) starts at thread e % 256, register e / 256.  A DIF stage of half
// size h pairs e with e + h and multiplies the difference by
// w_{2h}^(e mod h) = T[(e mod h) N / h].
__global__ __launch_bounds__(kThreads) void k_enc_inner(const double2* __restrict__ X,
                                                        const double2* __restrict__ T,
                                                        const double2* __restrict__ row_tw,
                                                        int64_t* __restrict__ mt, uint32_t n,
                                                        uint32_t M, double scale) {
  __shared__ double lre[kLdsC], lim[kLdsC];
  const uint32_t t = threadIdx.x, k1 = blockIdx.x, b = blockIdx.y;
  const double2* row = X + (size_t)b * n + (size_t)k1 * kRow;
  double2 x[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) x[r] = row[t + 256 * r];
  // bits 11..8 in registers: h = 256 H, e mod h = t + 256 (r mod H)
  const uint32_t aa = t >> 4, bb = t & 15;
  const Tw16 w1(row_tw + t, 256);
  // bits 7..4: thread t = 16 a + bb holds e = 256 a + 16 r + bb;
  // h = 16 H, e mod h = 16 (r mod H) + bb
  const Tw16 w2(row_tw + 15 * 256 + bb, 16);
  dif16(x, w1);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const uint32_t a = lds_e(t + 256 * r);
    lre[a] = x[r].x;
    lim[a] = x[r].y;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const uint32_t a = lds_e(256 * aa + 16 * r + bb);
    x[r] = double2{lre[a], lim[a]};
  }
  dif16(x, w2);
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
  dif16(x, Tw16(row_tw + 15 * 272, 1));
  // position e holds Y'[bitrev12(e)]: frequency k = k1 + M k2
  const double f = scale / (double)n;
  int64_t* out = mt + (size_t)b * n + (size_t)k1 * kRow;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const uint32_t e = 16 * t + r;
    const uint32_t k2 = __builtin_bitreverse32(e) >> 20;
    const uint32_t k = k1 + M * k2;
    const double2 w = T[k];
    out[e] = round_half_away((x[r].x * w.x - x[r].y * w.y) * f);
  }
}

// A coefficient |v| < 2^63 modulo the prime, within q / 2 (exact: v = hi 2^32 +
// lo, each part reduced).
__device__ __forceinline__ double lift_any(int64_t v, double two32, double q, double qinv) {
  const double hi = (double)(int32_t)(v >> 32);
  const double lo = (double)(uint32_t)(v & 0xffffffffu);
  return red_bal(mm_var(red_full(hi, q, qinv), two32, q, qinv) + lo, q, qinv);
}

// Lift, N = 4096 (one row, m at position bitrev12(k)): coefficient k of plaintext
// blockIdx.z reduced into row i = blockIdx.y of pt[b][rows][N]; row i uses prime
// i below `split`, prime1 + (i - split) from there (the special primes of an
// extended-basis plaintext).
__global__ __launch_bounds__(kThreads) void k_enc_lift(const int64_t* __restrict__ mt,
                                                       uint64_t* __restrict__ pt, uint32_t rows,
                                                       uint32_t split, uint32_t prime1,
                                                       const PrimeK* __restrict__ pk) {
  const uint32_t i = blockIdx.y, b = blockIdx.z;
  const uint32_t k = blockIdx.x * kThreads + threadIdx.x;
  const PrimeK P = pk[i < split ? i : prime1 + (i - split)];
  const int64_t v = mt[(size_t)b * kRow + (__builtin_bitreverse32(k) >> 20)];
  const double r = lift_any(v, red_full(4294967296.0, P.q, P.qinv), P.q, P.qinv);
  pt[((size_t)b * rows + i) * kRow + k] = to_res_2q(r, P.q, P.qinv);
}

// Lift fused with the first forward NTT pass (N > 4096, M = 2^LOGM): a thread
// takes C = 16 / M columns c, values c + 4096 m, of plaintext blockIdx.z and
// carries them through `per` rows from row blockIdx.y * per on.  Coefficient k = c +
// 4096 m sits in row k % M = c % M of m at position bitrev12(k / M), k / M = c / M +
// (4096 / M) m, i.e. at M bitrev(c / M) + bitrev(m): the M values of a column are
// adjacent, and are read once for all rows instead of once per row in
// bit-reversed order.
template <int LOGM>
__global__ __launch_bounds__(kThreads) void k_enc_lift_outer(const int64_t* __restrict__ mt,
                                                             uint64_t* __restrict__ pt,
                                                             uint32_t rows, uint32_t per,
                                                             uint32_t split, uint32_t prime1,
                                                             const PrimeK* __restrict__ pk,
                                                             const double* __restrict__ twf) {
  constexpr int M = 1 << LOGM, C = 16 / M;
  constexpr uint32_t n = kRow << LOGM;
  const uint32_t b = blockIdx.z;
  const uint32_t c0 = blockIdx.x * (kThreads * C) + threadIdx.x;
  int64_t v[16];  // v[j M + m]: value m of column c0 + 256 j
  bool small = true;
#pragma unroll
  for (int j = 0; j < C; ++j) {
    const uint32_t c = c0 + kThreads * j;
    const int64_t* src = mt + (size_t)b * n + (size_t)(c % M) * kRow +
                         M * (__builtin_bitreverse32(c / M) >> (20 + LOGM));
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int64_t x = src[__builtin_bitreverse32(m) >> (32 - LOGM)];
      v[j * M + m] = x;
      small = small && x > -(1ll << 51) && x < (1ll << 51);
    }
  }
  // coefficients below 2^51 (any plaintext at a scale the levels are made for)
  // are exact doubles; decided per wavefront
  const bool all_small = __all(small);
  const uint32_t end = min((blockIdx.y + 1) * per, rows);
  for (uint32_t i = blockIdx.y * per; i < end; ++i) {
    const uint32_t prime = i < split ? i : prime1 + (i - split);
    const double q = pk[prime].q, qinv = pk[prime].qinv;
    const double* tw = twf + (size_t)prime * n;
    double x[16];
    if (all_small) {
#pragma unroll
      for (int r = 0; r < 16; ++r)  // 1.5 2^52 + v holds v in its low bits
        x[r] = red_bal(__longlong_as_double(v[r] + 0x4338000000000000ll) - 6755399441055744.0, q,
                       qinv);
    } else {
      const double two32 = red_full(4294967296.0, q, qinv);
#pragma unroll
      for (int r = 0; r < 16; ++r) x[r] = lift_any(v[r], two32, q, qinv);
    }
    fwd_columns<LOGM>(x, tw, q, qinv);
    double* out = reinterpret_cast<double*>(pt) + ((size_t)b * rows + i) * n + c0;
#pragma unroll
    for (int j = 0; j < C; ++j)
#pragma unroll
      for (int m = 0; m < M; ++m) out[kThreads * j + kRow * m] = x[j * M + m];
  }
}

constexpr size_t kRoundBytes = (size_t)256 << 20;

template <int LOGM>
void launch_lift_outer(const Context* c, const int64_t* mt, uint64_t* pt, uint32_t m,
                       uint32_t rows, uint32_t level, hipStream_t s) {
  // rows per thread: as many as leave four workgroups per CU, so that a
  // column's coefficients are read rarely
  const uint32_t groups = (m << LOGM), want = std::max(1u, 1024u / groups);
  const uint32_t per = (rows + want - 1) / want;
  k_enc_lift_outer<LOGM><<<dim3(1u << LOGM, (rows + per - 1) / per, m), kThreads, 0, s>>>(
      mt, pt, rows, per, level, c->L, c->d_pk, c->d_tw_fwd);
}

}  // namespace

// Encodes `count` slot vectors z[count][N/2] (complex, device) at scale
// `scale` into evaluation-form plaintexts pt[count][rows][N], in rounds through the
// scratch ciphertext region (X and m of each plaintext, 3N words) of at least one
// plaintext per ciphertext slot (3N <= 2 L N) and up to 256 MB of plaintexts, what
// the Infinity Cache holds between the NTT's passes; rows = level, or level + alpha over
// the extended basis q_0 .. q_{level-1}, p_0 .. p_{alpha-1} (ext).
int op_encode_plain(Context* c, const double2* z, uint32_t count, double scale, uint64_t* pt,
                    uint32_t level, uint64_t* slots, uint32_t nslots, hipStream_t s, bool ext) {
  const uint32_t n = c->n, M = n / kRow;
  const uint32_t rows = ext ? level + c->alpha : level;
  const size_t W = (size_t)2 * c->L * n;
  const uint32_t fit = (uint32_t)std::min<size_t>(W * nslots / ((size_t)3 * n), 65535);
  const uint32_t cap = std::min(fit, std::max(nslots, (uint32_t)(kRoundBytes / ((size_t)rows * n * 8))));
  if (cap == 0) return fail(FESC_ERR_ARG, "encode scratch too small");
  for (uint32_t b0 = 0; b0 < count; b0 += cap) {
    const uint32_t m = std::min(cap, count - b0);
    double2* X = reinterpret_cast<double2*>(slots);   // [m][N] complex
    int64_t* mt = reinterpret_cast<int64_t*>(slots + (size_t)2 * n * m);  // [m][N]
    const dim3 g1(kRow * std::min(M, 4u) / kThreads, m);
    const double2* zb = z + (size_t)b0 * (n / 2);
    const auto outer = [&](auto kernel) {
      kernel<<<g1, kThreads, 0, s>>>(zb, c->d_enc_inv, c->d_enc_tw, X, n);
    };
    switch (M) {
      case 1: outer(k_enc_outer<1>); break;
      case 2: outer(k_enc_outer<2>); break;
      case 4: outer(k_enc_outer<4>); break;
      case 8: outer(k_enc_outer<8>); break;
      case 16: outer(k_enc_outer<16>); break;
      default: return fail(FESC_ERR_ARG, "ring degree outside 2^12 .. 2^16");
    }
    if (int rc = hip_check(hipGetLastError(), "k_enc_outer")) return rc;
    k_enc_inner<<<dim3(M, m), kThreads, 0, s>>>(X, c->d_enc_tw, c->d_enc_row, mt, n, M, scale);
    if (int rc = hip_check(hipGetLastError(), "k_enc_inner")) return rc;
    uint64_t* pb = pt + (size_t)b0 * rows * n;
    const RowSel rs{pb, (size_t)rows * n, (size_t)n, 0, level, c->L, 0, 0, 0};
    switch (M) {
      case 1:
        k_enc_lift<<<dim3(kRow / kThreads, rows, m), kThreads, 0, s>>>(mt, pb, rows, level, c->L,
                                                                       c->d_pk);
        break;
      case 2: launch_lift_outer<1>(c, mt, pb, m, rows, level, s); break;
      case 4: launch_lift_outer<2>(c, mt, pb, m, rows, level, s); break;
      case 8: launch_lift_outer<3>(c, mt, pb, m, rows, level, s); break;
      default: launch_lift_outer<4>(c, mt, pb, m, rows, level, s); break;
    }
    if (int rc = hip_check(hipGetLastError(), "k_enc_lift")) return rc;
    // N = 4096: the inner pass is the whole transform
    if (int rc = hip_check(launch_ntt_fwd_inner_rows(c, rs, m, rows, s), "encode NTT")) return rc;
  }
  return FESC_OK;
}

}  // namespace fesc
