// Negacyclic NTT / inverse NTT over word-sized primes, batched over rows.
//
// Definition (the forward transform's output order is bit-reversed):
//     A[j] = sum_k a_k psi^((2 brv(j) + 1) k)  mod q,
// psi the smallest primitive 2N-th root of unity mod q.  The transform is the
// radix-2 Cooley-Tukey network whose butterfly on the pair (j, j + t) uses the
// twiddle psi^brv((N + j) / 2t); the inverse is the Gentleman-Sande network
// with psi^-1 and a final scaling by N^-1.
//
// gfx950 mapping.  N = M * 4096 with M = 2^(log N - 12) in [1, 16].  At most
// two passes over HBM, each over independent sub-transforms held on chip:
//   outer pass (M > 1): the first log M stages couple only indices that agree
//               mod 4096, i.e. M-point "columns" at stride 4096.  A thread
//               keeps whole columns in registers; a wavefront reads and writes
//               64 adjacent columns, so every access is a contiguous 512-byte
//               run (2 KB per workgroup) and no LDS is needed.  The twiddles of
//               these stages do not depend on the column (M - 1 values).
//   inner pass: the last 12 stages couple only indices inside a contiguous
//               4096-element block, one block per 256-thread workgroup.  The
//               block is processed as three radix-16 register steps on index
//               bits 11..8, 7..4 and 3..0, with LDS transposes in between, so
//               loads and stores of the forward pass are fully coalesced.
// Between the passes the row holds the signed fp64 intermediate in place of
// the uint64 residues (same 8 bytes per value), so no conversion or full
// reduction is spent on it.  For N = 4096 the inner pass alone is the whole
// transform.
//
// Twiddles: the outer passes read the bit-reversed power table (uniform per
// stage); an inner pass reads its block's 15 twiddles of bits 11..8 through the
// scalar cache, stages those of bits 7..4 in LDS next to the data and generates
// those of bits 3..0 from one power per thread (Context::d_tw3_*), so that no
// vector load is waited on between its butterflies.
#include <algorithm>
#include <type_traits>

#include "block4096.hpp"
#include "butterfly.hpp"
#include "conversion_rule.hpp"
#include "fesc_internal.hpp"
#include "ops.hpp"

namespace fesc {

// Row selection of a batched transform launch.  blockIdx.y = batch index b,
// blockIdx.z = limb index i (the batch varies fastest between workgroups, so
// the twiddle tables of one prime stay resident in L2 across the batch).
// Limb i < split uses prime prime0 + i, limb i >= split prime1 + (i - split).
// If skip_alpha != 0, limbs [d*skip_alpha, min((d+1)*skip_alpha, skip_limit))
// of batch element b, d = b mod skip_mod, are left untouched (the own-digit
// rows of digit d in a batch of ModUp outputs).
__device__ __forceinline__ uint64_t* RowSel::row() const {
  return base + (size_t)blockIdx.y * batch_stride + (size_t)blockIdx.z * limb_stride;
}
__device__ __forceinline__ uint32_t RowSel::prime() const {
  const uint32_t i = blockIdx.z;
  return i < split ? prime0 + i : prime1 + (i - split);
}
__device__ __forceinline__ bool RowSel::skip() const {
  if (!skip_alpha) return false;
  const uint32_t lo = (blockIdx.y % skip_mod) * skip_alpha;
  const uint32_t hi = min(lo + skip_alpha, skip_limit);
  return blockIdx.z >= lo && blockIdx.z < hi;
}

namespace {

// ------------------------------------------------------------- outer pass

// M = 2^LOGM point columns at stride 4096; a thread holds C = 16/M columns,
// c0 + 256 j (j < C), value m of column j in x[j*M + m].  Grid x = M.
// Stage s has distance 4096 * M/2^(s+1).
template <int LOGM>
__global__ __launch_bounds__(kThreads) void k_fwd_outer(RowSel rs, uint32_t log_n,
                                                        const PrimeK* __restrict__ pk,
                                                        const double* __restrict__ twf) {
  constexpr int M = 1 << LOGM, C = 16 / M;
  if (rs.skip()) return;
  const uint32_t n = 1u << log_n;
  const uint32_t prime = rs.prime();
  const double q = pk[prime].q, qinv = pk[prime].qinv;
  const double* tw = twf + (size_t)prime * n;
  uint64_t* row = rs.row();
  const uint32_t c0 = blockIdx.x * (kThreads * C) + threadIdx.x;
  double x[16];
#pragma unroll
  for (int j = 0; j < C; ++j)
#pragma unroll
    for (int m = 0; m < M; ++m) x[j * M + m] = u2d(row[c0 + kThreads * j + kBlock * m]);
  fwd_columns<LOGM>(x, tw, q, qinv);
  double* rowd = reinterpret_cast<double*>(row);
#pragma unroll
  for (int j = 0; j < C; ++j)
#pragma unroll
    for (int m = 0; m < M; ++m) rowd[c0 + kThreads * j + kBlock * m] = x[j * M + m];
}

// Final store of an inverse transform: N^-1 x as a canonical uint64 residue.
struct InvCanon {
  __device__ __forceinline__ void operator()(uint64_t* row, uint32_t k, double x,
                                             const PrimeK& P) const {
    row[k] = to_res_2q(mm_shoup(x, P.ninv, P.ninvp, P.q), P.q, P.qinv);
  }
};

// Final store of an inverse transform that feeds a fast basis conversion: the
// centred digit [N^-1 f_i x]_q in (-q/2, q/2), stored as fp64 in place of the
// residue.  f holds {N^-1 f_i mod q_i (balanced), /q_i} per limb i (blockIdx.z),
// where f_i is the conversion's (Q_D/q_i)^-1.  The product lies within 1.2 q
// (|x| < 5 q), near enough for red_bal's quotient to be the nearest integer:
// x / q is at least 1 / 2q > 2^-51 away from a half, its error below 2^-51.
struct InvDigit {
  const double2* f;
  __device__ __forceinline__ void operator()(uint64_t* row, uint32_t k, double x,
                                             const PrimeK& P) const {
    const double2 c = f[blockIdx.z];
    reinterpret_cast<double*>(row)[k] = red_bal(mm_shoup(x, c.x, c.y, P.q), P.q, P.qinv);
  }
};

// Inverse: the columns, then the final store (N^-1 scaling included).
template <int LOGM, class St>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(5))) void k_inv_outer(
    RowSel rs, uint32_t log_n, const PrimeK* __restrict__ pk, const double* __restrict__ twi,
    St st) {
  constexpr int M = 1 << LOGM, C = 16 / M;
  if (rs.skip()) return;
  const uint32_t n = 1u << log_n;
  const uint32_t prime = rs.prime();
  const PrimeK P = pk[prime];
  uint64_t* row = rs.row();
  const double* rowd = reinterpret_cast<const double*>(row);
  const uint32_t c0 = blockIdx.x * (kThreads * C) + threadIdx.x;
  double x[16];
#pragma unroll
  for (int j = 0; j < C; ++j)
#pragma unroll
    for (int m = 0; m < M; ++m) x[j * M + m] = rowd[c0 + kThreads * j + kBlock * m];
  inv_columns<LOGM>(x, twi + (size_t)prime * n, P.q, P.qinv);
#pragma unroll
  for (int j = 0; j < C; ++j)
#pragma unroll
    for (int m = 0; m < M; ++m) st(row, c0 + kThreads * j + kBlock * m, x[j * M + m], P);
}

// ------------------------------------------ basis conversion + outer pass

// Fused fast basis conversion and first forward pass.  For group g
// (blockIdx.z) and targets t = T blockIdx.y .. T blockIdx.y + T - 1 of the
// map, value k of target row t (prime m) is
//     y_k = sum_{a < aj} x_a[k] * hat_a  mod m,
// x_a the centred digits stored by the inverse transform (InvDigit, fp64).
// The first log M forward stages then run on the thread's columns exactly as
// in k_fwd_outer and the fp64 intermediate is stored; for M = 1 (no outer
// pass) the canonical residue is stored instead.  FUSE: the digit rows still
// hold the inverse transform's intermediate; its columns are finished here
// (inv_columns and InvDigit's factor), which saves a launch and is done again by
// every workgroup of a column, so only where that costs less (valu_conversion).
// Targets vary fastest after
// the column block, so all targets of a column block run together and read
// its digit rows from L2; with M a multiple of 8 a column block also stays on
// one XCD (workgroups are dealt to the 8 XCDs round-robin).
template <int LOGM>
__device__ __forceinline__ void finish_digits(double (&x)[16], uint32_t prime, double2 f,
                                              const PrimeK* __restrict__ pk,
                                              const double* __restrict__ twi) {
  const double q = pk[prime].q, qinv = pk[prime].qinv;
  inv_columns<LOGM>(x, twi + ((size_t)prime << (12 + LOGM)), q, qinv);
#pragma unroll
  for (int v = 0; v < 16; ++v) x[v] = red_bal(mm_shoup(x[v], f.x, f.y, q), q, qinv);
}

template <int LOGM, int T, bool FUSE, class Map>
__global__ __launch_bounds__(kThreads) void k_bconv_outer(Map map, uint32_t log_n,
                                                          const PrimeK* __restrict__ pk,
                                                          const double* __restrict__ twf,
                                                          const double* __restrict__ twi) {
  constexpr int M = 1 << LOGM, C = 16 / M;
  const uint32_t g = blockIdx.z, t0 = blockIdx.y * T;
  const uint32_t nt = map.targets(g);
  if (t0 >= nt) return;
  const uint32_t n = 1u << log_n;
  const uint32_t aj = map.aj(g);
  uint32_t prime[T];
  const double2* hat[T];
#pragma unroll
  for (int i = 0; i < T; ++i) {
    const uint32_t row = map.row(g, min(t0 + i, nt - 1));
    prime[i] = map.prime(row);
    hat[i] = map.hat(g, row);
  }
  const double* dig = map.digits(g);
  const uint32_t c0 = blockIdx.x * (kThreads * C) + threadIdx.x;
  double y[T][16];
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) y[i][v] = 0.0;
  // |x_a| < 2^49 and hat_a < m: each Shoup product lies within 0.625 m, so
  // eight terms and a carried reduced sum stay below 2^53
  for (uint32_t a = 0; a < aj; ++a) {
    const double* da = dig + (size_t)a * n + c0;
    double x[16];
#pragma unroll
    for (int j = 0; j < C; ++j)
#pragma unroll
      for (int m = 0; m < M; ++m) x[j * M + m] = da[kThreads * j + kBlock * m];
    if constexpr (FUSE) finish_digits<LOGM>(x, map.src_prime(g, a), map.factor(g, a), pk, twi);
#pragma unroll
    for (int i = 0; i < T; ++i) {
      const double q = pk[prime[i]].q;
      const double2 h = hat[i][a];
#pragma unroll
      for (int v = 0; v < 16; ++v) y[i][v] += mm_shoup(x[v], h.x, h.y, q);
    }
    if ((a & 7) == 7) {
#pragma unroll
      for (int i = 0; i < T; ++i) {
        const double q = pk[prime[i]].q, qinv = pk[prime[i]].qinv;
#pragma unroll
        for (int v = 0; v < 16; ++v) y[i][v] = red_bal(y[i][v], q, qinv);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < T; ++i) {
    if (t0 + i >= nt) break;
    const uint32_t row = map.row(g, t0 + i);
    const double q = pk[prime[i]].q, qinv = pk[prime[i]].qinv;
    uint64_t* out = map.out(g, row);
    double (&x)[16] = y[i];
    if constexpr (LOGM == 0) {
#pragma unroll
      for (int v = 0; v < 16; ++v) out[c0 + kThreads * v] = to_res(x[v], q, qinv);
    } else {
      const double* tw = twf + (size_t)prime[i] * n;
#pragma unroll
      for (int v = 0; v < 16; ++v) x[v] = red_bal(x[v], q, qinv);
      fwd_columns<LOGM>(x, tw, q, qinv);
      double* outd = reinterpret_cast<double*>(out);
#pragma unroll
      for (int j = 0; j < C; ++j)
#pragma unroll
        for (int m = 0; m < M; ++m) outd[c0 + kThreads * j + kBlock * m] = x[j * M + m];
    }
  }
}

// ModUp: group g = s * dnum + j (source s, digit j = primes [lo, lo + aj)),
// targets = the extended rows outside the digit, digits = cc[s][lo ..].
struct ModupMap {
  const double* cc;
  uint64_t* ext;
  const double2* mu_hat;
  uint32_t level, L, alpha, dnum_l, n;
  const int8_t* mu_bytes;  // matrix-core operands (LevelTables::mu_bytes), or null
  const double2* f;        // InvDigit's factors of the digit rows (mu_inv_n)
  __device__ uint32_t src_prime(uint32_t g, uint32_t a) const { return lo(g) + a; }
  __device__ double2 factor(uint32_t g, uint32_t a) const { return f[lo(g) + a]; }
  __device__ uint32_t lo(uint32_t g) const { return (g % dnum_l) * alpha; }
  __device__ uint32_t aj(uint32_t g) const { return min(alpha, level - lo(g)); }
  __device__ uint32_t targets(uint32_t g) const { return level + alpha - aj(g); }
  __device__ uint32_t row(uint32_t g, uint32_t t) const {
    const uint32_t l = lo(g);
    return t < l ? t : t + aj(g);
  }
  __device__ uint32_t prime(uint32_t r) const { return r < level ? r : L + (r - level); }
  __device__ const double* digits(uint32_t g) const {
    return cc + ((size_t)(g / dnum_l) * level + lo(g)) * n;
  }
  __device__ const double2* hat(uint32_t g, uint32_t r) const {
    return mu_hat + ((size_t)(g % dnum_l) * (level + alpha) + r) * alpha;
  }
  __device__ uint64_t* out(uint32_t g, uint32_t r) const {
    return ext + ((size_t)g * (level + alpha) + r) * n;
  }
  __device__ const int8_t* bytes(uint32_t g, uint32_t r) const {
    return mu_bytes + ((size_t)(g % dnum_l) * (level + alpha) + r) * 512;
  }
};

// ModDown: group g = 2 * job + component, digits = the alpha special-prime
// rows of acc[g], targets = the level rows of y[g].
struct ModdownMap {
  const uint64_t* acc;
  uint64_t* y;
  const double2* md_hat;
  uint32_t level, alpha, n;
  const int8_t* md_bytes;  // matrix-core operands (LevelTables::md_bytes), or null
  const double2* f;        // md_inv_n
  uint32_t L;
  __device__ uint32_t src_prime(uint32_t, uint32_t a) const { return L + a; }
  __device__ double2 factor(uint32_t, uint32_t a) const { return f[a]; }
  __device__ uint32_t aj(uint32_t) const { return alpha; }
  __device__ uint32_t targets(uint32_t) const { return level; }
  __device__ uint32_t row(uint32_t, uint32_t t) const { return t; }
  __device__ uint32_t prime(uint32_t r) const { return r; }
  __device__ const double* digits(uint32_t g) const {
    return reinterpret_cast<const double*>(acc + ((size_t)g * (level + alpha) + level) * n);
  }
  __device__ const double2* hat(uint32_t, uint32_t r) const { return md_hat + (size_t)r * alpha; }
  __device__ uint64_t* out(uint32_t g, uint32_t r) const {
    return y + ((size_t)g * level + r) * n;
  }
  __device__ const int8_t* bytes(uint32_t, uint32_t r) const { return md_bytes + (size_t)r * 512; }
};

// ModDown merged with the rescale: group g = 2 * job + component, digits =
// the alpha + 1 rows level-1 .. level+alpha-1 of acc[g] (q_{level-1}, then the
// special primes), targets = rows 0 .. rows-1 (< level - 1) of y[g], stored
// [g][level-1][N].
struct ModdownRescaleMap {
  const uint64_t* acc;
  uint64_t* y;
  const double2* mr_hat;
  uint32_t level, E, alpha, rows, n;  // alpha = number of digits (special primes + 1)
  const int8_t* mr_bytes;  // matrix-core operands of digits 0..7 (LevelTables::mr_bytes), or null
  const double2* f;        // mr_inv_n
  uint32_t L;
  __device__ uint32_t src_prime(uint32_t, uint32_t a) const { return a ? L + a - 1 : level - 1; }
  __device__ double2 factor(uint32_t, uint32_t a) const { return f[a]; }
  __device__ uint32_t aj(uint32_t) const { return alpha; }
  __device__ uint32_t targets(uint32_t) const { return rows; }
  __device__ uint32_t row(uint32_t, uint32_t t) const { return t; }
  __device__ uint32_t prime(uint32_t r) const { return r; }
  __device__ const double* digits(uint32_t g) const {
    return reinterpret_cast<const double*>(acc + ((size_t)g * E + level - 1) * n);
  }
  __device__ const double2* hat(uint32_t, uint32_t r) const { return mr_hat + (size_t)r * alpha; }
  __device__ uint64_t* out(uint32_t g, uint32_t r) const {
    return y + ((size_t)g * (level - 1) + r) * n;
  }
  __device__ const int8_t* bytes(uint32_t, uint32_t r) const { return mr_bytes + (size_t)r * 512; }
};

// Rescale lift: group g = 2 b + t (component t of ciphertext b), one digit =
// the centred last limb v[g] (|v| < q_last / 2), weight 1 for every target,
// targets = rows 0 .. rows-1 of w[g]: each target row gets v mod q_i.
struct RescaleMap {
  const double* v;
  uint64_t* w;
  const double2* one;  // {1, 1/q_i}
  uint32_t last, rows, n;
  const double2* f;  // rs_ninv
  static constexpr uint32_t alpha = 1;
  __device__ uint32_t src_prime(uint32_t, uint32_t) const { return last; }
  __device__ double2 factor(uint32_t, uint32_t) const { return f[0]; }
  __device__ uint32_t aj(uint32_t) const { return 1; }
  __device__ uint32_t targets(uint32_t) const { return rows; }
  __device__ uint32_t row(uint32_t, uint32_t t) const { return t; }
  __device__ uint32_t prime(uint32_t r) const { return r; }
  __device__ const double* digits(uint32_t g) const { return v + (size_t)g * n; }
  __device__ const double2* hat(uint32_t, uint32_t r) const { return one + r; }
  __device__ uint64_t* out(uint32_t g, uint32_t r) const { return w + ((size_t)g * last + r) * n; }
};

// ------------------------------- basis conversion on the matrix cores

typedef int v4i __attribute__((ext_vector_type(4)));

// Balanced base-256 digits of an integer-valued x, |x| < 2^49, as 8 signed
// bytes (the top one zero): the bytes of x + B, B = 0x80 in each of the low
// seven bytes, each less 128 (x + 1.5 2^52 holds x in its low bits).
__device__ __forceinline__ uint64_t bal_bytes(double x) {
  const int64_t xi = __double_as_longlong(x + 6755399441055744.0) - 0x4338000000000000ll;
  return (uint64_t)(xi + 0x0080808080808080ll) ^ 0x0080808080808080ull;
}

// The conversion of k_bconv_outer for digits of at most 8 primes (a ninth
// source, for ModDown merged with the rescale, as one Shoup product per value
// on the VALU), as an integer matrix product.  With x_a = sum_s x_a^s 256^s and
// c_(a,s) = 256^s hat_a mod m = sum_tau c^tau_(a,s) 256^tau (balanced
// base-256 digits, LevelTables::mu_bytes),
//     y = sum_a x_a hat_a = sum_tau 256^tau Q_tau  (mod m),
//     Q_tau = sum_(a,s) x_a^s c^tau_(a,s),
// an exact int32 (56 products of magnitude <= 2^14).  A wavefront owns 16 C
// columns of the outer pass, C = 16 / M (values c + 4096 m, c = c0 + u + 16 j,
// j < C), i.e. 16 values per lane: value v = j M + m.  Per quad of targets and
// value v, two 16 x 16 x 64 int8 products (rows: 4 targets x tau 0..3, then
// tau 4..7; columns: u; k: 8 sources x 8 digit bytes) give every Q, so that
// lane (g, u) ends up with y of target g at all its 16 values: whole columns
// of the outer pass, which then runs in registers as in k_bconv_outer.
// The quads of a column share one load of the digits; blockIdx.y deals them out
// where one workgroup per column and group would leave the chip idle.
// FUSE as in k_bconv_outer: a lane holds whole columns of its two sources.
template <int LOGM, class Map, bool NINTH, bool FUSE>
__device__ __forceinline__ void bconv_mfma(const Map& map, const PrimeK* __restrict__ pk,
                                           const double* __restrict__ twf,
                                           const double* __restrict__ twi) {
  constexpr uint32_t n = kBlock << LOGM;
  constexpr int M = 1 << LOGM, C = 16 / M;
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const uint32_t lg = lane >> 4, col = lane & 15;
  const uint32_t g = blockIdx.z;
  // this lane's first column
  const uint32_t c = (blockIdx.x * (kThreads / 64) + wave) * (16 * C) + col;
  // offset of value v = j M + m
  auto at = [](int v) { return (uint32_t)(16 * (v / M)) + kBlock * (uint32_t)(v % M); };
  const uint32_t aj = map.aj(g), nt = map.targets(g);
  if (4 * blockIdx.y >= nt) return;
  // a ninth digit source (ModDown merged with the rescale: q_{l-1} and eight
  // special primes) is added on the VALU
  const double* d8 = map.digits(g) + (size_t)8 * n + c;  // read only with NINTH (aj = 9)
  // B operands: column col of product v holds value v of sources 2 lg (bytes
  // 0..7) and 2 lg + 1 (bytes 8..15); a source past the digit reads a valid
  // row and contributes zero
  v4i b[16];
  {
    const double* dig = map.digits(g);
    const uint32_t a0 = 2 * lg, a1 = a0 + 1;
    const double* r0 = dig + (size_t)min(a0, aj - 1) * n + c;
    const double* r1 = dig + (size_t)min(a1, aj - 1) * n + c;
    const uint64_t k0 = a0 < aj ? ~0ull : 0ull, k1 = a1 < aj ? ~0ull : 0ull;
    if constexpr (FUSE) {
      double x[16];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t a = min(h ? a1 : a0, aj - 1);
        const double* r = h ? r1 : r0;
#pragma unroll
        for (int v = 0; v < 16; ++v) x[v] = r[at(v)];
        finish_digits<LOGM>(x, map.src_prime(g, a), map.factor(g, a), pk, twi);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const uint64_t p = bal_bytes(x[v]) & (h ? k1 : k0);
          b[v][2 * h] = (int)(uint32_t)p;
          b[v][2 * h + 1] = (int)(uint32_t)(p >> 32);
        }
      }
    } else {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const uint64_t p0 = bal_bytes(r0[at(v)]) & k0, p1 = bal_bytes(r1[at(v)]) & k1;
        b[v] = v4i{(int)(uint32_t)p0, (int)(uint32_t)(p0 >> 32), (int)(uint32_t)p1,
                   (int)(uint32_t)(p1 >> 32)};
      }
    }
  }
  double x8[16];  // the ninth source's digits
  if constexpr (NINTH && FUSE) {
#pragma unroll
    for (int v = 0; v < 16; ++v) x8[v] = d8[at(v)];
    finish_digits<LOGM>(x8, map.src_prime(g, 8), map.factor(g, 8), pk, twi);
  }
  for (uint32_t q0 = 4 * blockIdx.y; q0 < nt; q0 += 4 * gridDim.y) {
    // A operands: product row col = target q0 + col / 4, digit tau = col % 4
    // (first product) or 4 + col % 4 (second)
    const int8_t* tb = map.bytes(g, map.row(g, min(q0 + col / 4, nt - 1)));
    const v4i alo = *reinterpret_cast<const v4i*>(tb + ((col % 4) * 4 + lg) * 16);
    const v4i ahi = *reinterpret_cast<const v4i*>(tb + ((4 + col % 4) * 4 + lg) * 16);
    // this lane's results: target q0 + lg (rows 4 lg .. 4 lg + 3 of each
    // product); in a partial last quad the idle lane groups still join the
    // products (a product needs the whole wavefront) and store nothing
    const uint32_t tt = q0 + lg;
    const uint32_t trow = map.row(g, min(tt, nt - 1));
    const uint32_t prime = map.prime(trow);
    const double q = pk[prime].q, qinv = pk[prime].qinv;
    double2 h8{0.0, 0.0};
    if constexpr (NINTH) h8 = map.hat(g, trow)[8];
    const v4i zero = {0, 0, 0, 0};
    double x[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const v4i dl = __builtin_amdgcn_mfma_i32_16x16x64_i8(alo, b[v], zero, 0, 0, 0);
      const v4i dh = __builtin_amdgcn_mfma_i32_16x16x64_i8(ahi, b[v], zero, 0, 0, 0);
      // R = hi + lo exactly (|lo| < 2^45, |hi| < 2^69), each |Q_tau| <=
      // 64 * 2^14 = 2^20, so digit pairs Q_t + 256 Q_t+1 still fit an int32
      // and are combined before the conversion to fp64; y = R - c q with
      // c = round(R / q), formed exactly (the fma's result is below 2^51)
      const double lo = __builtin_fma((double)(dl[2] + dl[3] * 256), 65536.0,
                                      (double)(dl[0] + dl[1] * 256));
      const double hi = __builtin_fma((double)dh[2], 65536.0, (double)(dh[0] + dh[1] * 256)) *
                        4294967296.0;
      const double cq = __builtin_rint(__builtin_fma(hi, qinv, lo * qinv));
      double r = __builtin_fma(-cq, q, hi) + lo;
      if constexpr (NINTH)  // |r| < 1.2 q before the reduction, 0.5 q without it
        r = red_bal(r + mm_shoup(FUSE ? x8[v] : d8[at(v)], h8.x, h8.y, q), q, qinv);
      x[v] = r;
      // consume each pair of products here: otherwise the combination sinks
      // below the branch on tt and all 32 products (128 registers of
      // results) are held at once
      asm volatile("" : "+v"(x[v]));
    }
    if (tt >= nt) continue;
    if constexpr (LOGM == 0) {
      uint64_t* out = map.out(g, trow);
#pragma unroll
      for (int v = 0; v < 16; ++v) out[c + at(v)] = to_res_2q(x[v], q, qinv);
    } else {
      const double* tw = twf + (size_t)prime * n;
      fwd_columns<LOGM>(x, tw, q, qinv);
      double* outd = reinterpret_cast<double*>(map.out(g, trow));
#pragma unroll
      for (int v = 0; v < 16; ++v) outd[c + at(v)] = x[v];
    }
  }
}

// Three waves per SIMD fit without spilling; the ninth-digit variant keeps
// two (its extra loads would spill at three).
template <int LOGM, bool FUSE, class Map>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3))) void k_bconv_mfma(
    Map map, const PrimeK* __restrict__ pk, const double* __restrict__ twf,
    const double* __restrict__ twi) {
  bconv_mfma<LOGM, Map, false, FUSE>(map, pk, twf, twi);
}

template <int LOGM, bool FUSE, class Map>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_bconv_mfma9(
    Map map, const PrimeK* __restrict__ pk, const double* __restrict__ twf,
    const double* __restrict__ twi) {
  bconv_mfma<LOGM, Map, true, FUSE>(map, pk, twf, twi);
}

// ------------------------------------------------------------- inner pass

// Thread t's values t + 256 r of block B: uint64 residues (SINGLE) or the
// outer pass's fp64 intermediate.
template <bool SINGLE>
__device__ __forceinline__ void fwd_load(const uint64_t* row, uint32_t B, double (&x)[16]) {
  const uint32_t t = threadIdx.x;
  if constexpr (SINGLE) {
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = u2d(row[B + t + 256 * r]);
  } else {
    const double* src = reinterpret_cast<const double*>(row) + B + t;
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = src[256 * r];
  }
}

// An epilogue with nothing to load ahead of the transform.
struct NoPre {};

// Forward 4096-point blocks.  Thread t starts with values t + 256 r (bits
// 11..8 in registers), moves to a*256 + 16 r + b (a = t/16, b = t%16; bits
// 7..4) and to 16 t + r (bits 3..0); fwd_transform ends there.  Each transpose
// writes exactly the LDS words the thread read in the previous one, so only
// the reads need ordering: a barrier of the workgroup for the first and the
// last, the middle one stays inside a wavefront.  The kernel hands values
// t + 256 r to the epilogue.
//
// SINGLE: N = 4096, the pass reads uint64 residues; otherwise it reads the
// outer pass's fp64 intermediate.  No global load is waited on inside the
// transform: its twiddles of bits 11..4 are loaded with the data, those of
// bits 3..0 generated from one loaded power.
template <bool SINGLE, class Epi>
__global__ __launch_bounds__(kThreads) void k_fwd_inner(RowSel rs, uint32_t log_n,
                                                        const PrimeK* __restrict__ pk,
                                                        const double* __restrict__ twf,
                                                        const double* __restrict__ tw3, Epi epi) {
  __shared__ double lds[kLds];
  __shared__ double lt[kTwL];
  if (rs.skip()) return;
  const uint32_t n = 1u << log_n;
  const uint32_t prime = rs.prime();
  const double q = pk[prime].q, qinv = pk[prime].qinv;
  uint64_t* row = rs.row();
  const uint32_t t = threadIdx.x;
  const uint32_t B = blockIdx.x * kBlock;
  const double* tw = twf + (size_t)prime * n;
  UniTw u(tw, n + B);
  const StagedTwiddle st = load_staged(tw, n + B);
  // psi_rev[(N + B) / 2 + 8 t]
  const double b = tw3[((size_t)prime * (n / kBlock) + blockIdx.x) * kThreads + t];
  // operands of the epilogue loaded before the transform, so that their
  // latency overlaps the butterflies
  const typename Epi::Pre pv = epi.pre(B + t, n);
  double x[16];
  fwd_load<SINGLE>(row, B, x);
  u.settle();
  lt[st.at] = st.w;
  fwd_transform(u, lt, b, q, qinv, lds, x);
#pragma unroll
  for (int r = 0; r < 16; ++r) lds[lds_col(t, r)] = x[r];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) x[r] = lds[lds_row(t, r)];
  epi(row, B + t, x, q, qinv, n, pv);
}

// Epilogue of the forward transform: canonical residues, value r at k0 + 256 r.
struct StoreResidues {
  using Pre = NoPre;
  __device__ __forceinline__ Pre pre(uint32_t, uint32_t) const { return {}; }
  __device__ __forceinline__ void operator()(uint64_t* row, uint32_t k0, const double (&x)[16],
                                             double q, double qinv, uint32_t, Pre) const {
#pragma unroll
    for (int r = 0; r < 16; ++r) row[k0 + 256 * r] = to_res_2q(x[r], q, qinv);
  }
};

// Source of the inverse inner pass: the row itself (in place).
struct LoadRow {
  __device__ __forceinline__ void operator()(const uint64_t* row, uint32_t off, double (&x)[16],
                                             double, double) const {
    load16(row + off, x);
  }
};

// Source of the inverse inner pass: rows [blockIdx.y][blockIdx.z][N] of a buffer
// (out of place).
struct LoadFrom {
  const uint64_t* in;
  uint32_t rows, n;
  __device__ __forceinline__ void operator()(const uint64_t*, uint32_t off, double (&x)[16],
                                             double, double) const {
    load16(in + ((size_t)blockIdx.y * rows + blockIdx.z) * n + off, x);
  }
};

// Source of the inverse inner pass: row blockIdx.z of source blockIdx.y of a
// key-switch table (out of place; the row receives the result).  A product
// source (src_y set) is formed here, x y mod q within 0.875 q (mul_bound of two
// canonical operands), inside the bound q from which the inverse stages start.
struct LoadSources {
  KsTable tab;
  __device__ __forceinline__ void operator()(const uint64_t*, uint32_t off, double (&x)[16],
                                             double q, double qinv) const {
    const size_t o = (size_t)blockIdx.z * tab.src_stride[blockIdx.y] + off;
    load16(tab.src_in[blockIdx.y] + o, x);
    if (const uint64_t* y = tab.src_y[blockIdx.y]) {
      double z[16];
      load16(y + o, z);
#pragma unroll
      for (int r = 0; r < 16; ++r) x[r] = mm_var(x[r], z[r], q, qinv);
    }
  }
};

// Inverse 4096-point blocks: the mirror image of k_fwd_inner, with one barrier
// of the workgroup, before the last transpose.  Reads uint64
// residues (16 consecutive values per thread), writes fp64 for the outer pass
// or, if SINGLE, applies the final store St.
template <bool SINGLE, class Ld, class St>
__global__ __launch_bounds__(kThreads) void k_inv_inner(RowSel rs, uint32_t log_n,
                                                        const PrimeK* __restrict__ pk,
                                                        const double* __restrict__ twi,
                                                        const double* __restrict__ tw3, Ld ld,
                                                        St st) {
  __shared__ double lds[kLds];
  __shared__ double lt[kTwL];
  if (rs.skip()) return;
  const uint32_t n = 1u << log_n;
  const uint32_t prime = rs.prime();
  const PrimeK P = pk[prime];
  const double q = P.q, qinv = P.qinv;
  const double* tw = twi + (size_t)prime * n;
  uint64_t* row = rs.row();
  const uint32_t t = threadIdx.x;
  const uint32_t B = blockIdx.x * kBlock;
  UniTw u(tw, n + B);
  const StagedTwiddle sw = load_staged(tw, n + B);
  // psi_rev[(N + B) / 2 + 8 t] (inverse powers)
  const double b1 = tw3[((size_t)prime * (n / kBlock) + blockIdx.x) * kThreads + t];
  double x[16];
  ld(row, B + 16 * t, x, q, qinv);
  u.settle();
  lt[sw.at] = sw.w;
  inv_transform(u, lt, b1, q, qinv, lds, x);
  if constexpr (SINGLE) {
#pragma unroll
    for (int r = 0; r < 16; ++r) st(row, B + t + 256 * r, x[r], P);
  } else {
    double* dst = reinterpret_cast<double*>(row) + B + t;
#pragma unroll
    for (int r = 0; r < 16; ++r) dst[256 * r] = x[r];
  }
}

}  // namespace

// Epilogue fusing the key-switch combine into the forward transform of the
// ModDown conversion y: for u = 2*job + t (blockIdx.y) and limb i
// (blockIdx.z), out_job[i][t] = (acc[u][i] - NTT(y)[u][i]) * P^-1 + adds,
// with the adds of the job table (sigma_g-permuted `add`, plain `add2`).  If
// tab.fold the inner product has already stored acc * P^-1 + add, and only
// NTT(y) * P^-1 is subtracted here.  With qlinv (ModDown merged with the
// rescale, fold only) the difference is also multiplied by q_{level-1}^-1
// before add2 is added.
struct KsCombine {
  KsTable tab;
  const uint64_t* acc;
  const double2* pinv;
  const double2* qlinv;
  uint32_t level, alpha, log_n;
  struct Pre {
    uint64_t a[16];  // acc[u][i] at k0 + 256 r
    uint64_t b[16];  // add2[i][t] there, if given
  };
  __device__ __forceinline__ Pre pre(uint32_t k0, uint32_t n) const {
    const uint32_t u = blockIdx.y, i = blockIdx.z;
    const uint64_t* a = acc + ((size_t)u * (level + alpha) + i) * n + k0;
    const uint64_t* add2 = tab.add2[u >> 1];
    Pre p;
#pragma unroll
    for (int r = 0; r < 16; ++r) p.a[r] = a[256 * r];
    if (add2) {
      add2 += ((size_t)2 * i + (u & 1)) * n + k0;
#pragma unroll
      for (int r = 0; r < 16; ++r) p.b[r] = add2[256 * r];
    }
    return p;
  }
  __device__ __forceinline__ void operator()(uint64_t*, uint32_t k0, const double (&x)[16],
                                             double q, double qinv, uint32_t n,
                                             const Pre& pa) const {
    const uint32_t u = blockIdx.y, i = blockIdx.z, job = u >> 1, t = u & 1;
    const double2 f = pinv[i];
    const size_t o = ((size_t)2 * i + t) * n;
    const bool use_add = (tab.add_mask[job] >> t) & 1u;
    const uint32_t g = tab.add_galois[job];
    const uint64_t* add = use_add ? tab.add[job] + o : nullptr;
    const uint64_t* add2 = tab.add2[job];
    uint64_t* out = tab.out[job] + o;
    if (tab.fold) {
      // |x| < 1.9 q, f < q: the product lies within (0.5 + 0.25 * 1.9) q, so
      // |v| < 2 q, the product with h (and add2) again; a bare v + add2 may not
      const double2 h = qlinv ? qlinv[i] : double2{0.0, 0.0};
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const uint32_t k = k0 + 256 * r;
        double v = u2d(pa.a[r]) - mm_shoup(x[r], f.x, f.y, q);
        if (qlinv) {
          v = mm_shoup(v, h.x, h.y, q);
          if (add2) v += u2d(pa.b[r]);
          out[k] = to_res_2q(v, q, qinv);
        } else {
          out[k] = add2 ? to_res(v + u2d(pa.b[r]), q, qinv) : to_res_2q(v, q, qinv);
        }
      }
      return;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const uint32_t k = k0 + 256 * r;
      double v = mm_shoup(u2d(pa.a[r]) - x[r], f.x, f.y, q);
      if (use_add) v += u2d(add[g ? galois_src(k, g, log_n) : k]);
      if (add2) v += u2d(pa.b[r]);
      out[k] = to_res(v, q, qinv);
    }
  }
};

// Epilogue fusing the rescale combine into the forward transform of the
// lifted last limbs: for u = 2 b + t (blockIdx.y) and limb i (blockIdx.z),
// out_b[i][t] = (in_b[i][t] - NTT(w)[u][i]) * q_last^-1 (+ add_b[i][t]).
// out_b may alias in_b or add_b (same element, same thread).
struct RsCombine {
  RsTable tab;
  const double2* qlinv;
  struct Pre {
    uint64_t in[16], add[16];  // in_b[i][t], add_b[i][t] at k0 + 256 r
  };
  __device__ __forceinline__ Pre pre(uint32_t k0, uint32_t n) const {
    const uint32_t u = blockIdx.y, i = blockIdx.z, b = u >> 1, t = u & 1;
    const size_t o = ((size_t)2 * i + t) * n + k0;
    const uint64_t *in = tab.in[b] + o, *add = tab.add[b];
    Pre p;
#pragma unroll
    for (int r = 0; r < 16; ++r) p.in[r] = in[256 * r];
    if (add) {
#pragma unroll
      for (int r = 0; r < 16; ++r) p.add[r] = (add + o)[256 * r];
    }
    return p;
  }
  __device__ __forceinline__ void operator()(uint64_t*, uint32_t k0, const double (&x)[16],
                                             double q, double qinv, uint32_t n,
                                             const Pre& p) const {
    const uint32_t u = blockIdx.y, i = blockIdx.z, b = u >> 1, t = u & 1;
    const double2 f = qlinv[i];
    uint64_t* out = tab.out[b] + ((size_t)2 * i + t) * n + k0;
    const bool add = tab.add[b];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const double v = mm_shoup(u2d(p.in[r]) - x[r], f.x, f.y, q);  // within 1.3 q
      out[256 * r] = add ? to_res(v + u2d(p.add[r]), q, qinv) : to_res_2q(v, q, qinv);
    }
  }
};

namespace {

hipError_t launch_fwd_outer(const Context* c, const RowSel& rs, uint32_t batch, uint32_t limbs,
                            hipStream_t s) {
  const dim3 grid(c->n / kBlock, batch, limbs), blk(kThreads);
  const double* tw = c->d_tw_fwd;
  switch (c->log_n) {
    case 12: return hipSuccess;
    case 13: hipLaunchKernelGGL(k_fwd_outer<1>, grid, blk, 0, s, rs, c->log_n, c->d_pk, tw); break;
    case 14: hipLaunchKernelGGL(k_fwd_outer<2>, grid, blk, 0, s, rs, c->log_n, c->d_pk, tw); break;
    case 15: hipLaunchKernelGGL(k_fwd_outer<3>, grid, blk, 0, s, rs, c->log_n, c->d_pk, tw); break;
    case 16: hipLaunchKernelGGL(k_fwd_outer<4>, grid, blk, 0, s, rs, c->log_n, c->d_pk, tw); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <class St>
hipError_t launch_inv_outer(const Context* c, const RowSel& rs, uint32_t batch, uint32_t limbs,
                            const St& st, hipStream_t s) {
  const dim3 grid(c->n / kBlock, batch, limbs), blk(kThreads);
  const double* tw = c->d_tw_inv;
  switch (c->log_n) {
    case 12: return hipSuccess;
    case 13: k_inv_outer<1, St><<<grid, blk, 0, s>>>(rs, c->log_n, c->d_pk, tw, st); break;
    case 14: k_inv_outer<2, St><<<grid, blk, 0, s>>>(rs, c->log_n, c->d_pk, tw, st); break;
    case 15: k_inv_outer<3, St><<<grid, blk, 0, s>>>(rs, c->log_n, c->d_pk, tw, st); break;
    case 16: k_inv_outer<4, St><<<grid, blk, 0, s>>>(rs, c->log_n, c->d_pk, tw, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <class Epi>
hipError_t launch_fwd_inner(const Context* c, const RowSel& rs, uint32_t batch, uint32_t limbs,
                            const Epi& epi, hipStream_t s) {
  const uint32_t nblk = c->n / kBlock;
  const dim3 blk(kThreads);
  if (c->log_n == 12) {
    k_fwd_inner<true, Epi><<<dim3(nblk, batch, limbs), blk, 0, s>>>(
        rs, c->log_n, c->d_pk, c->d_tw_fwd, c->d_tw3_fwd, epi);
  } else {
    k_fwd_inner<false, Epi><<<dim3(nblk, batch, limbs), blk, 0, s>>>(
        rs, c->log_n, c->d_pk, c->d_tw_fwd, c->d_tw3_fwd, epi);
  }
  return hipGetLastError();
}

// Inverse transform: inner pass (reading through Ld), then the outer pass; St
// is the final store of whichever pass is last.
template <class Ld, class St>
hipError_t launch_inv_first(const Context* c, const RowSel& rs, uint32_t batch, uint32_t limbs,
                            const Ld& ld, const St& st, hipStream_t s) {
  const dim3 grid(c->n / kBlock, batch, limbs), blk(kThreads);
  if (c->log_n == 12)
    k_inv_inner<true, Ld, St><<<grid, blk, 0, s>>>(rs, c->log_n, c->d_pk, c->d_tw_inv,
                                                    c->d_tw3_inv, ld, st);
  else
    k_inv_inner<false, Ld, St><<<grid, blk, 0, s>>>(rs, c->log_n, c->d_pk, c->d_tw_inv,
                                                     c->d_tw3_inv, ld, st);
  return hipGetLastError();
}
template <class Ld, class St>
hipError_t launch_inverse(const Context* c, const RowSel& rs, uint32_t batch, uint32_t limbs,
                          const Ld& ld, const St& st, hipStream_t s) {
  const hipError_t e = launch_inv_first(c, rs, batch, limbs, ld, st, s);
  if (e != hipSuccess) return e;
  return launch_inv_outer(c, rs, batch, limbs, st, s);
}

// The matrix-core conversion serves the maps that carry its operand tables
// (ModUp, ModDown and ModDown merged with the rescale, with digits of at most
// 8 primes plus at most one on the VALU).
template <class Map>
constexpr bool kMfmaMap = false;
template <>
constexpr bool kMfmaMap<ModupMap> = true;
template <>
constexpr bool kMfmaMap<ModdownMap> = true;
template <>
constexpr bool kMfmaMap<ModdownRescaleMap> = true;

__host__ inline const int8_t* mfma_bytes(const ModupMap& m) { return m.mu_bytes; }
__host__ inline const int8_t* mfma_bytes(const ModdownMap& m) { return m.md_bytes; }
__host__ inline const int8_t* mfma_bytes(const ModdownRescaleMap& m) {
  return m.alpha <= 9 ? m.mr_bytes : nullptr;  // at most one digit past the eight
}

// Digits of fewer primes leave most of the product's 64-deep sums empty and
// cost less as Shoup products on the VALU.  Rotations, matrix cores against
// VALU (one / 30 at a time, us): alpha = 3, N = 2^15: 68 / 534 against
// 66 / 518, N = 2^16: 90 / 1100 against 87 / 1055; alpha = 4, N = 2^14: 60 /
// 360 against 64 / 365, N = 2^16: 98 / 1415 against 99 / 1405; alpha = 8,
// N = 2^12: 49 / 199 against 59 / 235, N = 2^15: 95 / 1339 against 107 / 1452.
constexpr uint32_t kMfmaMinDigit = 4;

template <class Map>
bool on_matrix_cores(const Map& map) {
  if constexpr (kMfmaMap<Map>) return mfma_bytes(map) && map.alpha >= kMfmaMinDigit;
  return false;
}

template <class Map>
uint32_t longest_digit(const Map& map) {
  if constexpr (std::is_same_v<Map, ModupMap>) return std::min(map.alpha, map.level);
  return map.alpha;
}

// Whether a conversion finishes its digits' inverse transform itself, repeating
// the columns in every workgroup that reads them.  On the VALU: valu_conversion.
// On the matrix cores a lane finishes two sources whatever the digit's length;
// it pays while the launch leaves the chip room: one rotation at N = 2^16, 24
// limbs, alpha = 8: 139 -> 130 us, two 244 -> 226 us, not with the chip full (30
// rotations).  (N = 4096 has no outer pass.)
template <class Map>
bool fuse_digits(const Context* c, const Map& map, uint32_t targets, uint32_t groups) {
  const uint32_t M = c->n / kBlock;
  if (M == 1) return false;
  return on_matrix_cores(map)
             ? 4 * M * groups * 2 <= kBconvFill
             : valu_conversion(c->log_n - 12, longest_digit(map), targets, groups).fuse;
}

template <int LOGM, class Map>
hipError_t launch_bconv_logm(const Context* c, const Map& map, uint32_t targets, uint32_t groups,
                             hipStream_t s) {
  constexpr uint32_t M = 1u << LOGM;
  constexpr bool CAN = LOGM > 0;
  const double *tw = c->d_tw_fwd, *ti = c->d_tw_inv;
  const bool fuse = fuse_digits(c, map, targets, groups);
  if constexpr (kMfmaMap<Map>) {
    if (on_matrix_cores(map)) {
      // A batch of one key switch has far fewer (column block, digit) pairs than
      // fill the chip, so its quads of targets go to different workgroups; each of
      // those loads the digits again, from L2: one rotation at N = 2^16, 24 limbs,
      // alpha = 8: 151 -> 138 us.
      const uint32_t quads = (targets + 3) / 4, cols = 4 * M * groups;
      const uint32_t split = std::min(quads, std::max(1u, kBconvFill / cols));
      const dim3 grid(4 * M, split, groups);
      if constexpr (std::is_same_v<Map, ModdownRescaleMap>) {
        if (map.alpha > 8) {  // q_{l-1} and eight special primes
          if (fuse)
            k_bconv_mfma9<LOGM, CAN, Map><<<grid, kThreads, 0, s>>>(map, c->d_pk, tw, ti);
          else
            k_bconv_mfma9<LOGM, false, Map><<<grid, kThreads, 0, s>>>(map, c->d_pk, tw, ti);
          return hipGetLastError();
        }
      }
      if (fuse)
        k_bconv_mfma<LOGM, CAN, Map><<<grid, kThreads, 0, s>>>(map, c->d_pk, tw, ti);
      else
        k_bconv_mfma<LOGM, false, Map><<<grid, kThreads, 0, s>>>(map, c->d_pk, tw, ti);
      return hipGetLastError();
    }
  }
  const ValuConversion v = valu_conversion(LOGM, longest_digit(map), targets, groups);
  const dim3 grid(M, (targets + v.targets - 1) / v.targets, groups);
  if (v.targets == 3)
    k_bconv_outer<LOGM, 3, false, Map><<<grid, kThreads, 0, s>>>(map, c->log_n, c->d_pk, tw, ti);
  else if (fuse)
    k_bconv_outer<LOGM, 1, CAN, Map><<<grid, kThreads, 0, s>>>(map, c->log_n, c->d_pk, tw, ti);
  else
    k_bconv_outer<LOGM, 1, false, Map><<<grid, kThreads, 0, s>>>(map, c->log_n, c->d_pk, tw, ti);
  return hipGetLastError();
}

// Inverse transform of the rows rs selects (read through ld) to the centred
// digits of `map`, and their conversion fused with the targets' first forward
// pass.
template <class Ld, class Map>
hipError_t launch_convert(const Context* c, const RowSel& rs, uint32_t batch, uint32_t limbs,
                          const Ld& ld, const Map& map, uint32_t targets, uint32_t groups,
                          hipStream_t s) {
  const InvDigit st{map.f};
  hipError_t e = launch_inv_first(c, rs, batch, limbs, ld, st, s);
  if (e == hipSuccess && !fuse_digits(c, map, targets, groups))
    e = launch_inv_outer(c, rs, batch, limbs, st, s);
  if (e != hipSuccess) return e;
  switch (c->log_n) {
    case 12: return launch_bconv_logm<0>(c, map, targets, groups, s);
    case 13: return launch_bconv_logm<1>(c, map, targets, groups, s);
    case 14: return launch_bconv_logm<2>(c, map, targets, groups, s);
    case 15: return launch_bconv_logm<3>(c, map, targets, groups, s);
    case 16: return launch_bconv_logm<4>(c, map, targets, groups, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// ModUp of every key-switch source: inverse transform of its first `level` rows
// into cc[s][level][N] (out of place: the first pass reads the sources
// directly) to the centred digits [N^-1 (Q_D/q_i)^-1 x]_{q_i} (fp64), and their
// conversion fused with the first forward pass of the extended rows (own-digit
// rows are not written).
hipError_t launch_modup(const Context* c, const LevelTables& T, const KsTable& tab, uint32_t nsrc,
                        uint64_t* cc, uint64_t* ext, uint32_t level, hipStream_t s) {
  const RowSel rs{cc, (size_t)level * c->n, (size_t)c->n, 0, level, 0, 0, 0, 0};
  const uint32_t dnum_l = (level + c->alpha - 1) / c->alpha;
  const uint32_t aj_min = level - (dnum_l - 1) * c->alpha;
  const ModupMap map{reinterpret_cast<const double*>(cc), ext, T.mu_hat, level, c->L, c->alpha,
                     dnum_l, c->n, T.mu_bytes, T.mu_inv_n};
  return launch_convert(c, rs, nsrc, level, LoadSources{tab}, map, level + c->alpha - aj_min,
                        nsrc * dnum_l, s);
}

// Rescale, steps 1 and 2: inverse transform of nrows single rows under prime
// `last`, row r read from tab.src_in[r], into v[r][N] as centred coefficients
// [N^-1 x]_{q_last} (fp64), and their lift to rows 0 .. rows-1 (a conversion with
// one digit and weight 1) fused with the first forward pass, into w[r][last][N].
hipError_t launch_rescale_lift(const Context* c, const LevelTables& T, const KsTable& tab,
                               uint32_t nrows, uint64_t* v, uint64_t* w, uint32_t last,
                               uint32_t rows, hipStream_t s) {
  const RowSel rs{v, (size_t)c->n, (size_t)c->n, last, 1, 0, 0, 0, 0};
  const RescaleMap map{reinterpret_cast<const double*>(v), w, T.one, last, rows, c->n, T.rs_ninv};
  return launch_convert(c, rs, nrows, 1, LoadSources{tab}, map, rows, nrows, s);
}

// Rescale, step 3: second forward pass of w with the combine
// out_b = (in_b - w) * q_last^-1 (+ add_b) as the epilogue, first `rows` limbs.
hipError_t launch_ntt_fwd_rs_combine(const Context* c, uint64_t* w, uint32_t count, uint32_t last,
                                     uint32_t rows, const RsTable& tab, const double2* qlinv,
                                     hipStream_t s) {
  RowSel rs{w, (size_t)last * c->n, (size_t)c->n, 0, rows, 0, 0, 0, 0};
  return launch_fwd_inner(c, rs, 2 * count, rows, RsCombine{tab, qlinv}, s);
}

// ModDown of the special-prime rows of acc: inverse transform in place to
// centred digits, conversion fused with the first forward pass of y.
hipError_t launch_moddown(const Context* c, const LevelTables& T, uint64_t* acc, uint64_t* y,
                          uint32_t njobs, uint32_t level, hipStream_t s) {
  const size_t n = c->n;
  const RowSel rs{acc + level * n, (level + c->alpha) * n, n, c->L, c->alpha, 0, 0, 0, 0};
  const ModdownMap map{acc, y, T.md_hat, level, c->alpha, c->n, T.md_bytes, T.md_inv_n, c->L};
  return launch_convert(c, rs, 2 * njobs, c->alpha, LoadRow{}, map, level, 2 * njobs, s);
}

// Second forward pass of rows whose first pass has run (launch_modup, the encoder's lift).
hipError_t launch_ntt_fwd_inner_rows(const Context* c, const RowSel& rs, uint32_t batch,
                                     uint32_t limbs, hipStream_t s) {
  return launch_fwd_inner(c, rs, batch, limbs, StoreResidues{}, s);
}

// ModDown merged with the rescale: rows q_{level-1}, p_0 .. p_{alpha-1} (adjacent
// in acc) to the centred digits of M = P q_{level-1}, their conversion to rows 0
// .. rows-1 fused with the first forward pass of y[2*njobs][level-1][N].
hipError_t launch_moddown_rescale(const Context* c, const LevelTables& T, uint64_t* acc,
                                  uint64_t* y, uint32_t njobs, uint32_t level, uint32_t rows,
                                  hipStream_t s) {
  const size_t n = c->n;
  const RowSel rs{acc + (level - 1) * n, (level + c->alpha) * n, n, level - 1, 1, c->L, 0, 0, 0};
  const ModdownRescaleMap map{acc,  y,    T.mr_hat,   level,      level + c->alpha, c->alpha + 1,
                              rows, c->n, T.mr_bytes, T.mr_inv_n, c->L};
  return launch_convert(c, rs, 2 * njobs, c->alpha + 1, LoadRow{}, map, rows, 2 * njobs, s);
}

// Second forward pass of the ModDown conversions y[2*njobs][ystride][N]
// (first pass: launch_moddown or launch_moddown_rescale) with the
// key-switch combine as the epilogue; writes rows 0 .. rows-1 of the jobs'
// outputs.  qlinv: null, or q_{level-1}^-1 per row (merged rescale).
hipError_t launch_ntt_fwd_ks_combine(const Context* c, uint64_t* y, uint32_t njobs,
                                     uint32_t level, uint32_t rows, uint32_t ystride,
                                     const KsTable& tab, const uint64_t* acc,
                                     const double2* pinv, const double2* qlinv, hipStream_t s) {
  RowSel rs{y, (size_t)ystride * c->n, (size_t)c->n, 0, rows, 0, 0, 0, 0};
  return launch_fwd_inner(c, rs, 2 * njobs, rows,
                          KsCombine{tab, acc, pinv, qlinv, level, c->alpha, c->log_n}, s);
}

// (Splitting a large batch into cache-sized chunks, so that the second pass
// would read the first pass's output back from the 256 MB Infinity Cache, a launch
// per pass and chunk, measured no faster than one launch per pass over the whole
// batch.  With a chunk's second pass and the next one's first in one launch 64 x 24
// limbs gained 3%, 1463 -> 1413 us with the MAC, and 25 x 24 lost 6%, 550 -> 584; not
// taken.)
hipError_t launch_ntt_rows(const Context* c, const RowSel& rs, uint32_t batch, uint32_t limbs,
                           bool inverse, hipStream_t s) {
  if (inverse) return launch_inverse(c, rs, batch, limbs, LoadRow{}, InvCanon{}, s);
  hipError_t e = launch_fwd_outer(c, rs, batch, limbs, s);
  if (e != hipSuccess) return e;
  return launch_fwd_inner(c, rs, batch, limbs, StoreResidues{}, s);
}

// Inverse transform of in[batch][limbs][N] into out (primes 0 .. limbs - 1).
hipError_t launch_ntt_inv_from(const Context* c, const uint64_t* in, uint64_t* out, uint32_t batch,
                               uint32_t limbs, hipStream_t s) {
  RowSel rs{out, (size_t)limbs * c->n, (size_t)c->n, 0, limbs, 0, 0, 0, 0};
  return launch_inverse(c, rs, batch, limbs, LoadFrom{in, limbs, c->n}, InvCanon{}, s);
}

hipError_t launch_ntt(const Context* c, uint64_t* d, uint32_t batch, size_t batch_stride,
                      uint32_t limbs, size_t limb_stride, uint32_t prime0, bool inverse,
                      hipStream_t s) {
  RowSel rs{d, batch_stride, limb_stride, prime0, limbs, 0, 0, 0, 0};
  return launch_ntt_rows(c, rs, batch, limbs, inverse, s);
}

}  // namespace fesc
