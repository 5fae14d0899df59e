// Key switching and rescaling at N = 4096 in few launches.  A row of this ring is
// one 4096-value block, so a workgroup can hold a whole row through an inverse
// transform, a basis conversion and a forward transform.  The general pipeline
// (ntt.hip, keyswitch.hip) takes seven launches of a few workgroups each here,
// whose latency (launch, loads, one transform, stores: 3 to 9 us) is all that a
// small batch costs: one rotation over 3 + 1 primes 40 us.  Fused:
//   k_small_modup    inverse transform of the digit's rows, ModUp to one target
//                    row, forward transform (the digit's rows are transformed
//                    again for every target);
//   k_small_moddown  the same from the special primes (and q_{l-1} when merged with
//                    the rescale) to one level row, ending in the combine.
// The key inner product stays a launch of its own between them: it has 16 times
// the threads that way, and held by the workgroups of a transform (which saves a
// launch more) its loads took longer than the launch, 45 us for that rotation.
// The same residues: every step is exact modulo its prime.  The repeated
// transforms pay while the launches are small (kSmallFill) and at most three primes
// are converted; larger batches take the general pipeline.
#include "block4096.hpp"
#include "fesc_internal.hpp"
#include "ops.hpp"
#include "small_ring_rule.hpp"

namespace fesc {

namespace {

constexpr uint32_t kN = 4096;

// Twiddle tables of one direction.  The kernels take the pointers by themselves,
// __restrict__: the uniform twiddles stay scalar loads behind a barrier then.
struct Tables {
  const double *tw, *tw3;
};

// x: values 16 t + r under the prime -> values t + 256 r.  again: the LDS has been
// read by other wavefronts since the workgroup started.
__device__ __forceinline__ void inverse_row(const Tables& T, uint32_t prime, const PrimeK& P,
                                            double* lds, double* lt, bool again, double (&x)[16]) {
  const double* tw = T.tw + (size_t)prime * kN;
  UniTw u(tw, kN);
  const StagedTwiddle st = load_staged(tw, kN);
  const double b = T.tw3[(size_t)prime * kThreads + threadIdx.x];
  u.settle();
  if (again) __syncthreads();
  lt[st.at] = st.w;
  wave_sync();
  inv_transform(u, lt, b, P.q, P.qinv, lds, x);
}

// x: values t + 256 r -> transform, values t + 256 r (below 1.9 q).
__device__ __forceinline__ void forward_row(const Tables& T, uint32_t prime, const PrimeK& P,
                                            double* lds, double* lt, bool again, double (&x)[16]) {
  const uint32_t t = threadIdx.x;
  const double* tw = T.tw + (size_t)prime * kN;
  UniTw u(tw, kN);
  const StagedTwiddle st = load_staged(tw, kN);
  const double b = T.tw3[(size_t)prime * kThreads + t];
  u.settle();
  if (again) __syncthreads();
  lt[st.at] = st.w;
  fwd_transform(u, lt, b, P.q, P.qinv, lds, x);
#pragma unroll
  for (int r = 0; r < 16; ++r) lds[lds_col(t, r)] = x[r];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) x[r] = lds[lds_row(t, r)];
}

// Row a of source s of the table, values 16 t + r (a product source formed here).
__device__ __forceinline__ void load_source(const KsTable& tab, uint32_t s, uint32_t a,
                                            const PrimeK& P, double (&x)[16]) {
  const size_t o = (size_t)a * tab.src_stride[s] + 16 * threadIdx.x;
  load16(tab.src_in[s] + o, x);
  if (const uint64_t* y = tab.src_y[s]) {
    double z[16];
    load16(y + o, z);
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = mm_var(x[r], z[r], P.q, P.qinv);
  }
}

// Target row blockIdx.x (of those outside the digit) of digit g = blockIdx.y =
// source * dnum + j.
__global__ __launch_bounds__(kThreads) void k_small_modup(KsTable tab, uint64_t* __restrict__ ext,
                                                          uint32_t level, uint32_t L,
                                                          uint32_t alpha, uint32_t dnum,
                                                          const double2* __restrict__ hat,
                                                          const double2* __restrict__ f,
                                                          const PrimeK* __restrict__ pk,
                                                          const double* __restrict__ itw,
                                                          const double* __restrict__ itw3,
                                                          const double* __restrict__ ftw,
                                                          const double* __restrict__ ftw3) {
  const Tables inv{itw, itw3}, fwd{ftw, ftw3};
  __shared__ double lds[kLds];
  __shared__ double lt[kTwL];
  const uint32_t g = blockIdx.y, s = g / dnum, j = g % dnum, t = threadIdx.x;
  const uint32_t E = level + alpha, lo = j * alpha, aj = min(alpha, level - lo);
  if (blockIdx.x >= E - aj) return;
  const uint32_t row = blockIdx.x < lo ? blockIdx.x : blockIdx.x + aj;
  const uint32_t prime = row < level ? row : L + (row - level);
  const PrimeK M = pk[prime];
  double y[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) y[r] = 0.0;
  for (uint32_t a = 0; a < aj; ++a) {
    const PrimeK P = pk[lo + a];
    const double2 c = f[lo + a], h = hat[((size_t)j * E + row) * alpha + a];
    double x[16];
    load_source(tab, s, lo + a, P, x);
    inverse_row(inv, lo + a, P, lds, lt, a > 0, x);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const double d = red_bal(mm_shoup(x[r], c.x, c.y, P.q), P.q, P.qinv);  // centred digit
      y[r] += mm_shoup(d, h.x, h.y, M.q);
    }
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) y[r] = red_bal(y[r], M.q, M.qinv);
  forward_row(fwd, prime, M, lds, lt, true, y);
  uint64_t* out = ext + ((size_t)g * E + row) * kN + t;
#pragma unroll
  for (int r = 0; r < 16; ++r) out[256 * r] = to_res_2q(y[r], M.q, M.qinv);
}

// ModDown: component blockIdx.y & 1 of job blockIdx.y / 2 to level row blockIdx.x:
// out = (F - y P^-1) (times q_{l-1}^-1 when merged) + add2, F the folded inner
// product of that row in acc, y the conversion of the special-prime rows (before
// them q_{l-1} when merged), transformed here.
__global__ __launch_bounds__(kThreads) void k_small_moddown(
    KsTable tab, const uint64_t* __restrict__ acc, uint32_t level, uint32_t L, uint32_t alpha,
    uint32_t merged, const double2* __restrict__ pinv, const double2* __restrict__ qlinv,
    const double2* __restrict__ hat, const double2* __restrict__ f, const PrimeK* __restrict__ pk,
    const double* __restrict__ itw, const double* __restrict__ itw3,
    const double* __restrict__ ftw, const double* __restrict__ ftw3) {
  const Tables inv{itw, itw3}, fwd{ftw, ftw3};
  __shared__ double lds[kLds];
  __shared__ double lt[kTwL];
  const uint32_t t = threadIdx.x, i = blockIdx.x, comp = blockIdx.y & 1u, job = blockIdx.y >> 1;
  const uint32_t first = level - merged, nd = alpha + merged;
  const PrimeK M = pk[i];
  const uint64_t* rows = acc + (size_t)blockIdx.y * (level + alpha) * kN;
  double y[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) y[r] = 0.0;
  for (uint32_t a = 0; a < nd; ++a) {  // at most three digits: below 2 q
    const uint32_t row = first + a, prime = row < level ? row : L + (row - level);
    const PrimeK P = pk[prime];
    const double2 c = f[a], h = hat[(size_t)i * nd + a];
    double x[16];
    load16(rows + (size_t)row * kN + 16 * t, x);
    inverse_row(inv, prime, P, lds, lt, a > 0, x);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const double d = red_bal(mm_shoup(x[r], c.x, c.y, P.q), P.q, P.qinv);  // centred digit
      y[r] += mm_shoup(d, h.x, h.y, M.q);
    }
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) y[r] = red_bal(y[r], M.q, M.qinv);
  const size_t o = ((size_t)2 * i + comp) * kN + t;
  const uint64_t* add2 = tab.add2[job];
  uint64_t* out = tab.out[job] + o;
  uint64_t F[16], A[16];  // on their way during the transform
#pragma unroll
  for (int r = 0; r < 16; ++r) F[r] = rows[(size_t)i * kN + t + 256 * r];
  if (add2) {
#pragma unroll
    for (int r = 0; r < 16; ++r) A[r] = add2[o + 256 * r];
  }
  forward_row(fwd, i, M, lds, lt, true, y);
  const double2 p = pinv[i], h = merged ? qlinv[i] : double2{0.0, 0.0};
#pragma unroll
  for (int r = 0; r < 16; ++r) {  // |v| < 2 q before add2
    double v = u2d(F[r]) - mm_shoup(y[r], p.x, p.y, M.q);
    if (merged) v = mm_shoup(v, h.x, h.y, M.q);
    if (add2) v += u2d(A[r]);
    out[256 * r] = to_res(v, M.q, M.qinv);
  }
}

// Rescale: row blockIdx.x of component blockIdx.y & 1 of ciphertext blockIdx.y / 2:
// inverse transform of the last limb, lift, forward transform, combine.
__global__ __launch_bounds__(kThreads) void k_small_rescale(RsTable tab, uint32_t last,
                                                            const double2* __restrict__ ninv,
                                                            const double2* __restrict__ qlinv,
                                                            const PrimeK* __restrict__ pk,
                                                            const double* __restrict__ itw,
                                                            const double* __restrict__ itw3,
                                                            const double* __restrict__ ftw,
                                                            const double* __restrict__ ftw3) {
  const Tables inv{itw, itw3}, fwd{ftw, ftw3};
  __shared__ double lds[kLds];
  __shared__ double lt[kTwL];
  const uint32_t t = threadIdx.x, i = blockIdx.x, comp = blockIdx.y & 1u, b = blockIdx.y >> 1;
  const PrimeK P = pk[last], M = pk[i];
  const size_t o = ((size_t)2 * i + comp) * kN + t;
  const uint64_t *in = tab.in[b], *add = tab.add[b];
  double x[16];
  load16(in + ((size_t)2 * last + comp) * kN + 16 * t, x);
  uint64_t c[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) c[r] = in[o + 256 * r];
  inverse_row(inv, last, P, lds, lt, false, x);
  const double2 f = ninv[0], h = qlinv[i];
#pragma unroll
  for (int r = 0; r < 16; ++r)  // centred coefficient, reduced for the row
    x[r] = red_bal(red_bal(mm_shoup(x[r], f.x, f.y, P.q), P.q, P.qinv), M.q, M.qinv);
  forward_row(fwd, i, M, lds, lt, true, x);
  uint64_t* out = tab.out[b] + o;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    double v = mm_shoup(u2d(c[r]) - x[r], h.x, h.y, M.q);
    if (add) v += u2d(add[o + 256 * r]);
    out[256 * r] = to_res(v, M.q, M.qinv);
  }
}

}  // namespace

bool small_modup_fits(const Context* c, uint32_t nsrc, uint32_t level) {
  return small_modup_pays(c->log_n, c->alpha, nsrc, level);
}

hipError_t launch_small_modup(const Context* c, const LevelTables& T, const KsTable& tab,
                              uint32_t nsrc, uint64_t* ext, uint32_t level, hipStream_t s) {
  const uint32_t dnum = (level + c->alpha - 1) / c->alpha;
  k_small_modup<<<dim3(level + c->alpha, nsrc * dnum), kThreads, 0, s>>>(
      tab, ext, level, c->L, c->alpha, dnum, T.mu_hat, T.mu_inv_n, c->d_pk, c->d_tw_inv,
      c->d_tw3_inv, c->d_tw_fwd, c->d_tw3_fwd);
  return hipGetLastError();
}

bool small_moddown_fits(const Context* c, const KsTable& t, uint32_t njobs, uint32_t level,
                        uint32_t rescale_rows) {
  return t.fold == 1 && small_moddown_pays(c->log_n, c->alpha, rescale_rows != 0, njobs,
                                           rescale_rows ? rescale_rows : level);
}

hipError_t launch_small_moddown(const Context* c, const LevelTables& T, const KsTable& tab,
                                uint32_t njobs, const uint64_t* acc, uint32_t level,
                                uint32_t rescale_rows, hipStream_t s) {
  const uint32_t merged = rescale_rows ? 1 : 0;
  k_small_moddown<<<dim3(merged ? rescale_rows : level, 2 * njobs), kThreads, 0, s>>>(
      tab, acc, level, c->L, c->alpha, merged, T.md_pinv, T.rs_inv, merged ? T.mr_hat : T.md_hat,
      merged ? T.mr_inv_n : T.md_inv_n, c->d_pk, c->d_tw_inv, c->d_tw3_inv, c->d_tw_fwd,
      c->d_tw3_fwd);
  return hipGetLastError();
}

bool small_rescale_fits(const Context* c, const RsTable& t, uint32_t count, uint32_t last,
                        uint32_t rows) {
  if (!small_rescale_pays(c->log_n, count, rows)) return false;
  for (uint32_t i = 0; i < count; ++i)  // every row's workgroup reads the last limbs
    for (uint32_t j = 0; j < count; ++j)
      if (overlap(t.out[i], (size_t)2 * rows * kN, t.in[j] + (size_t)2 * last * kN, 2 * kN))
        return false;
  return true;
}

hipError_t launch_small_rescale(const Context* c, const LevelTables& T, const RsTable& tab,
                                uint32_t count, uint32_t last, uint32_t rows, hipStream_t s) {
  k_small_rescale<<<dim3(rows, 2 * count), kThreads, 0, s>>>(
      tab, last, T.rs_ninv, T.rs_inv, c->d_pk, c->d_tw_inv, c->d_tw3_inv, c->d_tw_fwd,
      c->d_tw3_fwd);
  return hipGetLastError();
}

}  // namespace fesc
