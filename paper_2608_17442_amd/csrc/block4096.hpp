// The 12 NTT stages inside a 4096-value block, one block per 256-thread workgroup:
// the inner passes of the transforms (ntt.hip), and, a row of N = 4096 being one
// block, the whole transform inside the fused kernels of small_ring.hip.
#pragma once

#include "butterfly.hpp"
#include "fesc_internal.hpp"

namespace fesc {

constexpr int kThreads = 256;
constexpr uint32_t kBlock = 4096;

// LDS layout of a 4096-value block: one pad word after every 16 values, so
// value k sits at k + k/16.  All three access patterns below then reduce to a
// per-thread base plus a compile-time offset (no address arithmetic per
// access), and 16 consecutive lanes always hit 16 distinct 8-byte bank slots.
//   lds_row(t, r):    value t + 256 r        (bits 11..8 in registers)
//   lds_mid(a, b, r): value 256 a + 16 r + b (bits 7..4 in registers)
//   lds_col(t, r):    value 16 t + r         (bits 3..0 in registers)
__device__ __forceinline__ uint32_t lds_row(uint32_t t, uint32_t r) {
  return (t + (t >> 4)) + 272 * r;
}
__device__ __forceinline__ uint32_t lds_mid(uint32_t a, uint32_t b, uint32_t r) {
  return (272 * a + b) + 17 * r;
}
__device__ __forceinline__ uint32_t lds_col(uint32_t t, uint32_t r) { return 17 * t + r; }
constexpr int kLds = kBlock + kBlock / 16;

// Inner passes, twiddles.  For index bits 11..8 (register distance H, distance
// 256 H) the group twiddle is psi_rev[(N + B) / 512H + gi] (B the block offset in
// the row): the same for the whole workgroup, so it comes through the scalar
// cache into scalar registers (TwU).  For bits 7..4 (distance 16 H) with a =
// bits 11..8 of the thread's values it is psi_rev[(N + B) / 32H + a * 8/H + gi].
// A wavefront holds the values of four a's, so it stages its own 60 of them in
// LDS (TwL) and no barrier of the workgroup stands before their use: entry
// 2^k + a 2^(k-4) + gi - 1 (k = 4 + log2(8/H)) is psi_rev[(N + B) / 2^(12 - k) +
// a 2^(k-4) + gi].
constexpr int kTwL = 255;
struct StagedTwiddle {
  double w;
  uint32_t at;
};
__device__ __forceinline__ StagedTwiddle load_staged(const double* tw, uint32_t nb) {
  const uint32_t wave = threadIdx.x >> 6, lane = min(threadIdx.x & 63, 59u);
  const uint32_t k = 4 + (31 - __builtin_clz(lane / 4 + 1));  // 4, 8, 16, 32 lanes
  const uint32_t i = lane + 4 - (1u << (k - 2)) + (wave << (k - 2));
  return {tw[(nb >> (12 - k)) + i], (1u << k) - 1 + i};
}
struct TwL {
  const double* lt;
  uint32_t off;
  __device__ __forceinline__ double operator()(int gi) const { return lt[off + gi]; }
};
// Uniform twiddles in scalar registers: the 15 of bits 11..8 (entry 2^k - 1 +
// gi: psi_rev[(N + B) / 2^(12 - k) + gi], k = log2(8/H)) and psi_rev[1..7].
struct UniTw {
  double top[15], c[7];
  __device__ __forceinline__ UniTw(const double* tw, uint32_t nb) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int i = 0; i < (1 << k); ++i) top[(1 << k) - 1 + i] = tw[(nb >> (12 - k)) + i];
#pragma unroll
    for (int i = 0; i < 7; ++i) c[i] = tw[i + 1];
  }
  // waits for them here, where the block's values are still on their way,
  // instead of between the butterflies
  __device__ __forceinline__ void settle() {
#pragma unroll
    for (int i = 0; i < 15; ++i) asm volatile("" : "+s"(top[i]));
#pragma unroll
    for (int i = 0; i < 7; ++i) asm volatile("" : "+s"(c[i]));
  }
};
struct TwU {
  const double* w;
  __device__ __forceinline__ double operator()(int gi) const { return w[gi]; }
};

// Orders a wavefront's LDS accesses where its lanes exchange values among
// themselves (the hardware performs them in program order).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Bits 3..0, generated instead of loaded: thread t's 16 consecutive values
// are positions 16 j + r with j = (N + B) / 16 + t; brv(j) has its three low
// bits clear, so psi_rev[j 8/H + gi] = psi_rev[j 8/H] psi_rev[gi] and
// psi_rev[j 8/H] = b^(8/H) with b = psi_rev[8 j].  The products are used as they
// come, within kTwGen q.
struct TwGen {
  double base;      // psi_rev[j 8/H]
  const double* c;  // psi_rev[1..7] (uniform)
  double q, qinv;
  __device__ __forceinline__ double operator()(int gi) const {
    return gi == 0 ? base : mm_var(base, c[gi - 1], q, qinv);
  }
};

// The 12 forward stages: thread t comes with the values t + 256 r of the block in
// x[r] and ends with those at 16 t + r.  u: the uniform twiddles, lt: the staged ones
// (written before the first barrier), b: psi_rev[(N + B) / 2 + 8 t].  Uses all of
// `lds`; the caller needs a barrier before touching it again unless it only
// writes the words it is handed (positions 16 t + r).
__device__ __forceinline__ void fwd_transform(const UniTw& u, const double* lt, double b,
                                              double q, double qinv, double* lds,
                                              double (&x)[16]) {
  const uint32_t t = threadIdx.x, a = t >> 4, bb = t & 15;
  // bits 11..8
  ct_st<8, kCtRed[0]>(x, TwU{u.top}, q, qinv);
  ct_st<4, kCtRed[1]>(x, TwU{u.top + 1}, q, qinv);
  ct_st<2, kCtRed[2]>(x, TwU{u.top + 3}, q, qinv);
  ct_st<1, kCtRed[3]>(x, TwU{u.top + 7}, q, qinv);
#pragma unroll
  for (int r = 0; r < 16; ++r) lds[lds_row(t, r)] = x[r];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) x[r] = lds[lds_mid(a, bb, r)];
  // bits 7..4
  ct_st<8, kCtRed[4]>(x, TwL{lt, 15 + a}, q, qinv);
  ct_st<4, kCtRed[5]>(x, TwL{lt, 31 + 2 * a}, q, qinv);
  ct_st<2, kCtRed[6]>(x, TwL{lt, 63 + 4 * a}, q, qinv);
  ct_st<1, kCtRed[7]>(x, TwL{lt, 127 + 8 * a}, q, qinv);
  // the 16 threads of one a exchange their 256 values: one wavefront
#pragma unroll
  for (int r = 0; r < 16; ++r) lds[lds_mid(a, bb, r)] = x[r];
  wave_sync();
#pragma unroll
  for (int r = 0; r < 16; ++r) x[r] = lds[lds_col(t, r)];
  // bits 3..0
  const double b2 = mm_var(b, b, q, qinv), b4 = mm_var(b2, b2, q, qinv);
  ct_st<8, kCtRed[8]>(x, TwGen{mm_var(b4, b4, q, qinv), u.c, q, qinv}, q, qinv);
  ct_st<4, kCtRed[9]>(x, TwGen{b4, u.c, q, qinv}, q, qinv);
  ct_st<2, kCtRed[10]>(x, TwGen{b2, u.c, q, qinv}, q, qinv);
  ct_st<1, kCtRed[11]>(x, TwGen{b, u.c, q, qinv}, q, qinv);
}

// The 12 inverse stages, the mirror image: from values 16 t + r (canonical
// residues or less than q in magnitude) to values t + 256 r, below kGsB2 q.  lt is
// written and read within each wavefront.
__device__ __forceinline__ void inv_transform(const UniTw& u, const double* lt, double b1, double q,
                                              double qinv, double* lds, double (&x)[16]) {
  const uint32_t t = threadIdx.x, a = t >> 4, bb = t & 15;
  // bits 3..0
  const double b2 = mm_var(b1, b1, q, qinv), b4 = mm_var(b2, b2, q, qinv);
  gs_st<1, kGs0.m[0]>(x, TwGen{b1, u.c, q, qinv}, q, qinv);
  gs_st<2, kGs0.m[1]>(x, TwGen{b2, u.c, q, qinv}, q, qinv);
  gs_st<4, kGs0.m[2]>(x, TwGen{b4, u.c, q, qinv}, q, qinv);
  gs_st<8, kGs0.m[3]>(x, TwGen{mm_var(b4, b4, q, qinv), u.c, q, qinv}, q, qinv);
#pragma unroll
  for (int r = 0; r < 16; ++r) lds[lds_col(t, r)] = x[r];
  wave_sync();
#pragma unroll
  for (int r = 0; r < 16; ++r) x[r] = lds[lds_mid(a, bb, r)];
  // bits 7..4
  gs_st<1, kGs1.m[0]>(x, TwL{lt, 127 + 8 * a}, q, qinv);
  gs_st<2, kGs1.m[1]>(x, TwL{lt, 63 + 4 * a}, q, qinv);
  gs_st<4, kGs1.m[2]>(x, TwL{lt, 31 + 2 * a}, q, qinv);
  gs_st<8, kGs1.m[3]>(x, TwL{lt, 15 + a}, q, qinv);
#pragma unroll
  for (int r = 0; r < 16; ++r) lds[lds_mid(a, bb, r)] = x[r];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) x[r] = lds[lds_row(t, r)];
  // bits 11..8
  gs_st<1, kGs2.m[0]>(x, TwU{u.top + 7}, q, qinv);
  gs_st<2, kGs2.m[1]>(x, TwU{u.top + 3}, q, qinv);
  gs_st<4, kGs2.m[2]>(x, TwU{u.top + 1}, q, qinv);
  gs_st<8, kGs2.m[3]>(x, TwU{u.top}, q, qinv);
}

// 16 consecutive residues at p, in 16-byte loads.  Callers' buffers are as aligned as
// their 64-bit words, which is all that the loads ask for.
typedef uint64_t u64x2 __attribute__((ext_vector_type(2), aligned(8)));
__device__ __forceinline__ void load16(const uint64_t* p, double (&x)[16]) {
  const u64x2* v = reinterpret_cast<const u64x2*>(p);
#pragma unroll
  for (int r = 0; r < 16; r += 2) {
    const u64x2 w = v[r / 2];
    x[r] = u2d(w.x);
    x[r + 1] = u2d(w.y);
  }
}

}  // namespace fesc
