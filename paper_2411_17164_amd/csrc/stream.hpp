// Wave-private chains with streamed weights (BF16, H = 256 and 512; see
// chain.hpp).
//
// At these widths the weights do not fit in LDS.  The workgroup's waves walk
// the same sequence of weight slabs (the MFMA fragments of one 32-wide k chunk,
// 16 or 32 KiB), which travel from L2 straight into a ring of four LDS slots,
// three slabs ahead of their use; one barrier per slab.  A wave's rows,
// accumulators and LayerNorm stay in its registers.
#pragma once

#include "chain.hpp"

namespace xmgn {

// A sequence of S weight slabs in global memory, in fragment order (k chunk by
// k chunk, block by block, 1 KiB each), cycled through by a workgroup of NW
// waves by way of a ring of four slots in LDS.  For every slab s: begin(s)
// sends slab s + 3 (of the next cycle past the end) on its way into the slot
// that slab s - 1 left, the products read frags(s), and end(s) makes slab
// s + 1 whole for every wave.
//
// The loads go to LDS without passing through registers, so the compiler does
// not track them; end() waits by count.  Memory operations of a wave complete
// in order, so `2 K newer ones may be outstanding` (K of each of the two slabs
// behind s + 1) never waits too little; other loads and stores in between only
// make it wait for more.  At the end of a product (slabs [s0, s1), back to
// back) it waits for everything, so that the first two slabs of the next need
// no wait behind the loads and stores between the products.
template <int NW, int S, int MBS>
struct WStream {
  static constexpr int SLAB = MBS * 1024, K = MBS / NW;  // K loads of 1 KiB per wave and slab
  static_assert(S % 4 == 0, "a slab's slot is s % 4");
  const unsigned char* base;  // (uniform)
  unsigned char* ring;        // LDS, 4 SLAB bytes
  __device__ __forceinline__ void send(int s) const {
    const int w = __builtin_amdgcn_readfirstlane(wave_id()) * K;
    const unsigned char* g = base + (size_t)(s % S) * SLAB + w * 1024;
    const unsigned dst = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)(ring) + (s & 3) * SLAB + w * 1024;
#pragma unroll
    for (int k = 0; k < K; ++k)
      asm volatile(
          "s_mov_b32 m0, %0\n\t"
          "s_nop 0\n\t"
          "global_load_lds_dwordx4 %1, %2"
          :
          : "s"(dst + k * 1024), "v"(lane_id() * 16), "s"(g + k * 1024)
          : "memory", "m0");
  }
  __device__ __forceinline__ void start() const {  // slabs 0, 1 and 2, whole at the next barrier
    send(0);
    send(1);
    send(2);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  __device__ __forceinline__ void begin(int s) const { send(s + 3); }
  __device__ __forceinline__ void end(int s, int s0, int s1) const {
    if (s == s1 - 1)
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else if (s >= s0 + 2) {
      if constexpr (K == 2)
        asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
      else
        asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
    }
    lds_sync();
  }
  __device__ __forceinline__ const bf16x8* frags(int s) const { return (const bf16x8*)(ring + (s & 3) * SLAB); }
  static_assert(K == 2 || K == 8, "waits are written for these counts");
};

// acc[t][mb] += W x over one k chunk; fragments are read D ahead of their
// products.
template <int ET, int MBS>
__device__ __forceinline__ void slab_gemm(f32x4 (&acc)[ET][MBS], const bf16x8* f, const bf16x8 (&x)[ET]) {
  constexpr int D = 6, N = MBS;
  f += lane_id();
  bf16x8 a[D];
#pragma unroll
  for (int i = 0; i < D; ++i) a[i] = f[i * 64];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const bf16x8 cur = a[i % D];
    if (i + D < N) a[i % D] = f[(i + D) * 64];
#pragma unroll
    for (int t = 0; t < ET; ++t) acc[t][i] = mma(cur, x[t], acc[t][i]);
  }
  __builtin_amdgcn_sched_group_barrier(0x100, D, 0);  // DS reads
#pragma unroll
  for (int i = 0; i < N - D; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, ET, 0);  // MFMA
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
  }
  __builtin_amdgcn_sched_group_barrier(0x008, D * ET, 0);
  __builtin_amdgcn_sched_barrier(0);
}

// LayerNorm of a row of H in the accumulator layout (in place -> xhat),
// returning 1 / std: (mean, M2) of each span of SW features, merged pairwise;
// every sum in the order ln_normalize takes it with H / SW waves.
template <int H, int SW>
__device__ __forceinline__ float ln_chain(f32x4 (&u)[H / 16], float eps) {
  constexpr int NS = H / SW, NB = SW / 16;
  float mw[NS], q[NS];
#pragma unroll
  for (int w = 0; w < NS; ++w) {
    float a[4], d[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      a[r] = u[NB * w][r] + u[NB * w + 1][r];
#pragma unroll
      for (int nb = 2; nb < NB; ++nb) a[r] += u[NB * w + nb][r];
    }
    mw[w] = add_xor32(add_xor16((a[0] + a[1]) + (a[2] + a[3]))) * (1.f / SW);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float d0 = u[NB * w][r] - mw[w], d1 = u[NB * w + 1][r] - mw[w];
      d[r] = __builtin_fmaf(d0, d0, d1 * d1);
#pragma unroll
      for (int nb = 2; nb < NB; ++nb) {
        const float dn = u[NB * w + nb][r] - mw[w];
        d[r] = __builtin_fmaf(dn, dn, d[r]);
      }
    }
    q[w] = add_xor32(add_xor16((d[0] + d[1]) + (d[2] + d[3])));
  }
  float mean = mw[0];
#pragma unroll
  for (int w = 1; w < NS; ++w) mean += mw[w];
  mean *= 1.f / NS;
  float m2 = 0.f;
#pragma unroll
  for (int w = 0; w < NS; ++w) {
    const float dm = mw[w] - mean;
    m2 += __builtin_fmaf((float)SW * dm, dm, q[w]);
  }
  const float inv = rsqrtf(__builtin_fmaf(m2, 1.f / H, eps));
#pragma unroll
  for (int mb = 0; mb < H / 16; ++mb)
#pragma unroll
    for (int r = 0; r < 4; ++r) u[mb][r] = (u[mb][r] - mean) * inv;
  return inv;
}

}  // namespace xmgn
