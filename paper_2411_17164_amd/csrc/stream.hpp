// Wave-private chains with streamed weights (see chain.hpp): BF16 at H = 256
// and 512, FP32 at H = 128 and 256.
//
// In these forms the weights do not fit in LDS.  The workgroup's waves walk
// the same sequence of weight slabs (the MFMA fragments of one or two k chunks,
// 16 or 32 KiB), which travel from L2 straight into a ring of four LDS slots,
// three slabs ahead of their use; one barrier per slab.  A wave's rows,
// accumulators and LayerNorm stay in its registers.
#pragma once

#include "chain.hpp"

namespace xmgn {

// One k chunk of a row's operand: 16 bytes per lane, features KW c + E g .. + E
// - 1 (g = lane / 16).  BF16: a 32-feature chunk, two accumulator blocks; FP32:
// 16 features, where the operand is the accumulator block itself.
template <typename T>
struct Chunk;
template <>
struct Chunk<bf16> {
  using V = bf16x8;
  static constexpr int KW = 32, E = 8, BLK = 2, MF = 1;  // MF: MFMAs per fragment
  static __device__ __forceinline__ V of(const f32x4 (&a)[2]) { return to_natural(a[0], a[1]); }
  static __device__ __forceinline__ void to(const V& v, f32x4 (&a)[2]) { from_natural(v, a[0], a[1]); }
};
template <>
struct Chunk<float> {
  using V = f32x4;
  static constexpr int KW = 16, E = 4, BLK = 1, MF = 4;
  static __device__ __forceinline__ V of(const f32x4 (&a)[1]) { return a[0]; }
  static __device__ __forceinline__ void to(const V& v, f32x4 (&a)[1]) { a[0] = v; }
};

// Shape of a streamed chain of width H: eight waves of 256 registers where a
// row's operand takes at most 32 of them, else four of 512.  W: so many waves
// instead.
template <typename T, int H, int W = 0>
struct StreamDims {
  using C = Chunk<T>;
  static constexpr int NW = W ? W : H * (int)sizeof(T) <= 512 ? 8 : 4, NT = 64 * NW;
  static constexpr int MBS = H / 16, KC = H / C::KW;       // output blocks; k chunks of an H-wide operand
  static constexpr int CPS = MBS < 16 ? 16 / MBS : 1;      // chunks per slab (16 or 32 KiB)
  static constexpr int FR = MBS * CPS, SP = KC / CPS;      // fragments per slab; slabs of an H x H matrix
  static constexpr size_t RING = 4 * FR * 1024;
};

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
// SLOTS == S: the sequence stays in LDS, and none of this is needed.
template <int NW, int S, int FR, int SLOTS = 4>
struct WStream {
  static constexpr int SLAB = FR * 1024, K = FR / NW;  // K loads of 1 KiB per wave and slab
  static constexpr bool STAY = SLOTS == S;
  static_assert(STAY || (SLOTS == 4 && S % 4 == 0), "a slab's slot is s % 4");
  const unsigned char* base;  // (uniform)
  unsigned char* ring;        // LDS, 4 SLAB bytes
  __device__ __forceinline__ void send(int s) const {
    const int w = __builtin_amdgcn_readfirstlane(wave_id()) * K;
    const unsigned char* g = base + (size_t)(s % S) * SLAB + w * 1024;
    const unsigned dst = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)(ring) + s % SLOTS * SLAB + w * 1024;
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
  __device__ __forceinline__ void start() const {  // slabs 0, 1 and 2 (or all), whole at the next barrier
#pragma unroll
    for (int s = 0; s < (STAY ? S : 3); ++s) send(s);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  __device__ __forceinline__ void begin(int s) const {
    if constexpr (!STAY) send(s + 3);
  }
  __device__ __forceinline__ void end(int s, int s0, int s1) const {
    if constexpr (STAY) return;
    if (s == s1 - 1)
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else if (s >= s0 + 2) {
      if constexpr (K == 2)
        asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
      else if constexpr (K == 4)
        asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
      else
        asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
    }
    lds_sync();
  }
  // fragment f of slab s
  template <typename V>
  __device__ __forceinline__ const V* frag(int s, int f) const {
    return (const V*)(ring + s % SLOTS * SLAB) + f * 64;
  }
  static_assert(K == 2 || K == 4 || K == 8, "waits are written for these counts");
};

// acc[mb] += W x over one k chunk; fragments are read D ahead of their
// products.
template <typename T, int MBS>
__device__ __forceinline__ void chunk_gemm(f32x4 (&acc)[MBS], const typename Chunk<T>::V* f,
                                           const typename Chunk<T>::V& x) {
  using V = typename Chunk<T>::V;
  constexpr int D = 6, MF = Chunk<T>::MF;
  f += lane_id();
  V a[D];
#pragma unroll
  for (int i = 0; i < D; ++i) a[i] = f[i * 64];
#pragma unroll
  for (int i = 0; i < MBS; ++i) {
    const V cur = a[i % D];
    if (i + D < MBS) a[i % D] = f[(i + D) * 64];
    acc[i] = mma(cur, x, acc[i]);
  }
  __builtin_amdgcn_sched_group_barrier(0x100, D, 0);  // DS reads
#pragma unroll
  for (int i = 0; i < MBS - D; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, MF, 0);  // MFMA
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
  }
  __builtin_amdgcn_sched_group_barrier(0x008, D * MF, 0);
  __builtin_amdgcn_sched_barrier(0);
}

// x += W xs for an H-wide operand, its weights in slabs [s, s + SP) of a
// product over slabs [s0, s1).
template <typename T, int H, int NW, int S, int SLOTS>
__device__ __forceinline__ void stream_gemm(const WStream<NW, S, StreamDims<T, H>::FR, SLOTS>& ws, int s,
                                            int s0, int s1, f32x4 (&x)[H / 16],
                                            const typename Chunk<T>::V (&xs)[StreamDims<T, H>::KC]) {
  using L = StreamDims<T, H>;
#pragma unroll
  for (int c = 0; c < L::SP; ++c) {
    ws.begin(s + c);
#pragma unroll
    for (int j = 0; j < L::CPS; ++j)
      chunk_gemm<T>(x, ws.template frag<typename Chunk<T>::V>(s + c, j * L::MBS), xs[c * L::CPS + j]);
    ws.end(s + c, s0, s1);
  }
}
// a product of one operand: x = W xs, slabs [s0, s0 + SP)
template <typename T, int H, int NW, int S, int SLOTS>
__device__ __forceinline__ void stream_product(const WStream<NW, S, StreamDims<T, H>::FR, SLOTS>& ws, int s0,
                                               f32x4 (&x)[H / 16],
                                               const typename Chunk<T>::V (&xs)[StreamDims<T, H>::KC]) {
  zero_blocks(x);
  stream_gemm<T, H>(ws, s0, s0, s0 + StreamDims<T, H>::SP, x, xs);
}

// A row's operand from and to global memory (p: the row's first element).
template <typename T, int KC>
__device__ __forceinline__ void load_row(typename Chunk<T>::V (&v)[KC], const T* p, int lg) {
#pragma unroll
  for (int c = 0; c < KC; ++c) v[c] = *(const typename Chunk<T>::V*)(p + Chunk<T>::KW * c + Chunk<T>::E * lg);
}
template <typename T, int KC>
__device__ __forceinline__ void store_row(T* p, const typename Chunk<T>::V (&v)[KC], int lg) {
#pragma unroll
  for (int c = 0; c < KC; ++c) *(typename Chunk<T>::V*)(p + Chunk<T>::KW * c + Chunk<T>::E * lg) = v[c];
}
template <typename V, int KC>
__device__ __forceinline__ void arrived_row(V (&v)[KC]) {
#pragma unroll
  for (int c = 0; c < KC; ++c) arrived(v[c]);
}

// A row held in FP32 as an operand: load, then get once it is needed (rounded to
// T, waiting for it at once: the compiler's counted waits do not know of the
// weight loads behind it).
template <typename T, int H>
struct F32Row {
  using C = Chunk<T>;
  static constexpr int KC = H / C::KW, N = C::E / 4;
  f32x4 v[KC][N];
  __device__ __forceinline__ void load(const float* p, int lg) {
#pragma unroll
    for (int c = 0; c < KC; ++c)
#pragma unroll
      for (int k = 0; k < N; ++k) v[c][k] = *(const f32x4*)(p + C::KW * c + C::E * lg + 4 * k);
  }
  __device__ __forceinline__ void get(typename C::V (&x)[KC]) {
#pragma unroll
    for (int c = 0; c < KC; ++c) {
#pragma unroll
      for (int k = 0; k < N; ++k) arrived(v[c][k]);
      if constexpr (N == 1) {
        x[c] = v[c][0];
      } else {
        const u32x4 u = {pack2(v[c][0][0], v[c][0][1]), pack2(v[c][0][2], v[c][0][3]), pack2(v[c][1][0], v[c][1][1]),
                         pack2(v[c][1][2], v[c][1][3])};
        x[c] = __builtin_bit_cast(bf16x8, u);
      }
    }
  }
};

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

// The rows of one wave: [begin, end) of R, and the workgroup's common number
// of 16-row steps.
struct WaveRows {
  int begin, end, steps;
  __device__ WaveRows(int R, int nw_wg) {
    const int nw = gridDim.x * nw_wg, w0 = blockIdx.x * nw_wg, wv = w0 + __builtin_amdgcn_readfirstlane(wave_id());
    begin = (int)((long long)R * wv / nw);
    end = (int)((long long)R * (wv + 1) / nw);
    steps = R > 0 ? (R / nw + 1 + 15) >> 4 : 0;  // (no range is longer than R / nw + 1)
  }
};

// Adds the NW waves' column sums of one vector (each lane gives its values
// through put(double* row of H)) and writes them to dst[f * stride].
template <int H, int NW, typename PutFn>
__device__ __forceinline__ void wg_colsum(double* ds, float* dst, int stride, PutFn put) {
  __syncthreads();
  put(ds + wave_id() * H);
  __syncthreads();
  for (int f = threadIdx.x; f < H; f += 64 * NW) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < NW; ++k) s += ds[k * H + f];
    dst[(size_t)f * stride] = (float)s;
  }
}
// ... of totals in colsum64's layout, one per 64 features
template <int H, int NW>
__device__ __forceinline__ void wg_colsum64(double* ds, float* dst, const double (&v)[H / 64]) {
  wg_colsum<H, NW>(ds, dst, 1, [&](double* d) {
    const int l = lane_id(), li = l & 15, lg = l >> 4;
#pragma unroll
    for (int gr = 0; gr < H / 64; ++gr) d[64 * gr + 16 * (li >> 2) + 4 * lg + (li & 3)] = v[gr];
  });
}

}  // namespace xmgn
