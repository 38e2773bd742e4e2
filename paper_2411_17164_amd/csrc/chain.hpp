// Wave-private MLP chains (BF16, gfx950): a wave takes 16 rows (edges or
// nodes) at a time through every product of an MLP with no workgroup
// barrier.  The products are formed transposed, C^T = W X^T: the A operand is
// the weight (rows = output features), the B operand the rows' features, so
// a lane holds features of ONE row (row = lane % 16) and LayerNorm's row sums
// are mostly sums inside a lane.
//
// Layouts of a row's H features over the 4 lanes g = lane / 16 that hold it:
//   natural:     chunk c (32 features), lane g: features 32 c + 8 g .. + 7,
//                16 bytes of BF16: the MFMA B operand, and 16-byte global
//                loads and stores;
//   accumulator: block mb (16 features), lane g: features 16 mb + 4 g .. + 3,
//                the MFMA result, and 16-byte loads and stores of FP32 rows.
// Blocks 2c and 2c + 1 hold chunk c; four lane swaps per chunk convert
// between the two.
#pragma once

#include "common.hpp"

namespace xmgn {

typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

// The same value, opaque to the compiler (what is formed from it inside a
// loop stays there).
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Has the compiler wait for a loaded value here.
template <typename V>
__device__ __forceinline__ void arrived(V& v) {
  u32x4 u = __builtin_bit_cast(u32x4, v);
  asm volatile("" : "+v"(u));
  v = __builtin_bit_cast(V, u);
}

// Ordering of LDS accesses between the lanes of one wave (a wave's LDS
// instructions execute in order; this holds the compiler to it).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Swap of the odd 16-lane rows of a with the even rows of b.
__device__ __forceinline__ void swap16(unsigned& a, unsigned& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
// Swap of the upper 32 lanes of a with the lower 32 of b.
__device__ __forceinline__ void swap32(unsigned& a, unsigned& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
// x + (x of lane ^ 16), x + (x of lane ^ 32)
__device__ __forceinline__ float add_xor16(float x) {
  unsigned a = __builtin_bit_cast(unsigned, x), b = a;
  swap16(a, b);
  return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}
__device__ __forceinline__ float add_xor32(float x) {
  unsigned a = __builtin_bit_cast(unsigned, x), b = a;
  swap32(a, b);
  return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}

__device__ __forceinline__ unsigned pack2(float lo, float hi) {
  const bf16x2 p = {(bf16)lo, (bf16)hi};
  return __builtin_bit_cast(unsigned, p);
}
__device__ __forceinline__ float unpack_lo(unsigned v) { return __builtin_bit_cast(float, v << 16); }
__device__ __forceinline__ float unpack_hi(unsigned v) { return __builtin_bit_cast(float, v & 0xffff0000u); }

// Chunk c of a row, accumulator layout (blocks lo = 2c, hi = 2c + 1) rounded
// to BF16 -> natural layout.
__device__ __forceinline__ bf16x8 to_natural(const f32x4& lo, const f32x4& hi) {
  unsigned a0 = pack2(lo[0], lo[1]), a1 = pack2(lo[2], lo[3]);
  unsigned b0 = pack2(hi[0], hi[1]), b1 = pack2(hi[2], hi[3]);
  swap32(a0, b0);
  swap32(a1, b1);
  swap16(a0, b0);
  swap16(a1, b1);
  const u32x4 v = {a0, a1, b0, b1};
  return __builtin_bit_cast(bf16x8, v);
}
// The inverse: natural BF16 chunk -> the two accumulator-layout blocks.
__device__ __forceinline__ void from_natural(const bf16x8& x, f32x4& lo, f32x4& hi) {
  const u32x4 v = __builtin_bit_cast(u32x4, x);
  unsigned a0 = v[0], a1 = v[1], b0 = v[2], b1 = v[3];
  swap16(a0, b0);
  swap16(a1, b1);
  swap32(a0, b0);
  swap32(a1, b1);
  lo = f32x4{unpack_lo(a0), unpack_hi(a0), unpack_lo(a1), unpack_hi(a1)};
  hi = f32x4{unpack_lo(b0), unpack_hi(b0), unpack_lo(b1), unpack_hi(b1)};
}

// Weight fragments in LDS: fragment (mb, c) of W[out][in] is the A operand of
// rows 16 mb .. + 15 and k = 32 c .. + 31 as one contiguous KiB in lane order,
// so a fragment read is conflict-free with an immediate offset.  Copies the
// MBS x KC fragments of W (row stride ldw) with NT threads.
template <int MBS, int KC, int NT>
__device__ __forceinline__ void stage_frags(bf16x8* dst, const bf16* __restrict__ W, int ldw) {
  static_assert(MBS * KC % (NT / 64) == 0, "whole steps of the workgroup");
  const int l = lane_id(), li = l & 15, lg = l >> 4;
#pragma unroll 4
  for (int f = wave_id(); f < MBS * KC; f += NT / 64) {
    const int mb = f / KC, c = f - mb * KC;
    dst[f * 64 + l] = *(const bf16x8*)(W + (size_t)(mb * 16 + li) * ldw + c * 32 + lg * 8);
  }
}

template <int N>
__device__ __forceinline__ void zero_blocks(f32x4 (&x)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) x[i] = f32x4{0.f, 0.f, 0.f, 0.f};
}

// acc[mb] += W X^T over the KC chunks of the fragments F (KC per block): x[c]
// is chunk c of the rows, natural layout.
// BOUND: keep the fragment reads of one chunk from being hoisted over the
// chunk before (bounds their registers to 4 MBS).
template <bool BOUND = false, int MBS, int KC>
__device__ __forceinline__ void chain_gemm(f32x4 (&acc)[MBS], const bf16x8* F, const bf16x8 (&x)[KC]) {
  const bf16x8* f = F + lane_id();
#pragma unroll
  for (int c = 0; c < KC; ++c) {
    if constexpr (BOUND) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int mb = 0; mb < MBS; ++mb) acc[mb] = mma(f[(mb * KC + c) * 64], x[c], acc[mb]);
  }
  if constexpr (BOUND) __builtin_amdgcn_sched_barrier(0);
}

// One exchange of a sum across lanes that halves the values a lane keeps: of
// x[0 .. 2N), the lanes with `up` keep the upper half and send the lower to
// their DPP partner, the others the reverse.
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float s) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, s), CTRL, 0xF, 0xF, false));
}
template <int CTRL, int N>
__device__ __forceinline__ void half_reduce(const float (&x)[2 * N], float (&y)[N], bool up) {
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const float keep = up ? x[N + k] : x[k], send = up ? x[k] : x[N + k];
    y[k] = keep + dpp_mov<CTRL>(send);
  }
}
// Column sums over the 16 rows of 64 features (four blocks): each lane ends
// with one total, of feature 16 (li / 4) + 4 lg + li % 4 (li = lane % 16).
__device__ __forceinline__ float colsum64(const f32x4 (&x)[4]) {
  const int li = lane_id() & 15;
  float v[16], a[8], b[4], c[2], d[1];
#pragma unroll
  for (int k = 0; k < 16; ++k) v[k] = x[k >> 2][k & 3];
  half_reduce<0x140, 8>(v, a, li & 8);  // row_mirror: lane 15 - li
  half_reduce<0x141, 4>(a, b, li & 4);  // row_half_mirror: lane 7 - li of its half
  half_reduce<0x4E, 2>(b, c, li & 2);   // quad_perm [2,3,0,1]
  half_reduce<0xB1, 1>(c, d, li & 1);   // quad_perm [1,0,3,2]
  return d[0];
}

// Sum over the 16 columns (features 32 w .. 32 w + 31 taken as li and
// li + 16) of one 32-feature span, in the pairwise order of sum16 on a row
// held one feature per lane: features li and li + 16 first, then pairs, quads,
// halves.  lo, hi: blocks 2w and 2w + 1.
__device__ __forceinline__ float span_sum(const f32x4& lo, const f32x4& hi) {
  const float s = ((lo[0] + hi[0]) + (lo[1] + hi[1])) + ((lo[2] + hi[2]) + (lo[3] + hi[3]));
  return add_xor32(add_xor16(s));
}

}  // namespace xmgn
