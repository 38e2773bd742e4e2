// Weight gradients fused into the wave-private chains (BF16, H = 128, eight
// waves): the waves lay their 16 rows of two operands in LDS as one 128-row
// tile, and each accumulates a 32 x 64 block of the product from all of it.
#pragma once

#include "chain.hpp"

namespace xmgn {

constexpr size_t kTileReg = 8192;  // bytes per wave: 16 rows of two 128-wide BF16 operands

// A wave's share of the 128-row tile: 16 rows x 128 BF16 in 256-byte rows,
// 32-byte units swizzled by row so that neither the row writes nor the
// transposing reads meet in a bank.
__device__ __forceinline__ int tile_off(int row, int unit16) {  // in bytes
  return row * 256 + ((((unit16 >> 1) ^ row) & 7) << 5) + ((unit16 & 1) << 4);
}
__device__ __forceinline__ void tile_put(unsigned char* reg, const bf16x8 (&x)[4], int l) {
  const int li = l & 15, lg = l >> 4;
#pragma unroll
  for (int c = 0; c < 4; ++c) *(bf16x8*)(reg + tile_off(li, 4 * c + lg)) = x[c];
}
// Fragment [features c0 .. + 15][rows 32 c .. + 31] of the tile at byte offset
// `off` of every wave's region (k order: rows 4 g + r, 16 + 4 g + r).
__device__ __forceinline__ bf16x8 tile_frag(const unsigned char* regs, int off, int c, int c0, int l) {
  const int L = l & 15, lg = l >> 4;
  const int row = 4 * lg + (L >> 2);
  const int f = c0 + 4 * (L & 3);
  const unsigned char* p = regs + (size_t)(2 * c) * kTileReg + off + tile_off(row, f >> 3) + (f & 7) * 2;
  const bf16x4_lds lo = lds_read_tr4((const bf16*)p), hi = lds_read_tr4((const bf16*)(p + kTileReg));
  return bf16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
}
// acc[i][j] += block (32 wm + 16 i, 64 wn + 16 j) of the sum over the tile's
// 128 rows of (row of the tile at offA)^T (row of the tile at offB).
__device__ __forceinline__ void tile_wgrad(f32x4 (&acc)[2][4], const unsigned char* regs, int offA, int offB, int wm,
                                           int wn, int l) {
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 a[2], b[4];
#pragma unroll
    for (int i = 0; i < 2; ++i) a[i] = tile_frag(regs, offA, c, 32 * wm + 16 * i, l);
#pragma unroll
    for (int j = 0; j < 4; ++j) b[j] = tile_frag(regs, offB, c, 64 * wn + 16 * j, l);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = mma(a[i], b[j], acc[i][j]);
  }
  __builtin_amdgcn_sched_barrier(0);
}

}  // namespace xmgn
