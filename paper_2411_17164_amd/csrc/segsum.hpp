// Work split and receiver sums of the wave-private edge kernels.
#pragma once

#include "chain.hpp"
#include "kernels.hpp"

namespace xmgn {

// The range of edges of wave `wv` of `nw`: E wv / nw and E (wv + 1) / nw, each
// moved on to the next segment start, so a wave holds whole receiver segments.
struct WaveEdges {
  int begin, end;
  __device__ static int align(const int* __restrict__ recv, int E, int t) {
    if (t <= 0) return 0;
    for (; t < E; t += 64) {
      const int i = t + lane_id();
      const bool start = i < E && recv[i] != recv[i - 1];
      const unsigned long long m = __ballot(start);
      if (m) return t + __builtin_ctzll(m);
    }
    return E;
  }
  __device__ WaveEdges(const BatchView& b, int wv, int nw) {
    begin = align(b.recv, b.E, (int)((long long)b.E * wv / nw));
    end = align(b.recv, b.E, (int)((long long)b.E * (wv + 1) / nw));
  }
};

// Position of this wave among the grid's waves: workgroup b runs on XCD b % 8,
// and each XCD takes a contiguous part of the edges.
__device__ __forceinline__ int wave_rank(int nw_wg) {
  const int G = gridDim.x, b = blockIdx.x;
  const int per = (G + 7) >> 3, full = G - 8 * (per - 1);  // XCDs with `per` workgroups
  const int x = b & 7, j = b >> 3;
  const int base = x < full ? x * per : full * per + (x - full) * (per - 1);
  return (base + j) * nw_wg + __builtin_amdgcn_readfirstlane(wave_id());
}

// Rows without in-edges: their sums are zero.
__device__ __forceinline__ void zero_empty_rows(const BatchView& b, float* __restrict__ m, int H, int wv, int nw) {
  for (int r0 = wv * 64; r0 < b.n; r0 += nw * 64) {
    const int r = r0 + lane_id();
    unsigned long long em = __ballot(r < b.n && b.row_ptr[r] == b.row_ptr[r + 1]);
    while (em) {
      const int i = __builtin_ctzll(em);
      em &= em - 1;
      for (int c = lane_id(); c < H; c += 64) m[(size_t)(r0 + i) * H + c] = 0.f;
    }
  }
}

// Steps of `rows` rows that the longest of the workgroup's NW ranges needs
// (its waves meet at barriers, so all take as many).  slots: LDS, one int per
// wave at this stride (in ints), free before and after.
template <int NW>
__device__ __forceinline__ int wg_steps(int len, int rows, int* slots, int stride) {
  if (lane_id() == 0) slots[wave_id() * stride] = len;
  __syncthreads();
  int longest = 0;
#pragma unroll
  for (int k = 0; k < NW; ++k) longest = max(longest, slots[k * stride]);
  __syncthreads();
  return (__builtin_amdgcn_readfirstlane(longest) + rows - 1) / rows;
}

// Receiver sums of rows held in the accumulator layout, added one edge after
// the other in edge order (ascending sender), through a wave-private LDS
// buffer of 16 rows x 128 FP32.  A segment may continue from the previous
// tile: its running sum is carried in registers (lane l: features 2 l, 2 l + 1
// of every 128).
template <int H>
struct SegSum {
  float2 s[H / 128];
  __device__ SegSum() {
#pragma unroll
    for (int p = 0; p < H / 128; ++p) s[p] = float2{0.f, 0.f};
  }
  // x: 16 edges; ends: bit i set where edge i is its receiver's last; rv: the
  // lane's edge's receiver; valid: edges in the group (may be <= 0).  done(p,
  // sum) sees every finished sum of a pass.
  template <typename Done>
  __device__ __forceinline__ void add(const f32x4 (&x)[H / 16], unsigned ends, int rv, int valid, float* buf,
                                      float* __restrict__ m, Done done) {
    const int l = opaque(lane_id()), li = l & 15, lg = l >> 4;
#pragma unroll
    for (int p = 0; p < H / 128; ++p) {
      wave_sync();
      // 16-byte unit u of row i at unit u ^ i: no bank conflict on either side
#pragma unroll
      for (int k = 0; k < 8; ++k) *(f32x4*)(buf + li * 128 + (((4 * k + lg) ^ li) << 2)) = x[8 * p + k];
      wave_sync();
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        if (i < valid) {
          const float2 v = *(const float2*)(buf + i * 128 + ((((l >> 1) ^ i) << 2) | ((l & 1) << 1)));
          s[p].x += v.x;
          s[p].y += v.y;
          if (ends >> i & 1) {
            const int r = __builtin_amdgcn_readlane(rv, i);
            *(float2*)(m + (size_t)r * H + 128 * p + 2 * l) = s[p];
            done(p, s[p]);
            s[p] = float2{0.f, 0.f};
          }
        }
      }
    }
    wave_sync();
  }
  __device__ __forceinline__ void add(const f32x4 (&x)[H / 16], unsigned ends, int rv, int valid, float* buf,
                                      float* __restrict__ m) {
    add(x, ends, rv, valid, buf, m, [](int, const float2&) {});
  }
};

}  // namespace xmgn
