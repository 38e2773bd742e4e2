// Edge kernels as wave-private chains (BF16, H = 128; see chain.hpp).
#include <algorithm>
#include <type_traits>

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

// Ordering of LDS accesses between the lanes of one wave (a wave's LDS
// instructions execute in order; this holds the compiler to it).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
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

// Receiver sums of rows held in the accumulator layout, added one edge after
// the other in edge order (ascending sender), through a wave-private LDS
// buffer of 16 rows x 64 features.  A segment may continue from the previous
// tile: its running sum is carried in registers (lane l: features l, 64 + l).
struct SegSum128 {
  float s[2] = {0.f, 0.f};
  // x: 16 edges; ends: bit i set where edge i is its receiver's last; rv: the
  // lane's edge's receiver; valid: edges in the group
  __device__ __forceinline__ void add(const f32x4 (&x)[8], unsigned ends, int rv, int valid, float* buf,
                                      float* __restrict__ m) {
    const int l = lane_id(), li = l & 15, lg = l >> 4;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      wave_sync();
      // 16-byte unit u of row i at unit u ^ i: no bank conflict on either side
#pragma unroll
      for (int k = 0; k < 4; ++k) *(f32x4*)(buf + li * 64 + (((4 * k + lg) ^ li) << 2)) = x[4 * p + k];
      wave_sync();
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        if (i < valid) {
          s[p] += buf[i * 64 + (l ^ (i << 2))];
          if (ends >> i & 1) {
            const int r = __builtin_amdgcn_readlane(rv, i);
            m[(size_t)r * 128 + 64 * p + l] = s[p];
            s[p] = 0.f;
          }
        }
      }
    }
  }
};

// LayerNorm of a row of 128 in the accumulator layout (in place -> xhat),
// returning 1 / std: (mean, M2) of each 32-feature span, merged pairwise like
// ln_normalize does across four waves (the same order of every sum).
__device__ __forceinline__ float ln128(f32x4 (&u)[8], float eps) {
  constexpr float CPW = 32.f;
  float mw[4], q[4];
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    mw[w] = span_sum(u[2 * w], u[2 * w + 1]) * (1.f / CPW);
    float d[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float a = u[2 * w][r] - mw[w], c = u[2 * w + 1][r] - mw[w];
      d[r] = __builtin_fmaf(a, a, c * c);
    }
    q[w] = add_xor32(add_xor16((d[0] + d[1]) + (d[2] + d[3])));
  }
  const float mean = (((mw[0] + mw[1]) + mw[2]) + mw[3]) * 0.25f;
  float m2 = 0.f;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float dm = mw[w] - mean;
    m2 += q[w] + CPW * dm * dm;
  }
  const float inv = rsqrtf(m2 * (1.f / 128) + eps);
#pragma unroll
  for (int mb = 0; mb < 8; ++mb)
#pragma unroll
    for (int r = 0; r < 4; ++r) u[mb][r] = (u[mb][r] - mean) * inv;
  return inv;
}

// The four 128-vectors of an MLP (b1, b2, gamma, beta) travel with the wave:
// lane l holds 8 of the 512 floats and puts them into the wave's LDS buffer
// at the start of a tile, from where each is read as the accumulator layout
// needs it (16 lanes read the same 16 bytes).
struct Vecs128 {
  f32x4 a, b;
  __device__ __forceinline__ void load(const float* b1, const float* b2, const float* g, const float* be) {
    const int l = lane_id();
    a = *(const f32x4*)((l < 32 ? b1 : b2) + 4 * (l & 31));
    b = *(const f32x4*)((l < 32 ? g : be) + 4 * (l & 31));
  }
  __device__ __forceinline__ void put(float* buf) const {
    wave_sync();
    *(f32x4*)(buf + 4 * lane_id()) = a;
    *(f32x4*)(buf + 256 + 4 * lane_id()) = b;
    wave_sync();
  }
  // vector v (0..3), block mb
  __device__ static __forceinline__ f32x4 get(const float* buf, int v, int mb) {
    return *(const f32x4*)(buf + 128 * v + 16 * mb + 4 * (lane_id() >> 4));
  }
};

// ---------------------------------------------------------------------------
// Fused edge processor, forward, BF16 H = 128 (the gathered form): the MLP of
// k_edge_fwd with each wave taking 16 edges of its own range at a time through
// both products, the LayerNorm and the receiver sums, and the next 16 edges'
// rows in flight meanwhile.  Both weights stay in LDS (128 KiB, one workgroup
// of eight waves per CU), so nothing but edge data crosses the memory system
// and no barrier follows the staging.  It is bound by HBM: on 3.55M edges and
// 400k nodes (keeping z) 968 us, 3.9 GB algorithmic, 4.0 TB/s where a large
// copy reaches 4.9; the workgroup-tile kernel it replaces took 1,818 us, most
// of it waiting at seven barriers per 64 edges.  32 edges per step need 100
// more registers than there are.  Every sum is taken in that kernel's order,
// and the results are the same bits.
// ---------------------------------------------------------------------------
template <int NW>
struct EdgeFwdChain {
  static constexpr size_t W1S = 96 * 1024, W2S = 32 * 1024;  // weight fragments
  static constexpr size_t BUF = 4096;                        // per wave
  static constexpr size_t bytes = W1S + W2S + NW * BUF;
};

template <int ACT, int AGG, int NW, int ET>
__global__ __launch_bounds__(64 * NW, NW / 4) void k_edge_fwd_chain(BatchView b, MlpW w, const bf16* __restrict__ h,
                                                                    const bf16* __restrict__ e,
                                                                    bf16* __restrict__ e_out, float* __restrict__ m,
                                                                    bf16* __restrict__ z_out,
                                                                    bf16* __restrict__ a_out, float eps) {
  constexpr int H = 128, MT = 16 * ET;
  using L = EdgeFwdChain<NW>;
  __shared__ __align__(16) unsigned char smem[L::bytes];
  bf16x8* F1 = (bf16x8*)smem;
  bf16x8* F2 = (bf16x8*)(smem + L::W1S);
  float* buf = (float*)(smem + L::W1S + L::W2S + wave_id() * L::BUF);
  const int l = lane_id(), li = l & 15, lg = l >> 4;
  const int nw = gridDim.x * NW, wv = wave_rank(NW);

  stage_frags<8, 12, 64 * NW>(F1, (const bf16*)w.W1, 3 * H);
  stage_frags<8, 4, 64 * NW>(F2, (const bf16*)w.W2, H);
  Vecs128 vec;
  vec.load(w.b1, w.b2, w.gamma, w.beta);
  const WaveEdges we(b, wv, nw);

  // indices of a tile: this lane's edge of every 16-row group (clamped to the
  // wave's last edge), its receiver, sender and the next edge's receiver
  int rv[ET], cv[ET], rn[ET];
  auto load_idx = [&](int e0) {
#pragma unroll
    for (int t = 0; t < ET; ++t) {
      const int k = min(e0 + 16 * t + li, we.end - 1);
      rv[t] = b.recv[k];
      cv[t] = b.col[k];
      rn[t] = k + 1 < b.E ? b.recv[k + 1] : -1;
    }
  };
  bf16x8 x[ET][12];
  auto load_rows = [&](int e0) {
#pragma unroll
    for (int t = 0; t < ET; ++t) {
      const int k = min(e0 + 16 * t + li, we.end - 1);
      const bf16* pr = h + (size_t)rv[t] * H + 8 * lg;
      const bf16* ps = h + (size_t)cv[t] * H + 8 * lg;
      const bf16* pe = e + (size_t)k * H + 8 * lg;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        x[t][c] = *(const bf16x8*)(pr + 32 * c);
        x[t][4 + c] = *(const bf16x8*)(ps + 32 * c);
        x[t][8 + c] = *(const bf16x8*)(pe + 32 * c);
      }
    }
  };
  const bool any = we.begin < we.end;
  if (any) {
    load_idx(we.begin);
    load_rows(we.begin);
  }
  __syncthreads();
  SegSum128 seg;
  for (int e0 = we.begin; e0 < we.end; e0 += MT) {
    const int ne = min(MT, we.end - e0);
    int rc[ET];
    unsigned ends[ET];
#pragma unroll
    for (int t = 0; t < ET; ++t) {
      rc[t] = rv[t];
      ends[t] = (unsigned)__ballot(rv[t] != rn[t]) & 0xffffu;
    }
    const bool more = e0 + MT < we.end;
    if (more) load_idx(e0 + MT);
    vec.put(buf);
    f32x4 acc[ET][8];
    zero_acc(acc);
    chain_gemm<ET, 8, 12, 0, 12>(acc, F1, x, 0);
    bf16x8 ec[ET][4];
#pragma unroll
    for (int t = 0; t < ET; ++t)
#pragma unroll
      for (int c = 0; c < 4; ++c) ec[t][c] = x[t][8 + c];
    if (more) load_rows(e0 + MT);  // the next tile's rows, in flight from here
    bf16x8 z[ET][4];
#pragma unroll
    for (int mb = 0; mb < 8; ++mb) {
      const f32x4 bb = Vecs128::get(buf, 0, mb);
#pragma unroll
      for (int t = 0; t < ET; ++t) acc[t][mb] += bb;
    }
    if (a_out) {
#pragma unroll
      for (int t = 0; t < ET; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const bf16x8 v = to_natural(acc[t][2 * c], acc[t][2 * c + 1]);
          if (16 * t + li < ne) *(bf16x8*)(a_out + (size_t)(e0 + 16 * t + li) * H + 32 * c + 8 * lg) = v;
        }
    }
#pragma unroll
    for (int t = 0; t < ET; ++t)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          acc[t][2 * c][r] = act_f<ACT>(acc[t][2 * c][r]);
          acc[t][2 * c + 1][r] = act_f<ACT>(acc[t][2 * c + 1][r]);
        }
        z[t][c] = to_natural(acc[t][2 * c], acc[t][2 * c + 1]);
        if (z_out && 16 * t + li < ne) *(bf16x8*)(z_out + (size_t)(e0 + 16 * t + li) * H + 32 * c + 8 * lg) = z[t][c];
      }
    zero_acc(acc);
    chain_gemm<ET, 8, 4, 0, 4>(acc, F2, z, 0);
#pragma unroll
    for (int mb = 0; mb < 8; ++mb) {
      const f32x4 bb = Vecs128::get(buf, 1, mb);
#pragma unroll
      for (int t = 0; t < ET; ++t) acc[t][mb] += bb;
    }
#pragma unroll
    for (int t = 0; t < ET; ++t) ln128(acc[t], eps);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const f32x4 g0 = Vecs128::get(buf, 2, 2 * c), g1 = Vecs128::get(buf, 2, 2 * c + 1);
      const f32x4 b0 = Vecs128::get(buf, 3, 2 * c), b1 = Vecs128::get(buf, 3, 2 * c + 1);
#pragma unroll
      for (int t = 0; t < ET; ++t) {
        f32x4 e_lo, e_hi;
        from_natural(ec[t][c], e_lo, e_hi);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float v0 = g0[r] * acc[t][2 * c][r] + b0[r], v1 = g1[r] * acc[t][2 * c + 1][r] + b1[r];
          e_lo[r] += v0;
          e_hi[r] += v1;
          acc[t][2 * c][r] = AGG ? e_lo[r] : v0;  // the summand of m
          acc[t][2 * c + 1][r] = AGG ? e_hi[r] : v1;
        }
        if (e_out) {
          const bf16x8 v = to_natural(e_lo, e_hi);
          if (16 * t + li < ne) *(bf16x8*)(e_out + (size_t)(e0 + 16 * t + li) * H + 32 * c + 8 * lg) = v;
        }
      }
    }
#pragma unroll
    for (int t = 0; t < ET; ++t) seg.add(acc[t], ends[t], rc[t], ne - 16 * t, buf, m);
  }
  zero_empty_rows(b, m, H, wv, nw);
}

bool edge_fwd_chain(const Shape& s) { return s.prec == 1 && s.H == 128; }

void launch_edge_fwd_chain(const Shape& s, const BatchView& b, const MlpW& w, const void* h, const void* e, void* e_out,
                           float* m, void* z_out, void* a_out, hipStream_t st) {
  constexpr int NW = 8, ET = 1;
  const int grid = std::max(1, std::min(256, (b.E + NW * 16 * ET - 1) / (NW * 16 * ET)));
  auto go = [&](auto act, auto agg) {
    k_edge_fwd_chain<decltype(act)::value, decltype(agg)::value, NW, ET><<<grid, 64 * NW, 0, st>>>(
        b, w, (const bf16*)h, (const bf16*)e, (bf16*)e_out, m, (bf16*)z_out, (bf16*)a_out, s.eps);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  if (s.act) {
    if (s.agg) go(I1{}, I1{}); else go(I1{}, I0{});
  } else {
    if (s.agg) go(I0{}, I1{}); else go(I0{}, I0{});
  }
}

}  // namespace xmgn
