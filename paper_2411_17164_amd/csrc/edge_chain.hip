// Edge kernels as wave-private chains (BF16, H = 128; see chain.hpp).
#include <algorithm>
#include <type_traits>

#include "chain.hpp"
#include "kernels.hpp"
#include "segsum.hpp"
#include "tile.hpp"

namespace xmgn {

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
// Fused edge processor, forward, BF16 H = 128 (the gathered form):
//   x = [h_r ; h_s ; e],  v = LN(W2 act(W1 x + b1) + b2),  e' = e + v,
//   m_r = sum over the edges into r of v (or of e'),
// each wave taking 16 edges of its own range at a time through both products, the LayerNorm and the receiver sums, and the next 16 edges'
// rows in flight meanwhile.  Both weights stay in LDS (128 KiB, one workgroup
// of eight waves per CU), so nothing but edge data crosses the memory system
// and no barrier follows the staging.  It is bound by HBM: on 3.54M edges and
// 400k nodes (keeping z) 970 to 990 us, 3.96 GB by counters (3.93 algorithmic),
// 4.0 TB/s where a large copy reaches 4.9; the workgroup-tile kernel it replaces
// took 1,818 us, most of it waiting at seven barriers per 64 edges.  32 edges per step need 100
// more registers than there are.  Every sum is taken in that kernel's order,
// and the results are the same bits.
// ---------------------------------------------------------------------------
template <int NW>
struct EdgeFwdChain {
  static constexpr size_t W1S = 96 * 1024, W2S = 32 * 1024;  // weight fragments
  static constexpr size_t BUF = 4096;                        // per wave
  static constexpr size_t bytes = W1S + W2S + NW * BUF;
};

template <int ACT, int AGG, int NW>
__global__ __launch_bounds__(64 * NW, NW / 4) void k_edge_fwd_chain(BatchView b, MlpW w, const bf16* __restrict__ h,
                                                                    const bf16* __restrict__ e,
                                                                    bf16* __restrict__ e_out, float* __restrict__ m,
                                                                    bf16* __restrict__ z_out,
                                                                    bf16* __restrict__ a_out, float eps) {
  constexpr int H = 128;
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

  // indices of a tile: this lane's edge (clamped to the wave's last edge), its
  // receiver, sender and the next edge's receiver
  int rv = 0, cv = 0, rn = 0;
  auto load_idx = [&](int e0) {
    const int k = min(e0 + li, we.end - 1);
    rv = b.recv[k];
    cv = b.col[k];
    rn = k + 1 < b.E ? b.recv[k + 1] : -1;
  };
  bf16x8 x[12];
  auto load_rows = [&](int e0) {
    const int k = min(e0 + li, we.end - 1);
    const bf16* pr = h + (size_t)rv * H + 8 * lg;
    const bf16* ps = h + (size_t)cv * H + 8 * lg;
    const bf16* pe = e + (size_t)k * H + 8 * lg;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      x[c] = *(const bf16x8*)(pr + 32 * c);
      x[4 + c] = *(const bf16x8*)(ps + 32 * c);
      x[8 + c] = *(const bf16x8*)(pe + 32 * c);
    }
  };
  const bool any = we.begin < we.end;
  if (any) {
    load_idx(we.begin);
    load_rows(we.begin);
  }
  __syncthreads();
  SegSum128 seg;
  for (int e0 = we.begin; e0 < we.end; e0 += 16) {
    const int ne = min(16, we.end - e0);
    const bool ok = li < ne;
    const size_t row = (size_t)(e0 + li) * H + 8 * lg;
    const int rc = rv;
    const unsigned ends = (unsigned)__ballot(rv != rn) & 0xffffu;
    const bool more = e0 + 16 < we.end;
    if (more) load_idx(e0 + 16);
    vec.put(buf);
    f32x4 acc[8];
    zero_blocks(acc);
    chain_gemm(acc, F1, x);
    bf16x8 ec[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) ec[c] = x[8 + c];
    if (more) load_rows(e0 + 16);  // the next tile's rows, in flight from here
    bf16x8 z[4];
#pragma unroll
    for (int mb = 0; mb < 8; ++mb) acc[mb] += Vecs128::get(buf, 0, mb);
    if (a_out) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const bf16x8 v = to_natural(acc[2 * c], acc[2 * c + 1]);
        if (ok) *(bf16x8*)(a_out + row + 32 * c) = v;
      }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        acc[2 * c][r] = act_f<ACT>(acc[2 * c][r]);
        acc[2 * c + 1][r] = act_f<ACT>(acc[2 * c + 1][r]);
      }
      z[c] = to_natural(acc[2 * c], acc[2 * c + 1]);
      if (z_out && ok) *(bf16x8*)(z_out + row + 32 * c) = z[c];
    }
    zero_blocks(acc);
    chain_gemm(acc, F2, z);
#pragma unroll
    for (int mb = 0; mb < 8; ++mb) acc[mb] += Vecs128::get(buf, 1, mb);
    ln128(acc, eps);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const f32x4 g0 = Vecs128::get(buf, 2, 2 * c), g1 = Vecs128::get(buf, 2, 2 * c + 1);
      const f32x4 b0 = Vecs128::get(buf, 3, 2 * c), b1 = Vecs128::get(buf, 3, 2 * c + 1);
      f32x4 e_lo, e_hi;
      from_natural(ec[c], e_lo, e_hi);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float v0 = g0[r] * acc[2 * c][r] + b0[r], v1 = g1[r] * acc[2 * c + 1][r] + b1[r];
        e_lo[r] += v0;
        e_hi[r] += v1;
        acc[2 * c][r] = AGG ? e_lo[r] : v0;  // the summand of m
        acc[2 * c + 1][r] = AGG ? e_hi[r] : v1;
      }
      if (e_out) {
        const bf16x8 v = to_natural(e_lo, e_hi);
        if (ok) *(bf16x8*)(e_out + row + 32 * c) = v;
      }
    }
    seg.add(acc, ends, rc, ne, buf, m);
  }
  zero_empty_rows(b, m, H, wv, nw);
}

bool edge_fwd_chain(const Shape& s) { return s.prec == 1 && s.H == 128; }

void launch_edge_fwd_chain(const Shape& s, const BatchView& b, const MlpW& w, const void* h, const void* e, void* e_out,
                           float* m, void* z_out, void* a_out, hipStream_t st) {
  constexpr int NW = 8;
  const int grid = edge_bwd_chain_grid(s, b.E);
  auto go = [&](auto act, auto agg) {
    k_edge_fwd_chain<decltype(act)::value, decltype(agg)::value, NW><<<grid, 64 * NW, 0, st>>>(
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

// ---------------------------------------------------------------------------
// Edge adjoint with z (and a) from the tape, BF16 H = 128.
// ---------------------------------------------------------------------------
// Eight waves, each 16 edges of its own range at a time, go through the three
// products (u = W2 z, dz = W2^T du, de = W1e^T da) as private chains; dW2 and
// the e-block of dW1 are sums over edges, so the waves lay [du | z], then
// [da | e], in LDS as one 128-row tile and each accumulates a 32 x 64 block of
// either matrix from all of it: four barriers per 128 edges.  W2, W2^T and the
// e-block of W1^T stay in LDS (96 KiB); z comes a step ahead, de' and dm_r
// during u and its statistics.  Column sums over edges (db2, dgamma, dbeta)
// are taken across the 16 lanes of a DPP row; db1 is the total of the receiver
// sums.  On 3.54M edges and 400k nodes 1,740 us; the 64-row workgroup-tile kernel
// it replaces took 3,345 us, and its 32-row form 2,430 us plus a product of 300 us
// for the e-block.  Bound by HBM: by counters it moves 8.5 GB at 4.9 TB/s, a large
// copy's rate.  6.75 GB are algorithmic; de' is read twice (for dv and for de), as
// it does not fit in the registers between.  Sums keep that kernel's order: da, de and S_r
// are the same bits.
struct EdgeBwdChain {
  static constexpr int NW = 8;
  static constexpr size_t WS = 32 * 1024;  // one matrix of fragments
  static constexpr size_t REG = kTileReg;
  static constexpr size_t bytes = 3 * WS + NW * REG;
};

// Sum over the 16 lanes of a DPP row of each of a lane's 32 values (x in the
// accumulator layout: value 4 mb + r), halving the values a lane keeps at each
// exchange: lane li ends with the totals of two values, 2 k and 2 k + 1 with
// k = colsum_slot(li).
// value index of the first of lane li's two totals
__device__ __forceinline__ int colsum_slot(int li) {
  return ((li >> 3) & 1) * 16 + ((li >> 2) & 1) * 8 + ((li >> 1) & 1) * 4 + (li & 1) * 2;
}
__device__ __forceinline__ void colsum16(const f32x4 (&x)[8], double (&tot)[2]) {
  const int li = lane_id() & 15;
  float v[32], a[16], b[8], c[4], d[2];
#pragma unroll
  for (int k = 0; k < 32; ++k) v[k] = x[k >> 2][k & 3];
  half_reduce<0x140, 16>(v, a, li & 8);   // row_mirror: lane 15 - li
  half_reduce<0x141, 8>(a, b, li & 4);    // row_half_mirror: lane 7 - li of its half
  half_reduce<0x4E, 4>(b, c, li & 2);     // quad_perm [2,3,0,1]
  half_reduce<0xB1, 2>(c, d, li & 1);     // quad_perm [1,0,3,2]
  tot[0] += (double)d[0];
  tot[1] += (double)d[1];
}

template <int ACT, int AGG>
__global__ __launch_bounds__(512, 2) void k_edge_bwd_chain(BatchView b, MlpW w, const bf16* __restrict__ e,
                                                           const bf16* __restrict__ zt, const bf16* __restrict__ at,
                                                           const float* __restrict__ de_in,
                                                           const float* __restrict__ dm, EdgeBwdOut o, float eps) {
  constexpr int H = 128, NW = EdgeBwdChain::NW;
  using L = EdgeBwdChain;
  __shared__ __align__(16) unsigned char smem[L::bytes];
  bf16x8* F2 = (bf16x8*)smem;                  // W2: rows u, k = z
  bf16x8* F2T = (bf16x8*)(smem + L::WS);       // W2^T: rows z, k = u
  bf16x8* F1T = (bf16x8*)(smem + 2 * L::WS);   // e-block of W1, transposed: rows e, k = a
  unsigned char* regs = smem + 3 * L::WS;
  unsigned char* reg = regs + wave_id() * L::REG;
  float* fr = (float*)reg;
  const int l = lane_id(), li = l & 15, lg = l >> 4;
  const int nw = gridDim.x * NW, wv = wave_rank(NW);
  const int wm = wave_id() & 3, wn = wave_id() >> 2;

  stage_frags<8, 4, 512>(F2, (const bf16*)w.W2, H);
  stage_frags<8, 4, 512>(F2T, (const bf16*)w.W2T, H);
  stage_frags<8, 4, 512>(F1T, (const bf16*)w.W1T, H);
  // b2 and gamma: lane l holds 4 of the 256 floats
  const f32x4 vec = *(const f32x4*)((l < 32 ? w.b2 : w.gamma) + 4 * (l & 31));
  const WaveEdges we(b, wv, nw);
  // every wave of the workgroup takes as many steps as its longest range needs
  if (l == 0) *(int*)reg = we.end - we.begin;
  __syncthreads();
  int longest = 0;
#pragma unroll
  for (int k = 0; k < NW; ++k) longest = max(longest, *(const int*)(regs + k * L::REG));
  const int steps = (__builtin_amdgcn_readfirstlane(longest) + 15) >> 4;
  __syncthreads();

  const int last = max(we.end - 1, 0);  // rows past the range repeat its last edge and count as zero
  int rv = 0, rn = 0;
  auto load_idx = [&](int e0) {
    const int k = min(e0 + li, last);
    rv = b.recv[k];
    rn = k + 1 < b.E ? b.recv[k + 1] : -1;
  };
  bf16x8 z[4], av[4];
  auto load_rows = [&](int e0) {
    const int k = min(e0 + li, last);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      z[c] = *(const bf16x8*)(zt + (size_t)k * H + 32 * c + 8 * lg);
      if constexpr (ACT != 0) av[c] = *(const bf16x8*)(at + (size_t)k * H + 32 * c + 8 * lg);
    }
  };
  f32x4 accW2[2][4], accW1[2][4];
  zero_acc(accW2);
  zero_acc(accW1);
  double cb2[2] = {}, cg[2] = {}, cbt[2] = {}, cb1[2] = {};
  float s0 = 0.f, s1 = 0.f;  // running receiver sum (lane l: features 2 l, 2 l + 1)
  if (steps) {
    load_idx(we.begin);
    load_rows(we.begin);
  }
  for (int it = 0; it < steps; ++it) {
    // lane numbers the compiler cannot see through: the LDS addresses made of
    // them are formed again in every step instead of spilled
    const int l = opaque(lane_id()), li = l & 15, lg = l >> 4;
    const int e0 = we.begin + 16 * it;
    const int ne = min(16, we.end - e0);  // may be <= 0
    const bool ok = li < ne;
    const int rc = rv;
    const unsigned ends = (unsigned)__ballot(rv != rn) & 0xffffu;
    const bool more = it + 1 < steps;
    f32x4 dve[8];  // de', in flight during u and its statistics
    if (de_in) {
      const float* p = de_in + (size_t)min(e0 + li, last) * H + 4 * lg;
#pragma unroll
      for (int mb = 0; mb < 8; ++mb) dve[mb] = *(const f32x4*)(p + 16 * mb);
    } else {
#pragma unroll
      for (int mb = 0; mb < 8; ++mb) dve[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    if (more) load_idx(e0 + 16);
    wave_sync();
    *(f32x4*)(fr + 4 * l) = vec;
    wave_sync();
    auto vget = [&](int v, int mb) { return *(const f32x4*)(fr + 128 * v + 16 * mb + 4 * lg); };
    // u = W2 z + b2, xhat
    f32x4 x[8];
    zero_blocks(x);
    chain_gemm<true>(x, F2, z);
    f32x4 dvm[8];  // dm_r, in flight during the statistics
#pragma unroll
    for (int mb = 0; mb < 8; ++mb) dvm[mb] = *(const f32x4*)(dm + (size_t)rc * H + 16 * mb + 4 * lg);
#pragma unroll
    for (int mb = 0; mb < 8; ++mb) x[mb] += vget(0, mb);
    const float inv = ln128(x, eps);
    // dv = dm_r + de'
    f32x4 g[8];
#pragma unroll
    for (int mb = 0; mb < 8; ++mb)
#pragma unroll
      for (int r = 0; r < 4; ++r) g[mb][r] = ok ? dvm[mb][r] + dve[mb][r] : 0.f;
    // LayerNorm adjoint: g = du
    {
      f32x4 t[8];
#pragma unroll
      for (int mb = 0; mb < 8; ++mb) t[mb] = g[mb] * x[mb];
      colsum16(t, cg);
    }
    colsum16(g, cbt);
    float sg = 0.f, sgx = 0.f;  // row sums of dv gamma and of dv gamma xhat
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 g0 = vget(1, 2 * q), g1 = vget(1, 2 * q + 1);
      f32x4 &lo = g[2 * q], &hi = g[2 * q + 1];
      const f32x4 &xl = x[2 * q], &xu = x[2 * q + 1];
      float a[4], d[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float dv1 = hi[r];
        lo[r] *= g0[r];
        hi[r] = dv1 * g1[r];
        a[r] = __builtin_fmaf(dv1, g1[r], lo[r]);
        d[r] = __builtin_fmaf(xu[r], hi[r], xl[r] * lo[r]);
      }
      sg += add_xor32(add_xor16((a[0] + a[1]) + (a[2] + a[3])));
      sgx += add_xor32(add_xor16((d[0] + d[1]) + (d[2] + d[3])));
    }
#pragma unroll
    for (int mb = 0; mb < 8; ++mb)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        g[mb][r] = __builtin_fmaf(sgx * (-1.f / H), x[mb][r], __builtin_fmaf(sg, -1.f / H, g[mb][r])) * inv;
    colsum16(g, cb2);
    bf16x8 du[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) du[c] = to_natural(g[2 * c], g[2 * c + 1]);
    // [du | z] of the 128 edges; act'(a) from z (ReLU: a > 0 exactly where z > 0) or a
    wave_sync();
    tile_put(reg, du, l);
    tile_put(reg + 4096, z, l);
    bf16x8 az[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) az[c] = ACT ? av[c] : z[c];
    bf16x8 er[4];
    {
      const int k = min(e0 + li, last);
#pragma unroll
      for (int c = 0; c < 4; ++c) er[c] = *(const bf16x8*)(e + (size_t)max(k, 0) * H + 32 * c + 8 * lg);
    }
    lds_sync();
    tile_wgrad(accW2, regs, 0, 4096, wm, wn, l);  // dW2 += du^T z
    // dz = W2^T du ; da = dz * act'(a)
    zero_blocks(x);
    chain_gemm<true>(x, F2T, du);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      f32x4 lo, hi;
      from_natural(az[c], lo, hi);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        x[2 * c][r] *= act_d<ACT>(lo[r]);
        x[2 * c + 1][r] *= act_d<ACT>(hi[r]);
      }
    }
    bf16x8 da[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      da[c] = to_natural(x[2 * c], x[2 * c + 1]);
      if (ok) *(bf16x8*)((bf16*)o.da + (size_t)(e0 + li) * H + 32 * c + 8 * lg) = da[c];
    }
    lds_sync();  // every wave is done with [du | z]
    // S_r: receiver sums of da in edge order; their total is db1
#pragma unroll
    for (int mb = 0; mb < 8; ++mb) *(f32x4*)(fr + li * 128 + (((4 * mb + lg) ^ li) << 2)) = x[mb];
    wave_sync();
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (i < ne) {
        const float2 v = *(const float2*)(fr + i * 128 + ((((l >> 1) ^ i) << 2) | ((l & 1) << 1)));
        s0 += v.x;
        s1 += v.y;
        if (ends >> i & 1) {
          const int r = __builtin_amdgcn_readlane(rc, i);
          *(float2*)(o.S_r + (size_t)r * H + 2 * l) = float2{s0, s1};
          cb1[0] += (double)s0;
          cb1[1] += (double)s1;
          s0 = 0.f;
          s1 = 0.f;
        }
      }
    }
    wave_sync();
    tile_put(reg, da, l);
    tile_put(reg + 4096, er, l);
    if (more) load_rows(e0 + 16);  // the next step's rows, in flight from here
    lds_sync();
    tile_wgrad(accW1, regs, 0, 4096, wm, wn, l);  // dW1[:, 2H:3H] += da^T e
    // de = de' (+ dm_r) + (W1^T da)[2H:3H]
    zero_blocks(x);
    chain_gemm<true>(x, F1T, da);
    if (ok) {
      const size_t at_ = (size_t)(e0 + li) * H + 4 * lg;
      f32x4 v[8];
      if (de_in) {
#pragma unroll
        for (int mb = 0; mb < 8; ++mb) v[mb] = *(const f32x4*)(de_in + at_ + 16 * mb);
      } else {
#pragma unroll
        for (int mb = 0; mb < 8; ++mb) v[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int mb = 0; mb < 8; ++mb) {
        if (AGG) v[mb] += *(const f32x4*)(dm + (size_t)rc * H + 16 * mb + 4 * lg);
        *(f32x4*)(o.de_out + at_ + 16 * mb) = x[mb] + v[mb];
      }
    }
    lds_sync();  // every wave is done with [da | e]
  }
  zero_empty_rows(b, o.S_r, H, wv, nw);
  // column sums of the workgroup's eight waves: lane li of group lg holds
  // values 2k, 2k + 1 of block layout (feature 16 (v / 4) + 4 lg + v % 4)
  double* ds = (double*)smem;  // [8 waves][4][128]; the weights are done with
  __syncthreads();
  {
    double* d = ds + wave_id() * 512;
    const int v = colsum_slot(li), f = 16 * (v >> 2) + 4 * lg + (v & 3);
    d[2 * l] = cb1[0];
    d[2 * l + 1] = cb1[1];
    d[128 + f] = cb2[0];
    d[128 + f + 1] = cb2[1];
    d[256 + f] = cg[0];
    d[256 + f + 1] = cg[1];
    d[384 + f] = cbt[0];
    d[384 + f + 1] = cbt[1];
  }
  __syncthreads();
  {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < NW; ++k) s += ds[k * 512 + threadIdx.x];
    o.partial[(size_t)blockIdx.x * 512 + threadIdx.x] = (float)s;
  }
  float* q2 = o.wpart + (size_t)blockIdx.x * 2 * H * H;
  float* q1 = q2 + H * H;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int at_ = (32 * wm + 16 * i + 4 * lg + r) * H + 64 * wn + 16 * j + li;
        q2[at_] = accW2[i][j][r];
        q1[at_] = accW1[i][j][r];
      }
}

int edge_bwd_chain_grid(const Shape& s, int E) {
  return edge_stream(s) ? edge_stream_grid(s, E) : std::max(1, std::min(256, (E + 47) / 48));
}

void launch_edge_bwd_chain(const Shape& s, const BatchView& b, const MlpW& w, const void* e, const void* zt,
                           const void* at, const float* de_in, const float* dm, const EdgeBwdOut& o, hipStream_t st) {
  if (s.act != 0 && !at) {
    g_config_error = 1;
    return;
  }
  auto go = [&](auto act, auto agg) {
    k_edge_bwd_chain<decltype(act)::value, decltype(agg)::value><<<edge_bwd_chain_grid(s, b.E), 512, 0, st>>>(
        b, w, (const bf16*)e, (const bf16*)zt, (const bf16*)at, de_in, dm, o, s.eps);
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
