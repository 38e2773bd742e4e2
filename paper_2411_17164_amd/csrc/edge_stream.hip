// Edge kernels with streamed weights (BF16, H = 256 and 512; see stream.hpp).
#include <algorithm>
#include <type_traits>

#include "kernels.hpp"
#include "segsum.hpp"
#include "stream.hpp"

namespace xmgn {

// ---------------------------------------------------------------------------
// Fused edge processor, forward, gathered form.  H = 256: eight waves of 256
// registers; H = 512: four of 512, since a wave's accumulators and operands
// alone take 320.  A wave's h_r and h_s rows come a tile ahead, e at the
// tile's start.  On 100k nodes, H = 256, 886k edges: 774 us (600 TFLOP/s)
// where the workgroup-tile kernel took 2,170 us on its 32-row tiles; weights
// kept in registers on their way to LDS (one slab ahead) gave 1,064 us, 400 us
// of it waiting for them.  On 50k nodes, H = 512, SiLU, 444k edges: 1,844 us
// (505 TFLOP/s) against 2,477 us in the 64-row K-sliced kernel.  What bounds it
// now is the weight traffic: every 128 (64) rows read 0.5 (2) MB of fragments
// from L2 into LDS and each wave reads all of it again from there.
// ---------------------------------------------------------------------------
template <int H>
struct EdgeFwdStream {
  static constexpr int NW = H == 256 ? 8 : 4, NT = 64 * NW, ET = 1;
  static constexpr int MBS = H / 16, KC = H / 32;  // output blocks, k chunks of one H-wide operand
  static constexpr int S = 4 * KC;                 // slabs: W1 (3 H), then W2
  static constexpr size_t RING = 4 * MBS * 1024;
  static constexpr size_t VEC = 4 * H * 4;         // b1, b2, gamma, beta
  static constexpr size_t BUF = 8192;              // per wave: 16 rows x 128 FP32
  // where it does not fit behind the ring (H = 512), the waves' buffers lie in
  // the slot of the cycle's last slab, free from its products to the next tile
  static constexpr bool ALIAS = RING + VEC + NW * BUF > 160 * 1024;
  static constexpr size_t bytes = RING + VEC + (ALIAS ? 0 : NW * BUF);
  static_assert(!ALIAS || NW * BUF <= RING / 4, "the buffers fit in one slot");
};

template <int H, int ACT, int AGG>
__global__ __launch_bounds__(EdgeFwdStream<H>::NT, EdgeFwdStream<H>::NW / 4) void k_edge_fwd_stream(BatchView b, MlpW w, const bf16* __restrict__ h,
                                                            const bf16* __restrict__ e, bf16* __restrict__ e_out,
                                                            float* __restrict__ m, bf16* __restrict__ z_out,
                                                            bf16* __restrict__ a_out, float eps) {
  using L = EdgeFwdStream<H>;
  constexpr int NW = L::NW, NT = L::NT, ET = L::ET, MT = 16 * ET, MBS = L::MBS, KC = L::KC;
  constexpr int SW = 64;  // LayerNorm span
  __shared__ __align__(16) unsigned char smem[L::bytes];
  float* vec = (float*)(smem + L::RING);
  unsigned char* bufs = smem + (L::ALIAS ? L::RING / 4 * 3 : L::RING + L::VEC);
  float* buf = (float*)(bufs + wave_id() * L::BUF);
  const int l = lane_id(), li = l & 15, lg = l >> 4;
  const int nw = gridDim.x * NW, wv = wave_rank(NW);
  const WStream<NW, L::S, MBS> ws{(const unsigned char*)w.FS, smem};
  for (int c = threadIdx.x; c < H; c += NT) {
    vec[c] = w.b1[c];
    vec[H + c] = w.b2[c];
    vec[2 * H + c] = w.gamma[c];
    vec[3 * H + c] = w.beta[c];
  }
  auto vget = [&](int v, int mb) { return *(const f32x4*)(vec + v * H + 16 * mb + 4 * lg); };
  const WaveEdges we(b, wv, nw);
  const int steps = wg_steps<NW>(we.end - we.begin, MT, (int*)bufs, L::BUF / 4);
  const int last = max(we.end - 1, 0);

  int rv[ET], cv[ET], rn[ET];
  auto load_idx = [&](int e0) {
#pragma unroll
    for (int t = 0; t < ET; ++t) {
      const int k = min(e0 + 16 * t + li, last);
      rv[t] = b.recv[k];
      cv[t] = b.col[k];
      rn[t] = k + 1 < b.E ? b.recv[k + 1] : -1;
    }
  };
  // the rows' operands [h_r ; h_s] a tile ahead, e at the tile's start
  bf16x8 xr[KC][ET], xs[KC][ET], ec[KC][ET];
  auto load_rows = [&]() {
#pragma unroll
    for (int t = 0; t < ET; ++t) {
      const bf16* pr = h + (size_t)rv[t] * H + 8 * lg;
      const bf16* ps = h + (size_t)cv[t] * H + 8 * lg;
#pragma unroll
      for (int c = 0; c < KC; ++c) {
        xr[c][t] = *(const bf16x8*)(pr + 32 * c);
        xs[c][t] = *(const bf16x8*)(ps + 32 * c);
      }
    }
  };
  if (steps) {
    load_idx(we.begin);
    load_rows();
  }
  ws.start();
  lds_sync();
  SegSum<H> seg;
  for (int it = 0; it < steps; ++it) {
    const int e0 = we.begin + MT * it, ne = min(MT, we.end - e0);
    int rc[ET];
    unsigned ends[ET];
#pragma unroll
    for (int t = 0; t < ET; ++t) {
      rc[t] = rv[t];
      ends[t] = (unsigned)__ballot(rv[t] != rn[t]) & 0xffffu;
    }
    const bool more = it + 1 < steps;
    if (more) load_idx(e0 + MT);
    // the rows are needed from here, e two thirds into the first product (each
    // waited for at once: the compiler's counted waits do not know of the
    // weight loads in between)
#pragma unroll
    for (int c = 0; c < KC; ++c)
#pragma unroll
      for (int t = 0; t < ET; ++t) {
        arrived(xr[c][t]);
        arrived(xs[c][t]);
      }
#pragma unroll
    for (int t = 0; t < ET; ++t)
#pragma unroll
      for (int c = 0; c < KC; ++c)
        ec[c][t] = *(const bf16x8*)(e + (size_t)min(e0 + 16 * t + li, last) * H + 32 * c + 8 * lg);
    if constexpr (L::ALIAS) lds_sync();  // every wave is done with its buffer
    f32x4 acc[ET][MBS];
    zero_acc(acc);
    // one H-wide operand's chunks, from slab s0 on
    auto product = [&](int s0, int p0, int p1, bf16x8(&xs)[KC][ET]) {
#pragma unroll
      for (int c = 0; c < KC; ++c) {
        ws.begin(s0 + c);
        slab_gemm(acc, ws.frags(s0 + c), xs[c]);
        ws.end(s0 + c, p0, p1);
      }
    };
    product(0, 0, 3 * KC, xr);
    product(KC, 0, 3 * KC, xs);
#pragma unroll
    for (int c = 0; c < KC; ++c)
#pragma unroll
      for (int t = 0; t < ET; ++t) arrived(ec[c][t]);
    product(2 * KC, 0, 3 * KC, ec);
#pragma unroll
    for (int mb = 0; mb < MBS; ++mb) {
      const f32x4 bb = vget(0, mb);
#pragma unroll
      for (int t = 0; t < ET; ++t) acc[t][mb] += bb;
    }
    if (a_out) {
#pragma unroll
      for (int t = 0; t < ET; ++t)
#pragma unroll
        for (int c = 0; c < KC; ++c) {
          const bf16x8 v = to_natural(acc[t][2 * c], acc[t][2 * c + 1]);
          if (16 * t + li < ne) *(bf16x8*)(a_out + (size_t)(e0 + 16 * t + li) * H + 32 * c + 8 * lg) = v;
        }
    }
    bf16x8 z[KC][ET];
#pragma unroll
    for (int t = 0; t < ET; ++t)
#pragma unroll
      for (int c = 0; c < KC; ++c) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          acc[t][2 * c][r] = act_f<ACT>(acc[t][2 * c][r]);
          acc[t][2 * c + 1][r] = act_f<ACT>(acc[t][2 * c + 1][r]);
        }
        z[c][t] = to_natural(acc[t][2 * c], acc[t][2 * c + 1]);
      }
    // second product
    zero_acc(acc);
    product(3 * KC, 3 * KC, 4 * KC, z);
    if (z_out) {  // (stores ahead of the second product would hold up its weights' waits)
#pragma unroll
      for (int t = 0; t < ET; ++t)
#pragma unroll
        for (int c = 0; c < KC; ++c)
          if (16 * t + li < ne) *(bf16x8*)(z_out + (size_t)(e0 + 16 * t + li) * H + 32 * c + 8 * lg) = z[c][t];
    }
    if (more) load_rows();  // the next tile's, in flight during the epilogue
#pragma unroll
    for (int mb = 0; mb < MBS; ++mb) {
      const f32x4 bb = vget(1, mb);
#pragma unroll
      for (int t = 0; t < ET; ++t) acc[t][mb] += bb;
    }
#pragma unroll
    for (int t = 0; t < ET; ++t) ln_chain<H, SW>(acc[t], eps);
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      const f32x4 g0 = vget(2, 2 * c), g1 = vget(2, 2 * c + 1), b0 = vget(3, 2 * c), b1 = vget(3, 2 * c + 1);
#pragma unroll
      for (int t = 0; t < ET; ++t) {
        f32x4 e_lo, e_hi;
        from_natural(ec[c][t], e_lo, e_hi);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float v0 = __builtin_fmaf(g0[r], acc[t][2 * c][r], b0[r]);
          const float v1 = __builtin_fmaf(g1[r], acc[t][2 * c + 1][r], b1[r]);
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

bool edge_fwd_stream(const Shape& s) { return s.prec == 1 && (s.H == 256 || s.H == 512); }

void launch_edge_fwd_stream(const Shape& s, const BatchView& b, const MlpW& w, const void* h, const void* e,
                            void* e_out, float* m, void* z_out, void* a_out, hipStream_t st) {
  auto go = [&](auto hh, auto act, auto agg) {
    constexpr int H = decltype(hh)::value, NT = EdgeFwdStream<H>::NT, RW = NT / 4 * EdgeFwdStream<H>::ET;
    const int grid = std::max(1, std::min(256, (b.E + RW - 1) / RW));
    k_edge_fwd_stream<H, decltype(act)::value, decltype(agg)::value><<<grid, NT, 0, st>>>(
        b, w, (const bf16*)h, (const bf16*)e, (bf16*)e_out, m, (bf16*)z_out, (bf16*)a_out, s.eps);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  auto by_h = [&](auto act, auto agg) {
    if (s.H == 256)
      go(std::integral_constant<int, 256>{}, act, agg);
    else
      go(std::integral_constant<int, 512>{}, act, agg);
  };
  if (s.act) {
    if (s.agg) by_h(I1{}, I1{}); else by_h(I1{}, I0{});
  } else {
    if (s.agg) by_h(I0{}, I1{}); else by_h(I0{}, I0{});
  }
}

// ---------------------------------------------------------------------------
// Edge adjoint with z (and a) from the tape; du and da go out for the separate
// weight-gradient products (256 x 256 accumulators do not fit beside a wave's
// rows).  Waves as in the forward; z comes a tile ahead, dm_r and de' two
// groups of 64 features ahead of their use.  On 100k nodes, H = 256, 886k
// edges: 1,165 us (3.9 GB, 3.3 TB/s) where the 32-row workgroup-tile kernel
// took 2,717 us; on 50k nodes, H = 512, SiLU, 444k edges: 2,151 us (4.0 GB,
// 1.9 TB/s) against 5,094 us.  H = 256 is bound by HBM and the barriers around
// its LayerNorm, H = 512 by the 1.5 MB of weight fragments that every 64 rows
// read.  da, du, de and S_r are the same bits as that kernel's.
// ---------------------------------------------------------------------------
template <int H>
struct EdgeBwdStream {
  static constexpr int NW = H == 256 ? 8 : 4, NT = 64 * NW;
  static constexpr int MBS = H / 16, KC = H / 32;
  static constexpr int S = 3 * KC;  // W2, W2^T, e-block of W1^T
  static constexpr size_t RING = 4 * MBS * 1024;
  static constexpr size_t VEC = 2 * H * 4;  // b2, gamma
  static constexpr size_t BUF = 8192;       // per wave: 16 rows x 128 FP32
  // H = 512: in the slot of W2^T's last slab, free from its products to the
  // next product's first
  static constexpr bool ALIAS = RING + VEC + NW * BUF > 160 * 1024;
  static constexpr size_t bytes = RING + VEC + (ALIAS ? 0 : NW * BUF);
  static_assert(!ALIAS || NW * BUF <= RING / 4, "the buffers fit in one slot");
  static_assert(NW * 4 * H * 8 <= RING, "the column sums fit in the ring");
};

template <int H, int ACT, int AGG>
__global__ __launch_bounds__(EdgeBwdStream<H>::NT, EdgeBwdStream<H>::NW / 4) void k_edge_bwd_stream(
    BatchView b, MlpW w, const bf16* __restrict__ zt, const bf16* __restrict__ at, const float* __restrict__ de_in,
    const float* __restrict__ dm, EdgeBwdOut o, float eps) {
  using L = EdgeBwdStream<H>;
  constexpr int NW = L::NW, NT = L::NT, MBS = L::MBS, KC = L::KC;
  constexpr int SW = 64, NG = H / 64;  // LayerNorm spans: groups of four blocks
  __shared__ __align__(16) unsigned char smem[L::bytes];
  float* vec = (float*)(smem + L::RING);
  unsigned char* bufs = smem + (L::ALIAS ? (2 * KC - 1) % 4 * (L::RING / 4) : L::RING + L::VEC);
  float* buf = (float*)(bufs + wave_id() * L::BUF);
  const int nw = gridDim.x * NW, wv = wave_rank(NW);
  const WStream<NW, L::S, MBS> ws{(const unsigned char*)w.BS, smem};
  for (int c = threadIdx.x; c < H; c += NT) {
    vec[c] = w.b2[c];
    vec[H + c] = w.gamma[c];
  }
  const WaveEdges we(b, wv, nw);
  const int steps = wg_steps<NW>(we.end - we.begin, 16, (int*)bufs, L::BUF / 4);
  const int last = max(we.end - 1, 0);  // rows past the range repeat its last edge and count as zero

  int rv = 0, rn = 0;
  bf16x8 z[1][KC];
  auto load_tile = [&](int e0) {
    const int li = lane_id() & 15, lg = lane_id() >> 4;
    const int k = min(e0 + li, last);
    rv = b.recv[k];
    rn = k + 1 < b.E ? b.recv[k + 1] : -1;
#pragma unroll
    for (int c = 0; c < KC; ++c) z[0][c] = *(const bf16x8*)(zt + (size_t)k * H + 32 * c + 8 * lg);
  };
  if (steps) load_tile(we.begin);
  ws.start();
  lds_sync();
  SegSum<H> seg;
  double cb2[NG] = {}, cg[NG] = {}, cbt[NG] = {}, cb1[H / 128][2] = {};
  for (int it = 0; it < steps; ++it) {
    const int l = opaque(lane_id()), li = l & 15, lg = l >> 4;
    const int e0 = we.begin + 16 * it;
    const int ne = min(16, we.end - e0);  // may be <= 0
    const bool ok = li < ne;
    const int rc = rv;
    const unsigned ends = (unsigned)__ballot(rv != rn) & 0xffffu;
    const bool more = it + 1 < steps;
    const size_t row = (size_t)min(e0 + li, last) * H;
    auto vget = [&](int v, int mb) { return *(const f32x4*)(vec + v * H + 16 * mb + 4 * lg); };
    f32x4 x[1][MBS];
    auto product = [&](int s0, const bf16x8(&xs)[KC]) {
      zero_acc(x);
#pragma unroll
      for (int c = 0; c < KC; ++c) {
        const bf16x8 xc[1] = {xs[c]};
        ws.begin(s0 + c);
        slab_gemm(x, ws.frags(s0 + c), xc);
        ws.end(s0 + c, s0, s0 + KC);
      }
    };
#pragma unroll
    for (int c = 0; c < KC; ++c) arrived(z[0][c]);
    // u = W2 z + b2, xhat
    product(0, z[0]);
    // dv = dm_r + de', two groups of blocks in flight
    f32x4 pm[2][4], pe[2][4];
    auto load_dv = [&](int s, int gr) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        pm[s][k] = *(const f32x4*)(dm + (size_t)rc * H + 64 * gr + 16 * k + 4 * lg);
        pe[s][k] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      if (de_in) {
#pragma unroll
        for (int k = 0; k < 4; ++k) pe[s][k] = *(const f32x4*)(de_in + row + 64 * gr + 16 * k + 4 * lg);
      }
    };
    load_dv(0, 0);
    load_dv(1, 1);
#pragma unroll
    for (int mb = 0; mb < MBS; ++mb) x[0][mb] += vget(0, mb);
    const float inv = ln_chain<H, SW>(x[0], eps);
    f32x4 g[MBS];
    float sg = 0.f, sgx = 0.f;  // row sums of dv gamma and of dv gamma xhat
#pragma unroll
    for (int gr = 0; gr < NG; ++gr) {
      f32x4 dv[4], t[4];
      float a[4], d[4];
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) dv[k][r] = ok ? pm[gr & 1][k][r] + pe[gr & 1][k][r] : 0.f;
      if (gr + 2 < NG) load_dv(gr & 1, gr + 2);
#pragma unroll
      for (int k = 0; k < 4; ++k) t[k] = dv[k] * x[0][4 * gr + k];
      cg[gr] += (double)colsum64(t);
      cbt[gr] += (double)colsum64(dv);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const f32x4 gm = vget(1, 4 * gr + k);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float p = dv[k][r] * gm[r];
          a[r] = k ? __builtin_fmaf(dv[k][r], gm[r], a[r]) : p;
          d[r] = k ? __builtin_fmaf(x[0][4 * gr + k][r], p, d[r]) : x[0][4 * gr][r] * p;
          g[4 * gr + k][r] = p;
        }
      }
      sg += add_xor32(add_xor16((a[0] + a[1]) + (a[2] + a[3])));
      sgx += add_xor32(add_xor16((d[0] + d[1]) + (d[2] + d[3])));
    }
    bf16x8 du[KC];
#pragma unroll
    for (int gr = 0; gr < NG; ++gr) {
      f32x4 t[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          t[k][r] = __builtin_fmaf(sgx * (-1.f / H), x[0][4 * gr + k][r], __builtin_fmaf(sg, -1.f / H, g[4 * gr + k][r])) * inv;
      }
      cb2[gr] += (double)colsum64(t);
      du[2 * gr] = to_natural(t[0], t[1]);
      du[2 * gr + 1] = to_natural(t[2], t[3]);
    }
    if (ok) {
#pragma unroll
      for (int c = 0; c < KC; ++c) *(bf16x8*)((bf16*)o.du + row + 32 * c + 8 * lg) = du[c];
    }
    bf16x8 av[KC];
    if constexpr (ACT != 0) {
#pragma unroll
      for (int c = 0; c < KC; ++c) av[c] = *(const bf16x8*)(at + row + 32 * c + 8 * lg);
    }
    // dz = W2^T du ; da = dz * act'(a)  (ReLU: a > 0 exactly where z > 0)
    product(KC, du);
    bf16x8 da[KC];
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      f32x4 lo, hi;
      from_natural(ACT ? av[c] : z[0][c], lo, hi);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        x[0][2 * c][r] *= act_d<ACT>(lo[r]);
        x[0][2 * c + 1][r] *= act_d<ACT>(hi[r]);
      }
      da[c] = to_natural(x[0][2 * c], x[0][2 * c + 1]);
      if (ok) *(bf16x8*)((bf16*)o.da + row + 32 * c + 8 * lg) = da[c];
    }
    // S_r: receiver sums of da in edge order; their total is db1
    seg.add(x[0], ends, rc, ne, buf, o.S_r, [&](int p, const float2& s) {
      cb1[p][0] += (double)s.x;
      cb1[p][1] += (double)s.y;
    });
    if constexpr (L::ALIAS) lds_sync();  // every wave is done with its buffer
    if (more) load_tile(e0 + 16);        // the next tile's, in flight during the last product
    // de = de' (+ dm_r) + (W1^T da)[2H:3H]
    product(2 * KC, da);
    if (ok) {
#pragma unroll
      for (int m0 = 0; m0 < MBS; m0 += 8) {
        f32x4 v[8];
        if (de_in) {
#pragma unroll
          for (int k = 0; k < 8; ++k) v[k] = *(const f32x4*)(de_in + row + 16 * (m0 + k) + 4 * lg);
        } else {
#pragma unroll
          for (int k = 0; k < 8; ++k) v[k] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          if (AGG) v[k] += *(const f32x4*)(dm + (size_t)rc * H + 16 * (m0 + k) + 4 * lg);
          *(f32x4*)(o.de_out + row + 16 * (m0 + k) + 4 * lg) = x[0][m0 + k] + v[k];
        }
      }
    }
  }
  zero_empty_rows(b, o.S_r, H, wv, nw);
  // column sums of the workgroup's waves, over the ring
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (weights still on their way into it)
  __syncthreads();
  double* ds = (double*)smem;  // [NW][4][H]
  {
    const int l = lane_id(), li = l & 15, lg = l >> 4;
    double* d = ds + wave_id() * 4 * H;
#pragma unroll
    for (int p = 0; p < H / 128; ++p) {
      d[128 * p + 2 * l] = cb1[p][0];
      d[128 * p + 2 * l + 1] = cb1[p][1];
    }
#pragma unroll
    for (int gr = 0; gr < NG; ++gr) {
      const int f = 64 * gr + 16 * (li >> 2) + 4 * lg + (li & 3);
      d[H + f] = cb2[gr];
      d[2 * H + f] = cg[gr];
      d[3 * H + f] = cbt[gr];
    }
  }
  __syncthreads();
  for (int c = threadIdx.x; c < 4 * H; c += NT) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < NW; ++k) s += ds[k * 4 * H + c];
    o.partial[(size_t)blockIdx.x * 4 * H + c] = (float)s;
  }
}

int edge_bwd_stream_grid(int H, int E) {
  const int rows = H == 256 ? 128 : 64;
  return std::max(1, std::min(256, (E + rows - 1) / rows));
}

void launch_edge_bwd_stream(const Shape& s, const BatchView& b, const MlpW& w, const void* zt, const void* at,
                            const float* de_in, const float* dm, const EdgeBwdOut& o, hipStream_t st) {
  if (s.act != 0 && !at) {
    g_config_error = 1;
    return;
  }
  auto go = [&](auto hh, auto act, auto agg) {
    constexpr int H = decltype(hh)::value;
    k_edge_bwd_stream<H, decltype(act)::value, decltype(agg)::value>
        <<<edge_bwd_stream_grid(H, b.E), EdgeBwdStream<H>::NT, 0, st>>>(b, w, (const bf16*)zt, (const bf16*)at, de_in, dm,
                                                                       o, s.eps);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  auto by_h = [&](auto act, auto agg) {
    if (s.H == 256)
      go(std::integral_constant<int, 256>{}, act, agg);
    else
      go(std::integral_constant<int, 512>{}, act, agg);
  };
  if (s.act) {
    if (s.agg) by_h(I1{}, I1{}); else by_h(I1{}, I0{});
  } else {
    if (s.agg) by_h(I0{}, I1{}); else by_h(I0{}, I0{});
  }
}

}  // namespace xmgn
