// Edge kernels with streamed weights (see stream.hpp).
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
// (505 TFLOP/s) against 2,477 us in the 64-row K-sliced kernel.  FP32 at
// H = 128 on 50k nodes, 443k edges: 590 to 610 us (98 TFLOP/s, an FP32 library
// product here reaches 152) against 831 us.  Every 128 (64) rows bring 0.5 (2) MB
// of fragments from L2 into LDS, and each wave reads all of it again from there.
// By counters, of the cycles that a CU is busy: H = 256 30% MFMA, 37% LDS, its
// waves waiting (slabs, rows, barriers) for 42% of theirs; H = 512 22%, 25% and
// 41%, with one wave per SIMD to hide it; FP32 73% MFMA.
// ---------------------------------------------------------------------------
template <typename T, int H, int W>
struct EdgeFwdStream : StreamDims<T, H, W> {
  using D = StreamDims<T, H, W>;
  static constexpr int S = 4 * D::SP;              // slabs: W1 (3 H), then W2
  static constexpr size_t VEC = 4 * H * 4;         // b1, b2, gamma, beta
  static constexpr size_t BUF = 8192;              // per wave: 16 rows x 128 FP32
  // where it does not fit behind the ring (H = 512), the waves' buffers lie in
  // the slot of the cycle's last slab, free from its products to the next tile
  static constexpr bool ALIAS = D::RING + VEC + D::NW * BUF > 160 * 1024;
  static constexpr size_t bytes = D::RING + VEC + (ALIAS ? 0 : D::NW * BUF);
  static_assert(!ALIAS || D::NW * BUF <= D::RING / 4, "the buffers fit in one slot");
};
// LayerNorm spans of the edge MLP: the columns of one of four waves (H = 128
// and 256) or eight (H = 512)
template <int H>
constexpr int edge_span() {
  return H == 128 ? 32 : 64;
}

template <typename T, int H, int W, int ACT, int AGG>
__global__ __launch_bounds__((StreamDims<T, H, W>::NT), (StreamDims<T, H, W>::NW / 4)) void k_edge_fwd_stream(
    BatchView b, MlpW w, const T* __restrict__ h, const T* __restrict__ e, T* __restrict__ e_out,
    float* __restrict__ m, T* __restrict__ z_out, T* __restrict__ a_out, float eps) {
  using L = EdgeFwdStream<T, H, W>;
  using C = Chunk<T>;
  using V = typename C::V;
  constexpr int NW = L::NW, NT = L::NT, MBS = L::MBS, KC = L::KC, BLK = C::BLK;
  __shared__ __align__(16) unsigned char smem[L::bytes];
  float* vec = (float*)(smem + L::RING);
  unsigned char* bufs = smem + (L::ALIAS ? L::RING / 4 * 3 : L::RING + L::VEC);
  float* buf = (float*)(bufs + wave_id() * L::BUF);
  const int l = lane_id(), li = l & 15, lg = l >> 4;
  const int nw = gridDim.x * NW, wv = wave_rank(NW);
  const WStream<NW, L::S, L::FR> ws{(const unsigned char*)w.FS, smem};
  for (int c = threadIdx.x; c < H; c += NT) {
    vec[c] = w.b1[c];
    vec[H + c] = w.b2[c];
    vec[2 * H + c] = w.gamma[c];
    vec[3 * H + c] = w.beta[c];
  }
  auto vget = [&](int v, int mb) { return *(const f32x4*)(vec + v * H + 16 * mb + 4 * lg); };
  const WaveEdges we(b, wv, nw);
  const int steps = wg_steps<NW>(we.end - we.begin, 16, (int*)bufs, L::BUF / 4);
  const int last = max(we.end - 1, 0);

  int rv = 0, cv = 0, rn = 0;
  auto load_idx = [&](int e0) {
    const int k = min(e0 + li, last);
    rv = b.recv[k];
    cv = b.col[k];
    rn = k + 1 < b.E ? b.recv[k + 1] : -1;
  };
  // the rows' operands [h_r ; h_s] a tile ahead, e behind h_r's part
  V xr[KC], xs[KC], ec[KC];
  auto load_rows = [&]() {
    load_row(xr, h + (size_t)rv * H, lg);
    load_row(xs, h + (size_t)cv * H, lg);
  };
  if (steps) {
    load_idx(we.begin);
    load_rows();
  }
  ws.start();
  lds_sync();
  SegSum<H> seg;
  for (int it = 0; it < steps; ++it) {
    const int e0 = we.begin + 16 * it, ne = min(16, we.end - e0);
    const bool ok = li < ne;
    const size_t row = (size_t)min(e0 + li, last) * H;
    const int rc = rv;
    const unsigned ends = (unsigned)__ballot(rv != rn) & 0xffffu;
    const bool more = it + 1 < steps;
    if (more) load_idx(e0 + 16);
    // (waited for at once: the compiler's counted waits do not know of the
    // weight loads behind them; e likewise below)
    arrived_row(xr);
    arrived_row(xs);
    if constexpr (L::ALIAS) lds_sync();  // every wave is done with its buffer
    f32x4 acc[MBS];
    zero_blocks(acc);
    stream_gemm<T, H>(ws, 0, 0, 3 * L::SP, acc, xr);
    load_row(ec, e + row, lg);
    stream_gemm<T, H>(ws, L::SP, 0, 3 * L::SP, acc, xs);
    arrived_row(ec);
    stream_gemm<T, H>(ws, 2 * L::SP, 0, 3 * L::SP, acc, ec);
#pragma unroll
    for (int mb = 0; mb < MBS; ++mb) acc[mb] += vget(0, mb);
    if (a_out && ok) {
#pragma unroll
      for (int c = 0; c < KC; ++c)
        *(V*)(a_out + row + C::KW * c + C::E * lg) = C::of(*(const f32x4(*)[BLK])(acc + BLK * c));
    }
    V z[KC];
#pragma unroll
    for (int c = 0; c < KC; ++c) {
#pragma unroll
      for (int k = 0; k < BLK; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[BLK * c + k][r] = act_f<ACT>(acc[BLK * c + k][r]);
      z[c] = C::of(*(const f32x4(*)[BLK])(acc + BLK * c));
    }
    // second product
    zero_blocks(acc);
    stream_gemm<T, H>(ws, 3 * L::SP, 3 * L::SP, 4 * L::SP, acc, z);
    // (stores ahead of the second product would hold up its weights' waits)
    if (z_out && ok) store_row(z_out + row, z, lg);
    if (more) load_rows();  // the next tile's, in flight during the epilogue
#pragma unroll
    for (int mb = 0; mb < MBS; ++mb) acc[mb] += vget(1, mb);
    ln_chain<H, edge_span<H>()>(acc, eps);
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      f32x4 en[BLK];
      C::to(ec[c], en);
#pragma unroll
      for (int k = 0; k < BLK; ++k) {
        const int mb = BLK * c + k;
        const f32x4 g = vget(2, mb), be = vget(3, mb);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float v = __builtin_fmaf(g[r], acc[mb][r], be[r]);
          en[k][r] += v;
          acc[mb][r] = AGG ? en[k][r] : v;  // the summand of m
        }
      }
      if (e_out && ok) *(V*)(e_out + row + C::KW * c + C::E * lg) = C::of(en);
    }
    seg.add(acc, ends, rc, ne, buf, m);
  }
  zero_empty_rows(b, m, H, wv, nw);
}

// The forms with streamed weights: all but BF16 at H = 128, whose weights fit
// in LDS.
bool edge_stream(const Shape& s) { return !(s.prec == 1 && s.H == 128); }

// FP32 at H = 128 with at most 12 rows for each of 1024 waves: four waves per
// workgroup.  One 16-row step is all there is to do then, and its FP32 MFMAs
// take 14 us on a SIMD.  Four against eight waves, us a launch: edge forward on
// 1,500 edges 26 / 40, on 9,000 28 / 42, on 12,000 30 / 43 where every node has
// six in-edges, but 47 / 44 where in-degrees vary and some ranges of whole
// segments take a second step, on 16,000 50 / 45.  Rows without segments gain up
// to 16,000, but lie on either side of the line at little cost: node adjoint 48 /
// 73 on 12,000 rows, 50 / 75 on 16,000, 87 / 78 on 24,000; edge encoder adjoint
// 41 / 57 on 12,000, 67 / 59 on 20,000.
bool stream_small(const Shape& s, int rows) { return s.prec == 0 && s.H == 128 && rows <= 1024 * 12; }

// One workgroup per CU as soon as there are 6 rows for each of its waves: a
// wave's time goes by its 16-row steps, so a few rows on every CU beat full
// steps on some, and ranges that end on whole segments stay within one step
// (12,000 edges, FP32, H = 128: 78 us on 94 full workgroups).
int stream_grid(int rows, int waves) { return std::max(1, std::min(256, (rows + 6 * waves - 1) / (6 * waves))); }
int edge_stream_grid(const Shape& s, int rows) {
  return stream_grid(rows, s.H * (s.prec == 1 ? 2 : 4) <= 512 && !stream_small(s, rows) ? 8 : 4);
}

// f(T{}, H, W) with the form's type, width and waves for so many rows
template <typename F>
static void by_form(const Shape& s, int rows, F f) {
  using std::integral_constant;
  using W0 = integral_constant<int, 0>;
  if (s.prec == 1) {
    if (s.H == 256)
      f(bf16{}, integral_constant<int, 256>{}, W0{});
    else
      f(bf16{}, integral_constant<int, 512>{}, W0{});
  } else {
    if (s.H == 128 && stream_small(s, rows))
      f(float{}, integral_constant<int, 128>{}, integral_constant<int, 4>{});
    else if (s.H == 128)
      f(float{}, integral_constant<int, 128>{}, W0{});
    else
      f(float{}, integral_constant<int, 256>{}, W0{});
  }
}
template <typename F>
static void by_act_agg(const Shape& s, F f) {
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  if (s.act) {
    if (s.agg) f(I1{}, I1{}); else f(I1{}, I0{});
  } else {
    if (s.agg) f(I0{}, I1{}); else f(I0{}, I0{});
  }
}

void launch_edge_fwd_stream(const Shape& s, const BatchView& b, const MlpW& w, const void* h, const void* e,
                            void* e_out, float* m, void* z_out, void* a_out, hipStream_t st) {
  by_form(s, b.E, [&](auto t, auto hh, auto ww) {
    using T = decltype(t);
    constexpr int H = decltype(hh)::value, W = decltype(ww)::value;
    by_act_agg(s, [&](auto act, auto agg) {
      k_edge_fwd_stream<T, H, W, decltype(act)::value, decltype(agg)::value>
          <<<edge_stream_grid(s, b.E), StreamDims<T, H, W>::NT, 0, st>>>(b, w, (const T*)h, (const T*)e, (T*)e_out, m,
                                                                     (T*)z_out, (T*)a_out, s.eps);
    });
  });
}

// ---------------------------------------------------------------------------
// Edge adjoint with z (and a) from the tape; du and da go out for the separate
// weight-gradient products (256 x 256 accumulators do not fit beside a wave's
// rows).  Waves as in the forward; z comes a tile ahead, dm_r and de' two
// groups of 64 features ahead of their use.  On 100k nodes, H = 256, 886k
// edges: 1,165 us (3.9 GB, 3.3 TB/s) where the 32-row workgroup-tile kernel
// took 2,717 us; on 50k nodes, H = 512, SiLU, 444k edges: 2,151 us (4.0 GB,
// 1.9 TB/s) against 5,094 us; FP32, H = 128, 443k edges: 515 to 540 us against 789.
// By counters H = 256 moves 4.9 GB (de' twice) at 4.35 TB/s, near a large copy's
// 4.9: bound by HBM.  H = 512 moves 6.2 GB (de' twice, and spills of 544 bytes a
// lane under SiLU) at 3.05 TB/s, its one wave per SIMD waiting for 35% of its
// cycles; FP32 is busy with MFMA for 61%.  da, du, de and S_r are the same bits as
// that kernel's.
// ---------------------------------------------------------------------------
template <typename T, int H, int W>
struct EdgeBwdStream : StreamDims<T, H, W> {
  using D = StreamDims<T, H, W>;
  static constexpr int S = 3 * D::SP;  // W2, W2^T, e-block of W1^T
  static constexpr size_t VEC = 2 * H * 4;  // b2, gamma
  static constexpr size_t BUF = 8192;       // per wave: 16 rows x 128 FP32
  // H = 512: in the slot of W2^T's last slab, free from its products to the
  // next product's first
  static constexpr bool ALIAS = D::RING + VEC + D::NW * BUF > 160 * 1024;
  static constexpr size_t bytes = D::RING + VEC + (ALIAS ? 0 : D::NW * BUF);
  static_assert(D::SP % 4 == 0, "whole rounds of the ring");
  static_assert(!ALIAS || D::NW * BUF <= D::RING / 4, "the buffers fit in one slot");
  static_assert(D::NW * 4 * H * 8 <= D::RING, "the column sums fit in the ring");
};

template <typename T, int H, int W, int ACT, int AGG>
__global__ __launch_bounds__((StreamDims<T, H, W>::NT), (StreamDims<T, H, W>::NW / 4)) void k_edge_bwd_stream(
    BatchView b, MlpW w, const T* __restrict__ zt, const T* __restrict__ at, const float* __restrict__ de_in,
    const float* __restrict__ dm, EdgeBwdOut o, float eps) {
  using L = EdgeBwdStream<T, H, W>;
  using C = Chunk<T>;
  using V = typename C::V;
  constexpr int NW = L::NW, NT = L::NT, MBS = L::MBS, KC = L::KC, BLK = C::BLK;
  constexpr int NB = edge_span<H>() / 16, NG = H / 64;  // blocks per LayerNorm span; groups of four blocks
  __shared__ __align__(16) unsigned char smem[L::bytes];
  float* vec = (float*)(smem + L::RING);
  unsigned char* bufs = smem + (L::ALIAS ? (2 * L::SP - 1) % 4 * (L::RING / 4) : L::RING + L::VEC);
  float* buf = (float*)(bufs + wave_id() * L::BUF);
  const int nw = gridDim.x * NW, wv = wave_rank(NW);
  const WStream<NW, L::S, L::FR> ws{(const unsigned char*)w.BS, smem};
  for (int c = threadIdx.x; c < H; c += NT) {
    vec[c] = w.b2[c];
    vec[H + c] = w.gamma[c];
  }
  const WaveEdges we(b, wv, nw);
  const int steps = wg_steps<NW>(we.end - we.begin, 16, (int*)bufs, L::BUF / 4);
  const int last = max(we.end - 1, 0);  // rows past the range repeat its last edge and count as zero

  int rv = 0, rn = 0;
  V z[KC];
  auto load_tile = [&](int e0) {
    const int li = lane_id() & 15, lg = lane_id() >> 4;
    const int k = min(e0 + li, last);
    rv = b.recv[k];
    rn = k + 1 < b.E ? b.recv[k + 1] : -1;
    load_row(z, zt + (size_t)k * H, lg);
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
    f32x4 x[MBS];
    arrived_row(z);
    // u = W2 z + b2, xhat
    stream_product<T, H>(ws, 0, x, z);
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
    for (int mb = 0; mb < MBS; ++mb) x[mb] += vget(0, mb);
    const float inv = ln_chain<H, edge_span<H>()>(x, eps);
    f32x4 g[MBS];
    float sg = 0.f, sgx = 0.f, a[4], d[4];  // row sums of dv gamma and of dv gamma xhat, span by span
#pragma unroll
    for (int gr = 0; gr < NG; ++gr) {
      f32x4 dv[4], t[4];
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) dv[k][r] = ok ? pm[gr & 1][k][r] + pe[gr & 1][k][r] : 0.f;
      if (gr + 2 < NG) load_dv(gr & 1, gr + 2);
#pragma unroll
      for (int k = 0; k < 4; ++k) t[k] = dv[k] * x[4 * gr + k];
      cg[gr] += (double)colsum64(t);
      cbt[gr] += (double)colsum64(dv);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int mb = 4 * gr + k;
        const f32x4 gm = vget(1, mb);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float p = dv[k][r] * gm[r];
          a[r] = mb % NB ? __builtin_fmaf(dv[k][r], gm[r], a[r]) : p;
          d[r] = mb % NB ? __builtin_fmaf(x[mb][r], p, d[r]) : x[mb][r] * p;
          g[mb][r] = p;
        }
        if (mb % NB == NB - 1) {
          sg += add_xor32(add_xor16((a[0] + a[1]) + (a[2] + a[3])));
          sgx += add_xor32(add_xor16((d[0] + d[1]) + (d[2] + d[3])));
        }
      }
    }
    V du[KC];
#pragma unroll
    for (int gr = 0; gr < NG; ++gr) {
      f32x4 t[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          t[k][r] = __builtin_fmaf(sgx * (-1.f / H), x[4 * gr + k][r], __builtin_fmaf(sg, -1.f / H, g[4 * gr + k][r])) * inv;
      }
      cb2[gr] += (double)colsum64(t);
#pragma unroll
      for (int k = 0; k < 4 / BLK; ++k) du[4 / BLK * gr + k] = C::of(*(const f32x4(*)[BLK])(t + BLK * k));
    }
    if (ok) store_row((T*)o.du + row, du, lg);
    V av[KC];
    if constexpr (ACT != 0) load_row(av, at + row, lg);
    // dz = W2^T du ; da = dz * act'(a)  (ReLU: a > 0 exactly where z > 0)
    stream_product<T, H>(ws, L::SP, x, du);
    V da[KC];
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      f32x4 p[BLK];
      C::to(ACT ? av[c] : z[c], p);
#pragma unroll
      for (int k = 0; k < BLK; ++k) {
#pragma unroll
        for (int r = 0; r < 4; ++r) x[BLK * c + k][r] *= act_d<ACT>(p[k][r]);
        p[k] = x[BLK * c + k];
      }
      da[c] = C::of(p);
    }
    if (ok) store_row((T*)o.da + row, da, lg);
    // S_r: receiver sums of da in edge order; their total is db1
    seg.add(x, ends, rc, ne, buf, o.S_r, [&](int p, const float2& s) {
      cb1[p][0] += (double)s.x;
      cb1[p][1] += (double)s.y;
    });
    if constexpr (L::ALIAS) lds_sync();  // every wave is done with its buffer
    if (more) load_tile(e0 + 16);        // the next tile's, in flight during the last product
    // de = de' (+ dm_r) + (W1^T da)[2H:3H]
    stream_product<T, H>(ws, 2 * L::SP, x, da);
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
          *(f32x4*)(o.de_out + row + 16 * (m0 + k) + 4 * lg) = x[m0 + k] + v[k];
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

void launch_edge_bwd_stream(const Shape& s, const BatchView& b, const MlpW& w, const void* zt, const void* at,
                            const float* de_in, const float* dm, const EdgeBwdOut& o, hipStream_t st) {
  if (s.act != 0 && !at) {
    g_config_error = 1;
    return;
  }
  by_form(s, b.E, [&](auto t, auto hh, auto ww) {
    using T = decltype(t);
    constexpr int H = decltype(hh)::value, W = decltype(ww)::value;
    by_act_agg(s, [&](auto act, auto agg) {
      k_edge_bwd_stream<T, H, W, decltype(act)::value, decltype(agg)::value>
          <<<edge_stream_grid(s, b.E), StreamDims<T, H, W>::NT, 0, st>>>(b, w, (const T*)zt, (const T*)at, de_in, dm, o,
                                                                     s.eps);
    });
  });
}

}  // namespace xmgn
