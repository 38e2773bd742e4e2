// Node kernels as wave-private chains (see chain.hpp and stream.hpp): the
// weights are streamed through LDS, or, in the BF16 forward at H = 128 (96
// KiB), kept there.
#include <algorithm>
#include <type_traits>

#include "kernels.hpp"
#include "stream.hpp"

namespace xmgn {

template <typename T, int H, int W>
struct NodeFwd : StreamDims<T, H, W> {
  static constexpr int S = 3 * StreamDims<T, H>::SP;  // slabs: W1 (2 H), then W2
  // weights that fit stay; a cycle of 6 slabs would not go round a ring of 4
  static constexpr int SLOTS = S * StreamDims<T, H>::FR <= 96 ? S : 4;
  static constexpr size_t RING = (size_t)SLOTS * StreamDims<T, H>::FR * 1024;
  static constexpr int SW = H / 4;  // LayerNorm span: the sums of four waves
};

// ---------------------------------------------------------------------------
// Node processor, forward (Eq. 3): h' = h + LN(W2 act(W1 [h ; m] + b1) + b2)
// Bound by HBM at H = 128, by the weight fragments beyond.  The workgroup-tile
// kernel read the weights from L2 for every 32 (16 at H = 512) rows, with a
// barrier between any two products.  BF16, H = 128, 400k nodes: 163 -> 99 us
// (0.41 GB, 4.1 TB/s); H = 256, 100k: 203 -> 85 us; H = 512, 50k: 595 -> 177 us;
// FP32, H = 128, 50k: 88 -> 64 us.
// ---------------------------------------------------------------------------
template <typename T, int H, int W, int ACT>
__global__ __launch_bounds__((StreamDims<T, H, W>::NT), (StreamDims<T, H, W>::NW / 4)) void k_node_fwd_stream(
    int n, MlpW w, const T* __restrict__ h, const float* __restrict__ m, T* __restrict__ h_out, float eps) {
  using L = NodeFwd<T, H, W>;
  using C = Chunk<T>;
  using V = typename C::V;
  constexpr int NW = L::NW, NT = L::NT, MBS = L::MBS, KC = L::KC, BLK = C::BLK;
  constexpr bool AHEAD = H == 128;  // m a step ahead too (wider rows: at the step's start)
  __shared__ __align__(16) unsigned char smem[L::RING + 4 * H * 4];
  float* vec = (float*)(smem + L::RING);
  const WStream<NW, L::S, L::FR, L::SLOTS> ws{(const unsigned char*)w.FS, smem};
  for (int c = threadIdx.x; c < H; c += NT) {
    vec[c] = w.b1[c];
    vec[H + c] = w.b2[c];
    vec[2 * H + c] = w.gamma[c];
    vec[3 * H + c] = w.beta[c];
  }
  const WaveRows wr(n, NW);
  const int last = max(wr.end - 1, 0);
  V hr[KC];
  F32Row<T, H> mr;
  auto load = [&](int r0) {
    const int l = lane_id(), k = min(r0 + (l & 15), last);
    load_row(hr, h + (size_t)k * H, l >> 4);
    if constexpr (AHEAD) mr.load(m + (size_t)k * H, l >> 4);
  };
  if (wr.steps) load(wr.begin);
  ws.start();
  lds_sync();
  for (int it = 0; it < wr.steps; ++it) {
    const int l = opaque(lane_id()), li = l & 15, lg = l >> 4;
    const int r0 = wr.begin + 16 * it;
    const bool ok = r0 + li < wr.end;
    const size_t row = (size_t)min(r0 + li, last) * H;
    auto vget = [&](int v, int mb) { return *(const f32x4*)(vec + v * H + 16 * mb + 4 * lg); };
    f32x4 x[MBS];
    V z[KC], hc[KC];
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      arrived(hr[c]);
      hc[c] = hr[c];
    }
    if constexpr (!AHEAD) mr.load(m + row, lg);
    zero_blocks(x);
    stream_gemm<T, H>(ws, 0, 0, 2 * L::SP, x, hc);
    mr.get(z);
    if constexpr (AHEAD) {
      if (it + 1 < wr.steps) load(r0 + 16);
    }
    stream_gemm<T, H>(ws, L::SP, 0, 2 * L::SP, x, z);
#pragma unroll
    for (int c = 0; c < KC; ++c) {
#pragma unroll
      for (int k = 0; k < BLK; ++k) {
        x[BLK * c + k] += vget(0, BLK * c + k);
#pragma unroll
        for (int r = 0; r < 4; ++r) x[BLK * c + k][r] = act_f<ACT>(x[BLK * c + k][r]);
      }
      z[c] = C::of(*(const f32x4(*)[BLK])(x + BLK * c));
    }
    stream_product<T, H>(ws, 2 * L::SP, x, z);
    if constexpr (!AHEAD) {
      if (it + 1 < wr.steps) load(r0 + 16);
    }
#pragma unroll
    for (int mb = 0; mb < MBS; ++mb) x[mb] += vget(1, mb);
    ln_chain<H, L::SW>(x, eps);
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      f32x4 hv[BLK];
      C::to(hc[c], hv);
#pragma unroll
      for (int k = 0; k < BLK; ++k) {
        const f32x4 g = vget(2, BLK * c + k), be = vget(3, BLK * c + k);
#pragma unroll
        for (int r = 0; r < 4; ++r) hv[k][r] = __builtin_fmaf(g[r], x[BLK * c + k][r], hv[k][r]) + be[r];
      }
      if (ok) *(V*)(h_out + row + C::KW * c + C::E * lg) = C::of(hv);
    }
  }
}

// ---------------------------------------------------------------------------
// Node adjoint with recompute; DH: first the upstream gradient's part through
// the layer above's edge products, dh' = dh_mid + [S_r | S_s] B_rs^T.  Then
// dh_mid = dh' + (W1^T da)[0:H], dm = (W1^T da)[H:2H]; da, du and z go out for
// the weight gradients.  dh' and z stay in registers at H = 128, else they are
// read back from o.dh_mid and o.z; the pre-activations a (SiLU) wait in o.dm.
// Taking in the edge products of the layer above saves dh' a trip to memory.
// BF16, H = 128, 400k nodes: 410 us (1.6 GB, 4.0 TB/s) where two workgroup-tile
// kernels took 693 + 232; H = 256, 100k: 281 us (543 + 200); H = 512, SiLU, 50k:
// 533 us (2,279 + 441); FP32, H = 128, 50k: 156 us (191 + 74).  Bound by HBM at
// H = 128, by the weight fragments and the products' barriers beyond.
// ---------------------------------------------------------------------------
template <typename T, int H, int W, int ACT, int DH>
__global__ __launch_bounds__((StreamDims<T, H, W>::NT), (StreamDims<T, H, W>::NW / 4)) void k_node_bwd_stream(
    int n, MlpW w, const T* __restrict__ h, const float* __restrict__ m, const float* dh_in,
    const float* __restrict__ S_r, const float* __restrict__ S_s, NodeBwdOut o, float eps) {
  using L = StreamDims<T, H, W>;
  using C = Chunk<T>;
  using V = typename C::V;
  constexpr int NW = L::NW, NT = L::NT, MBS = L::MBS, KC = L::KC, BLK = C::BLK, SP = L::SP, SW = H / 4, NB = SW / 16;
  constexpr int S0 = DH ? 2 * SP : 0, S = S0 + 6 * SP;  // slabs: B_rs, W1, W2, W2^T, W1^T
  constexpr bool KEEP = H == 128;
  __shared__ __align__(16) unsigned char smem[L::RING + 3 * H * 4];
  float* vec = (float*)(smem + L::RING);
  const WStream<NW, S, L::FR> ws{(const unsigned char*)w.BS, smem};
  for (int c = threadIdx.x; c < H; c += NT) {
    vec[c] = w.b1[c];
    vec[H + c] = w.b2[c];
    vec[2 * H + c] = w.gamma[c];
  }
  const WaveRows wr(n, NW);
  const int last = max(wr.end - 1, 0);
  V hr[KC];
  // S_r's row, S_s's, then m's; in flight over a product, and the first loads a
  // step ahead, at H = 128 only: with the operands and the sums a wider row's
  // 64 or 128 registers spill
  F32Row<T, H> fr;
  auto load_first = [&](int r0) {
    const int l = lane_id(), k = min(r0 + (l & 15), last);
    if constexpr (DH)
      fr.load(S_r + (size_t)k * H, l >> 4);
    else
      load_row(hr, h + (size_t)k * H, l >> 4);
  };
  if (KEEP && wr.steps) load_first(wr.begin);
  ws.start();
  lds_sync();
  double cb1[H / 64] = {}, cb2[H / 64] = {}, cg[H / 64] = {}, cbt[H / 64] = {};
  for (int it = 0; it < wr.steps; ++it) {
    const int l = opaque(lane_id()), li = l & 15, lg = l >> 4;
    const int r0 = wr.begin + 16 * it;
    const bool ok = r0 + li < wr.end;
    const size_t row = (size_t)min(r0 + li, last) * H;
    auto vget = [&](int v, int mb) { return *(const f32x4*)(vec + v * H + 16 * mb + 4 * lg); };
    auto at = [&](const float* p, int mb) { return *(const f32x4*)(p + row + 16 * mb + 4 * lg); };
    auto put = [&](float* p, int mb, const f32x4& v) {
      if (ok) *(f32x4*)(p + row + 16 * mb + 4 * lg) = v;
    };
    // o.dh_mid = v + the row of p, eight blocks at a time (all loads at once spill)
    auto add_dh = [&](const f32x4(&v)[MBS], const float* p) {
#pragma unroll
      for (int m0 = 0; m0 < MBS; m0 += 8) {
        __builtin_amdgcn_sched_barrier(0);
        f32x4 t[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) t[k] = at(p, m0 + k);
#pragma unroll
        for (int k = 0; k < 8; ++k) put(o.dh_mid, m0 + k, v[m0 + k] + t[k]);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    f32x4 x[MBS], dh[KEEP ? MBS : 1];
    V z[KC];
    if constexpr (!KEEP) load_first(r0);
    if constexpr (DH) {
      fr.get(z);
      if constexpr (KEEP) fr.load(S_s + row, lg);
      zero_blocks(x);
      stream_gemm<T, H>(ws, 0, 0, 2 * SP, x, z);
      if constexpr (!KEEP) fr.load(S_s + row, lg);
      fr.get(z);
      load_row(hr, h + row, lg);
      if constexpr (KEEP) {
#pragma unroll
        for (int mb = 0; mb < MBS; ++mb) dh[mb] = at(dh_in, mb);
      }
      stream_gemm<T, H>(ws, SP, 0, 2 * SP, x, z);
      if constexpr (KEEP) {
#pragma unroll
        for (int mb = 0; mb < MBS; ++mb) dh[mb] = x[mb] + dh[mb];
      } else {
        add_dh(x, dh_in);
      }
    }
    if constexpr (KEEP) fr.load(m + row, lg);
    arrived_row(hr);
    zero_blocks(x);
    stream_gemm<T, H>(ws, S0, S0, S0 + 2 * SP, x, hr);
    if constexpr (!KEEP) fr.load(m + row, lg);
    fr.get(z);
    if constexpr (KEEP && !DH) {
#pragma unroll
      for (int mb = 0; mb < MBS; ++mb) dh[mb] = at(dh_in, mb);
    }
    stream_gemm<T, H>(ws, S0 + SP, S0, S0 + 2 * SP, x, z);
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      f32x4 t[BLK];
#pragma unroll
      for (int k = 0; k < BLK; ++k) {
        const int mb = BLK * c + k;
        t[k] = x[mb] + vget(0, mb);
        if constexpr (ACT != 0) put(o.dm, mb, t[k]);
#pragma unroll
        for (int r = 0; r < 4; ++r) t[k][r] = act_f<ACT>(t[k][r]);
      }
      z[c] = C::of(t);
    }
    stream_product<T, H>(ws, S0 + 2 * SP, x, z);
    if (ok) store_row((T*)o.z + row, z, lg);
    // dh', one group of four blocks ahead
    const float* dv_from = DH ? o.dh_mid : dh_in;
    f32x4 pd[2][4];
    auto load_dv = [&](int s, int gr) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if constexpr (KEEP)
          pd[s][k] = dh[4 * gr + k];
        else
          pd[s][k] = at(dv_from, 4 * gr + k);
      }
    };
    load_dv(0, 0);
    load_dv(1, 1);
#pragma unroll
    for (int mb = 0; mb < MBS; ++mb) x[mb] += vget(1, mb);
    const float inv = ln_chain<H, SW>(x, eps);
    f32x4 g[MBS];
    float sg = 0.f, sgx = 0.f, sa[4], sd[4];
#pragma unroll
    for (int gr = 0; gr < H / 64; ++gr) {
      f32x4 dv[4], t[4];
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) dv[k][r] = ok ? pd[gr & 1][k][r] : 0.f;
      if (gr + 2 < H / 64) load_dv(gr & 1, gr + 2);
#pragma unroll
      for (int k = 0; k < 4; ++k) t[k] = dv[k] * x[4 * gr + k];
      cg[gr] += (double)colsum64(t);
      cbt[gr] += (double)colsum64(dv);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int mb = 4 * gr + k;
        const f32x4 gm = vget(2, mb);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float p = dv[k][r] * gm[r];
          sa[r] = mb % NB ? __builtin_fmaf(dv[k][r], gm[r], sa[r]) : p;
          sd[r] = mb % NB ? __builtin_fmaf(x[mb][r], p, sd[r]) : x[mb][r] * p;
          g[mb][r] = p;
        }
        if (mb % NB == NB - 1) {  // a span is whole
          sg += add_xor32(add_xor16((sa[0] + sa[1]) + (sa[2] + sa[3])));
          sgx += add_xor32(add_xor16((sd[0] + sd[1]) + (sd[2] + sd[3])));
        }
      }
    }
    V du[KC];
#pragma unroll
    for (int gr = 0; gr < H / 64; ++gr) {
      f32x4 t[4];
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          t[k][r] = __builtin_fmaf(sgx * (-1.f / H), x[4 * gr + k][r], __builtin_fmaf(sg, -1.f / H, g[4 * gr + k][r])) * inv;
      cb2[gr] += (double)colsum64(t);
#pragma unroll
      for (int k = 0; k < 4 / BLK; ++k) du[4 / BLK * gr + k] = C::of(*(const f32x4(*)[BLK])(t + BLK * k));
    }
    stream_product<T, H>(ws, S0 + 3 * SP, x, du);
    if (ok) store_row((T*)o.du + row, du, lg);
#pragma unroll
    for (int gr = 0; gr < H / 64; ++gr) {
      f32x4 t[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if constexpr (ACT != 0) t[k] = at(o.dm, 4 * gr + k);
      }
      if constexpr (ACT == 0) {  // a > 0 exactly where z > 0
#pragma unroll
        for (int k = 0; k < 4 / BLK; ++k) {
          const int c = 4 / BLK * gr + k;
          C::to(KEEP ? z[c] : *(const V*)((const T*)o.z + row + C::KW * c + C::E * lg), *(f32x4(*)[BLK])(t + BLK * k));
        }
      }
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          t[k][r] = x[4 * gr + k][r] * act_d<ACT>(t[k][r]);
          // (a wave without rows looks at another's, whose a may not be written yet)
          if (ACT != 0 && !ok) t[k][r] = 0.f;
        }
      cb1[gr] += (double)colsum64(t);
#pragma unroll
      for (int k = 0; k < 4 / BLK; ++k) du[4 / BLK * gr + k] = C::of(*(const f32x4(*)[BLK])(t + BLK * k));
    }
    stream_product<T, H>(ws, S0 + 4 * SP, x, du);
    if (ok) store_row((T*)o.da + row, du, lg);
    if constexpr (KEEP) {
      if (it + 1 < wr.steps) load_first(r0 + 16);
#pragma unroll
      for (int mb = 0; mb < MBS; ++mb) put(o.dh_mid, mb, x[mb] + dh[mb]);
    } else {
      add_dh(x, dv_from);
    }
    stream_product<T, H>(ws, S0 + 5 * SP, x, du);
#pragma unroll
    for (int mb = 0; mb < MBS; ++mb) put(o.dm, mb, x[mb]);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (no weights on their way into the ring)
  float* p = o.partial + (size_t)blockIdx.x * 4 * H;
  double* ds = (double*)smem;
  wg_colsum64<H, NW>(ds, p, cb1);
  wg_colsum64<H, NW>(ds, p + H, cb2);
  wg_colsum64<H, NW>(ds, p + 2 * H, cg);
  wg_colsum64<H, NW>(ds, p + 3 * H, cbt);
}

// ---------------------------------------------------------------------------
// f(T{}, H, W, ACT) of the form with the waves for so many rows
template <typename F>
static void node_form(const Shape& s, int rows, F f) {
  using std::integral_constant;
  using W0 = integral_constant<int, 0>;
  auto go = [&](auto t, auto hh, auto ww) {
    if (s.act)
      f(t, hh, ww, integral_constant<int, 1>{});
    else
      f(t, hh, ww, integral_constant<int, 0>{});
  };
  if (s.prec == 1) {
    if (s.H == 128)
      go(bf16{}, integral_constant<int, 128>{}, W0{});
    else if (s.H == 256)
      go(bf16{}, integral_constant<int, 256>{}, W0{});
    else
      go(bf16{}, integral_constant<int, 512>{}, W0{});
  } else {
    if (s.H == 128 && stream_small(s, rows))
      go(float{}, integral_constant<int, 128>{}, integral_constant<int, 4>{});
    else if (s.H == 128)
      go(float{}, integral_constant<int, 128>{}, W0{});
    else
      go(float{}, integral_constant<int, 256>{}, W0{});
  }
}

void launch_node_fwd(const Shape& s, const BatchView& b, const MlpW& w, const void* h, const float* m, void* h_out,
                     hipStream_t st) {
  if (b.n == 0) return;
  if (row_tiles(s, b.n)) {
    launch_node_fwd_tiles(s, b, w, h, m, h_out, st);
    return;
  }
  node_form(s, b.n, [&](auto t, auto hh, auto ww, auto act) {
    using T = decltype(t);
    constexpr int H = decltype(hh)::value, W = decltype(ww)::value;
    k_node_fwd_stream<T, H, W, decltype(act)::value>
        <<<edge_stream_grid(s, b.n), StreamDims<T, H, W>::NT, 0, st>>>(b.n, w, (const T*)h, m, (T*)h_out, s.eps);
  });
}

void launch_node_bwd(const Shape& s, const BatchView& b, const MlpW& w, const void* h, const float* m,
                     const float* dh_in, const float* S_r, const float* S_s, const NodeBwdOut& o, hipStream_t st) {
  node_form(s, b.n, [&](auto t, auto hh, auto ww, auto act) {
    using T = decltype(t);
    constexpr int H = decltype(hh)::value, W = decltype(ww)::value, A = decltype(act)::value;
    const int grid = edge_stream_grid(s, b.n);
    if (S_r)
      k_node_bwd_stream<T, H, W, A, 1>
          <<<grid, StreamDims<T, H, W>::NT, 0, st>>>(b.n, w, (const T*)h, m, dh_in, S_r, S_s, o, s.eps);
    else
      k_node_bwd_stream<T, H, W, A, 0>
          <<<grid, StreamDims<T, H, W>::NT, 0, st>>>(b.n, w, (const T*)h, m, dh_in, S_r, S_s, o, s.eps);
  });
}

}  // namespace xmgn
