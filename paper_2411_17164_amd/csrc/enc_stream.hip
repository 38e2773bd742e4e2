// Encoders with streamed weights (see stream.hpp):
// y = LN(W3 act(W2 act(W1 x + b1) + b2) + b3), the input layer (at most 32
// inputs) as FMA in the accumulator layout.  The workgroup-tile kernels they
// replace loaded each H x H matrix from L2 for every 32 (16 at H = 512) rows
// and spilled in the adjoint.  Edge encoder, 886k rows at H = 256: forward
// 1,353 -> 322 us, adjoint 3,359 -> 1,121 us (its two kernels and their
// reductions; FP32 dout in, z1, z2, du3, da2 out: bound by HBM); 442k rows at
// H = 512, SiLU: 3,462 -> 866 us and 14,703 -> 2,604 us (bound by the weight
// fragments, as the edge kernels); FP32, 443k rows at H = 128: 345 -> 269 us and
// 1,015 -> 687 us.  The adjoint is two kernels because xhat,
// the upstream gradient and both FP32 pre-activations of a row do not fit in a
// wave's registers together.
#include <algorithm>
#include <type_traits>

#include "kernels.hpp"
#include "stream.hpp"
#include "tile.hpp"

namespace xmgn {

template <typename T, int H, int W>
struct EncStream : StreamDims<T, H, W> {
  static constexpr int S = 2 * StreamDims<T, H>::SP;  // two H x H matrices (BF16 at H = 128: the ring holds both)
  static constexpr size_t VEC = 5 * H * 4;  // b1, b2, b3, gamma, beta
  static constexpr size_t BUF = 8192;       // per wave (second adjoint kernel): 16 rows x 128 FP32
  static constexpr int SW = H / 4;          // LayerNorm span: the sums of four waves
};
// Input weights in LDS, [k][H]: 4 or 8 inputs; more are read from global memory.
template <int H, int KIN>
constexpr size_t enc_w1_bytes() {
  return KIN <= 8 ? (size_t)KIN * H * 4 : 0;
}

// The input layer and its data: KIN = 4 (edge features), 8 (up to 8 node
// inputs) or 32.
template <int H, int KIN, int KIND>
struct EncIn {
  static constexpr int MBS = H / 16;
  const float* src;
  const int* gid;
  const float* W1f;  // [H][in_dim]
  const float* w1s;  // LDS [KIN][H] (KIN <= 8)
  int in_dim;
  float x[KIN];
  // stage W1 (a barrier follows)
  __device__ __forceinline__ void stage(float* dst, int nt) {
    w1s = dst;
    if constexpr (KIN <= 8)
      for (int c = threadIdx.x; c < KIN * H; c += nt) {
        const int k = c / H, f = c - k * H;
        dst[c] = k < in_dim ? W1f[f * in_dim + k] : 0.f;
      }
  }
  __device__ __forceinline__ void load(int row) {
    if constexpr (KIND == 1) {
      const float4 f = ((const float4*)src)[row];
      x[0] = f.x;
      x[1] = f.y;
      x[2] = f.z;
      x[3] = f.w;
    } else {
      const float* p = src + (size_t)gid[row] * in_dim;
#pragma unroll
      for (int k = 0; k < KIN; ++k) x[k] = k < in_dim ? p[k] : 0.f;
    }
  }
  // block mb of a1 = b1 + W1 x
  __device__ __forceinline__ f32x4 layer(const float* b1, int mb, int lg) const {
    f32x4 a = *(const f32x4*)(b1 + 16 * mb + 4 * lg);
    if constexpr (KIN <= 8) {
#pragma unroll
      for (int k = 0; k < KIN; ++k) {
        const f32x4 wk = *(const f32x4*)(w1s + k * H + 16 * mb + 4 * lg);
#pragma unroll
        for (int r = 0; r < 4; ++r) a[r] = __builtin_fmaf(wk[r], x[k], a[r]);
      }
    } else {
      const float* p = W1f + (size_t)(16 * mb + 4 * lg) * in_dim;
#pragma unroll
      for (int k = 0; k < KIN; k += 4)
        if (k < in_dim) {  // (a multiple of 4)
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int j = 0; j < 4; ++j) a[r] = __builtin_fmaf(p[r * in_dim + k + j], x[k + j], a[r]);
        }
    }
    return a;
  }
};

template <int H>
__device__ __forceinline__ void stage_vecs(float* vec, const MlpW& w, int nt) {
  for (int c = threadIdx.x; c < H; c += nt) {
    vec[c] = w.b1[c];
    vec[H + c] = w.b2[c];
    vec[2 * H + c] = w.b3[c];
    vec[3 * H + c] = w.gamma[c];
    vec[4 * H + c] = w.beta[c];
  }
}

template <typename T, int H, int W, int ACT, int KIN, int KIND>
__global__ __launch_bounds__((StreamDims<T, H, W>::NT), (StreamDims<T, H, W>::NW / 4)) void k_enc_fwd_stream(
    int rows, const int* __restrict__ gid, MlpW w, const float* __restrict__ src, int in_dim, T* __restrict__ out,
    float eps) {
  using L = EncStream<T, H, W>;
  using C = Chunk<T>;
  using V = typename C::V;
  constexpr int NW = L::NW, NT = L::NT, MBS = L::MBS, KC = L::KC, BLK = C::BLK;
  __shared__ __align__(16) unsigned char smem[L::RING + L::VEC + enc_w1_bytes<H, KIN>()];
  float* vec = (float*)(smem + L::RING);
  const WStream<NW, L::S, L::FR> ws{(const unsigned char*)w.FS, smem};
  EncIn<H, KIN, KIND> in{src, gid, w.W1f, nullptr, in_dim};
  in.stage(vec + 5 * H, NT);
  stage_vecs<H>(vec, w, NT);
  const WaveRows wr(rows, NW);
  const int last = max(wr.end - 1, 0);
  if (wr.steps) in.load(min(wr.begin + (lane_id() & 15), last));
  ws.start();
  lds_sync();
  for (int it = 0; it < wr.steps; ++it) {
    const int l = opaque(lane_id()), li = l & 15, lg = l >> 4;
    const int r0 = wr.begin + 16 * it;
    const bool ok = r0 + li < wr.end;
    auto vget = [&](int v, int mb) { return *(const f32x4*)(vec + v * H + 16 * mb + 4 * lg); };
    f32x4 x[MBS];
    V z[KC];
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      f32x4 a[BLK];
#pragma unroll
      for (int k = 0; k < BLK; ++k) {
        a[k] = in.layer(vec, BLK * c + k, lg);
#pragma unroll
        for (int r = 0; r < 4; ++r) a[k][r] = act_f<ACT>(a[k][r]);
      }
      z[c] = C::of(a);
    }
    in.load(min(r0 + 16 + li, last));
    stream_product<T, H>(ws, 0, x, z);
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      f32x4 a[BLK];
#pragma unroll
      for (int k = 0; k < BLK; ++k) {
        a[k] = x[BLK * c + k] + vget(1, BLK * c + k);
#pragma unroll
        for (int r = 0; r < 4; ++r) a[k][r] = act_f<ACT>(a[k][r]);
      }
      z[c] = C::of(a);
    }
    stream_product<T, H>(ws, L::SP, x, z);
#pragma unroll
    for (int mb = 0; mb < MBS; ++mb) x[mb] += vget(2, mb);
    ln_chain<H, L::SW>(x, eps);
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      f32x4 y[BLK];
#pragma unroll
      for (int k = 0; k < BLK; ++k) {
        const f32x4 gm = vget(3, BLK * c + k), be = vget(4, BLK * c + k);
#pragma unroll
        for (int r = 0; r < 4; ++r) y[k][r] = __builtin_fmaf(gm[r], x[BLK * c + k][r], be[r]);
      }
      if (ok) *(V*)(out + (size_t)(r0 + li) * H + C::KW * c + C::E * lg) = C::of(y);
    }
  }
}

// ---------------------------------------------------------------------------
// Adjoint, first kernel: recomputes the chain to xhat, takes the LayerNorm
// adjoint of dout and writes z1, z2 and du3 (and, under SiLU, a2 in FP32 for
// the second kernel's derivative).
// ---------------------------------------------------------------------------
template <typename T, int H, int W, int ACT, int KIN, int KIND>
__global__ __launch_bounds__((StreamDims<T, H, W>::NT), (StreamDims<T, H, W>::NW / 4)) void k_enc_bwd1_stream(
    int rows, const int* __restrict__ gid, MlpW w, const float* __restrict__ src, int in_dim,
    const float* __restrict__ dout, EncBwdOut o, float* __restrict__ a2_out, float eps) {
  using L = EncStream<T, H, W>;
  using C = Chunk<T>;
  using V = typename C::V;
  constexpr int NW = L::NW, NT = L::NT, MBS = L::MBS, KC = L::KC, BLK = C::BLK, SW = L::SW, NB = SW / 16;
  __shared__ __align__(16) unsigned char smem[L::RING + L::VEC + enc_w1_bytes<H, KIN>()];
  float* vec = (float*)(smem + L::RING);
  const WStream<NW, L::S, L::FR> ws{(const unsigned char*)w.FS, smem};
  EncIn<H, KIN, KIND> in{src, gid, w.W1f, nullptr, in_dim};
  in.stage(vec + 5 * H, NT);
  stage_vecs<H>(vec, w, NT);
  const WaveRows wr(rows, NW);
  const int last = max(wr.end - 1, 0);
  if (wr.steps) in.load(min(wr.begin + (lane_id() & 15), last));
  ws.start();
  lds_sync();
  double cb3[H / 64] = {}, cg[H / 64] = {}, cbt[H / 64] = {};
  for (int it = 0; it < wr.steps; ++it) {
    const int l = opaque(lane_id()), li = l & 15, lg = l >> 4;
    const int r0 = wr.begin + 16 * it;
    const bool ok = r0 + li < wr.end;
    const size_t row = (size_t)min(r0 + li, last) * H;
    auto vget = [&](int v, int mb) { return *(const f32x4*)(vec + v * H + 16 * mb + 4 * lg); };
    f32x4 x[MBS];
    V z[KC];
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      f32x4 a[BLK];
#pragma unroll
      for (int k = 0; k < BLK; ++k) {
        a[k] = in.layer(vec, BLK * c + k, lg);
#pragma unroll
        for (int r = 0; r < 4; ++r) a[k][r] = act_f<ACT>(a[k][r]);
      }
      z[c] = C::of(a);
    }
    in.load(min(r0 + 16 + li, last));
    stream_product<T, H>(ws, 0, x, z);
    if (ok) store_row((T*)o.z1 + row, z, lg);
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      f32x4 a[BLK];
#pragma unroll
      for (int k = 0; k < BLK; ++k) {
        a[k] = x[BLK * c + k] + vget(1, BLK * c + k);
        if (ACT != 0 && ok) *(f32x4*)(a2_out + row + 16 * (BLK * c + k) + 4 * lg) = a[k];
#pragma unroll
        for (int r = 0; r < 4; ++r) a[k][r] = act_f<ACT>(a[k][r]);
      }
      z[c] = C::of(a);
    }
    stream_product<T, H>(ws, L::SP, x, z);
    if (ok) store_row((T*)o.z2 + row, z, lg);
    // dout, one group of four blocks ahead
    f32x4 pd[2][4];
    auto load_dv = [&](int s, int gr) {
#pragma unroll
      for (int k = 0; k < 4; ++k) pd[s][k] = *(const f32x4*)(dout + row + 64 * gr + 16 * k + 4 * lg);
    };
    load_dv(0, 0);
    load_dv(1, 1);
#pragma unroll
    for (int mb = 0; mb < MBS; ++mb) x[mb] += vget(2, mb);
    const float inv = ln_chain<H, SW>(x, eps);
    f32x4 g[MBS];
    float sg = 0.f, sgx = 0.f, a[4], d[4];
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
        const f32x4 gm = vget(3, mb);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float p = dv[k][r] * gm[r];
          a[r] = mb % NB ? __builtin_fmaf(dv[k][r], gm[r], a[r]) : p;
          d[r] = mb % NB ? __builtin_fmaf(x[mb][r], p, d[r]) : x[mb][r] * p;
          g[mb][r] = p;
        }
        if (mb % NB == NB - 1) {  // a span is whole
          sg += add_xor32(add_xor16((a[0] + a[1]) + (a[2] + a[3])));
          sgx += add_xor32(add_xor16((d[0] + d[1]) + (d[2] + d[3])));
        }
      }
    }
#pragma unroll
    for (int gr = 0; gr < H / 64; ++gr) {
      f32x4 t[4];
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          t[k][r] = __builtin_fmaf(sgx * (-1.f / H), x[4 * gr + k][r], __builtin_fmaf(sg, -1.f / H, g[4 * gr + k][r])) * inv;
      cb3[gr] += (double)colsum64(t);
#pragma unroll
      for (int k = 0; k < 4 / BLK; ++k) z[4 / BLK * gr + k] = C::of(*(const f32x4(*)[BLK])(t + BLK * k));
    }
    if (ok) store_row((T*)o.du3 + row, z, lg);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (no weights on their way into the ring)
  float* p = o.partial + (size_t)blockIdx.x * 13 * H;
  wg_colsum64<H, NW>((double*)smem, p + 2 * H, cb3);
  wg_colsum64<H, NW>((double*)smem, p + 3 * H, cg);
  wg_colsum64<H, NW>((double*)smem, p + 4 * H, cbt);
}

// Adjoint, second kernel: dz2 = W3^T du3, da2, dz1 = W2^T da2, da1; writes da2,
// and the input layer's gradient as column sums (KIN <= 8) or da1 in FP32.
template <typename T, int H, int W, int ACT, int KIN, int KIND>
__global__ __launch_bounds__((StreamDims<T, H, W>::NT), (StreamDims<T, H, W>::NW / 4)) void k_enc_bwd2_stream(
    int rows, const int* __restrict__ gid, MlpW w, const float* __restrict__ src, int in_dim, EncBwdOut o,
    const float* __restrict__ a2) {
  using L = EncStream<T, H, W>;
  using C = Chunk<T>;
  using V = typename C::V;
  constexpr int NW = L::NW, NT = L::NT, MBS = L::MBS, KC = L::KC, BLK = C::BLK;
  constexpr int NP = H / 128, KW = KIN <= 8 ? KIN : 0;
  constexpr size_t HEAD = L::RING + L::VEC + enc_w1_bytes<H, KIN>();
  // H = 512: the waves' buffers lie in the slot of the cycle's last slab, free
  // from its products to the next step
  constexpr bool ALIAS = HEAD + NW * L::BUF > 160 * 1024;
  static_assert(!ALIAS || NW * L::BUF <= L::RING / 4, "the buffers fit in one slot");
  __shared__ __align__(16) unsigned char smem[HEAD + (ALIAS ? 0 : NW * L::BUF)];
  float* vec = (float*)(smem + L::RING);
  float* buf = (float*)(smem + (ALIAS ? L::RING / 4 * 3 : HEAD) + wave_id() * L::BUF);
  const WStream<NW, L::S, L::FR> ws{(const unsigned char*)w.BS, smem};
  EncIn<H, KIN, KIND> in{src, gid, w.W1f, nullptr, in_dim};
  in.stage(vec + 5 * H, NT);
  stage_vecs<H>(vec, w, NT);
  const WaveRows wr(rows, NW);
  const int last = max(wr.end - 1, 0);
  V du[KC];
  auto load_du = [&](int r0) {
    const int l = lane_id(), k = min(r0 + (l & 15), last);
    load_row(du, (const T*)o.du3 + (size_t)k * H, l >> 4);
  };
  if (wr.steps) load_du(wr.begin);
  ws.start();
  lds_sync();
  double cb2[H / 64] = {}, cb1[NP][2] = {}, cw[NP][KW > 0 ? KW : 1][2] = {};
  for (int it = 0; it < wr.steps; ++it) {
    const int l = opaque(lane_id()), li = l & 15, lg = l >> 4;
    const int r0 = wr.begin + 16 * it;
    const bool ok = r0 + li < wr.end;
    const size_t row = (size_t)min(r0 + li, last) * H;
    if constexpr (ALIAS) lds_sync();  // every wave is done with its buffer
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      arrived(du[c]);
      if (!ok) du[c] = V{};
    }
    in.load(min(r0 + li, last));
    f32x4 x[MBS];
    stream_product<T, H>(ws, 0, x, du);
    V da[KC];
#pragma unroll
    for (int gr = 0; gr < H / 64; ++gr) {
      f32x4 t[4];
      if constexpr (ACT == 0) {  // a2 > 0 exactly where z2 > 0
#pragma unroll
        for (int k = 0; k < 4 / BLK; ++k)
          C::to(*(const V*)((const T*)o.z2 + row + C::KW * (4 / BLK * gr + k) + C::E * lg), *(f32x4(*)[BLK])(t + BLK * k));
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) t[k] = *(const f32x4*)(a2 + row + 64 * gr + 16 * k + 4 * lg);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) t[k][r] = x[4 * gr + k][r] * act_d<ACT>(t[k][r]);
      cb2[gr] += (double)colsum64(t);
#pragma unroll
      for (int k = 0; k < 4 / BLK; ++k) da[4 / BLK * gr + k] = C::of(*(const f32x4(*)[BLK])(t + BLK * k));
    }
    if (ok) store_row((T*)o.da2 + row, da, lg);
    stream_product<T, H>(ws, L::SP, x, da);
    if (it + 1 < wr.steps) load_du(r0 + 16);  // in flight during the sums
#pragma unroll
    for (int mb = 0; mb < MBS; ++mb) {
      const f32x4 a = in.layer(vec, mb, lg);
#pragma unroll
      for (int r = 0; r < 4; ++r) x[mb][r] *= act_d<ACT>(a[r]);
      if (KIN > 8 && ok) *(f32x4*)(o.da1 + row + 16 * mb + 4 * lg) = x[mb];
    }
    // sums over the rows of da1 and da1 x^T, row by row through the wave's
    // buffer (lane l: features 2 l, 2 l + 1 of every 128)
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      wave_sync();
#pragma unroll
      for (int k = 0; k < 8; ++k) *(f32x4*)(buf + li * 128 + (((4 * k + lg) ^ li) << 2)) = x[8 * p + k];
      wave_sync();
      float2 s = {0.f, 0.f}, sw[KW > 0 ? KW : 1];
#pragma unroll
      for (int k = 0; k < KW; ++k) sw[k] = float2{0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float2 v = *(const float2*)(buf + i * 128 + ((((l >> 1) ^ i) << 2) | ((l & 1) << 1)));
        s.x += v.x;
        s.y += v.y;
#pragma unroll
        for (int k = 0; k < KW; ++k) {
          const float xi = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, in.x[k]), i));
          sw[k].x = __builtin_fmaf(v.x, xi, sw[k].x);
          sw[k].y = __builtin_fmaf(v.y, xi, sw[k].y);
        }
      }
      cb1[p][0] += (double)s.x;
      cb1[p][1] += (double)s.y;
#pragma unroll
      for (int k = 0; k < KW; ++k) {
        cw[p][k][0] += (double)sw[k].x;
        cw[p][k][1] += (double)sw[k].y;
      }
    }
    wave_sync();
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (no weights on their way into the ring)
  float* p = o.partial + (size_t)blockIdx.x * 13 * H;
  double* ds = (double*)smem;
  wg_colsum64<H, NW>(ds, p + H, cb2);
  wg_colsum<H, NW>(ds, p, 1, [&](double* d) {
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      d[128 * q + 2 * lane_id()] = cb1[q][0];
      d[128 * q + 2 * lane_id() + 1] = cb1[q][1];
    }
  });
#pragma unroll
  for (int k = 0; k < KW; ++k)
    wg_colsum<H, NW>(ds, p + 5 * H + k, 8, [&](double* d) {
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        d[128 * q + 2 * lane_id()] = cw[q][k][0];
        d[128 * q + 2 * lane_id() + 1] = cw[q][k][1];
      }
    });
}

// ---------------------------------------------------------------------------
// Edge encoder adjoint, BF16, H = 128: one kernel.  xhat, the upstream gradient
// and both hidden rows of 16 edges fit in a wave's registers there, so nothing
// but the column sums and the weight gradients leaves it: dW3 = du3^T z2 and
// dW2 = da2^T z1 are accumulated from 128-row tiles (tile.hpp).  The four
// matrices are streamed: with the tiles they do not fit in LDS.  3.55M edges:
// 3,556 -> 1,615 us against the workgroup-tile kernel with the same fusion,
// which passed every intermediate through LDS behind a barrier; its floor is
// reading dout (1.8 GB, 370 us).  Bound by issue and waits: by counters VALU and
// MFMA instructions issue in 57% of a SIMD's cycles, LDS is active in 31%, and a
// wave waits (slabs, barriers) for 35% of its own.
// ---------------------------------------------------------------------------
template <int ACT>
__global__ __launch_bounds__(512, 2) void k_enc_edge_bwd_chain(int rows, MlpW w, const float* __restrict__ src,
                                                               const float* __restrict__ dout, EncBwdOut o,
                                                               float* __restrict__ a2_out, float eps) {
  using T = bf16;
  constexpr int H = 128, KIN = 4, SW = 32;
  using L = StreamDims<T, H>;
  using C = Chunk<T>;
  constexpr int NW = L::NW, NT = L::NT, MBS = L::MBS, KC = L::KC, SP = L::SP;
  static_assert(NW == 8, "tiles of eight waves");
  constexpr size_t HEAD = L::RING + 5 * H * 4 + enc_w1_bytes<H, KIN>();
  __shared__ __align__(16) unsigned char smem[HEAD + NW * kTileReg];
  float* vec = (float*)(smem + L::RING);
  unsigned char* regs = smem + HEAD;
  unsigned char* reg = regs + wave_id() * kTileReg;
  float* buf = (float*)reg;
  const int wm = wave_id() & 3, wn = wave_id() >> 2;
  const WStream<NW, 4 * SP, L::FR> ws{(const unsigned char*)w.BS, smem};
  EncIn<H, KIN, 1> in{src, nullptr, w.W1f, nullptr, 4}, nx = in;
  in.stage(vec + 5 * H, NT);
  stage_vecs<H>(vec, w, NT);
  const WaveRows wr(rows, NW);
  const int last = max(wr.end - 1, 0);
  if (wr.steps) nx.load(min(wr.begin + (lane_id() & 15), last));
  ws.start();
  lds_sync();
  f32x4 accW3[2][4], accW2[2][4];
  zero_acc(accW3);
  zero_acc(accW2);
  double cb1[2] = {}, cb2[2] = {}, cb3[2] = {}, cg[2] = {}, cbt[2] = {}, cw[KIN][2] = {};
  for (int it = 0; it < wr.steps; ++it) {
    const int l = opaque(lane_id()), li = l & 15, lg = l >> 4;
    const int r0 = wr.begin + 16 * it;
    const bool ok = r0 + li < wr.end;
    const size_t row = (size_t)min(r0 + li, last) * H;
    auto vget = [&](int v, int mb) { return *(const f32x4*)(vec + v * H + 16 * mb + 4 * lg); };
#pragma unroll
    for (int k = 0; k < KIN; ++k) in.x[k] = nx.x[k];
    f32x4 x[MBS];
    bf16x8 z1[KC], z2[KC], d[KC];
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      f32x4 a[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        a[k] = in.layer(vec, 2 * c + k, lg);
#pragma unroll
        for (int r = 0; r < 4; ++r) a[k][r] = act_f<ACT>(a[k][r]);
      }
      z1[c] = C::of(a);
    }
    stream_product<T, H>(ws, 0, x, z1);
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      f32x4 a[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        a[k] = x[2 * c + k] + vget(1, 2 * c + k);
        if (ACT != 0 && ok) *(f32x4*)(a2_out + row + 16 * (2 * c + k) + 4 * lg) = a[k];
#pragma unroll
        for (int r = 0; r < 4; ++r) a[k][r] = act_f<ACT>(a[k][r]);
      }
      z2[c] = C::of(a);
    }
    f32x4 g[MBS];  // dout, in flight during the product
#pragma unroll
    for (int mb = 0; mb < MBS; ++mb) g[mb] = *(const f32x4*)(dout + row + 16 * mb + 4 * lg);
    stream_product<T, H>(ws, SP, x, z2);
#pragma unroll
    for (int mb = 0; mb < MBS; ++mb) x[mb] += vget(2, mb);
    const float inv = ln_chain<H, SW>(x, eps);
    float sg = 0.f, sgx = 0.f, sa[4], sd[4];
#pragma unroll
    for (int gr = 0; gr < 2; ++gr) {
      f32x4 dv[4], t[4];
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) dv[k][r] = ok ? g[4 * gr + k][r] : 0.f;
#pragma unroll
      for (int k = 0; k < 4; ++k) t[k] = dv[k] * x[4 * gr + k];
      cg[gr] += (double)colsum64(t);
      cbt[gr] += (double)colsum64(dv);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int mb = 4 * gr + k;
        const f32x4 gm = vget(3, mb);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float p = dv[k][r] * gm[r];
          sa[r] = mb % 2 ? __builtin_fmaf(dv[k][r], gm[r], sa[r]) : p;
          sd[r] = mb % 2 ? __builtin_fmaf(x[mb][r], p, sd[r]) : x[mb][r] * p;
          g[mb][r] = p;
        }
        if (mb % 2 == 1) {  // a span is whole
          sg += add_xor32(add_xor16((sa[0] + sa[1]) + (sa[2] + sa[3])));
          sgx += add_xor32(add_xor16((sd[0] + sd[1]) + (sd[2] + sd[3])));
        }
      }
    }
#pragma unroll
    for (int gr = 0; gr < 2; ++gr) {
      f32x4 t[4];
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          t[k][r] = __builtin_fmaf(sgx * (-1.f / H), x[4 * gr + k][r], __builtin_fmaf(sg, -1.f / H, g[4 * gr + k][r])) * inv;
      cb3[gr] += (double)colsum64(t);
#pragma unroll
      for (int k = 0; k < 2; ++k) d[2 * gr + k] = C::of(*(const f32x4(*)[2])(t + 2 * k));
    }
    // (the last product's barriers: every wave is done with its buffer)
    tile_put(reg, d, l);
    tile_put(reg + kTileReg / 2, z2, l);
    lds_sync();
    tile_wgrad(accW3, regs, 0, kTileReg / 2, wm, wn, l);  // dW3 += du3^T z2
    stream_product<T, H>(ws, 2 * SP, x, d);
#pragma unroll
    for (int gr = 0; gr < 2; ++gr) {
      f32x4 t[4];
      if constexpr (ACT == 0) {  // a2 > 0 exactly where z2 > 0
#pragma unroll
        for (int k = 0; k < 2; ++k) C::to(z2[2 * gr + k], *(f32x4(*)[2])(t + 2 * k));
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) t[k] = *(const f32x4*)(a2_out + row + 64 * gr + 16 * k + 4 * lg);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          t[k][r] = x[4 * gr + k][r] * act_d<ACT>(t[k][r]);
          // (a wave without rows looks at another's, whose a2 may not be written yet)
          if (ACT != 0 && !ok) t[k][r] = 0.f;
        }
      cb2[gr] += (double)colsum64(t);
#pragma unroll
      for (int k = 0; k < 2; ++k) d[2 * gr + k] = C::of(*(const f32x4(*)[2])(t + 2 * k));
    }
    // (that product's barriers: every wave is done with [du3 | z2])
    tile_put(reg, d, l);
    tile_put(reg + kTileReg / 2, z1, l);
    lds_sync();
    tile_wgrad(accW2, regs, 0, kTileReg / 2, wm, wn, l);  // dW2 += da2^T z1
    if (it + 1 < wr.steps) nx.load(min(r0 + 16 + li, last));
    stream_product<T, H>(ws, 3 * SP, x, d);
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      f32x4 a[2];
      if constexpr (ACT == 0)  // a1 > 0 exactly where z1 > 0
        C::to(z1[c], a);
      else {
        a[0] = in.layer(vec, 2 * c, lg);
        a[1] = in.layer(vec, 2 * c + 1, lg);
      }
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) x[2 * c + k][r] *= act_d<ACT>(a[k][r]);
    }
    // sums over the rows of da1 and da1 x^T, row by row through the wave's
    // buffer (that product's barriers: every wave is done with [da2 | z1])
    wave_sync();
#pragma unroll
    for (int k = 0; k < 8; ++k) *(f32x4*)(buf + li * 128 + (((4 * k + lg) ^ li) << 2)) = x[k];
    wave_sync();
    float2 s = {0.f, 0.f}, sw[KIN];
#pragma unroll
    for (int k = 0; k < KIN; ++k) sw[k] = float2{0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float2 v = *(const float2*)(buf + i * 128 + ((((l >> 1) ^ i) << 2) | ((l & 1) << 1)));
      s.x += v.x;
      s.y += v.y;
#pragma unroll
      for (int k = 0; k < KIN; ++k) {
        const float xi = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, in.x[k]), i));
        sw[k].x = __builtin_fmaf(v.x, xi, sw[k].x);
        sw[k].y = __builtin_fmaf(v.y, xi, sw[k].y);
      }
    }
    cb1[0] += (double)s.x;
    cb1[1] += (double)s.y;
#pragma unroll
    for (int k = 0; k < KIN; ++k) {
      cw[k][0] += (double)sw[k].x;
      cw[k][1] += (double)sw[k].y;
    }
    wave_sync();
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (no weights on their way into the ring)
  float* p = o.partial + (size_t)blockIdx.x * 13 * H;
  double* ds = (double*)smem;
  auto two = [&](float* dst, int stride, const double (&v)[2]) {  // lane l: features 2 l, 2 l + 1
    wg_colsum<H, NW>(ds, dst, stride, [&](double* q) {
      q[2 * lane_id()] = v[0];
      q[2 * lane_id() + 1] = v[1];
    });
  };
  two(p, 1, cb1);
  wg_colsum64<H, NW>(ds, p + H, cb2);
  wg_colsum64<H, NW>(ds, p + 2 * H, cb3);
  wg_colsum64<H, NW>(ds, p + 3 * H, cg);
  wg_colsum64<H, NW>(ds, p + 4 * H, cbt);
#pragma unroll
  for (int k = 0; k < KIN; ++k) two(p + 5 * H + k, 8, cw[k]);
  float* q2 = o.wpart + (size_t)blockIdx.x * 2 * H * H;
  float* q3 = q2 + H * H;
  const int li = lane_id() & 15, lg = lane_id() >> 4;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int at = (32 * wm + 16 * i + 4 * lg + r) * H + 64 * wn + 16 * j + li;
        q2[at] = accW2[i][j][r];
        q3[at] = accW3[i][j][r];
      }
}

void launch_enc_edge_bwd_chain(const Shape& s, int R, const MlpW& w, const float* xe, const float* dout,
                               const EncBwdOut& o, float* a2, hipStream_t st) {
  const int grid = edge_stream_grid(s, R);
  if (s.act)
    k_enc_edge_bwd_chain<1><<<grid, 512, 0, st>>>(R, w, xe, dout, o, a2, s.eps);
  else
    k_enc_edge_bwd_chain<0><<<grid, 512, 0, st>>>(R, w, xe, dout, o, a2, s.eps);
}

// ---------------------------------------------------------------------------
bool enc_stream(const Shape& s) { return edge_stream(s); }

// f(T{}, H, W, ACT, KIN, KIND) as constants
template <typename F>
static void enc_dispatch(const Shape& s, int R, int kind, int in_dim, F f) {
  using std::integral_constant;
  using I0 = integral_constant<int, 0>;
  using I1 = integral_constant<int, 1>;
  auto by = [&](auto t, auto hh, auto ww, auto act) {
    if (kind == 1)
      f(t, hh, ww, act, integral_constant<int, 4>{}, I1{});
    else if (in_dim <= 8)
      f(t, hh, ww, act, integral_constant<int, 8>{}, I0{});
    else
      f(t, hh, ww, act, integral_constant<int, 32>{}, I0{});
  };
  auto by_act = [&](auto t, auto hh, auto ww) {
    if (s.act)
      by(t, hh, ww, I1{});
    else
      by(t, hh, ww, I0{});
  };
  if (s.prec == 1) {
    if (s.H == 128)
      by_act(bf16{}, integral_constant<int, 128>{}, I0{});
    else if (s.H == 256)
      by_act(bf16{}, integral_constant<int, 256>{}, I0{});
    else
      by_act(bf16{}, integral_constant<int, 512>{}, I0{});
  } else {
    if (s.H == 128 && stream_small(s, R))
      by_act(float{}, integral_constant<int, 128>{}, integral_constant<int, 4>{});
    else if (s.H == 128)
      by_act(float{}, integral_constant<int, 128>{}, I0{});
    else
      by_act(float{}, integral_constant<int, 256>{}, I0{});
  }
}

static void launch_enc_fwd(const Shape& s, int kind, int R, const int* gid, const MlpW& w, const float* src, int in_dim,
                           void* out, hipStream_t st) {
  if (R == 0) return;
  if (row_tiles(s, R)) {
    launch_enc_fwd_tiles(s, kind, R, gid, w, src, in_dim, out, st);
    return;
  }
  enc_dispatch(s, R, kind, in_dim, [&](auto t, auto hh, auto ww, auto act, auto kin, auto kd) {
    using T = decltype(t);
    constexpr int H = decltype(hh)::value, W = decltype(ww)::value;
    // BF16 at H = 128 runs two workgroups per CU (70 KiB of LDS, 16 waves of 86
    // registers), its weights in LDS for good: 397 us for 3.55M edges (1.0 GB,
    // 2.5 TB/s; by counters LDS is active in 61% of a CU's cycles, and VALU and
    // MFMA issue fill the SIMDs') where the workgroup-tile kernel took 1,088
    const int grid = s.prec == 1 && s.H == 128 ? std::max(1, std::min(512, (R + 47) / 48)) : edge_stream_grid(s, R);
    k_enc_fwd_stream<T, H, W, decltype(act)::value, decltype(kin)::value, decltype(kd)::value>
        <<<grid, StreamDims<T, H, W>::NT, 0, st>>>(R, gid, w, src, in_dim, (T*)out, s.eps);
  });
}

void launch_enc_node_fwd(const Shape& s, const BatchView& b, const MlpW& w, const float* node_in, int in_dim,
                         void* h0, hipStream_t st) {
  launch_enc_fwd(s, 0, b.n, b.gid, w, node_in, in_dim, h0, st);
}

void launch_enc_edge_fwd(const Shape& s, const BatchView& b, const MlpW& w, const float* xe, void* e0,
                         hipStream_t st) {
  launch_enc_fwd(s, 1, b.E, nullptr, w, xe, 4, e0, st);
}

void launch_enc_bwd_stream(const Shape& s, int kind, int R, const int* gid, const MlpW& w, const float* src, int in_dim,
                           const float* dout, const EncBwdOut& o, float* a2, hipStream_t st) {
  enc_dispatch(s, R, kind, in_dim, [&](auto t, auto hh, auto ww, auto act, auto kin, auto kd) {
    using T = decltype(t);
    constexpr int H = decltype(hh)::value, W = decltype(ww)::value, A = decltype(act)::value, KIN = decltype(kin)::value,
                  KD = decltype(kd)::value;
    if constexpr (sizeof(T) == 4 || H > 128) {  // (enc_stream)
      const int grid = edge_stream_grid(s, R);
      k_enc_bwd1_stream<T, H, W, A, KIN, KD>
          <<<grid, StreamDims<T, H, W>::NT, 0, st>>>(R, gid, w, src, in_dim, dout, o, a2, s.eps);
      k_enc_bwd2_stream<T, H, W, A, KIN, KD><<<grid, StreamDims<T, H, W>::NT, 0, st>>>(R, gid, w, src, in_dim, o, a2);
    }
  });
}

}  // namespace xmgn
