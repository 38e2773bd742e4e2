// Edge kernels as wave-private chains with streamed weights (BF16, H = 256
// and 512; see chain.hpp).
//
// At these widths the weights do not fit in LDS.  The workgroup's waves walk
// the same sequence of weight slabs (the MFMA fragments of one 32-wide k chunk,
// 16 or 32 KiB), which travel from L2 straight into a ring of four LDS slots,
// three slabs ahead of their use; one barrier per slab.  A wave's rows,
// accumulators and LayerNorm stay in its registers.
#include <algorithm>
#include <type_traits>

#include "chain.hpp"
#include "kernels.hpp"
#include "segsum.hpp"

namespace xmgn {

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
// behind s + 1) is always enough and never too little; other loads and stores
// in between only make it wait for more.  At the end of a cycle it waits for
// everything, so that the first two slabs of the next need no wait behind the
// stores of the epilogue.
template <int NW, int S, int MBS>
struct WStream {
  static constexpr int SLAB = MBS * 1024, K = MBS / NW;  // K loads of 1 KiB per wave and slab
  static_assert(S % 4 == 0, "a slab's slot is s % 4");
  const unsigned char* base;  // (uniform)
  unsigned char* ring;        // LDS, 4 SLAB bytes
  __device__ __forceinline__ void send(int s) const {
    const int w = __builtin_amdgcn_readfirstlane(wave_id()) * K;
    const unsigned char* g = base + (size_t)(s % S) * SLAB + w * 1024;
    const unsigned dst = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)(ring) + (s & 3) * SLAB + w * 1024;
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
  __device__ __forceinline__ void start() const {  // slabs 0, 1 and 2, whole at the next barrier
    send(0);
    send(1);
    send(2);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  __device__ __forceinline__ void begin(int s) const { send(s + 3); }
  __device__ __forceinline__ void end(int s) const {
    if (s == S - 1)
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else if (s >= 2) {
      if constexpr (K == 2)
        asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
      else
        asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
    }
    lds_sync();
  }
  __device__ __forceinline__ const bf16x8* frags(int s) const { return (const bf16x8*)(ring + (s & 3) * SLAB); }
  static_assert(K == 2 || K == 8, "waits are written for these counts");
};

// acc[t][mb] += W x over one k chunk; fragments are read D ahead of their
// products.
template <int ET, int MBS>
__device__ __forceinline__ void slab_gemm(f32x4 (&acc)[ET][MBS], const bf16x8* f, const bf16x8 (&x)[ET]) {
  constexpr int D = 6, N = MBS;
  f += lane_id();
  bf16x8 a[D];
#pragma unroll
  for (int i = 0; i < D; ++i) a[i] = f[i * 64];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const bf16x8 cur = a[i % D];
    if (i + D < N) a[i % D] = f[(i + D) * 64];
#pragma unroll
    for (int t = 0; t < ET; ++t) acc[t][i] = mma(cur, x[t], acc[t][i]);
  }
  __builtin_amdgcn_sched_group_barrier(0x100, D, 0);  // DS reads
#pragma unroll
  for (int i = 0; i < N - D; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, ET, 0);  // MFMA
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
  }
  __builtin_amdgcn_sched_group_barrier(0x008, D * ET, 0);
  __builtin_amdgcn_sched_barrier(0);
}

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
    auto product = [&](int s0, bf16x8(&xs)[KC][ET]) {
#pragma unroll
      for (int c = 0; c < KC; ++c) {
        ws.begin(s0 + c);
        slab_gemm(acc, ws.frags(s0 + c), xs[c]);
        ws.end(s0 + c);
      }
    };
    product(0, xr);
    product(KC, xs);
#pragma unroll
    for (int c = 0; c < KC; ++c)
#pragma unroll
      for (int t = 0; t < ET; ++t) arrived(ec[c][t]);
    product(2 * KC, ec);
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
    product(3 * KC, z);
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

}  // namespace xmgn
