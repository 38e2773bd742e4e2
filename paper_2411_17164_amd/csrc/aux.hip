// Auxiliary kernels: weight gradients as row-sums of outer products
// (split over row chunks, reduced in a fixed order), fixed-order reductions
// of per-workgroup partial vectors, weight preparation (cast / transpose into
// the compute type), the masked MSE and gradient accumulation.
#include <algorithm>
#include <mutex>
#include <stdexcept>
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace xmgn {

int g_config_error = 0;

// ---------------------------------------------------------------------------
// wgrad: C[m][n] = sum_r A[r][a0 + m] * B[r][b0 + n], several such products in
// one launch.  A workgroup owns one chunk of one product's rows and one block
// of its outputs: 128 x 128 by four waves, or, in the BF16 form from H = 256
// on, 256 x 256 by eight, which halves the reads of the operands.  Rows go to
// LDS as they lie in memory, 64 (FP32: 32) at a time, into two buffers in turn,
// with one barrier per stage and the loads of the next stage in flight behind
// it; the row index is the MFMA k dimension, so the BF16 fragments are
// transposing reads (32-byte units swizzled by row: no bank conflicts on either
// side) and the FP32 ones four reads of one word (rows padded by 16 bytes).
// Two products over 444k rows, BF16, H = 512: 480 us (970 TFLOP/s).  All weight
// gradients of a step with their sums, against a launch per product of 128-row
// stages transposed on their way into LDS (eight lanes to a bank) and two
// reductions each: 2,000 nodes, FP32: 441 -> 155 us; 50k nodes, FP32: 2.54 -> 1.78
// ms; 100k, BF16, H = 256: 3.26 -> 2.5; 50k, H = 512: 4.07 -> 2.9; 400k, H = 128
// (bound by reading its operands, 5.5 TB/s): 5.9 -> 4.4.  In FP32 MFMA is busy for
// 82% of the cycles that a CU is, but a launch's CUs end unevenly.  Loads under a condition, or
// behind a possible row index, each waited for the ones before: 20% slower.
// A chunk can be 20,000 rows, more than one running FP32 sum takes well: the
// FP32 form adds up runs of 64 MFMA steps (256 rows) in a second set of
// accumulators.  Gradient against 64 bits, 400k nodes, H = 128: 1.0e-7 (worst
// tensor 1.4e-7) where one sum a chunk left 3.8e-7 (1.1e-6); the 50k-node step
// takes 7.33 ms instead of 7.30.  Beside the rounding of BF16 operands the longer
// sum does not show (worst tensor, 400k nodes and edges, H = 128, 256 and 512:
// 1.85e-4, 1.39e-4 and 1.39e-4 here as with the shorter chunks of a launch per product).
// ---------------------------------------------------------------------------
template <typename T, int BLK, int ROWS = 64>
struct Wg {
  static constexpr int NW = BLK == 256 ? 8 : 4, NT = 64 * NW;
  static constexpr int KR = sizeof(T) == 2 ? ROWS : 32;     // rows per stage
  static constexpr int E = 16 / sizeof(T), UPR = BLK / E;   // elements per 16-byte unit; units per row
  static constexpr int RPP = NT / UPR, P = KR / RPP;        // rows per pass of the workgroup; passes
  static constexpr int LD = sizeof(T) == 2 ? BLK * 2 : BLK * 4 + 16;  // bytes per LDS row
  static constexpr int TILE = KR * LD;
  static constexpr int FM = BLK / 32, FN = 4;               // 16 x 16 blocks of a wave
  static constexpr int RUN = sizeof(T) == 4 ? 256 : 0;      // rows summed in one run (0: all)
  static __device__ __forceinline__ int off(int row, int u) {
    if constexpr (sizeof(T) == 2)
      return row * LD + (((u >> 1) ^ (row & 7)) << 5) + ((u & 1) << 4);
    else
      return row * LD + 16 * u;
  }
};

// One thread's share of a stage of one operand (source type S).
template <typename T, typename S, typename G, int BLK>
struct WgStage {
  static constexpr int N = sizeof(S) / sizeof(T);  // 16-byte loads per unit
  uint4 v[G::P][N];
  // (rows and columns out of range repeat one within; store() clears them)
  __device__ __forceinline__ void load(const S* base, int ld, int r0, int r_end, int c0, int C) {
    const int c = c0 + G::E * ((int)threadIdx.x % G::UPR), rr = (int)threadIdx.x / G::UPR;
    const char* s = (const char*)(base + (size_t)r0 * ld);  // (uniform; 32-bit offsets within a stage)
#pragma unroll
    for (int p = 0; p < G::P; ++p)
#pragma unroll
      for (int k = 0; k < N; ++k) {
        const int ck = c + k * (G::E / N);
        const unsigned o = (unsigned)(min(rr + p * G::RPP, r_end - 1 - r0) * ld + (ck < C ? ck : 0)) * (unsigned)sizeof(S);
        v[p][k] = *(const uint4*)(s + o);
      }
  }
  // rows taken through idx (their indices first, so that no load waits for another)
  __device__ __forceinline__ void load(const S* base, int ld, const int* idx, int r0, int r_end, int c0, int C) {
    const int c = c0 + G::E * ((int)threadIdx.x % G::UPR), rr = r0 + (int)threadIdx.x / G::UPR;
    int ri[G::P];
#pragma unroll
    for (int p = 0; p < G::P; ++p) ri[p] = idx[min(rr + p * G::RPP, r_end - 1)];
#pragma unroll
    for (int p = 0; p < G::P; ++p)
#pragma unroll
      for (int k = 0; k < N; ++k) {
        const int ck = c + k * (G::E / N);
        v[p][k] = *(const uint4*)(base + (size_t)ri[p] * ld + (ck < C ? ck : 0));
      }
  }
  __device__ __forceinline__ void store(unsigned char* tile, int r0, int r_end, int c0, int C) {
    const int u = (int)threadIdx.x % G::UPR, rr = (int)threadIdx.x / G::UPR;
    if (r0 + G::KR > r_end || c0 + BLK > C) {
#pragma unroll
      for (int p = 0; p < G::P; ++p)
#pragma unroll
        for (int k = 0; k < N; ++k)
          if (r0 + rr + p * G::RPP >= r_end || c0 + G::E * u + k * (G::E / N) >= C) v[p][k] = uint4{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int p = 0; p < G::P; ++p) {
      uint4 x = v[p][0];
      if constexpr (N == 2) {
        T h[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) h[k] = from_f<T>(((const float*)&v[p][k >> 2])[k & 3]);
        x = *(const uint4*)h;
      }
      *(uint4*)(tile + G::off(rr + p * G::RPP, u)) = x;
    }
  }
};

// Fragment [columns c0 .. + 15][k chunk c] of a tile; the k order of BF16
// (rows 4 g + r, 16 + 4 g + r of 32) is the same on both operands.
template <typename T, int BLK>
__device__ __forceinline__ typename TT<T>::V wg_frag(const unsigned char* tile, int c, int c0) {
  using G = Wg<T, BLK>;
  const int l = lane_id(), L = l & 15, lg = l >> 4;
  if constexpr (sizeof(T) == 2) {
    const int row = 32 * c + 4 * lg + (L >> 2), f = c0 + 4 * (L & 3);
    const unsigned char* p = tile + G::off(row, f >> 3) + (f & 7) * 2;
    const bf16x4_lds lo = lds_read_tr4((const bf16*)p), hi = lds_read_tr4((const bf16*)(p + 16 * G::LD));
    return bf16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  } else {
    const unsigned char* p = tile + (16 * c + 4 * lg) * G::LD + (c0 + L) * 4;
    return f32x4{*(const float*)p, *(const float*)(p + G::LD), *(const float*)(p + 2 * G::LD),
                 *(const float*)(p + 3 * G::LD)};
  }
}

template <typename T, int BLK, typename SA, typename SB, bool IDX>
__device__ __forceinline__ void wg_block(const WgradOp& op, int r_begin, int r_end, int m0, int n0, unsigned char* smem,
                                         float* __restrict__ out) {
  // (two FP32 sources of BF16 products: 32 rows, or their loads spill)
  using G = Wg<T, BLK, sizeof(SA) + sizeof(SB) == 8 ? 32 : 64>;
  using V = typename TT<T>::V;
  constexpr int KC = 4 * TT<T>::E;
  const int w = wave_id(), wm = (w & 1) * (BLK / 2), wn = (w >> 1) * 64;
  const int l = lane_id(), li = l & 15, lg = l >> 4;
  const SA* A = (const SA*)op.A + op.a0;
  const SB* B = (const SB*)op.B + op.b0;
  f32x4 acc[G::FM][G::FN], tot[G::RUN ? G::FM : 1][G::FN];
  zero_acc(acc);
  zero_acc(tot);
  WgStage<T, SA, G, BLK> sa;
  WgStage<T, SB, G, BLK> sb;
  auto load = [&](int r0) {
    if constexpr (IDX)
      sb.load(B, op.ldb, op.ib, r0, r_end, n0, op.N);
    else
      sb.load(B, op.ldb, r0, r_end, n0, op.N);
    sa.load(A, op.lda, r0, r_end, m0, op.M);
  };
  const bool live = m0 + wm < op.M && n0 + wn < op.N;  // (uniform)
  load(r_begin);
  int half = 0, run = 0;
  for (int r0 = r_begin; r0 < r_end; r0 += G::KR, half ^= 1) {
    unsigned char* At = smem + half * 2 * G::TILE;
    unsigned char* Bt = At + G::TILE;
    // this buffer was last read before the previous stage's barrier
    sa.store(At, r0, r_end, m0, op.M);
    sb.store(Bt, r0, r_end, n0, op.N);
    __syncthreads();
    if (r0 + G::KR < r_end) load(r0 + G::KR);
    if (live) {
#pragma unroll
      for (int c = 0; c < G::KR / KC; ++c) {
        V b[G::FN];
#pragma unroll
        for (int j = 0; j < G::FN; ++j) b[j] = wg_frag<T, BLK>(Bt, c, wn + 16 * j);
        V a = wg_frag<T, BLK>(At, c, wm);
#pragma unroll
        for (int i = 0; i < G::FM; ++i) {
          const V ai = a;
          if (i + 1 < G::FM) a = wg_frag<T, BLK>(At, c, wm + 16 * (i + 1));
#pragma unroll
          for (int j = 0; j < G::FN; ++j) acc[i][j] = mma(ai, b[j], acc[i][j]);
        }
      }
    }
    if constexpr (G::RUN > 0) {
      run += G::KR;
      if (run == G::RUN || r0 + G::KR >= r_end) {
        run = 0;
#pragma unroll
        for (int i = 0; i < G::FM; ++i)
#pragma unroll
          for (int j = 0; j < G::FN; ++j) tot[i][j] += acc[i][j];
        zero_acc(acc);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < G::FM; ++i)
#pragma unroll
    for (int j = 0; j < G::FN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + wm + 16 * i + 4 * lg + r, n = n0 + wn + 16 * j + li;
        if (m < op.M && n < op.N) out[(size_t)m * op.N + n] = (G::RUN ? tot : acc)[i][j][r];
      }
}

// Workgroup ids of a product go chunk by chunk in groups of eight, one per XCD,
// so that the blocks of one chunk, and the products over the same rows, meet
// their operands in one L2.
template <typename T, int BLK>
__global__ __launch_bounds__((Wg<T, BLK>::NT), 2) void k_wgrad(WgradBatch b) {
  using G = Wg<T, BLK>;
  __shared__ __align__(16) unsigned char smem[4 * G::TILE];
  int j = 0;
  while (j + 1 < b.n && (int)blockIdx.x >= b.job[j + 1].first) ++j;
  const WgradJob& jb = b.job[j];
  const WgradOp& op = jb.op;
  const int id = blockIdx.x - jb.first, nbm = (op.M + BLK - 1) / BLK, blocks = nbm * ((op.N + BLK - 1) / BLK);
  const int blk = (id >> 3) % blocks, chunk = (id >> 3) / blocks * 8 + (id & 7);
  if (chunk >= jb.chunks) return;
  const int r0 = chunk * jb.rows, r1 = min(op.R, r0 + jb.rows);
  const int m0 = blk % nbm * BLK, n0 = blk / nbm * BLK;
  float* out = jb.partial + (size_t)chunk * op.M * op.N;
  // (the combinations launch_wgrad lets through)
  if (op.ib) {
    if (op.b_f32) wg_block<T, BLK, float, float, true>(op, r0, r1, m0, n0, smem, out);
    else if constexpr (sizeof(T) == 2) wg_block<T, BLK, T, T, true>(op, r0, r1, m0, n0, smem, out);
  } else if constexpr (sizeof(T) == 4) {
    wg_block<T, BLK, float, float, false>(op, r0, r1, m0, n0, smem, out);
  } else {
    if (op.a_f32) wg_block<T, BLK, float, T, false>(op, r0, r1, m0, n0, smem, out);
    else if (op.b_f32) wg_block<T, BLK, T, float, false>(op, r0, r1, m0, n0, smem, out);
    else wg_block<T, BLK, T, T, false>(op, r0, r1, m0, n0, smem, out);
  }
}

// Fixed-order column sums of a [rows][stride] partial matrix, in two
// stages: stage 1 sums rows [s*per, (s+1)*per) of each column into
// tmp[s][col] (grid.y = split s); stage 2 adds the splits in order.  The
// result depends only on (rows, splits), never on scheduling.
constexpr int RED_SPLITS = 32;

// p[r stride] over [r0, r1): even and odd places apart (an order fixed by the
// range), eight loads in flight: two at a time, a 2,000-node graph's 21 weight
// gradients and their sums took 485 us a step where they take 439.
__device__ __forceinline__ float split_sum(const float* __restrict__ p, int stride, int r0, int r1) {
  float a0 = 0.f, a1 = 0.f;
  int r = r0;
  for (; r + 7 < r1; r += 8) {
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = p[(size_t)(r + k) * stride];
#pragma unroll
    for (int k = 0; k < 8; k += 2) {
      a0 += v[k];
      a1 += v[k + 1];
    }
  }
  for (; r + 1 < r1; r += 2) {
    a0 += p[(size_t)r * stride];
    a1 += p[(size_t)(r + 1) * stride];
  }
  if (r < r1) a0 += p[(size_t)r * stride];
  return a0 + a1;
}
// p[k stride] over k < n in order, eight loads in flight
__device__ __forceinline__ float order_sum(const float* __restrict__ p, size_t stride, int n) {
  float s = 0.f;
  int k = 0;
  for (; k + 7 < n; k += 8) {
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = p[(k + i) * stride];
#pragma unroll
    for (int i = 0; i < 8; ++i) s += v[i];
  }
  for (; k < n; ++k) s += p[k * stride];
  return s;
}

__global__ void k_colsum_stage1(const float* __restrict__ src, int rows, int stride, int ncol, int per,
                                float* __restrict__ tmp) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= ncol) return;
  const int s = blockIdx.y;
  const int r0 = s * per, r1 = min(rows, r0 + per);
  tmp[(size_t)s * ncol + j] = split_sum(src + j, stride, r0, r1);
}

size_t reduce_tmp_floats(int max_cols) { return (size_t)RED_SPLITS * (size_t)max_cols; }

// Two workgroups of 128 x 128 blocks per CU, one of 256 x 256 (from H = 256 on
// in BF16: 2.6 ms in all on 100k nodes where 128 x 128 took 3.26; an FP32 block
// of 256 x 256 would leave no room for a second buffer)
static int wgrad_block(const Shape& s) { return s.prec == 1 && s.H >= 256 ? 256 : 128; }
static int wgrad_target(const Shape& s) { return wgrad_block(s) == 256 ? 256 : 512; }

size_t wgrad_partial_floats(const Shape& s) {
  const int blk = wgrad_block(s), nb = (s.H + blk - 1) / blk;
  return (size_t)std::max(wgrad_target(s), kMaxWgradJobs * nb * nb) * blk * blk;
}

void launch_wgrad(const Shape& s, WgradBatch& b, float* partial, RedBatch& red, hipStream_t st) {
  // the fewest rows per chunk, in whole stages, with which no workgroup waits
  // for another to end (a launch a little over that takes twice as long)
  const int blk = wgrad_block(s), kr = s.prec == 1 ? 64 : 32, target = wgrad_target(s);
  auto blocks = [&](const WgradOp& o) { return ((o.M + blk - 1) / blk) * ((o.N + blk - 1) / blk); };
  // a row of which one operand is to be rounded from FP32 takes about twice as
  // long (H = 512: 68 against 35 ns in a workgroup).  With this weight against
  // none, us a layer with its sums: H = 512, 50k nodes 667 / 712; H = 256, 100k
  // 424 / 443; H = 128, 400k 165 / 182, 60k 48 / 47.
  auto weight = [&](const WgradOp& o) { return s.prec == 1 && (o.a_f32 || o.b_f32) ? 2 : 1; };
  long long rows = 0;
  for (int j = 0; j < b.n; ++j) rows += (long long)b.job[j].op.R * weight(b.job[j].op) * blocks(b.job[j].op);
  long long rpc = std::max<long long>(kr, ((rows + target - 1) / target + kr - 1) / kr * kr);
  for (;; rpc += kr) {
    long long wgs = 0;
    for (int j = 0; j < b.n; ++j)
      wgs += (b.job[j].op.R * (long long)weight(b.job[j].op) + rpc - 1) / rpc * blocks(b.job[j].op);
    if (wgs <= target) break;
  }
  int grid = 0;
  size_t at = 0;
  for (int j = 0; j < b.n; ++j) {
    WgradJob& jb = b.job[j];
    WgradOp& o = jb.op;
    if (s.prec == 0) o.a_f32 = o.b_f32 = 1;
    if (o.ib ? o.a_f32 != o.b_f32 : s.prec == 1 && o.a_f32 && o.b_f32)
      throw std::logic_error("no weight-gradient kernel for these operands");
    jb.chunks = (int)((o.R * (long long)weight(o) + rpc - 1) / rpc);
    jb.rows = jb.chunks > 0 ? ((o.R + jb.chunks - 1) / jb.chunks + kr - 1) / kr * kr : 0;
    if (jb.rows) jb.chunks = (o.R + jb.rows - 1) / jb.rows;
    jb.first = grid;
    jb.partial = partial + at;
    grid += (jb.chunks + 7) / 8 * 8 * blocks(o);
    at += (size_t)jb.chunks * o.M * o.N;
    red.add(jb.partial, jb.chunks, o.M * o.N, o.M_valid, o.N, o.dst, o.ldd);
  }
  if (at > wgrad_partial_floats(s)) throw std::logic_error("weight-gradient partials exceed their scratch");
  if (grid == 0) return;
  if (s.prec == 0)
    k_wgrad<float, 128><<<grid, Wg<float, 128>::NT, 0, st>>>(b);
  else if (blk == 128)
    k_wgrad<bf16, 128><<<grid, Wg<bf16, 128>::NT, 0, st>>>(b);
  else
    k_wgrad<bf16, 256><<<grid, Wg<bf16, 256>::NT, 0, st>>>(b);
}

// Batched form: workgroups in job order (a grid of the largest job's size for
// all of them spent 100 us on empty workgroups at H = 512).  A job of at most
// RED_SPLITS rows has no first stage: the second reads its rows, in the same
// order.
// (the lanes look at one job each: one after the other they took half of a
// small workgroup's time)
__device__ __forceinline__ int red_job(const int* first, int n) {
  const int l = lane_id();
  return __popcll(__ballot(l < n && (int)blockIdx.x >= first[min(l, n - 1)])) - 1;
}
__global__ void k_colsum_batch1(RedBatch b, float* __restrict__ tmp) {
  const int job = __builtin_amdgcn_readfirstlane(red_job(b.first1, b.n));
  const RedJob& jb = b.job[job];
  const int ncol = jb.M_valid * jb.N, cb = (ncol + 255) / 256, id = blockIdx.x - b.first1[job];
  const int s = id / cb, j = (id - s * cb) * 256 + threadIdx.x;
  if (j >= ncol) return;
  const int r0 = s * jb.per, r1 = min(jb.rows, r0 + jb.per);
  tmp[jb.tmp_off + (size_t)s * ncol + j] = split_sum(jb.src + j, jb.stride, r0, r1);
}

__global__ void k_colsum_batch2(RedBatch b, const float* __restrict__ tmp) {
  const int job = __builtin_amdgcn_readfirstlane(red_job(b.first2, b.n));
  const RedJob& jb = b.job[job];
  const int ncol = jb.M_valid * jb.N, idx = (blockIdx.x - b.first2[job]) * 256 + threadIdx.x;
  if (idx >= ncol) return;
  const int m = idx / jb.N, n = idx - m * jb.N;
  jb.dst[(size_t)m * jb.ldd + n] =
      jb.per <= 1 ? order_sum(jb.src + idx, jb.stride, jb.rows) : order_sum(tmp + jb.tmp_off + idx, ncol, jb.splits);
}

void RedBatch::add(const float* src, int rows, int stride, int M_valid, int N, float* dst, int ldd) {
  if (n >= kMaxRedJobs) throw std::runtime_error("reduction batch is full");
  RedJob& j = job[n++];
  j.src = src;
  j.dst = dst;
  j.rows = rows;
  j.stride = stride;
  j.M_valid = M_valid;
  j.N = N;
  j.ldd = ldd;
  j.splits = rows < RED_SPLITS ? (rows > 0 ? rows : 1) : RED_SPLITS;
  j.per = rows > 0 ? (rows + j.splits - 1) / j.splits : 0;
  const int cb = (M_valid * N + 255) / 256;
  first1[n - 1] = grid1;
  first2[n - 1] = grid2;
  grid1 += j.per > 1 ? cb * j.splits : 0;
  grid2 += cb;
  j.tmp_off = tmp_floats;
  tmp_floats += (long long)j.splits * M_valid * N;
}

void RedBatch::add_vec(const float* partial, int G, int row, const VecSeg* segs, int n_seg) {
  for (int i = 0; i < n_seg; ++i) add(partial + segs[i].src, G, row, 1, segs[i].len, segs[i].dst, 0);
}

void launch_reduce_batch(const RedBatch& b, float* tmp, hipStream_t st) {
  if (b.n == 0) return;
  if (b.grid1) k_colsum_batch1<<<b.grid1, 256, 0, st>>>(b, tmp);
  k_colsum_batch2<<<b.grid2, 256, 0, st>>>(b, tmp);
}

// ---------------------------------------------------------------------------
// Fixed-order reduction of per-workgroup partial rows.
// ---------------------------------------------------------------------------
__global__ void k_vec_reduce(const float* __restrict__ tmp, int splits, int row, int src, int len, int inner,
                             int src_stride, float* __restrict__ dst, int dst_stride) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= len) return;
  const int run = j / inner, k = j - run * inner;
  dst[run * dst_stride + k] = order_sum(tmp + src + run * src_stride + k, row, splits);
}

void launch_vec_reduce_strided(const float* partial, int G, int row, int src, int runs, int inner, int src_stride,
                               float* dst, int dst_stride, float* tmp, hipStream_t st) {
  const int splits = G < RED_SPLITS ? G : RED_SPLITS, per = (G + splits - 1) / splits;
  k_colsum_stage1<<<dim3((row + 255) / 256, splits), 256, 0, st>>>(partial, G, row, row, per, tmp);
  k_vec_reduce<<<(runs * inner + 255) / 256, 256, 0, st>>>(tmp, splits, row, src, runs * inner, inner, src_stride, dst,
                                                           dst_stride);
}

// ---------------------------------------------------------------------------
// Weight preparation: cast (and transpose) FP32 parameter matrices into the
// compute blob.
// ---------------------------------------------------------------------------
template <typename T>
__global__ void k_prep(const float* __restrict__ params, T* __restrict__ blob, const PrepJob* __restrict__ jobs) {
  const PrepJob j = jobs[blockIdx.y];
  const int tot = j.rows * j.cols;
  for (int idx = blockIdx.x * blockDim.x + threadIdx.x; idx < tot; idx += gridDim.x * blockDim.x) {
    const int i = idx / j.cols, k = idx - i * j.cols;
    const float v = j.transpose ? params[j.src_off + (int64_t)k * j.src_ld + j.src_col0 + i]
                                : params[j.src_off + (int64_t)i * j.src_ld + j.src_col0 + k];
    int64_t at = j.dst_off;
    if (j.frag) {  // k chunk (4 E wide), block of 16 rows, then lane (k / E % 4, row % 16) with E k each
      constexpr int E = 16 / sizeof(T);
      at += (((int64_t)(k / (4 * E)) * (j.rows >> 4) + (i >> 4)) * 64 + (k / E % 4) * 16 + (i & 15)) * E + k % E;
    } else
      at += (int64_t)i * j.dst_ld + j.dst_col0 + k;
    blob[at] = from_f<T>(v);
  }
}

void launch_prep(const float* params, void* blob, int prec, const PrepJob* jobs_dev, int n_jobs, hipStream_t st) {
  if (n_jobs == 0) return;
  dim3 grid(64, n_jobs);
  if (prec == 1) k_prep<bf16><<<grid, 256, 0, st>>>(params, (bf16*)blob, jobs_dev);
  else k_prep<float><<<grid, 256, 0, st>>>(params, (float*)blob, jobs_dev);
}

// ---------------------------------------------------------------------------
__global__ void k_fill(float* p, size_t n, float v) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}
void launch_fill(float* p, size_t n, float v, hipStream_t st) {
  if (n == 0) return;
  size_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  k_fill<<<(unsigned)blocks, 256, 0, st>>>(p, n, v);
}

__global__ void k_accumulate(float* __restrict__ acc, const float* __restrict__ g, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    acc[i] += g[i];
}
void launch_accumulate(float* acc, const float* g, int64_t n, hipStream_t st) {
  if (n == 0) return;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  k_accumulate<<<(unsigned)blocks, 256, 0, st>>>(acc, g, n);
}

// ---------------------------------------------------------------------------
// Optimizer: global-norm clipping and Adam.  The squared norm is summed in
// FP64, per workgroup over a fixed index set and then over the workgroups in
// order, so the step is deterministic.
//
// Both kernels are bound by HBM (reads g; then reads p, g, m, v and writes p,
// m, v): elements go four at a time where every array is 16-byte aligned
// (VEC = 4; else and for a remainder one at a time), and every workgroup adds
// up the 256 partials as a tree instead of one thread walking them.  29.2M
// parameters: 181 us (0.93 GB, 5.2 TB/s), was 336 us with scalar accesses, one wave per
// SIMD in the norm and the serial walk.
// ---------------------------------------------------------------------------
constexpr int SUMSQ_THREADS = 1024;

// Sum over the workgroup's NT threads in a fixed order; every thread gets it.
template <int NT>
__device__ __forceinline__ double block_sum(double s, double* red) {
  red[threadIdx.x] = s;
  __syncthreads();
#pragma unroll
  for (int k = NT / 2; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
    __syncthreads();
  }
  const double t = red[0];
  __syncthreads();
  return t;
}

template <int VEC>
__global__ __launch_bounds__(SUMSQ_THREADS) void k_sumsq(const float* __restrict__ g, int64_t n,
                                                         double* __restrict__ partial) {
  __shared__ double red[SUMSQ_THREADS];
  const int64_t at = blockIdx.x * (int64_t)SUMSQ_THREADS + threadIdx.x, step = (int64_t)gridDim.x * SUMSQ_THREADS;
  double s = 0.0;
  const int64_t nv = VEC == 4 ? n / 4 : 0;
#pragma unroll 4
  for (int64_t i = at; i < nv; i += step) {
    const float4 v = ((const float4*)g)[i];
    const double x = v.x, y = v.y, z = v.z, w = v.w;
    s += (x * x + y * y) + (z * z + w * w);
  }
  for (int64_t i = nv * 4 + at; i < n; i += step) {
    const double x = g[i];
    s += x * x;
  }
  const double t = block_sum<SUMSQ_THREADS>(s, red);
  if (threadIdx.x == 0) partial[blockIdx.x] = t;
}

__device__ __forceinline__ void adam_one(float& p, float g, float& m, float& v, float sc, const AdamArgs& a) {
  const float gi = g * sc;
  const float mi = a.b1 * m + a.c1 * gi;
  const float vi = a.b2 * v + a.c2 * gi * gi;
  m = mi;
  v = vi;
  p -= a.lr * (mi / a.bc1) / (sqrtf(vi / a.bc2) + a.eps);
}

template <int VEC>
__global__ __launch_bounds__(256) void k_adam(float* __restrict__ p, const float* __restrict__ g,
                                              float* __restrict__ m, float* __restrict__ v, int64_t n,
                                              const double* __restrict__ partial, AdamArgs a,
                                              float* __restrict__ norm_out) {
  __shared__ double red[256];
  static_assert(kAdamScratchPartials == 256, "one partial per thread");
  const double norm = sqrt(block_sum<256>(partial[threadIdx.x], red));
  const float sc = a.clip > 0.0 ? (float)fmin(1.0, a.clip / (norm + 1e-6)) : 1.f;
  if (blockIdx.x == 0 && threadIdx.x == 0 && norm_out) norm_out[0] = (float)norm;
  const int64_t at = blockIdx.x * (int64_t)256 + threadIdx.x, step = (int64_t)gridDim.x * 256;
  const int64_t nv = VEC == 4 ? n / 4 : 0;
  for (int64_t i = at; i < nv; i += step) {
    float4 p4 = ((float4*)p)[i], m4 = ((float4*)m)[i], v4 = ((float4*)v)[i];
    const float4 g4 = ((const float4*)g)[i];
    adam_one(p4.x, g4.x, m4.x, v4.x, sc, a);
    adam_one(p4.y, g4.y, m4.y, v4.y, sc, a);
    adam_one(p4.z, g4.z, m4.z, v4.z, sc, a);
    adam_one(p4.w, g4.w, m4.w, v4.w, sc, a);
    ((float4*)m)[i] = m4;
    ((float4*)v)[i] = v4;
    ((float4*)p)[i] = p4;
  }
  for (int64_t i = nv * 4 + at; i < n; i += step) {
    float pi = p[i], mi = m[i], vi = v[i];
    adam_one(pi, g[i], mi, vi, sc, a);
    m[i] = mi;
    v[i] = vi;
    p[i] = pi;
  }
}

void launch_adam(float* p, const float* g, float* m, float* v, int64_t n, double* partial, const AdamArgs& a,
                 float* norm_out, hipStream_t st) {
  // any caller's pointer is taken: 16-byte accesses only where all four allow them
  const bool vec = (((uintptr_t)p | (uintptr_t)g | (uintptr_t)m | (uintptr_t)v) & 15) == 0;
  int64_t blocks = (n / (vec ? 4 : 1) + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  if (blocks < 1) blocks = 1;
  if (vec) {
    k_sumsq<4><<<kAdamScratchPartials, SUMSQ_THREADS, 0, st>>>(g, n, partial);
    k_adam<4><<<(unsigned)blocks, 256, 0, st>>>(p, g, m, v, n, partial, a, norm_out);
  } else {
    k_sumsq<1><<<kAdamScratchPartials, SUMSQ_THREADS, 0, st>>>(g, n, partial);
    k_adam<1><<<(unsigned)blocks, 256, 0, st>>>(p, g, m, v, n, partial, a, norm_out);
  }
}

// ---------------------------------------------------------------------------
// Allocation-free optimizer step.  The clipping norm's per-workgroup
// partials live in `scratch`, a fixed array of the library on every device
// it runs on (held until the process ends), instead of a context buffer.
// In host code `scratch` names a host-side stand-in: its device address is
// looked up once per device and only that address is ever used.
// ---------------------------------------------------------------------------
static __device__ __align__(256) double scratch[kAdamScratchPartials];

static std::mutex g_scratch_mu;
static double* g_scratch_dev[kMaxDevices] = {};

int adam_noalloc_scratch(int device, double** out, const char** err) {
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (device < 0 || device >= kMaxDevices) {
    *err = "device index out of range";
    return -1;
  }
  if (!g_scratch_dev[device]) {
    // with `device` current (the caller made it so): this device's copy
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) {
      *err = hipGetErrorString(e);
      return -3;
    }
    g_scratch_dev[device] = (double*)ptr;
  }
  *out = g_scratch_dev[device];
  return 0;
}

// Masked MSE over the batch's inner rows: per-workgroup partial sums in a
// fixed order, then a single-workgroup fixed-order total.
__global__ __launch_bounds__(256) void k_mse(const float* __restrict__ out, const float* __restrict__ target,
                                             const int* __restrict__ gid, const int* __restrict__ inner, int n_inner,
                                             int C, double inv_norm, float* __restrict__ d_out,
                                             float* __restrict__ partial) {
  __shared__ double red[256];
  double s = 0.0;
  const int tot = n_inner * C;
  for (int idx = blockIdx.x * 256 + threadIdx.x; idx < tot; idx += gridDim.x * 256) {
    const int i = idx / C, c = idx - i * C;
    const size_t o = (size_t)gid[inner[i]] * C + c;
    const double d = (double)out[o] - (double)target[o];
    s += d * d;
    d_out[o] = (float)(2.0 * d * inv_norm);
  }
  const double t = block_sum<256>(s, red);
  if (threadIdx.x == 0) partial[blockIdx.x] = (float)(t * inv_norm);
}
__global__ __launch_bounds__(256) void k_sum_partials(const float* __restrict__ partial, int G,
                                                      float* __restrict__ out) {
  __shared__ double red[256];
  double s = 0.0;
  for (int g = threadIdx.x; g < G; g += 256) s += partial[g];
  const double t = block_sum<256>(s, red);
  if (threadIdx.x == 0) out[0] = (float)t;
}

void launch_mse(const float* out, const float* target, const int* gid, const int* inner, int n_inner, int out_dim,
                double inv_norm, float* d_out, float* partial, int G, float* loss, hipStream_t st) {
  k_mse<<<G, 256, 0, st>>>(out, target, gid, inner, n_inner, out_dim, inv_norm, d_out, partial);
  k_sum_partials<<<1, 256, 0, st>>>(partial, G, loss);
}

}  // namespace xmgn
