// Kernel argument blocks and launcher declarations of the xmgn library.
#pragma once

#include <stdexcept>
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace xmgn {

// Set by a launcher when the requested tile configuration does not fit the
// hardware (LDS); the host turns it into XMGN_ERR_UNSUPPORTED.
extern int g_config_error;

constexpr int kMaxTiledEdges = 1 << 17;  // (see edge_tiles)

// Device view of a batch (disjoint union of partitions).
struct BatchView {
  int n;                 // nodes
  int E;                 // edges
  const int* gid;        // [n] global node id
  const int* row_ptr;    // [n+1] receiver CSR
  const int* col;        // [E] sender (batch index)
  const int* recv;       // [E] receiver (batch index)
  const int* csc_ptr;    // [n+1] sender CSR
  const int* csc_edge;   // [E] CSR edge of each sender slot
  const int* etiles;     // [n_etiles+1][2] (receiver, edge) bounds of edge tiles
  int n_etiles;
  int steps4, steps8;    // up to kMaxTiledEdges edges: 16-row steps of the longest range that a wave of the
                         // streaming kernels takes, with four and with eight waves per workgroup
  const int* inner;      // [n_inner] batch rows of inner nodes
  int n_inner;
};

// Per-MLP weight views.  W* are the compute-type copies ([out][in]);
// W*T are transposes ([in][out]) used by the backward products; vectors are
// FP32 views into the parameter blob.
struct MlpW {
  const void* W1;
  const void* W2;
  const void* W3;
  const void* W1T;  // edge: [H][H] block of W1^T for the e input; node/dec: full W1^T
  const void* W2T;
  const void* Brs;  // edge layers: [H][2H] = [W1_r^T | W1_s^T]
  const float* W1f; // FP32 first-layer weights (encoders) / last layer (decoder)
  const float* b1;
  const float* b2;
  const float* b3;
  const float* gamma;
  const float* beta;
  // kernels with streamed weights (the node MLP's; edge_stream): MFMA fragment
  // order, k chunk by k chunk, as the kernels walk them
  const void* FS;   // forward: W1, W2 (edge, node MLP); W2, W3 (encoder)
  const void* BS;   // adjoint: W2, W2^T, e-block of W1^T (edge MLP); W3^T, W2^T (encoder; BF16 H = 128 edges: W2, W3 ahead);
                    // B_rs of the edge layer above (if any), W1, W2, W2^T, W1^T (node MLP)
};

struct Shape {
  int H;
  int prec;     // 0 fp32, 1 bf16
  int act;      // 0 relu, 1 silu
  int agg;      // 0 message, 1 edge
  int mt_edge;  // rows per edge tile
  int mt_edge_bwd;  // rows per edge tile of the edge adjoint (its own tiling of the same edges)
  int mt_node;  // rows per node tile
  int grid;     // persistent grid (workgroups)
  int nw_edge;  // waves per workgroup of the edge kernels (4 or 8)
  int nw_edge_bwd;  // waves per workgroup of the edge adjoint
  float eps;
};

struct EdgeNorm {
  float mu[4];
  float sd[4];
};

// ---- forward ----
void launch_enc_node_fwd(const Shape& s, const BatchView& b, const MlpW& w, const float* node_in,
                         int in_dim, void* h0, hipStream_t st);
// Edge features ([x_s - x_r, |x_s - x_r|] - mu) / sd into xe[E][4].
void launch_edge_feat(const BatchView& b, const float* pos, EdgeNorm en, float* xe, hipStream_t st);
void launch_enc_edge_fwd(const Shape& s, const BatchView& b, const MlpW& w, const float* xe, void* e0,
                         hipStream_t st);
// z_out (or NULL): the hidden activation of every edge;
// a_out (or NULL): its pre-activation, for edge_a_tape forms.
// pr, ps (or NULL for the gathered form): the node projections of
// launch_node_proj for this layer's edge MLP.
void launch_edge_fwd(const Shape& s, const BatchView& b, const MlpW& w, const void* h,
                     const void* e, void* e_out, float* m, void* z_out, void* a_out, const float* pr,
                     const float* ps, hipStream_t st);
// The BF16 gathered forward at H = 128 runs as wave-private chains.
bool edge_fwd_chain(const Shape& s);
void launch_edge_fwd_chain(const Shape& s, const BatchView& b, const MlpW& w, const void* h, const void* e,
                           void* e_out, float* m, void* z_out, void* a_out, hipStream_t st);
// Every other form streams its weights (w.FS) through LDS.
bool edge_stream(const Shape& s);
bool stream_small(const Shape& s, int rows);     // so few rows that it runs four waves per workgroup
int stream_grid(int rows, int waves);            // workgroups of so many waves over so many rows
int edge_stream_grid(const Shape& s, int rows);  // workgroups of a streaming kernel over so many rows
void launch_edge_fwd_stream(const Shape& s, const BatchView& b, const MlpW& w, const void* h, const void* e,
                            void* e_out, float* m, void* z_out, void* a_out, hipStream_t st);
// Few rows run on tiles instead (why: at the definitions): the node processor and
// the encoders (FP32, H = 256), and the gathered edge processor.
bool row_tiles(const Shape& s, int rows);
bool edge_tiles(const Shape& s, const BatchView& b);
void launch_node_fwd_tiles(const Shape& s, const BatchView& b, const MlpW& w, const void* h, const float* m,
                           void* h_out, hipStream_t st);
void launch_enc_fwd_tiles(const Shape& s, int kind, int R, const int* gid, const MlpW& w, const float* src, int in_dim,
                          void* out, hipStream_t st);
// pr = W1_r h + b1, ps = W1_s h for every node (FP32 [n][H] each).
void launch_node_proj(const Shape& s, const BatchView& b, const MlpW& w, const void* h, float* pr, float* ps,
                      hipStream_t st);
void launch_node_fwd(const Shape& s, const BatchView& b, const MlpW& w, const void* h,
                     const float* m, void* h_out, hipStream_t st);
void launch_dec_fwd(const Shape& s, const BatchView& b, const MlpW& w, const void* h, float* out,
                    int out_dim, hipStream_t st);

// ---- backward ----
struct EdgeBwdOut {
  float* de_out;   // [E][H]
  float* S_r;      // [n][H] receiver sums of da
  void* da;        // [E][H] T
  void* du;        // [E][H] T
  void* z;         // [E][H] T
  float* partial;  // [grid][4H]: db1, db2, dgamma, dbeta
  float* wpart;    // fused weight gradients [grid][2][H][H] (dW2, e-block of dW1) or NULL
};
// True when the edge adjoint accumulates dW2 and the e-block of dW1 itself
// (then du and z are not written and wpart must be given).
bool edge_bwd_fuses_wgrad(const Shape& s);
// Scratch (floats) of the two-stage sums over the rows of partial matrices with
// so many columns.
size_t reduce_tmp_floats(int max_cols);
// True when the adjoint with z on the tape also needs a (SiLU).
bool edge_a_tape(const Shape& s);
// zt: z of every edge as the forward kept it, or NULL (recomputed; the unfused
// form then writes it to o.z for its dW2 product); at: a likewise, where
// edge_a_tape.
void launch_edge_bwd(const Shape& s, const BatchView& b, const MlpW& w, const void* h, const void* e,
                     const void* zt, const void* at, const float* de_in, const float* dm, const EdgeBwdOut& o,
                     hipStream_t st);

// With z on the tape the adjoint runs as wave-private chains: in the BF16 form
// at H = 128 they accumulate dW2 and the e-block of dW1, elsewhere they stream
// their weights (w.BS) and write du.  Their partials have
// edge_bwd_chain_grid(s, E) rows.
int edge_bwd_chain_grid(const Shape& s, int E);
void launch_edge_bwd_stream(const Shape& s, const BatchView& b, const MlpW& w, const void* zt, const void* at,
                            const float* de_in, const float* dm, const EdgeBwdOut& o, hipStream_t st);
void launch_edge_bwd_chain(const Shape& s, const BatchView& b, const MlpW& w, const void* e, const void* zt,
                           const void* at, const float* de_in, const float* dm, const EdgeBwdOut& o, hipStream_t st);

struct NodeBwdOut {
  float* dh_mid;   // [n][H]
  float* dm;       // [n][H]
  void* da;        // [n][H] T
  void* du;        // [n][H] T
  void* z;         // [n][H] T
  float* partial;  // [grid][4H]: db1, db2, dgamma, dbeta
};
// Upstream gradient dh_in, or with S_r and S_s dh_in + [S_r | S_s] * [W1_r ;
// W1_s] of the edge layer above (dh_in may be o.dh_mid then).  Partials have
// edge_stream_grid(s, b.n) rows.
void launch_node_bwd(const Shape& s, const BatchView& b, const MlpW& w, const void* h, const float* m,
                     const float* dh_in, const float* S_r, const float* S_s, const NodeBwdOut& o, hipStream_t st);
// dh_out = dh_mid + [S_r | S_s] * [W1_r ; W1_s]  (edge-layer input gradients)
void launch_node_dh(const Shape& s, const BatchView& b, const MlpW& w, const float* dh_mid,
                    const float* S_r, const float* S_s, float* dh_out, hipStream_t st);
void launch_sender_sum(const Shape& s, const BatchView& b, const void* da, float* S_s, hipStream_t st);

struct DecBwdOut {
  float* dh;       // [n][H], rows of inner nodes written (caller zeroes the rest)
  void* z1;        // [n_inner][H] T
  void* z2;
  void* da1;
  void* da2;
  float* dy;       // [n_inner][16]
  float* partial;  // [grid][2H + 16]
};
void launch_dec_bwd(const Shape& s, const BatchView& b, const MlpW& w, const void* h,
                    const float* d_out, int out_dim, const DecBwdOut& o, hipStream_t st);

struct EncBwdOut {
  void* z1;
  void* z2;
  void* da2;
  void* du3;
  float* partial;  // [grid][5H + 8H]: db1 db2 db3 dgamma dbeta dW1[H][8]
  float* wpart;    // fused weight gradients [grid][2][H][H] (dW2, dW3) or NULL
  float* da1;      // more than 8 inputs: adjoint of the input layer's output [rows][H] (FP32); dW1 not in partial
};
// True when the encoder adjoint accumulates dW2 and dW3 itself (then z1,
// z2, da2 and du3 are not written and wpart must be given).
bool enc_bwd_fuses_wgrad(const Shape& s);
void launch_enc_node_bwd(const Shape& s, const BatchView& b, const MlpW& w, const float* node_in,
                         int in_dim, const float* dh0, const EncBwdOut& o, float* a2, hipStream_t st);
void launch_enc_edge_bwd(const Shape& s, const BatchView& b, const MlpW& w, const float* xe, const float* de0,
                         const EncBwdOut& o, float* a2, hipStream_t st);

// True for the forms whose encoder adjoints stream their weights (w.BS): all but
// BF16 at H = 128.  kind 0: node inputs src[gid[row]], 1: edge features src[row].
// The adjoint's partials have edge_stream_grid(s, R) rows; a2: FP32 [R][H]
// scratch (SiLU).
bool enc_stream(const Shape& s);
void launch_enc_bwd_stream(const Shape& s, int kind, int R, const int* gid, const MlpW& w, const float* src, int in_dim,
                           const float* dout, const EncBwdOut& o, float* a2, hipStream_t st);

// The edge encoder's adjoint of the BF16 form at H = 128 (w.BS: W2, W3, W3^T,
// W2^T): accumulates dW2 and dW3 itself; partials have edge_stream_grid(s, R)
// rows; a2: FP32 [R][H] scratch (SiLU).
void launch_enc_edge_bwd_chain(const Shape& s, int R, const MlpW& w, const float* xe, const float* dout,
                               const EncBwdOut& o, float* a2, hipStream_t st);

// ---- auxiliary ----
// C[m][n] = sum_r A[r][a0 + m] * B[ib(r)][b0 + n] over r < R; partial
// sums per row chunk, then dst[m * ldd + n] = sum over chunks (m < M_valid).
struct WgradOp {
  const void* A;
  int a_f32;  // 1: A is FP32, else compute type
  int lda, a0;
  const void* B;
  int b_f32;
  int ldb, b0;
  const int* ib;
  int R, M, N, M_valid;
  float* dst;
  int ldd;
};
struct WgradJob {
  WgradOp op;
  int chunks, rows, first;  // (set by the launch: row chunks, rows in each, first workgroup, its partials)
  float* partial;
};
constexpr int kMaxWgradJobs = 7;
struct WgradBatch {
  int n = 0;
  WgradJob job[kMaxWgradJobs];
  void add(const WgradOp& op) {
    if (n >= kMaxWgradJobs) throw std::logic_error("weight-gradient batch is full");
    job[n++].op = op;
  }
};

struct VecSeg {
  int src;  // offset in the partial row
  int len;
  float* dst;
};
// Fixed-order two-stage sums over the rows of partial matrices: 32 equal groups
// of rows (fewer rows: one each), even and odd places of a group apart, then the
// groups in order.  The result depends on the row count only.
// dst[i * dst_stride + k] = sum over g < G of partial[g * row + src + i *
// src_stride + k] for i < runs, k < inner.
void launch_vec_reduce_strided(const float* partial, int G, int row, int src, int runs, int inner, int src_stride,
                               float* dst, int dst_stride, float* tmp, hipStream_t st);

// A batch of such sums in two launches in all: job j sets dst[m * ldd + n] =
// sum over r < rows of src[r * stride + m * N + n] (m < M_valid, n < N).
struct RedJob {
  const float* src;
  float* dst;
  int rows, stride, M_valid, N, ldd, splits, per;
  long long tmp_off;  // this job's stage-1 scratch, in floats
};
constexpr int kMaxRedJobs = 24;
struct RedBatch {
  int n = 0;
  long long tmp_floats = 0;  // scratch the batch needs
  int grid1 = 0, grid2 = 0;  // workgroups of the two launches, and each job's first
  int first1[kMaxRedJobs], first2[kMaxRedJobs];
  RedJob job[kMaxRedJobs];
  void add(const float* src, int rows, int stride, int M_valid, int N, float* dst, int ldd);
  // the segments of a per-workgroup partial row [G][row]
  void add_vec(const float* partial, int G, int row, const VecSeg* segs, int n_seg);
};
void launch_reduce_batch(const RedBatch& b, float* tmp, hipStream_t st);
// Runs the products of b in one launch and adds their reductions to red;
// partial: wgrad_partial_floats(s) floats of scratch, in use until red has run.
size_t wgrad_partial_floats(const Shape& s);
void launch_wgrad(const Shape& s, WgradBatch& b, float* partial, RedBatch& red, hipStream_t st);

struct PrepJob {
  int64_t src_off;   // element offset in the FP32 params
  int src_ld;        // row stride of the source matrix
  int src_col0;      // first source column
  int transpose;     // 0: dst[i][j] = src[i][col0 + j]; 1: dst[i][j] = src[j][col0 + i]
  int64_t dst_off;   // element offset in the compute blob
  int dst_ld;
  int dst_col0;
  int rows, cols;
  int frag;          // 1: dst in MFMA fragment order (rows, cols multiples of 16 and 32): k chunk, block, lane
};
void launch_prep(const float* params, void* blob, int prec, const PrepJob* jobs_dev, int n_jobs,
                 hipStream_t st);

void launch_fill(float* p, size_t n, float v, hipStream_t st);
void launch_accumulate(float* acc, const float* g, int64_t n, hipStream_t st);
// Adam constants of one step, each rounded to FP32 once from its FP64 value:
// c1 = 1 - b1, c2 = 1 - b2, bc1 = 1 - b1^t, bc2 = 1 - b2^t; clip <= 0: none.
struct AdamArgs {
  float lr, b1, b2, c1, c2, eps, bc1, bc2;
  double clip;
};
// partial: dev double [kAdamScratchPartials] scratch; norm_out: dev float [1] or NULL.
void launch_adam(float* p, const float* g, float* m, float* v, int64_t n, double* partial, const AdamArgs& a,
                 float* norm_out, hipStream_t st);
// Partials of the clipping norm: what launch_adam writes and reads, and the
// capacity of the library's fixed per-device array that the allocation-free
// entry point uses.
constexpr int kAdamScratchPartials = 256;
constexpr int kMaxDevices = 64;
// Device address (on `device`, which must be current) of that array; looked
// up on the first call per device.  Returns 0, or -1 (bad device) / -3
// (HIP error) with *err set.
int adam_noalloc_scratch(int device, double** out, const char** err);
void launch_mse(const float* out, const float* target, const int* gid, const int* inner, int n_inner,
                int out_dim, double inv_norm, float* d_out, float* partial, int G, float* loss,
                hipStream_t st);

// ---- kNN ----
int knn_build(const float* pos, int n, const int* level_end, int n_levels, int k_intra,
              int k_cross, int** row_ptr_out, int** col_out, long long* n_edges, hipStream_t st,
              const char** err);

}  // namespace xmgn
