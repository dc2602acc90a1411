// Internal launch interface between the stage driver and the kernel files.
// Everything here works on device pointers and enqueues on the given stream.
#pragma once
#include "common.h"

namespace swarm {

// ------------------------------------------------------------------ GEMM
// C[M,N] (+)= sum_k A(m,k) * B(n,k) with fp32 accumulation.
//   a_trans = false: A stored [M,K] (k contiguous, row pitch lda); true: stored [K,M].
//   b_trans = false: B stored [N,K] (k contiguous, row pitch ldb); true: stored [K,N].
// The three uses: forward  y = x W^T      (A = x [T,in],   B = W [out,in]:            F,F)
//                 dgrad    dx = dy W      (A = dy [T,out], B = W [out,in] as [K,N]:    F,T)
//                 wgrad    dW += dy^T x   (A = dy [T,out] as [K,M], B = x [T,in]:      T,T)
enum GemmEpilogue {
  EPI_STORE = 0,       // C = acc                                   (C in the activation dtype)
  EPI_BIAS = 1,        // C = acc + bias[n]
  EPI_BIAS_RESID = 2,  // C = acc + bias[n] + aux[m,n]
  EPI_BIAS_GELU = 3,   // u = acc + bias[n]; C = gelu(u); C2 = u when C2 != nullptr
  EPI_DGELU = 4,       // C = acc * gelu'(aux[m,n])
  EPI_ACCUM_F32 = 5,   // C (fp32) += acc
  EPI_BIAS_RESID_ENCODE = 6,  // x = acc + bias[n] + aux[m,n] rounded to bf16, stored int8-encoded: C = codes, scales
  // The three below exist in the bf16 MFMA kernels only; gemm_bf16 returns SWARM_ERR_SHAPE (nothing launched)
  // for a problem they cannot take, and the caller then uses the unfused kernels.
  EPI_BIAS_ROPE = 7,          // C = acc + bias[n], columns n < rope_cols rotated pairwise (rotary embedding)
  EPI_DGEGLU = 8,             // aux = u [M, 2*split]: C[m,n] = acc * u[m,split+n] * gelu'(u[m,n]),
                              //                       C[m,split+n] = acc * gelu(u[m,n])        (N = split)
  EPI_BIAS_GEGLU = 9          // B = W1 [2*split, K], N = 2*split: u = acc + bias over gate|up,
                              // C[m,j] = gelu(u[m,j]) * u[m,split+j] (C is [M,split]), C2 = u when C2 != nullptr
};

struct GemmArgs {
  int M, N, K;
  const void* A; int lda; bool a_trans;
  const void* B; int ldb; bool b_trans;
  void* C; int ldc;
  int epilogue;
  const void* bias;        // [N], activation dtype
  const void* aux; int ldaux;   // [M,N] residual or pre-activation, activation dtype
  void* C2; int ldc2;      // optional second output (pre-activation u)
  void* scales;            // EPI_BIAS_RESID_ENCODE: one scale per 64 consecutive elements of C (ldc == N): fp32, or
  bool scales16;           // (scales16) bf16 bit patterns, the codes then dividing by the rounded scale
  const float* rope;       // EPI_BIAS_ROPE: (cos, sin) table [rope_S, rope_dh/2]; row m is at position m % rope_S,
  int rope_S, rope_dh, rope_cols;   // a head spans rope_dh columns, columns >= rope_cols are left alone
  int split;               // EPI_DGEGLU / EPI_BIAS_GEGLU: f, the width of the gate (and of the up) half
  float* splitk_ws;        // optional scratch of splitk_floats floats (>= gemm_splitk_floats(M, N)): lets a product with
  size_t splitk_floats;    // few output tiles and a long K be cut along K (bf16 MFMA kernel only); nullptr: never cut
  float* rowsum;           // EPI_ACCUM_F32 with both operands transposed: rowsum[m] += sum_k A(m,k) (the bias gradient next
                           // to the weight gradient), where gemm_sums_rows says so; ignored elsewhere
  long long* stamps;       // instrumented build only: 16 int64 per workgroup of the 256 x 256 kernel (phase stamps)
};

// Sums over the rows of `parts` matrices [rows, stride] of partial sums, added to up to four vectors: out[2 i + j][c] += sum_q sum_p
// partial[i * set + q * part + p * stride + j * cols + c] (LayerNorm backward: dgamma, dbeta, of one or two norms, of one or
// more applications).
struct ColumnSums {
  const float* partial;
  int rows, cols, n_out;
  int parts;
  ptrdiff_t stride, set, part;
  float* out[4];
  int blocks;         // workgroups that do it: 64 columns of one vector each
};
inline ColumnSums column_sums_of(const float* partial, int rows, int cols, ptrdiff_t stride, float* o0, float* o1) {
  ColumnSums c{partial, rows, cols, o1 ? 2 : 1, 1, stride, 0, 0, {o0, o1, nullptr, nullptr}, 0};
  c.blocks = (cols + 63) / 64 * c.n_out;
  return c;
}
// One of those workgroups, of THREADS: vector o, 64 columns from c0 on x THREADS / 64 row groups, each with eight running sums (rows in a fixed
// assignment, a fixed combine order) that keep as many loads in flight.  Latency bound: with four row groups the 512 partial rows of a
// LayerNorm backward are sixteen dependent rounds of loads, with sixteen groups four.
// (PARTS: of any number of them; else of one.)
template <int THREADS, bool PARTS>
__device__ __forceinline__ void column_sums_of_vector(const ColumnSums& s, int o, int c0, float (*red)[64]) {
  constexpr int RG = THREADS / 64;
  const int l = threadIdx.x & 63, rg = threadIdx.x >> 6, c = c0 + l;
  const float* partial = s.partial + (o >> 1) * s.set + (ptrdiff_t)(o & 1) * s.cols;
  const int all = PARTS ? s.rows * s.parts : s.rows, per = (all + RG - 1) / RG, p0 = rg * per, p1 = min(all, p0 + per);
  float sum = 0.f;
  if (c < s.cols) {
    float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int p = p0; p < p1;) {                    // the rows of this group, part by part
      const int q = PARTS && s.parts > 1 ? p / s.rows : 0, end = min(p1, (q + 1) * s.rows);
      const float* at = partial + q * s.part + (ptrdiff_t)(p - q * s.rows) * s.stride + c;
      for (; p + 8 <= end; p += 8, at += 8 * s.stride) {
#pragma unroll
        for (int u = 0; u < 8; ++u) a[u] += at[u * s.stride];
      }
#pragma unroll
      for (int u = 0; u < 7; ++u)
        if (p + u < end) a[u] += at[u * s.stride];
      p = end;
    }
    sum = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
  }
  red[rg][l] = sum;
  __syncthreads();
  if (rg == 0 && c < s.cols) {
    sum = red[0][l];
#pragma unroll
    for (int g = 1; g < RG; ++g) sum += red[g][l];
    float* out = o == 0 ? s.out[0] : o == 1 ? s.out[1] : o == 2 ? s.out[2] : s.out[3];
    out[c] += sum;
  }
}
// The block-th of s.blocks, in the launch of something else.
template <int THREADS>
__device__ __forceinline__ void column_sums_block(const ColumnSums& s, int block, float (*red)[64]) {
  const int per_out = (s.cols + 63) / 64;
  column_sums_of_vector<THREADS, true>(s, block / per_out, block % per_out * 64, red);
}

// Weight-gradient products over the same token rows (one parameter set's four), as ONE launch of their kernel takes them.
constexpr int kMaxWgrads = 4;
struct WgradProduct {
  const void* A; const void* B;   // [K, M], [K, N]
  float* C;                       // [M, N] += A^T B
  float* rowsum;                  // [M] += column sums of A, or nullptr
  int M, N, lda, ldb, ldc;
  int tiles_m, tiles_n;
};
struct WgradGroup {
  // what a workgroup needs first, together: which product it works on is then two rounds of scalar loads away, not five
  int first[kMaxWgrads];          // product i's workgroups start at first[i], behind the column sums'; none: INT_MAX
  int K, workgroups;
  int stream;                     // bf16: see KArgs
  long long* stamps;              // bf16, instrumented build: see GemmArgs
  WgradProduct q[kMaxWgrads];
  ColumnSums sums;                // done by the workgroups in front of first[0]
};
inline WgradGroup wgrad_group_of(const GemmArgs* g, int n, const ColumnSums* sums, int tile_m, int tile_n) {
  WgradGroup w{};
  if (sums) w.sums = *sums;
  w.K = g[0].K; w.stamps = g[0].stamps;
  w.workgroups = w.sums.blocks;
  for (int i = 0; i < kMaxWgrads; ++i) w.first[i] = 0x7FFFFFFF;
  for (int i = 0; i < n; ++i) {
    WgradProduct& q = w.q[i];
    q.A = g[i].A; q.B = g[i].B; q.C = (float*)g[i].C; q.rowsum = g[i].rowsum; q.M = g[i].M; q.N = g[i].N; q.lda = g[i].lda;
    q.ldb = g[i].ldb; q.ldc = g[i].ldc;
    q.tiles_m = (q.M + tile_m - 1) / tile_m; q.tiles_n = (q.N + tile_n - 1) / tile_n;
    w.first[i] = w.workgroups;
    w.workgroups += (q.tiles_m * q.tiles_n + 7) / 8 * 8;
  }
  return w;
}
// Which product this workgroup (behind the column sums) works on, and which of its tiles.  Workgroups go to the 8 XCDs in turn;
// every XCD gets a contiguous band of every product's tiles, one product after the other, so that all XCDs read the same
// operands at a time (bands of the whole list instead: four gradients of a d_model 4096 block over 8192 tokens 2610 -> 3000
// us).  A product's share of the list is padded to a multiple of 8: tile >= its number means nothing to do.  A product alone whose
// tiles are no such multiple keeps their order (50432 x 1024 over 256 tokens, 788 tiles, in bands 101.9 us, in order 96.1; 20224 x 1024, 316,
// 41.8 and 39.0): the bands' ends would come in a last round of their own.
__device__ __forceinline__ int wgrad_of_block(const WgradGroup& g, int& tile) {
  static_assert(kMaxWgrads == 4, "the sum below");
  const int pid = blockIdx.x, i = (pid >= g.first[1]) + (pid >= g.first[2]) + (pid >= g.first[3]);
  const int tiles = g.q[i].tiles_m * g.q[i].tiles_n, at = pid - g.first[i];
  const bool in_order = (tiles & 7) && g.first[1] == 0x7FFFFFFF;
  tile = in_order ? at : (at & 7) * ((tiles + 7) >> 3) + (at >> 3);
  return i;
}

// Floats of split-K scratch that a bf16 product with an [M, N] output can make use of (0: it is never cut).
size_t gemm_splitk_floats(int M, int N);

// Whether the kernel that this product goes to adds up the rows of A on the way (see GemmArgs::rowsum).
bool gemm_sums_rows(const GemmArgs& g, bool bf16);

swarm_status gemm_f32(const GemmArgs& g, hipStream_t st);
// n <= kMaxWgrads weight-gradient products (both operands transposed, EPI_ACCUM_F32, the same K, row sums wherever rowsum is
// set) in one launch, column sums with them (sums != nullptr); SWARM_ERR_SHAPE (nothing launched) where they are only possible
// one by one.
swarm_status gemm_wgrads(const GemmArgs* g, int n, const ColumnSums* sums, bool bf16, hipStream_t st);
swarm_status gemm_bf16(const GemmArgs& g, hipStream_t st);
// Generic (slow, any shape, either dtype) kernel behind both; `bf16` selects the element type.
swarm_status gemm_generic(const GemmArgs& g, bool bf16, hipStream_t st);

// ------------------------------------------------------------------ LayerNorm / reductions
// y = (x - mean) * rstd * gamma + beta over the last dim d; mean, rstd [T] fp32 are written.
swarm_status layernorm_fwd(const void* x, const void* gamma, const void* beta, void* y, float* mean, float* rstd,
                           int T, int d, float eps, bool bf16, hipStream_t st);
// dx = dres + LN-backward(dy) (dres == nullptr: no residual), dgamma += sum_t dy*xhat, dbeta += sum_t dy.
// `partial` is scratch of layernorm_bwd_scratch_floats(T, d) floats.
size_t layernorm_bwd_scratch_floats(int T, int d);
// dgamma == nullptr: the sums stay in `partial`, [layernorm_bwd_partial_rows(T)][2 d] (dgamma | dbeta), for column_sums.
int layernorm_bwd_partial_rows(int T);
swarm_status column_sums(const ColumnSums& s, hipStream_t st);
// With codes != nullptr dx is not stored: its int8 blockwise encoding is (fused stage-exit encode, bf16 and
// d % 256 == 0 only).
swarm_status layernorm_bwd(const void* dy, const void* x, const float* mean, const float* rstd, const void* gamma,
                           const void* dres, void* dx, float* dgamma, float* dbeta, float* partial, int T, int d,
                           bool bf16, hipStream_t st, int8_t* codes = nullptr, void* scales = nullptr,
                           bool scales16 = false);
// LayerNorm fused with the maxout that follows it in the compression-aware sender (k in {2, 4, 8}; other k:
// SWARM_ERR_SHAPE and nothing launched): z [T, d/k] = maxout_k(LN(x)), the normalised row is never stored.  The
// window maximum is taken on the normalised values rounded to the dtype.  k = -1: mean and rstd only.
swarm_status layernorm_fwd_maxout(const void* x, const void* gamma, const void* beta, void* z, float* mean, float* rstd,
                                  int T, int d, int k, float eps, bool bf16, hipStream_t st);
// Its backward: recomputes the normalised row from x, mean, rstd, routes dz [T, d/k] to the first maximum of every
// window and applies the LayerNorm backward; dgamma, dbeta += as in layernorm_bwd.
swarm_status layernorm_bwd_maxout(const void* dz, const void* x, const float* mean, const float* rstd,
                                  const void* gamma, const void* beta, void* dx, float* dgamma, float* dbeta,
                                  float* partial, int T, int d, int k, bool bf16, hipStream_t st);
// LayerNorm of a row that arrives int8-encoded: xdec receives the decoded row (fused stage-entry decode, bf16 only).
swarm_status layernorm_fwd_decode(const int8_t* codes, const void* scales, void* xdec, const void* gamma,
                                  const void* beta, void* y, float* mean, float* rstd, int T, int d, float eps,
                                  bool bf16, hipStream_t st, bool scales16 = false);
// Stand-alone codec launches (same kernels as the C ABI entry points).
// (scales16: the scales are bf16 bit patterns, as in swarm_codec_encode_s16 / swarm_codec_decode_s16)
swarm_status codec_decode_launch(const int8_t* codes, const void* scales, size_t n, void* tensor, bool bf16,
                                 hipStream_t st, bool scales16 = false);
swarm_status codec_encode_launch(const void* tensor, size_t n, int8_t* codes, void* scales, bool bf16,
                                 hipStream_t st, bool scales16 = false);
// out[n] += sum_t X[t,n]  (X [T,N] in the activation dtype, out fp32); scratch of colsum_scratch_floats floats.
size_t colsum_scratch_floats(int T, int N);
swarm_status colsum_accum(const void* X, int T, int N, float* out, float* partial, bool bf16, hipStream_t st);

// ------------------------------------------------------------------ rotary embedding / GeGLU
// table [S, dh/2] of (cos, sin) fp32 pairs of pos * 10000^(-2i/dh); rope_table_floats(S, dh) floats.
size_t rope_table_floats(int S, int dh);
swarm_status rope_table(float* table, int S, int dh, hipStream_t st);
// Rotates the pairs (2i, 2i+1) of every head of the q and k columns of qkv [T,3d] in place;
// inverse = rotation by the negative angle (applied to dq, dk in the backward pass).
swarm_status rope_apply(void* qkv, const float* table, int T, int S, int d, int dh, bool inverse, bool bf16,
                        hipStream_t st);
// u [T,2f] = gate | up.  g [T,f] = gelu(gate) * up.
swarm_status geglu_fwd(const void* u, void* g, int T, int f, bool bf16, hipStream_t st);
// du [T,2f] = dg * up * gelu'(gate) | dg * gelu(gate).
swarm_status geglu_bwd(const void* dg, const void* u, void* du, int T, int f, bool bf16, hipStream_t st);

// ------------------------------------------------------------------ maxout
// z[t, j] = max_{i<k} a[t, j*k + i]  (a [T, n*k] -> z [T, n]).
swarm_status maxout_fwd(const void* a, void* z, int T, int n, int k, bool bf16, hipStream_t st);
// da[t, j*k + i] = dz[t, j] for the first i with a[t, j*k+i] == max of the window, else 0.
swarm_status maxout_bwd(const void* a, const void* dz, void* da, int T, int n, int k, bool bf16, hipStream_t st);

// ------------------------------------------------------------------ attention
// qkv [T,3d] (q | k | v along the last dim; head h = columns h*dh..), causal, scores scaled by 1/sqrt(dh).
// o [T,d]; lse [B,H,S] fp32 = log-sum-exp of the scaled scores of each query row.
swarm_status attention_fwd(const void* qkv, void* o, float* lse, int B, int S, int H, int dh, bool bf16,
                           hipStream_t st);
// dqkv [T,3d] from do [T,d]; delta [B,H,S] fp32 scratch.
swarm_status attention_bwd(const void* qkv, const void* o, const void* dout, const float* lse, float* delta,
                           void* dqkv, int B, int S, int H, int dh, bool bf16, hipStream_t st);

}  // namespace swarm
