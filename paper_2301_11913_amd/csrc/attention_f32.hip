// fp32 causal attention on the matrix cores (v_mfma_f32_32x32x2_f32), forward and backward, d_head 64 or 128.
//
// What bounds it: fp32 microbatches are small (tens of heads times a few hundred tokens), so a kernel has few blocks of
// work and each is a chain of dependent loads and products.  Tiles are therefore 32 queries (32 keys for dK / dV) and a
// workgroup's four wavefronts share one tile: each takes every fourth block of 32 keys (queries) with sums and softmax
// statistics of its own, and they meet once, in LDS.  Operands go from global memory straight into registers.
//
// One layout serves everything.  A score block is formed with the streamed rows as the first MFMA operand and the
// tile's rows as the second, so lane l holds column l % 32 (its own query, or key) and in register r row
// 8 (r / 4) + 4 (l / 32) + r % 4 of the streamed block; softmax statistics are then per lane.  As second operand of
// the product that follows (P V, dS K, P^T dO, dS^T Q), register r is exactly what MFMA number r wants from the lane
// when the first operand brings the same row: no transpose, no LDS.
//
// Measured against one workgroup per row (attention_naive.hip: forward 20, dK / dV 37, dQ 25 us at 4 sequences of 128
// tokens, 4 heads of 64, and growing with the square of the length): the training pass they are part of 302 -> 257 us.
// With the second product's rows requested beside the first's the forward went from 15 to 8 us (pass 204 -> 189 us).  The
// smallest calls stay with those kernels (attention.hip).
#include "kernels.h"

namespace swarm {
namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16_t;
constexpr int kWaves = 4, kNT = kWaves * 64;

__device__ __forceinline__ float comp(const float4& v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }
__device__ __forceinline__ int row_of(int r, int lg) { return 8 * (r >> 2) + 4 * lg + (r & 3); }
__device__ __forceinline__ f32x16_t zero16() {
  f32x16_t z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  return z;
}

// this lane's row of a [rows, DH] operand: DH values in 8-deep steps, four per half of the wavefront
template <int DH>
__device__ __forceinline__ void load_row(float4 (&f)[DH / 8], const float* row, int lg) {
#pragma unroll
  for (int s = 0; s < DH / 8; ++s) f[s] = *reinterpret_cast<const float4*>(row + 8 * s + 4 * lg);
}
// streamed rows (lane's own: `x`) times the tile's rows (`f`): a 32 x 32 block of dot products over DH
template <int DH>
__device__ __forceinline__ f32x16_t dots(const float4 (&x)[DH / 8], const float4 (&f)[DH / 8]) {
  f32x16_t acc = zero16();
#pragma unroll
  for (int s = 0; s < DH / 8; ++s)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(comp(x[s], c), comp(f[s], c), acc, 0, 0, 0);
  return acc;
}
// A block of 32 streamed rows as first operand of the second product: value (r, c) of a lane is X[first + row_of(r)][32 c +
// l32].  Rows past `last` read row `last` (their weights are zero).  At d_head 64 a kernel requests these together with the
// rows of the first product, whose multiplies and softmax then cover their latency; at 128 they do not fit beside them
// (a pass at 2 x 512 tokens, 4 heads of 128: 652 us against 639).
template <int DH>
constexpr bool kAhead = DH == 64;
template <int DH>
struct Streamed {
  float v[16][DH / 32];
  __device__ __forceinline__ void load(const float* x, size_t ld, int first, int last, int l32, int lg) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float* row = x + (size_t)min(first + row_of(r, lg), last) * ld + l32;
#pragma unroll
      for (int c = 0; c < DH / 32; ++c) v[r][c] = row[32 * c];
    }
  }
  // zeros in the place of rows past `last`: row `last`, which they repeat, may hold a value that is not finite
  __device__ __forceinline__ void drop_past(int first, int last, int lg) {
    if (first + 31 <= last) return;
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
      for (int c = 0; c < DH / 32; ++c) v[r][c] = first + row_of(r, lg) <= last ? v[r][c] : 0.f;
  }
};
// out^T [DH][tile column] += sum over the block's 32 streamed rows of X[row][:] w[row][column]
template <int DH>
__device__ __forceinline__ void accumulate(f32x16_t (&out)[DH / 32], const Streamed<DH>& x, const f32x16_t& w) {
#pragma unroll
  for (int r = 0; r < 16; ++r)
#pragma unroll
    for (int c = 0; c < DH / 32; ++c) out[c] = __builtin_amdgcn_mfma_f32_32x32x2f32(x.v[r][c], w[r], out[c], 0, 0, 0);
}
// On the diagonal some columns must not see some rows.  Their weight is zero, but zero times a value that is not finite is
// not, and a bad token would reach rows that do not depend on it.  The diagonal block is therefore a wavefront's first: if
// its sums are not all finite, they are formed again from the rows that a column sees, one by one.  `rows`: what the block
// streams; scratch: 32 x 33 floats of this wavefront's.  (Fifty to a hundred vector instructions on a finite block.)
template <int DH, typename Seen>
__device__ __forceinline__ void keep_unseen_apart(f32x16_t (&out)[DH / 32], const f32x16_t& w, const float* rows, size_t ld,
                                                  int first, int last, float* scratch, int l32, int lg, Seen&& seen) {
  float z = 0.f;
#pragma unroll
  for (int c = 0; c < DH / 32; ++c)
#pragma unroll
    for (int r = 0; r < 16; ++r) z = fmaf(out[c][r], 0.f, z);
  if (__builtin_amdgcn_ballot_w64(!(z == 0.f)) == 0) return;
#pragma unroll
  for (int c = 0; c < DH / 32; ++c) out[c] = zero16();
#pragma unroll
  for (int r = 0; r < 16; ++r) scratch[row_of(r, lg) * 33 + l32] = w[r];
#pragma unroll 1
  for (int j = 0; j < 32 && first + j <= last; ++j) {
    if (!seen(first + j)) continue;
    const float wj = scratch[j * 33 + l32];
    const float* row = rows + (size_t)(first + j) * ld;
#pragma unroll
    for (int c = 0; c < DH / 32; ++c)
#pragma unroll
      for (int r = 0; r < 16; ++r) out[c][r] = fmaf(wj, row[32 * c + row_of(r, lg)], out[c][r]);
  }
}
// The block of 32 keys that wavefront `wave` takes i-th for query tile qt: every fourth, the diagonal first; and how many.
__device__ __forceinline__ int key_block(int i, int qt, int wave) {
  const bool diagonal = wave == qt % kWaves;
  return diagonal ? (i == 0 ? qt : wave + kWaves * (i - 1)) : wave + kWaves * i;
}
__device__ __forceinline__ int key_blocks(int qt, int wave) { return wave <= qt ? (qt - wave) / kWaves + 1 : 0; }
// The wavefronts' out^T meet 64 of its DH rows at a time: each writes its own to patch[wave] ([64][33]), and
// emit(i, c, row) is called for every column i < columns of the tile and feature c, row = 33 (c % 64) + i.
template <int DH, typename F>
__device__ __forceinline__ void meet(const f32x16_t (&out)[DH / 32], float (*patch)[64 * 33], int wave, int l32, int lg,
                                     int columns, F&& emit) {
#pragma unroll
  for (int c0 = 0; c0 < DH; c0 += 64) {
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int r = 0; r < 16; ++r) patch[wave][(32 * c + row_of(r, lg)) * 33 + l32] = out[c0 / 32 + c][r];
    __syncthreads();
    for (int e = threadIdx.x; e < 64 * columns; e += kNT) emit(e / 64, c0 + e % 64, e % 64 * 33 + e / 64);
  }
}

// one workgroup per (32 queries, head, sequence), long rows first
template <int DH>
__global__ __launch_bounds__(kNT, 2) void attn_f32_fwd_kernel(const float* __restrict__ qkv, float* __restrict__ o,
                                                              float* __restrict__ lse, int S, int H) {
  __shared__ float patch[kWaves][64 * 33];
  __shared__ float stat[2][kWaves][32];
  const int qt = gridDim.x - 1 - blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int d = H * DH;
  const size_t ld = 3 * (size_t)d;
  const float* base = qkv + (size_t)b * S * ld + h * DH;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, lg = lane >> 5;
  const float scale = 1.0f / sqrtf((float)DH);
  const int query = qt * 32 + l32;
  float4 q[DH / 8];
  load_row<DH>(q, base + (size_t)min(query, S - 1) * ld, lg);

  float m = -__FLT_MAX__, l = 0.f;     // finite: the scores of a block may all be -inf
  f32x16_t out[DH / 32];
#pragma unroll
  for (int c = 0; c < DH / 32; ++c) out[c] = zero16();
  for (int i = 0; i < key_blocks(qt, wave); ++i) {
    const int kb = key_block(i, qt, wave);
    float4 k[DH / 8];
    Streamed<DH> v;
    load_row<DH>(k, base + (size_t)min(kb * 32 + l32, S - 1) * ld + d, lg);
    if constexpr (kAhead<DH>) {
      v.load(base + 2 * d, ld, kb * 32, S - 1, l32, lg);
      __builtin_amdgcn_sched_barrier(0);                   // requested here, not where they are used
    }
    f32x16_t s = dots<DH>(k, q);
    float top = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = kb * 32 + row_of(r, lg) <= query ? s[r] * scale : -INFINITY;
      top = fmaxf(top, s[r]);
    }
    top = fmaxf(m, fmaxf(top, __shfl_xor(top, 32, 64)));
    const float old = expf(m - top);
    m = top;
    float sum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = expf(s[r] - m);
      sum += s[r];
    }
    l = l * old + sum + __shfl_xor(sum, 32, 64);
#pragma unroll
    for (int c = 0; c < DH / 32; ++c)
#pragma unroll
      for (int r = 0; r < 16; ++r) out[c][r] *= old;
    if constexpr (!kAhead<DH>) v.load(base + 2 * d, ld, kb * 32, S - 1, l32, lg);
    accumulate<DH>(out, v, s);
    if (kb == qt)
      keep_unseen_apart<DH>(out, s, base + 2 * d, ld, kb * 32, S - 1, patch[wave], l32, lg,
                            [&](int key) __attribute__((always_inline)) { return key <= query; });
  }
  if (lg == 0) {
    stat[0][wave][l32] = m;
    stat[1][wave][l32] = l;
  }
  __syncthreads();
  // each wavefront's weight in its columns' sums, once per column and not once per value (forward at 4 sequences of 128
  // tokens, 4 heads of 64: 16.4 -> 15 us)
  if (threadIdx.x < 32) {
    const int i = threadIdx.x;
    float top = stat[0][0][i];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) top = fmaxf(top, stat[0][w][i]);
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float f = expf(stat[0][w][i] - top);
      sum += f * stat[1][w][i];
      stat[0][w][i] = f;
    }
    stat[1][0][i] = sum;
    // (a row in which every score is -inf has no weights: 0 / 0, and its lse is NaN)
    if (qt * 32 + i < S) lse[((size_t)b * H + h) * S + qt * 32 + i] = sum > 0.f ? top + logf(sum) : NAN;
  }                                                        // (meet begins with a barrier)
  meet<DH>(out, patch, wave, l32, lg, min(32, S - qt * 32), [&](int i, int c, int at) __attribute__((always_inline)) {
    float acc = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) acc += stat[0][w][i] * patch[w][at];
    o[((size_t)b * S + qt * 32 + i) * d + h * DH + c] = acc / stat[1][0][i];
  });
}

// dQ of 32 queries; leaves delta[b,h,i] = sum_c do[i,c] o[i,c] for dK and dV (with a kernel of its own
// for it the backward pass of one sequence of 512, 16 heads of 64 takes 63.7 us, without 61.4)
template <int DH>
__global__ __launch_bounds__(kNT, DH == 64 ? 2 : 1) void attn_f32_dq_kernel(const float* __restrict__ qkv,
                                                                            const float* __restrict__ dout,
                                                                            const float* __restrict__ o,
                                                                            const float* __restrict__ lse,
                                                                            float* __restrict__ delta,
                                                                            float* __restrict__ dqkv, int S, int H) {
  __shared__ float patch[kWaves][64 * 33];
  const int qt = gridDim.x - 1 - blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int d = H * DH;
  const size_t ld = 3 * (size_t)d;
  const float* base = qkv + (size_t)b * S * ld + h * DH;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, lg = lane >> 5;
  const float scale = 1.0f / sqrtf((float)DH);
  const int query = qt * 32 + l32, qrow = min(query, S - 1);
  float4 q[DH / 8], g[DH / 8];
  load_row<DH>(q, base + (size_t)qrow * ld, lg);
  load_row<DH>(g, dout + ((size_t)b * S + qrow) * d + h * DH, lg);
  const float L = lse[((size_t)b * H + h) * S + qrow];
  float D;
  {
    // halves are added to halves all the way, seven or eight roundings deep: a running sum of DH / 2 products would be 18
    float4 out[DH / 8];
    float t[8][4];
    load_row<DH>(out, o + ((size_t)b * S + qrow) * d + h * DH, lg);
#pragma unroll
    for (int c = 0; c < 8; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        t[c][e] = fmaf(comp(out[c], e), comp(g[c], e), 0.f);
        if constexpr (DH == 128) t[c][e] = fmaf(comp(out[c + 8], e), comp(g[c + 8], e), t[c][e]);
      }
#pragma unroll
    for (int half = 4; half >= 1; half /= 2)
#pragma unroll
      for (int c = 0; c < half; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) t[c][e] += t[c + half][e];
#pragma unroll
    for (int e = 0; e < 4; ++e) t[0][e] += __shfl_xor(t[0][e], 32, 64);
    D = (t[0][0] + t[0][2]) + (t[0][1] + t[0][3]);
  }
  if (wave == 0 && lg == 0 && query < S) delta[((size_t)b * H + h) * S + query] = D;
  f32x16_t out[DH / 32];
#pragma unroll
  for (int c = 0; c < DH / 32; ++c) out[c] = zero16();
  for (int i = 0; i < key_blocks(qt, wave); ++i) {
    const int kb = key_block(i, qt, wave);
    const float* krow = base + (size_t)min(kb * 32 + l32, S - 1) * ld + d;
    float4 k[DH / 8], v[DH / 8];
    Streamed<DH> kc;
    load_row<DH>(k, krow, lg);
    load_row<DH>(v, krow + d, lg);
    if constexpr (kAhead<DH>) {
      kc.load(base + d, ld, kb * 32, S - 1, l32, lg);
      __builtin_amdgcn_sched_barrier(0);
    }
    f32x16_t s = dots<DH>(k, q);
    const f32x16_t dp = dots<DH>(v, g);
#pragma unroll
    for (int r = 0; r < 16; ++r)
      s[r] = kb * 32 + row_of(r, lg) <= query ? expf(s[r] * scale - L) * (dp[r] - D) : 0.f;
    if constexpr (!kAhead<DH>) kc.load(base + d, ld, kb * 32, S - 1, l32, lg);
    accumulate<DH>(out, kc, s);
    if (kb == qt)
      keep_unseen_apart<DH>(out, s, base + d, ld, kb * 32, S - 1, patch[wave], l32, lg,
                            [&](int key) __attribute__((always_inline)) { return key <= query; });
  }
  meet<DH>(out, patch, wave, l32, lg, min(32, S - qt * 32), [&](int i, int c, int at) __attribute__((always_inline)) {
    float acc = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) acc += patch[w][at];
    dqkv[((size_t)b * S + qt * 32 + i) * ld + h * DH + c] = acc * scale;
  });
}

// dK and dV of 32 keys
template <int DH>
__global__ __launch_bounds__(kNT) void attn_f32_dkdv_kernel(const float* __restrict__ qkv, const float* __restrict__ dout,
                                                            const float* __restrict__ lse,
                                                            const float* __restrict__ delta, float* __restrict__ dqkv,
                                                            int S, int H) {
  __shared__ float patch[kWaves][64 * 33];
  const int kt = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int d = H * DH;
  const size_t ld = 3 * (size_t)d;
  const float* base = qkv + (size_t)b * S * ld + h * DH;
  const float* gout = dout + (size_t)b * S * d + h * DH;
  const float *L = lse + ((size_t)b * H + h) * S, *D = delta + ((size_t)b * H + h) * S;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, lg = lane >> 5;
  const float scale = 1.0f / sqrtf((float)DH);
  const int key = kt * 32 + l32, krow = min(key, S - 1);
  float4 k[DH / 8], v[DH / 8];
  load_row<DH>(k, base + (size_t)krow * ld + d, lg);
  load_row<DH>(v, base + (size_t)krow * ld + 2 * d, lg);
  f32x16_t dk[DH / 32], dv[DH / 32];
#pragma unroll
  for (int c = 0; c < DH / 32; ++c) dk[c] = dv[c] = zero16();
  const int blocks = (S + 31) / 32;
  for (int qb = kt + wave; qb < blocks; qb += kWaves) {
    const int qrow = min(qb * 32 + l32, S - 1);
    float4 q[DH / 8], g[DH / 8];
    Streamed<DH> gc, qc;
    load_row<DH>(q, base + (size_t)qrow * ld, lg);
    load_row<DH>(g, gout + (size_t)qrow * d, lg);
    if constexpr (kAhead<DH>) {
      gc.load(gout, d, qb * 32, S - 1, l32, lg);
      qc.load(base, ld, qb * 32, S - 1, l32, lg);
    }
    float Lq[16], Dq[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int at = min(qb * 32 + row_of(r, lg), S - 1);
      Lq[r] = L[at];
      Dq[r] = D[at];
    }
    if constexpr (kAhead<DH>) __builtin_amdgcn_sched_barrier(0);
    f32x16_t p = dots<DH>(q, k);
    f32x16_t ds = dots<DH>(g, v);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int query = qb * 32 + row_of(r, lg);
      const bool seen = query >= key && query < S;
      p[r] = seen ? expf(p[r] * scale - Lq[r]) : 0.f;
      ds[r] = seen ? p[r] * (ds[r] - Dq[r]) : 0.f;
    }
    if constexpr (!kAhead<DH>) gc.load(gout, d, qb * 32, S - 1, l32, lg);
    gc.drop_past(qb * 32, S - 1, lg);
    accumulate<DH>(dv, gc, p);
    if constexpr (!kAhead<DH>) qc.load(base, ld, qb * 32, S - 1, l32, lg);
    qc.drop_past(qb * 32, S - 1, lg);
    accumulate<DH>(dk, qc, ds);
    if (qb == kt) {
      auto seen = [&](int query) __attribute__((always_inline)) { return query >= key; };
      keep_unseen_apart<DH>(dv, p, gout, d, qb * 32, S - 1, patch[wave], l32, lg, seen);
      keep_unseen_apart<DH>(dk, ds, base, ld, qb * 32, S - 1, patch[wave], l32, lg, seen);
    }
  }
  auto emit = [&](int part, float factor) __attribute__((always_inline)) {
    return [=](int i, int c, int at) __attribute__((always_inline)) {
      float acc = 0.f;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) acc += patch[w][at];
      dqkv[((size_t)b * S + kt * 32 + i) * ld + part * d + h * DH + c] = acc * factor;
    };
  };
  meet<DH>(dk, patch, wave, l32, lg, min(32, S - kt * 32), emit(1, scale));
  meet<DH>(dv, patch, wave, l32, lg, min(32, S - kt * 32), emit(2, 1.0f));
}

template <int DH>
swarm_status bwd(const float* qkv, const float* o, const float* dout, const float* lse, float* delta, float* dqkv, int B,
                 int S, int H, hipStream_t st) {
  const dim3 grid((S + 31) / 32, H, B);
  hipLaunchKernelGGL(attn_f32_dq_kernel<DH>, grid, dim3(kNT), 0, st, qkv, dout, o, lse, delta, dqkv, S, H);
  hipLaunchKernelGGL(attn_f32_dkdv_kernel<DH>, grid, dim3(kNT), 0, st, qkv, dout, lse, delta, dqkv, S, H);
  return launch_status();
}

}  // namespace

// d_head 64 or 128
swarm_status attention_fwd_f32(const float* qkv, float* o, float* lse, int B, int S, int H, int dh, hipStream_t st) {
  const dim3 grid((S + 31) / 32, H, B);
  if (dh == 64) hipLaunchKernelGGL(attn_f32_fwd_kernel<64>, grid, dim3(kNT), 0, st, qkv, o, lse, S, H);
  else if (dh == 128) hipLaunchKernelGGL(attn_f32_fwd_kernel<128>, grid, dim3(kNT), 0, st, qkv, o, lse, S, H);
  else return SWARM_ERR_SHAPE;
  return launch_status();
}

swarm_status attention_bwd_f32(const float* qkv, const float* o, const float* dout, const float* lse, float* delta,
                               float* dqkv, int B, int S, int H, int dh, hipStream_t st) {
  if (dh == 64) return bwd<64>(qkv, o, dout, lse, delta, dqkv, B, S, H, st);
  if (dh == 128) return bwd<128>(qkv, o, dout, lse, delta, dqkv, B, S, H, st);
  return SWARM_ERR_SHAPE;
}

}  // namespace swarm
