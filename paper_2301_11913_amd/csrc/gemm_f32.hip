// fp32 GEMM on the matrix cores:  C[M,N] (+)= sum_k A(m,k) B(n,k), v_mfma_f32_32x32x2_f32 (fp32 products and sums).
//
// What bounds it: the fp32 products of this library are small (a few hundred to a few thousand rows, 256..4096
// columns), so the time is latency and idle compute units before it is arithmetic.  A wavefront therefore works
// alone on a 32 x 32 (or 64 x 64) block and on its own part of K: it loads its fragments straight from global memory
// into registers (one slice ahead, no LDS and no barrier in the loop, the L1 serves the wavefronts that share rows),
// and the K parts of a block meet once, in LDS, where they are added in a fixed order and the epilogue is applied to
// rows of four.  Lanes 0..31 / 32..63 take k 0..3 / 4..7 of an 8-deep step with one 16-byte load each and feed four
// MFMAs from it: which k meets which MFMA is free as long as both operands agree.
//
// Measured against the LDS-tiled FMA kernel of gemm_generic.hip, whose 64 x 64 tiles put 32..128 workgroups on 256
// compute units: one training pass of a d_model 256 block on 4 x 128 tokens 1712 -> 302 us, four applications of a
// d_model 768 rotary + GeGLU block on 384 tokens 14.38 -> 3.09 ms, a d_model 3072 maxout boundary on 352 tokens 1034 ->
// 251 us; distance from 64-bit sums 7e-7 -> 4e-7 (shorter chains of additions).
#include "gelu.h"
#include "kernels.h"

namespace swarm {
namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16_t;

// Four consecutive k of one row (or column) of an operand: k0 + 4 g + {0..3}, g = lane / 32.
template <bool TRANS>
struct Operand {
  const float* p;   // TRANS: column `row` of [K, ld]; else row `row` of [.., ld]
  size_t ld;
  __device__ __forceinline__ void init(const float* base, int ld_, int row) {
    ld = (size_t)ld_;
    p = TRANS ? base + row : base + (size_t)row * ld;
  }
  __device__ __forceinline__ float4 load(int k) const {
    if constexpr (!TRANS) return *reinterpret_cast<const float4*>(p + k);
    else {
      const float* q = p + (size_t)k * ld;
      return make_float4(q[0], q[ld], q[2 * ld], q[3 * ld]);
    }
  }
  // the same with everything at and behind kend replaced by zero (and not read)
  __device__ __forceinline__ float4 load_guarded(int k, int kend) const {
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int kk = min(k + i, kend - 1);
      const float x = TRANS ? p[(size_t)kk * ld] : p[kk];
      v[i] = k + i < kend ? x : 0.f;
    }
    return make_float4(v[0], v[1], v[2], v[3]);
  }
};

__device__ __forceinline__ float comp(const float4& v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }

// What a kernel is launched with.  GROUP: several weight gradients in a launch; one alone has a kernel of its own, since finding its
// place in a group's arguments takes 0.2 us (1024 x 512 over 128 tokens 4.60 -> 4.83).
template <bool GROUP> struct F32Args { typedef GemmArgs type; };
template <> struct F32Args<true> { typedef WgradGroup type; };

// A workgroup: WM x WN x WK wavefronts; wavefront (wm, wn, wk) multiplies block (wm, wn) of 32 FM x 32 FN over the
// wk-th part of K.
template <int FM, int FN, int WM, int WN, int WK, bool A_T, bool B_T, bool GROUP>
__global__ __launch_bounds__(WM* WN* WK * 64) void gemm_f32_kernel(typename F32Args<GROUP>::type args, int tiles_m, int tiles_n) {
  static_assert(!GROUP || (A_T && B_T), "groups are of weight gradients");
  constexpr int TM = 32 * FM * WM, TN = 32 * FN * WN, NT = WM * WN * WK * 64;
  constexpr int U = FM * FN == 1 ? 4 : 2;      // 8-deep steps per slice: 32 registers of fragments in flight
  constexpr int PITCH = TN + 4;
  extern __shared__ __attribute__((aligned(16))) float lds[];

  // contiguous bands of tiles per XCD, walked in groups of 8 tile rows
  int pid;
  GemmArgs g;
  if constexpr (GROUP) {
    if ((int)blockIdx.x < args.first[0]) {
      column_sums_block<NT>(args.sums, blockIdx.x, reinterpret_cast<float (*)[64]>(lds));
      return;
    }
    const WgradProduct& q = args.q[wgrad_of_block(args, pid)];
    g = GemmArgs{};
    g.M = q.M; g.N = q.N; g.K = args.K; g.A = q.A; g.lda = q.lda; g.B = q.B; g.ldb = q.ldb; g.C = q.C; g.ldc = q.ldc;
    g.epilogue = EPI_ACCUM_F32; g.rowsum = q.rowsum;
    tiles_m = q.tiles_m; tiles_n = q.tiles_n;
    if (pid >= tiles_m * tiles_n) return;
  } else {
    g = args;
    pid = blockIdx.x;
    const int ntiles = tiles_m * tiles_n;
    if ((ntiles & 7) == 0) pid = (pid & 7) * (ntiles >> 3) + (pid >> 3);
  }
  const int per_group = 8 * tiles_n, first = pid / per_group * 8, gsz = min(tiles_m - first, 8);
  const int m0 = (first + pid % per_group % gsz) * TM, n0 = pid % per_group / gsz * TN;

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wk = wave % WK, wn = wave / WK % WN, wm = wave / WK / WN;
  const int l32 = lane & 31, lg = lane >> 5;

  // Weight gradients of 32 x 32 blocks have a second set of sums, for every other MFMA: with K dealt to four, chains of additions
  // are then no longer than with K dealt to eight, which several products in a launch have too many tiles for (d_model 256, 512
  // tokens, distance from 64 bits 2.1e-7 -> 1.5e-7).
  constexpr bool TWO = A_T && FM * FN == 1;
  f32x16_t acc[FM][FN], odd;
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  if constexpr (TWO) odd = acc[0][0];

  // rows and columns past the end read the last one; what they produce is not stored
  Operand<A_T> a[FM];
  Operand<B_T> b[FN];
#pragma unroll
  for (int i = 0; i < FM; ++i) a[i].init((const float*)g.A, g.lda, min(m0 + (wm * FM + i) * 32 + l32, g.M - 1));
#pragma unroll
  for (int j = 0; j < FN; ++j) b[j].init((const float*)g.B, g.ldb, min(n0 + (wn * FN + j) * 32 + l32, g.N - 1));

  // Sum of this lane's values of A (a row's bias gradient beside its weight gradient).  In doubles, one addition per 8-deep
  // step: the rows of shared layers make one K of up to 2^22, where a running fp32 sum loses (32768 rows of mean 1 5.9e-7).
  double rsum[FM];
#pragma unroll
  for (int i = 0; i < FM; ++i) rsum[i] = 0.0;
  const int part = ((g.K + 7) / 8 + WK - 1) / WK * 8;
  const int kbeg = wk * part, kend = min(g.K, kbeg + part);
  auto multiply = [&](const float4 (&fa)[FM], const float4 (&fb)[FN]) __attribute__((always_inline)) {
    if constexpr (A_T) {
#pragma unroll
      for (int i = 0; i < FM; ++i) rsum[i] += (double)((fa[i].x + fa[i].y) + (fa[i].z + fa[i].w));
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
        {
          f32x16_t& sum = TWO && (c & 1) ? odd : acc[i][j];
          sum = __builtin_amdgcn_mfma_f32_32x32x2f32(comp(fa[i], c), comp(fb[j], c), sum, 0, 0, 0);
        }
  };
  const int nfull = max(kend - kbeg, 0) / (8 * U);
  if (nfull > 0) {
    float4 fa[U][FM], fb[U][FN];
    auto load = [&](int k, float4 (&va)[U][FM], float4 (&vb)[U][FN]) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int i = 0; i < FM; ++i) va[u][i] = a[i].load(k + 8 * u + 4 * lg);
#pragma unroll
        for (int j = 0; j < FN; ++j) vb[u][j] = b[j].load(k + 8 * u + 4 * lg);
      }
    };
    load(kbeg, fa, fb);
    for (int s = 1; s <= nfull; ++s) {
      float4 na[U][FM], nb[U][FN];
      load(kbeg + min(s, nfull - 1) * 8 * U, na, nb);     // the last pass requests its own slice again
      __builtin_amdgcn_sched_barrier(0);                  // requested before the multiplies, not where they are used
#pragma unroll
      for (int u = 0; u < U; ++u) multiply(fa[u], fb[u]);
#pragma unroll
      for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int i = 0; i < FM; ++i) fa[u][i] = na[u][i];
#pragma unroll
        for (int j = 0; j < FN; ++j) fb[u][j] = nb[u][j];
      }
    }
  }
  for (int k = kbeg + nfull * 8 * U; k < kend; k += 8) {
    float4 fa[FM], fb[FN];
#pragma unroll
    for (int i = 0; i < FM; ++i) fa[i] = a[i].load_guarded(k + 4 * lg, kend);
#pragma unroll
    for (int j = 0; j < FN; ++j) fb[j] = b[j].load_guarded(k + 4 * lg, kend);
    multiply(fa, fb);
  }

  if constexpr (TWO) acc[0][0] += odd;
  // acc[i][j][r] is the element (32 i + 8 (r / 4) + 4 lg + r % 4, 32 j + l32) of the block
  float* mine = lds + wk * TM * PITCH + wm * 32 * FM * PITCH + wn * 32 * FN;
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) mine[(32 * i + 8 * (r >> 2) + 4 * lg + (r & 3)) * PITCH + 32 * j + l32] = acc[i][j][r];
  const bool sum_rows = A_T && g.rowsum && n0 == 0;
  // into the columns behind the tile's, still in doubles: K parts rounded one by one leave the sums 6.2e-8 from 64 bits, so 4.6e-8
  if (sum_rows && wn == 0) {
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const double s = rsum[i] + __shfl_xor(rsum[i], 32, 64);
      if (lg == 0) *reinterpret_cast<double*>(&mine[(32 * i + l32) * PITCH + TN]) = s;
    }
  }
  __syncthreads();
  if (sum_rows && threadIdx.x < TM && m0 + (int)threadIdx.x < g.M) {
    double s = g.rowsum[m0 + threadIdx.x];
#pragma unroll
    for (int w = 0; w < WK; ++w) s += *reinterpret_cast<const double*>(&lds[(w * TM + threadIdx.x) * PITCH + TN]);
    g.rowsum[m0 + threadIdx.x] = (float)s;
  }
  for (int e = threadIdx.x; e < TM * TN / 4; e += NT) {
    const int rl = e / (TN / 4), cl = e % (TN / 4) * 4;
    const int row = m0 + rl, col = n0 + cl;
    if (row >= g.M || col >= g.N) continue;              // N % 4 == 0: all four columns or none
    float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < WK; ++w) {
      const float4 x = *reinterpret_cast<const float4*>(lds + w * TM * PITCH + rl * PITCH + cl);
      v[0] += x.x; v[1] += x.y; v[2] += x.z; v[3] += x.w;
    }
    float* c = (float*)g.C + (size_t)row * g.ldc + col;
    float bias[4], aux[4];
    auto get = [](float (&d)[4], const float* s) __attribute__((always_inline)) {
      const float4 t = *reinterpret_cast<const float4*>(s);
      d[0] = t.x; d[1] = t.y; d[2] = t.z; d[3] = t.w;
    };
    auto put = [](float* d, const float (&s)[4]) __attribute__((always_inline)) {
      *reinterpret_cast<float4*>(d) = make_float4(s[0], s[1], s[2], s[3]);
    };
    if (g.epilogue == EPI_BIAS || g.epilogue == EPI_BIAS_RESID || g.epilogue == EPI_BIAS_GELU) {
      get(bias, (const float*)g.bias + col);
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] += bias[q];
    }
    if (g.epilogue == EPI_BIAS_RESID || g.epilogue == EPI_DGELU) get(aux, (const float*)g.aux + (size_t)row * g.ldaux + col);
    if (g.epilogue == EPI_BIAS_RESID) {
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] += aux[q];
    } else if (g.epilogue == EPI_BIAS_GELU) {
      if (g.C2) put((float*)g.C2 + (size_t)row * g.ldc2 + col, v);
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = gelu_f(v[q]);
    } else if (g.epilogue == EPI_DGELU) {
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] *= gelu_grad_f(aux[q]);
    } else if (g.epilogue == EPI_ACCUM_F32) {
      get(aux, c);
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] += aux[q];
    }
    put(c, v);
  }
}

template <int FM, int FN, int WM, int WN, int WK, bool A_T, bool B_T, bool GROUP = false>
swarm_status launch(const typename F32Args<GROUP>::type& g, int tm, int tn, int tiles, hipStream_t st) {
  constexpr int TM = 32 * FM * WM, TN = 32 * FN * WN;
  constexpr size_t lds_bytes = (size_t)WK * TM * (TN + 4) * sizeof(float);
  auto kern = gemm_f32_kernel<FM, FN, WM, WN, WK, A_T, B_T, GROUP>;
  if constexpr (lds_bytes > 64 * 1024) {
    static LdsOptIn opted;   // per instantiation
    if (lds_opt_in((const void*)kern, lds_bytes, opted) != SWARM_OK) return SWARM_ERR_LAUNCH;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)tiles), dim3(WM * WN * WK * 64), lds_bytes, st, g, tm, tn);
  return launch_status();
}

// n > 1: weight gradients
template <int FM, int FN, int WM, int WN, int WK>
swarm_status launch_layout(const GemmArgs* g, int n, const ColumnSums* sums, hipStream_t st) {
  constexpr int TM = 32 * FM * WM, TN = 32 * FN * WN;
  if (n > 1 || sums) {
    const WgradGroup w = wgrad_group_of(g, n, sums, TM, TN);
    return launch<FM, FN, WM, WN, WK, true, true, true>(w, 0, 0, w.workgroups, st);
  }
  const int tm = (g->M + TM - 1) / TM, tn = (g->N + TN - 1) / TN;
  if (g->a_trans) return launch<FM, FN, WM, WN, WK, true, true>(*g, tm, tn, tm * tn, st);
  if (!g->b_trans) return launch<FM, FN, WM, WN, WK, false, false>(*g, tm, tn, tm * tn, st);
  return launch<FM, FN, WM, WN, WK, false, true>(*g, tm, tn, tm * tn, st);
}

}  // namespace

bool gemm_f32_takes(const GemmArgs& g) {
  auto al16 = [](const void* q) { return ((uintptr_t)q & 15) == 0; };
  auto row_ok = [&](const void* q, int ld) { return !q || (al16(q) && ld % 4 == 0); };
  // rows of four in the epilogue, 16-byte fragment loads where k is contiguous
  if (g.a_trans && (!g.b_trans || g.epilogue != EPI_ACCUM_F32)) return false;
  return g.epilogue <= EPI_ACCUM_F32 && g.N % 4 == 0 && al16(g.bias) &&
         row_ok(g.C, g.ldc) && row_ok(g.aux, g.ldaux) && row_ok(g.C2, g.ldc2) &&
         (g.a_trans || (g.K % 8 == 0 && row_ok(g.A, g.lda))) &&
         (g.b_trans || (g.K % 8 == 0 && row_ok(g.B, g.ldb)));
}

static swarm_status launch_by_size(const GemmArgs* g, int n, const ColumnSums* sums, hipStream_t st) {
  auto tiles = [&](int t) {
    long sum = 0;
    for (int i = 0; i < n; ++i) sum += (long)((g[i].M + t - 1) / t) * ((g[i].N + t - 1) / t);
    return sum;
  };
  // 64 x 64 per wavefront loads half the fragments per flop of 32 x 32, and K dealt to the four wavefronts of a workgroup makes a
  // 64 x 64 tile of it: four times as many workgroups as 128 x 128 tiles with K whole.  Measured in turn, us, on 64 x 64 tiles with K
  // dealt | 32 x 32 with K dealt | 64 x 64 of four 32 x 32 with K whole | 128 x 128 with K whole:
  //   forward         1292 x 3072, K = 768 (1008 tiles of 64)  62 | 105 | 95 | 108      2048 x 1024, K = 4096  143 | 242 | 231 | 325
  //                   1292 x 768, K = 3072 (252)  65 | 99 | 92 | 251                    381 x 2048, K = 512 (192)  14.1 | 16.5 | 18 | 44
  //                   512 x 1024, K = 256 (128)  9.3 | 8.1 | 11 | 25                    2048 x 4096, K = 1024 (2048)  152 | - | - | 143
  //   data gradient   the lanes of a load share rows already, so 32 x 32 holds out longer: (252) 66 | 75 | 90, (192) 13.9 | 12.3 | 16
  //   weight gradient the four of d_model 768 over 1292 tokens  182 | 207 | 212; 1024 over 2048  635 | 753 | 743 | 638;
  //                   256 over 512 (192)  15.9 | 13.5 | 18.7
  if (tiles(128) >= (g->a_trans ? 1024 : 448)) return launch_layout<2, 2, 2, 2, 1>(g, n, sums, st);
  if (tiles(64) >= (g->a_trans ? 400 : g->b_trans ? 240 : 160)) return launch_layout<2, 2, 1, 1, 4>(g, n, sums, st);
  // One 32 x 32 block per workgroup, its K dealt to so many wavefronts that every SIMD has one.
  if (tiles(32) >= 256) return launch_layout<1, 1, 1, 1, 4>(g, n, sums, st);
  return launch_layout<1, 1, 1, 1, 8>(g, n, sums, st);
}

swarm_status gemm_f32(const GemmArgs& g, hipStream_t st) {
  if (!gemm_f32_takes(g)) return gemm_generic(g, false, st);
  return launch_by_size(&g, 1, nullptr, st);
}

swarm_status gemm_f32_wgrads(const GemmArgs* g, int n, const ColumnSums* sums, hipStream_t st) {
  for (int i = 0; i < n; ++i)
    if (!gemm_f32_takes(g[i])) return SWARM_ERR_SHAPE;
  return launch_by_size(g, n, sums, st);
}

}  // namespace swarm
