// bf16 MFMA GEMM for products with few output tiles and for ragged ones:  C[M,N] (+)= sum_k A(m,k) B(n,k).
//
// What bounds such a product is latency: a launch of 32..256 workgroups (or a ragged one of more, whose 135 KB workgroups
// still run one to a unit) leaves every compute unit with one, and what that one waits for between two slices of K (about a
// microsecond from memory) is longer than what it multiplies in
// one.  So a workgroup keeps NS slices in LDS, NS - 1 of them in flight, and divides K as well as the tile: WM x WN x WK
// wavefronts, each multiplying a 64 x 64 block (or, for the fewest tiles, 16 or 32 rows of one) over its own 32 of the 32 * WK
// values of k in a slice.  That keeps the LDS bytes per flop of a 64 x 64 block (16 fragment reads for 32 MFMAs) on a tile as small
// as 64 x 64, and gives a 128 x 128 tile eight wavefronts, two per SIMD.  The WK partial blocks meet once, in LDS, and are added
// in index order; the epilogue then runs on rows of eight columns.
//
// Loads are buffer loads into LDS with the operand's exact size in the descriptor: what lies behind its last row reads
// as zero, so a ragged M or N costs nothing in the loop and only the stores are guarded.  The descriptor moves along K
// with scalar arithmetic; a lane's offset inside a slice never changes.  LDS layouts, swizzles and the transpose reads
// are those of gemm_bf16_dma.hip.
//
// One barrier per slice: behind it slice k + 1 is in LDS for everyone and everyone's fragments of slice k are in
// registers, so the reads of k + 1 and the refill of k's stage are issued there and the multiplies of k cover both.
// Measured against what these products ran on before, 128 x 128 tiles with two LDS stages (whole tiles) and a
// register-staged kernel (ragged ones): forward of one 512-token sequence at d_model 1024 119 -> 71 us, a training pass
// at d_model 768 on 5 x 333 tokens 660 -> 463 us, two d_model 1024 blocks on 4096 tokens 1954 -> 1504 us.
#include "gemm_bf16_common.h"

namespace swarm {
namespace {

typedef uint32_t u32x4_kw __attribute__((ext_vector_type(4)));

// One operand's tile: BR rows (of C's rows or columns) x BK k per slice.
//   !TRANS: BK / 64 sub-tiles [BR][64 k], 16-byte chunks of a row XOR-ed with row & 7
//    TRANS: [BK k][BR], chunks of a k-row XOR-ed so that the 8 k-rows x 32 bytes of one transpose-read pass hit all banks
template <int BR, int BK, int NW, bool TRANS>
struct KwOperand {
  static constexpr int NI = BR * BK / 512 / NW;   // 1 KiB load instructions per wavefront and slice
  static constexpr int BYTES = BR * BK * 2;
  const char* base;
  size_t step;          // bytes from slice to slice
  size_t left;          // bytes from `base` to the end of the operand
  int slices;           // still to come; behind the last one nothing is read and zeros arrive
  uint32_t off[NI];     // this lane's offset in every load of a slice
  uint32_t frag[4];     // this lane's LDS address of the four 16-row fragments of its block (relative to the tile)

  static __device__ __forceinline__ int swz(int krow) {
    return BR == 64 ? 4 * ((krow >> 1) & 1) ^ 2 * ((krow >> 3) & 1) : 4 * (krow & 3) ^ 2 * ((krow >> 3) & 1);
  }

  // rows r0 .. of an operand of `rows` rows and `kdim` k values; k starts at 0.  glu_split: see EPI_BIAS_GEGLU (B = W1,
  // every 64 tile rows are 32 gate rows and the 32 up rows of the same features; r0 counts features)
  __device__ __forceinline__ void init(const bf16_raw* p, int ld, int rows, int kdim, int r0, int glu_split, int wave,
                                       int lane, int block_row, int wk) {
    slices = (kdim + BK - 1) / BK;
    if constexpr (!TRANS) {
      base = reinterpret_cast<const char*>(p + (size_t)r0 * ld);
      left = ((size_t)(rows - 1 - r0) * ld + kdim) * 2;
      step = BK * 2;
#pragma unroll
      for (int t = 0; t < NI; ++t) {
        const int q = wave + t * NW, sub = q / (BR / 8), row = q % (BR / 8) * 8 + lane / 8;
        const int src = glu_split ? 32 * (row >> 6) + (row & 31) + ((row & 32) ? glu_split : 0) : row;
        off[t] = ((uint32_t)src * (uint32_t)ld + 64u * sub + 8u * ((lane % 8) ^ (row & 7))) * 2u;
      }
      const int l16 = lane & 15, c = 4 * (wk & 1) + (lane >> 4);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        frag[i] = (uint32_t)((wk >> 1) * BR * 64 + (block_row + 16 * i + l16) * 64 + 8 * (c ^ (l16 & 7))) * 2u;
    } else {
      base = reinterpret_cast<const char*>(p + r0);
      left = ((size_t)(kdim - 1) * ld + rows - r0) * 2;
      step = (size_t)BK * ld * 2;
      constexpr int CPR = BR / 8;
#pragma unroll
      for (int t = 0; t < NI; ++t) {
        const int krow = (wave + t * NW) * (64 / CPR) + lane / CPR;
        off[t] = ((uint32_t)krow * (uint32_t)ld + 8u * ((lane % CPR) ^ swz(krow))) * 2u;
      }
      const int l16 = lane & 15, krow = 32 * wk + 8 * (lane >> 4) + (l16 >> 2);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int col = block_row + 16 * i + 4 * (l16 & 3);
        frag[i] = (uint32_t)(krow * BR + 8 * ((col >> 3) ^ swz(krow)) + (col & 4)) * 2u;
      }
    }
  }
  // the t-th of this wavefront's loads of the next slice into the tile at `lds`
  __device__ __forceinline__ void issue_one(bf16_raw* lds, int wave, int t) const {
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass knows neither the descriptor type nor its builtins
    const uint32_t records = slices <= 0 ? 0u : left > 0xFFFFFFF0u ? 0xFFFFFFF0u : (uint32_t)left;
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), (short)0, (int)records, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        r, (__attribute__((address_space(3))) void*)(lds + (wave + t * NW) * 512), 16, off[t], 0, 0, 0);
#endif
  }
  // behind the last of them
  __device__ __forceinline__ void next_slice() {
    if (--slices > 0) {
      base += step;
      left -= step;
    }
  }
  // Fragment i of the slice whose tile starts at LDS byte `tile`.  Plain instructions: the compiler takes every load into
  // LDS as a possible writer of what an LDS read of its own returns and would wait for all of them.  The caller waits.
  __device__ __forceinline__ u32x4_kw read(uint32_t tile, int i) const {
    const uint32_t addr = tile + frag[i];
    if constexpr (!TRANS) {
      u32x4_kw v;
      asm volatile("ds_read_b128 %0, %1" : "=v"(v) : "v"(addr) : "memory");
      return v;
    } else {
      uint2 a, b;
      // k-rows krow and krow + 4: the swizzle depends on bits 0, 1 and 3 of krow, which the two share
      asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(a) : "v"(addr) : "memory");
      asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(b) : "v"(addr), "n"(8 * BR) : "memory");
      const u32x4_kw v = {a.x, a.y, b.x, b.y};
      return v;
    }
  }
};

template <int N>
__device__ __forceinline__ void kw_wait_loads() {   // at most N loads of this wavefront still on their way
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// NT: the bf16 epilogues' global accesses are non-temporal (see KArgs::stream; a kernel of its own, since two copies of the
// epilogue in one cost the small launches 0.2..0.5 us of instruction fetch).
template <int FM, int WM, int WN, int WK, int NS, bool A_T, bool B_T, bool NT>
__global__ __launch_bounds__(WM* WN* WK * 64) void gemm_bf16_kw_kernel(typename LaunchArgs<A_T>::type args) {
  constexpr int NW = WM * WN * WK, NTHR = NW * 64;
  constexpr int BM = 16 * FM * WM, BN = 64 * WN, BK = 32 * WK;
  static_assert(FM == 4 || !A_T, "weight gradients have enough tiles");
  static_assert(BK % 64 == 0 && BM * BK % (512 * NW) == 0 && BN * BK % (512 * NW) == 0, "loads split evenly");
  extern __shared__ __attribute__((aligned(1024))) bf16_raw lds[];

  int tile_m, tile_n;
  KArgs p;
  if constexpr (A_T) {
    if ((int)blockIdx.x < args.first[0]) {
      column_sums_block<NTHR>(args.sums, blockIdx.x, reinterpret_cast<float (*)[64]>(lds));
      return;
    }
    if (!tile_of_block(args, p, tile_m, tile_n)) return;
  } else {
    p = args;
    tile_of_block(p, tile_m, tile_n);
  }
  const int glu = (!B_T && p.epilogue == EPI_BIAS_GEGLU) ? p.split : 0;
  const int m0 = tile_m * BM, n0 = glu ? tile_n * (BN / 2) : tile_n * BN;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wk = wave % WK, wn = wave / WK % WN, wm = wave / WK / WN;

  KwOperand<BM, BK, NW, A_T> a;
  KwOperand<BN, BK, NW, B_T> b;
  a.init(p.A, p.lda, p.M, p.K, m0, 0, wave, lane, wm * 16 * FM, wk);
  b.init(p.B, p.ldb, glu ? 2 * glu : p.N, p.K, n0, glu, wave, lane, wn * 64, wk);
  constexpr int IPW = decltype(a)::NI + decltype(b)::NI;
  constexpr int STAGE = a.BYTES + b.BYTES;
  auto issue_one = [&](int stage, int t) __attribute__((always_inline)) {      // A's, then B's
    bf16_raw* s = lds + stage * (STAGE / 2);
    if (t < a.NI) a.issue_one(s, wave, t);
    else b.issue_one(s + a.BYTES / 2, wave, t - a.NI);
  };
  auto next_slice = [&]() __attribute__((always_inline)) {
    a.next_slice();
    b.next_slice();
  };

  f32x4 acc[FM][4];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;

  // Row sums of A (the bias gradient beside a weight gradient): one more MFMA against a column of ones per fragment row,
  // each of the four in another column of tiles (tile_n modulo four), by the first column of wavefronts.  Every 64 slices they
  // are moved to sums in doubles: a gradient over shared layers has up to 2^22 rows, and one running fp32 sum loses with their
  // number (131105 rows of mean 1: 3.4e-7 off, against 6e-8 of the column sum that this replaces).  It costs a product about
  // 0.4 us (768 x 3072, K = 1665: 21.7 -> 22.1); kept in LDS by the lanes that hold a sum, it costs the same.
  f32x4 rsum[4];
  double total[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) { rsum[i][r] = 0.f; total[i][r] = 0.0; }
  int sum_rows = 0;   // bit i: fragment row i is summed here
  if constexpr (A_T) {
    if (p.rowsum)
      for (int i = 0; i < 4; ++i) sum_rows |= (i % p.tiles_n == tile_n) << i;
  }
  const u32x4_kw ones = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};

  constexpr int NM = 4 * FM, NR = FM + 4;      // multiplies and fragment reads of a wavefront and slice
  struct Frags { u32x4_kw a[FM], b[4]; };
  auto read_one = [&](int stage, Frags& f, int n) __attribute__((always_inline)) {
    const uint32_t tile = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)lds + (uint32_t)stage * STAGE;
    if (n < FM) f.a[n % FM] = a.read(tile, n % FM);
    else f.b[(n - FM) & 3] = b.read(tile + a.BYTES, (n - FM) & 3);
  };
  // every fragment read so far has returned; nothing that uses one moves in front of this
  auto arrived = [&](Frags& f) __attribute__((always_inline)) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int i = 0; i < FM; ++i) asm volatile("" : "+v"(f.a[i])::"memory");
#pragma unroll
    for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(f.b[j])::"memory");
  };

#pragma unroll
  for (int s = 0; s < NS; ++s) {
#pragma unroll
    for (int t = 0; t < IPW; ++t) issue_one(s, t);
    next_slice();
  }
  kw_wait_loads<(NS - 1) * IPW>();
  __builtin_amdgcn_s_barrier();
  Frags f0, f1;
#pragma unroll
  for (int n = 0; n < NR; ++n) read_one(0, f0, n);

  // A unit takes in 64 bytes per clock, 512 clocks for a slice of 32 KB, as long as the multiplies and the fragment reads of a
  // slice together: so the loads are spread over the multiplies, the reads over the first half of them.  Requested in front of
  // them, a wavefront waits for its loads to be taken before it multiplies (K = 4096 on one 64 x 64 tile 16.7 us, of which 11.9
  // without the multiplies and reads; spread 13.2).
  int now = 0;      // stage of the current slice
  auto step = [&](Frags& cur, Frags& next, int k) __attribute__((always_inline)) {
    // this wavefront's fragments have arrived, and its part of the next slice
    arrived(cur);
    kw_wait_loads<(NS - 2) * IPW>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    const int after = now + 1 == NS ? 0 : now + 1;
    if (k < p.K) {   // K of a k-contiguous operand is a multiple of 32: a wavefront's 32 are all in or all out
#pragma unroll
      for (int n = 0; n < NM; ++n) {
        const int i = n >> 2, j = n & 3;
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, cur.a[i]),
                                                            __builtin_bit_cast(bf16x8, cur.b[j]), acc[i][j], 0, 0, 0);
        if (n < NM / 2) {
#pragma unroll
          for (int r = n * NR / (NM / 2); r < (n + 1) * NR / (NM / 2); ++r) read_one(after, next, r);
        }
#pragma unroll
        for (int t = n * IPW / NM; t < (n + 1) * IPW / NM; ++t) issue_one(now, t);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (A_T) {
        if (sum_rows && wn == 0) {
#pragma unroll
          for (int i = 0; i < FM; ++i)
            if (sum_rows & (1 << i))
              rsum[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, cur.a[i]),
                                                                __builtin_bit_cast(bf16x8, ones), rsum[i], 0, 0, 0);
        }
      }
    } else {
#pragma unroll
      for (int n = 0; n < NR; ++n) read_one(after, next, n);
#pragma unroll
      for (int t = 0; t < IPW; ++t) issue_one(now, t);
    }
    next_slice();
    now = after;
    __builtin_amdgcn_sched_barrier(0);
  };
  const int KT = (p.K + BK - 1) / BK;
  for (int kt = 0; kt < KT; kt += 2) {
    step(f0, f1, kt * BK + 32 * wk);
    step(f1, f0, (kt + 1) * BK + 32 * wk);
    if constexpr (A_T) {
      if (sum_rows && (kt & 62) == 62) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) { total[i][r] += (double)rsum[i][r]; rsum[i][r] = 0.f; }
      }
    }
  }
  // the fragments requested last are not used, but have to arrive before their registers are
  arrived(f0);
  kw_wait_loads<0>();
  __builtin_amdgcn_s_barrier();   // the stages are free: the partial blocks take their place

  constexpr int PITCH = BN + 4;
  float* sums = reinterpret_cast<float*>(lds);
  {
    float* mine = sums + (wk * BM + wm * 16 * FM) * PITCH + wn * 64;
    const int l16 = lane & 15, q = lane >> 4;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) mine[(16 * i + 4 * q + r) * PITCH + 16 * j + l16] = acc[i][j][r];
    if (A_T && sum_rows && wn == 0 && l16 == 0) {     // into the column behind the tile's
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) mine[(16 * i + 4 * q + r) * PITCH + BN] = (float)(total[i][r] + (double)rsum[i][r]);
    }
  }
  __syncthreads();
  if (A_T && sum_rows) {
    const int rl = threadIdx.x;
    if (rl < BM && m0 + rl < p.M && (sum_rows >> (rl % 64 / 16) & 1)) {
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < WK; ++w) s += sums[(w * BM + rl) * PITCH + BN];
      p.rowsum[m0 + rl] += s;
    }
  }
  auto sum8 = [&](int rl, int cl, float (&x)[8]) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = 0.f;
#pragma unroll
    for (int w = 0; w < WK; ++w) {
      const float* s = sums + (w * BM + rl) * PITCH + cl;
      const float4 u = *reinterpret_cast<const float4*>(s), v = *reinterpret_cast<const float4*>(s + 4);
      x[0] += u.x; x[1] += u.y; x[2] += u.z; x[3] += u.w; x[4] += v.x; x[5] += v.y; x[6] += v.z; x[7] += v.w;
    }
  };
  const int epi = p.epilogue;
  if (glu) {
    constexpr int CPR = BN / 16;         // chunks of 8 features per row
    for (int e = threadIdx.x; e < BM * CPR; e += NTHR) {
      const int rl = e / CPR, fl = e % CPR * 8;
      const int row = m0 + rl, feat = n0 + fl;
      if (row >= p.M || feat >= p.split) continue;
      float g[8], u[8], t[8];
      sum8(rl, fl / 32 * 64 + fl % 32, g);
      sum8(rl, fl / 32 * 64 + fl % 32 + 32, u);
      unpack8(*reinterpret_cast<const uint4*>(p.bias + feat), t);
#pragma unroll
      for (int i = 0; i < 8; ++i) g[i] += t[i];
      unpack8(*reinterpret_cast<const uint4*>(p.bias + p.split + feat), t);
#pragma unroll
      for (int i = 0; i < 8; ++i) u[i] += t[i];
      if (p.C2) {
        store_stream<NT>(p.C2 + (size_t)row * p.ldc2 + feat, pack8_bf16(g));
        store_stream<NT>(p.C2 + (size_t)row * p.ldc2 + p.split + feat, pack8_bf16(u));
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) g[i] = gelu_fast(g[i]) * u[i];
      store_stream<NT>(reinterpret_cast<bf16_raw*>(p.C) + (size_t)row * p.ldc + feat, pack8_bf16(g));
    }
    return;
  }
  constexpr int CPR = BN / 8;
  static_assert(NTHR % CPR == 0, "a thread stays in its columns");
  const int cl = threadIdx.x % CPR * 8, col = n0 + cl;
  if (col >= p.N) return;                // N is a multiple of 8
  float bias[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) bias[e] = 0.f;
  if (epilogue_has_bias(epi)) unpack8(*reinterpret_cast<const uint4*>(p.bias + col), bias);
  for (int rl = threadIdx.x / CPR; rl < BM && m0 + rl < p.M; rl += NTHR / CPR) {
    float x[8];
    sum8(rl, cl, x);
    if (epi == EPI_ACCUM_F32) {
      // (never streamed: what comes here mostly stays in the memory-side cache between microbatches; 4096 x 4096 over 513 tokens
      // 50 -> 63 us with non-temporal accesses)
      float4* c = reinterpret_cast<float4*>(reinterpret_cast<float*>(p.C) + (size_t)(m0 + rl) * p.ldc + col);
      const float4 u = c[0], v = c[1];
      c[0] = make_float4(u.x + x[0], u.y + x[1], u.z + x[2], u.w + x[3]);
      c[1] = make_float4(v.x + x[4], v.y + x[5], v.z + x[6], v.w + x[7]);
    } else {
      finish_chunk<NT>(p, epi, x, bias, m0 + rl, col);
    }
  }
}

template <int FM, int WM, int WN, int WK, int NS, bool A_T, bool B_T, bool NT = false>
swarm_status launch(const typename LaunchArgs<A_T>::type& k, int tiles, hipStream_t st) {
  constexpr int BM = 16 * FM * WM, BN = 64 * WN, BK = 32 * WK;
  constexpr size_t stages = (size_t)NS * (BM + BN) * BK * 2, sums = (size_t)WK * BM * (BN + 4) * 4;
  constexpr size_t lds_bytes = stages > sums ? stages : sums;
  auto kern = gemm_bf16_kw_kernel<FM, WM, WN, WK, NS, A_T, B_T, NT>;
  static LdsOptIn opted;   // per instantiation
  if (lds_opt_in((const void*)kern, lds_bytes, opted) != SWARM_OK) return SWARM_ERR_LAUNCH;
  hipLaunchKernelGGL(kern, dim3(tiles), dim3(WM * WN * WK * 64), lds_bytes, st, k);
  return launch_status();
}

template <int WM, int WN, int WK, int NS, int FM = 4>
swarm_status launch_layout(const GemmArgs& g, int stream, hipStream_t st) {
  KArgs k = kargs_of(g);
  k.stream = stream;
  k.tiles_m = (k.M + 16 * FM * WM - 1) / (16 * FM * WM);
  k.tiles_n = (k.N + 64 * WN - 1) / (64 * WN);
  const int tiles = k.tiles_m * k.tiles_n;
  if constexpr (WM == 2 && WN == 2) {      // an output of 64 MB has many tiles
    if (k.stream && !g.b_trans) return launch<FM, WM, WN, WK, NS, false, false, true>(k, tiles, st);
    if (k.stream) return launch<FM, WM, WN, WK, NS, false, true, true>(k, tiles, st);
  }
  if (!g.b_trans) return launch<FM, WM, WN, WK, NS, false, false>(k, tiles, st);
  return launch<FM, WM, WN, WK, NS, false, true>(k, tiles, st);
}

template <int WM, int WN, int WK, int NS>
swarm_status launch_wgrads(const GemmArgs* g, int n, const ColumnSums* sums, hipStream_t st) {
  const WgradGroup w = wgrad_group_of(g, n, sums, 64 * WM, 64 * WN);
  return launch<4, WM, WN, WK, NS, true, true>(w, w.workgroups, st);
}

}  // namespace

// Whether gemm_bf16_kw takes the product.
bool gemm_bf16_kw_takes(const GemmArgs& g) {
  if ((g.a_trans && !g.b_trans) || g.N % 8) return false;
  if (!(g.a_trans && g.b_trans) && g.K % 32) return false;
  if (g.epilogue == EPI_BIAS_GEGLU && (g.a_trans || g.b_trans || g.N != 2 * g.split || g.split % 32)) return false;
  const long long span = 128 + (g.epilogue == EPI_BIAS_GEGLU ? g.split : 0);   // rows a tile's offsets reach over
  return span * g.lda < (1ll << 30) && span * g.ldb < (1ll << 30);
}

// n weight gradients over the same rows, all of which gemm_bf16_kw_takes, in one launch; the rule of gemm_bf16_kw over the tiles
// of all of them.
swarm_status gemm_bf16_kw_wgrads(const GemmArgs* g, int n, const ColumnSums* sums, hipStream_t st) {
  long small = 0, mid = 0;
  for (int i = 0; i < n; ++i) {
    small += (long)((g[i].M + 63) / 64) * ((g[i].N + 63) / 64);
    mid += (long)((g[i].M + 127) / 128) * ((g[i].N + 63) / 64);
  }
  if (small > 512) return launch_wgrads<2, 2, 2, 4>(g, n, sums, st);
  if (small > 256 && mid <= 256) return launch_wgrads<2, 1, 4, 3>(g, n, sums, st);
  if (small > 256) return launch_wgrads<1, 1, 4, 2>(g, n, sums, st);
  return launch_wgrads<1, 1, 4, 4>(g, n, sums, st);
}

// SWARM_ERR_SHAPE (nothing launched): a k-contiguous operand whose K is no multiple of 32, or a tile whose offsets do
// not fit 32 bits.  The caller has checked alignment (16-byte rows, N % 8 == 0) and the layout.  stream: see KArgs (8100 x
// 16384, K = 4096 with GeLU 1224 -> 1180 us, its gradient 1284 -> 1208).
swarm_status gemm_bf16_kw(const GemmArgs& g, int stream, hipStream_t st) {
  if (!gemm_bf16_kw_takes(g)) return SWARM_ERR_SHAPE;
  // By rounds of workgroups.  A 64-deep slice takes 0.7 us on a 128 x 128 tile, of which a compute unit holds one, and
  // 0.47 us on two 64 x 64 tiles with two stages.  So 128 x 128 tiles where a round (512) of 64 x 64 ones does not hold the
  // product: the last 1280 columns of a 50432-row vocabulary on 2048 tokens, K = 4096, 640 small or 160 large tiles: 74 ->
  // 45 us.  Up to there one round of 128 x 64 tiles with eight wavefronts instead of two 64 x 64 ones per unit, unless half
  // of those tiles' rows would be empty (a pass at d_model 768 on 5 x 333 tokens, 324 small tiles: 362 -> 356 us).  One
  // 64 x 64 tile per unit has four stages; a fifth changes nothing (365 us).
  if (g.a_trans) return gemm_bf16_kw_wgrads(&g, 1, nullptr, st);
  //
  // Fewer 64 x 64 tiles than a quarter or half of the units: what bounds the workgroup is the bytes that its unit takes in, so it
  // gets 16 or 32 rows, and the 16 rows K over eight wavefronts, unless K is shorter than four slices of that.  On 64 | 32 | 16 rows:
  // 200 x 1024, K = 4096 14.3 | 10.7 | 9.4 us, K = 1024 7.0 | 5.4 | 5.1; 64 x 64, K = 256 4.9 | 4.0 | 4.2; 512 x 1024, K = 4096 15.1 |
  // 10.9 | 19.4 (two rounds).  (32 rows on eight wavefronts lie between: 10.2, 5.6, 4.6, 11.0.)
  const long cols = (g.N + 63) / 64;
  if ((g.M + 15) / 16 * cols <= 256 && g.K >= 1024) return launch_layout<1, 1, 8, 3, 1>(g, stream, st);
  if ((g.M + 31) / 32 * cols <= 256) return launch_layout<1, 1, 4, 4, 2>(g, stream, st);
  const long small = (g.M + 63) / 64 * cols, mid = (g.M + 127) / 128 * cols;
  if (small > 512) return launch_layout<2, 2, 2, 4>(g, stream, st);
  if (small > 256 && mid <= 256) return launch_layout<2, 1, 4, 3>(g, stream, st);
  if (small > 256) return launch_layout<1, 1, 4, 2>(g, stream, st);
  return launch_layout<1, 1, 4, 4>(g, stream, st);
}

}  // namespace swarm
