// bf16 MFMA GEMM on 128 x 128 tiles, two workgroups per compute unit:  C[M,N] (+)= sum_k A(m,k) B(n,k).
//
// For products with more 128 x 128 tiles than compute units and too few 256 x 256 ones.  Four wavefronts of 64 x 64 and two
// LDS stages of 64 k (64 KB) leave room for a second workgroup on the unit: what bounds a tile here is the fill of its first
// stages and its epilogue, and the other workgroup multiplies meanwhile.  gemm_bf16_kw.hip holds one workgroup per unit and
// hides the loads better, but has nothing to cover those two; its rounds of 256 tiles are 1.6..1.8 times as long as half
// of a round of 512 here.
//
// Loads go global -> LDS directly.  Tiles keep their memory layout, [rows][64 k] or, where the contraction is the slow index,
// [64 k][rows]; 16-byte chunks are XOR-ed so that ds_read_b128 resp. the LDS transpose read hit all banks.  The multiplies
// are v_mfma_f32_32x32x16_bf16: 2 % faster than 16 x 16 x 32 on this tile, and the K order is one chain, as in
// gemm_bf16_dma.hip, in steps of 16.
#include "gemm_bf16_common.h"

namespace swarm {
namespace {

constexpr int kTile = 128, kDepth = 64, kWaves = 4;
constexpr int kStage = 2 * kTile * kDepth;                      // elements
constexpr int kLoads = kTile * kDepth / 512 / kWaves;           // 1 KiB load instructions per wavefront, operand and slice

#define LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))
#define GLB_PTR(p) ((const __attribute__((address_space(1))) void*)(p))

__device__ __forceinline__ int swz_rows(int row) { return (row & 7) ^ ((row >> 3) & 1); }

// One operand's tile: rows (or, TRANS, columns) r0 .. r0 + 127 of it, kDepth of k per slice.
template <bool TRANS>
struct PairOperand {
  // k-rows as tile rows: the address is a scalar base and ONE 32-bit offset per lane.  Left whole, the compiler multiplies by
  // the leading dimension again for every load in the loop, quarter rate, rather than keep the address registers.
  uint32_t off;
  __device__ __forceinline__ void init(int ld, int wave, int lane) {
    const int krow = wave * 4 + lane / 16;
    off = TRANS ? (uint32_t)(krow * ld + 8 * ((lane % 16) ^ (4 * (krow & 3)))) * 2u : 0u;
  }
  // glu_split: see EPI_BIAS_GEGLU (every 64 tile rows are 32 gate rows and the 32 up rows of the same features; r0 counts
  // features)
  __device__ __forceinline__ void issue_one(const bf16_raw* __restrict__ g, int ld, int r0, int k0, bf16_raw* lds, int wave,
                                            int lane, int t, int glu_split) const {
    const int q = wave + t * kWaves;
    const char* src;
    if constexpr (!TRANS) {
      const int row = q * 8 + lane / 8;
      const int grow = glu_split ? r0 + 32 * (row >> 6) + (row & 31) + ((row & 32) ? glu_split : 0) : r0 + row;
      src = reinterpret_cast<const char*>(g + (size_t)grow * ld + k0 + 8 * ((lane % 8) ^ swz_rows(row)));
    } else {
      src = reinterpret_cast<const char*>(g) + ((size_t)(k0 + t * kWaves * 4) * ld + r0) * 2 + off;
    }
    __builtin_amdgcn_global_load_lds(GLB_PTR(src), LDS_PTR(lds + q * 512), 16, 0, 0);
  }
  // 32 rows (columns) from `base` x 16 k (the kk-th of the slice).  The transpose read is two plain instructions: behind the
  // compiler's builtin every pending global -> LDS load counts as a possible writer of the bytes read and is waited for.  The
  // stages are disjoint by construction; the compiler does not count these reads, so the caller waits for them before use.
  static __device__ __forceinline__ bf16x8 read(const bf16_raw* tile, int base, int kk, int lane) {
    if constexpr (!TRANS) {
      const int l32 = lane & 31, lg = lane >> 5;
      return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(tile + (base + l32) * kDepth +
                                                                        8 * ((2 * kk + lg) ^ swz_rows(l32))));
    } else {
      const int l16 = lane & 15, grp = lane >> 4, kq = l16 >> 2;
      const int col = base + 16 * (grp & 1) + 4 * (l16 & 3), krow = 16 * kk + 8 * (grp >> 1) + kq;
      const bf16_raw* p = tile + krow * kTile + 8 * ((col >> 3) ^ (4 * kq)) + (col & 4);
      const uint32_t addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
      uint2 a, b;
      asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(a) : "v"(addr) : "memory");
      asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(b) : "v"(addr), "n"(8 * kTile) : "memory");
      return __builtin_bit_cast(bf16x8, make_uint4(a.x, a.y, b.x, b.y));
    }
  }
};

template <bool A_T, bool B_T>
__global__ __launch_bounds__(kWaves * 64) void gemm_bf16_pair_kernel(KArgs p) {
  extern __shared__ __attribute__((aligned(1024))) bf16_raw lds[];
  int tile_m, tile_n;
  tile_of_block(p, tile_m, tile_n);
  const int glu = (!B_T && p.epilogue == EPI_BIAS_GEGLU) ? p.split : 0;
  // (weight gradients, which add to their output, come in whole tiles only)
  const int m0 = tile_origin(tile_m, kTile, p.M);
  const int n0 = glu ? tile_origin(tile_n, kTile / 2, glu) : tile_origin(tile_n, kTile, p.N);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  PairOperand<A_T> a;
  PairOperand<B_T> b;
  a.init(p.lda, wave, lane);
  b.init(p.ldb, wave, lane);
  // load t of slice kt into stage st: the A tile's, then the B tile's
  auto issue_one = [&](int t, int kt, bf16_raw* st) __attribute__((always_inline)) {
    if (t < kLoads) a.issue_one(p.A, p.lda, m0, kt * kDepth, st, wave, lane, t, 0);
    else b.issue_one(p.B, p.ldb, n0, kt * kDepth, st + kTile * kDepth, wave, lane, t - kLoads, glu);
  };
  // fragment n of a sub-step in the order its multiplies need them: A rows 0, B 0, B 1, A rows 1
  bf16x8 fa[2][2], fb[2][2];
  auto read_one = [&](const bf16_raw* st, int kk, int n, int buf) __attribute__((always_inline)) {
    if (n == 0 || n == 3) fa[buf][n == 3] = PairOperand<A_T>::read(st, wm * 64 + 32 * (n == 3), kk, lane);
    else fb[buf][n - 1] = PairOperand<B_T>::read(st + kTile * kDepth, wn * 64 + 32 * (n - 1), kk, lane);
  };

  const int KT = p.K / kDepth;
#pragma unroll
  for (int t = 0; t < 2 * kLoads; ++t) issue_one(t, 0, lds);
  __builtin_amdgcn_s_waitcnt(0x0F70);            // vmcnt(0)
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int n = 0; n < 4; ++n) read_one(lds, 0, n, 0);

  // One sub-step of 16 k: four multiplies of buffer `cur`; behind each one fragment of the next sub-step (`nkk` of the stage at
  // `next`) and, in the first of a slice, two loads of the slice after it.
  auto substep = [&](int cur, const bf16_raw* next, int nkk, bool loads, int kt, bf16_raw* st) __attribute__((always_inline)) {
    if constexpr (A_T || B_T) {                   // fragments read with plain instructions: all of them have returned
      __builtin_amdgcn_s_waitcnt(0xC07F);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      acc[n >> 1][n & 1] =
          __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[cur][n >> 1], fb[cur][n & 1], acc[n >> 1][n & 1], 0, 0, 0);
      read_one(next, nkk, n, cur ^ 1);
      if (loads) {
        issue_one(2 * n, kt, st);
        issue_one(2 * n + 1, kt, st);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  for (int kt = 0; kt < KT; ++kt) {
    bf16_raw* now = lds + (kt & 1) * kStage;
    bf16_raw* next = lds + ((kt + 1) & 1) * kStage;
    // (the last iteration fetches its own slice again instead of branching)
    substep(0, now, 1, true, min(kt + 1, KT - 1), next);
    substep(1, now, 2, false, 0, next);
    substep(0, now, 3, false, 0, next);
    // this wavefront's part of slice kt + 1 has landed and its reads of slice kt are complete; then all meet.  The slice's last
    // sub-step is multiplied behind the barrier, over the first reads of the next one.
    __builtin_amdgcn_s_waitcnt(0x0070);           // vmcnt(0), lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    substep(1, next, 0, false, 0, now);
  }
  // the fragments requested last are not used, but have to arrive before their registers are
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" : "+v"(fa[0][0]), "+v"(fa[0][1]), "+v"(fb[0][0]), "+v"(fb[0][1])::"memory");
  __builtin_amdgcn_s_barrier();                   // every read of the stages is done: they become the epilogue's patches
  gemm_epilogue<2, 2, false>(p, acc, m0 + wm * 64, glu ? n0 + wn * 32 : n0 + wn * 64, lane & 31, lane >> 5,
                             reinterpret_cast<float*>(lds) + wave * 32 * kEpiPitch);
}

template <bool A_T, bool B_T>
swarm_status launch(const KArgs& k, hipStream_t st) {
  constexpr size_t lds_bytes = (size_t)2 * kStage * sizeof(bf16_raw);
  static_assert(lds_bytes <= 64 * 1024 && kWaves * 32 * kEpiPitch * sizeof(float) <= lds_bytes, "two workgroups per unit");
  hipLaunchKernelGGL((gemm_bf16_pair_kernel<A_T, B_T>), dim3(k.tiles_m * k.tiles_n), dim3(kWaves * 64), lds_bytes, st, k);
  return launch_status();
}

}  // namespace

// M and N at least 128 (weight gradients: multiples of it), K a multiple of 64; the caller has checked alignment and the layout.
swarm_status gemm_bf16_pair(const GemmArgs& g, int stream, hipStream_t st) {
  KArgs k = kargs_of(g);
  k.stamps = nullptr;
  k.stream = stream;
  k.tiles_m = (g.M + kTile - 1) / kTile; k.tiles_n = (g.N + kTile - 1) / kTile;
  if (!g.a_trans && !g.b_trans) return launch<false, false>(k, st);
  if (!g.a_trans) return launch<false, true>(k, st);
  if (g.b_trans) return launch<true, true>(k, st);
  return SWARM_ERR_SHAPE;
}

}  // namespace swarm
