// LAMB step for one parameter tensor (appendix "Additional Details for Section 4.3").  Streaming kernels: moments + update
// direction + per-workgroup partial sums of |w|^2 and |u|^2; the trust ratio, their sum in a fixed order; the weight update (and
// the copy in the stage's dtype).  What bounds a short tensor is launches, 4 us each and more: one of at most kSmall elements (of a
// block's twelve seven at d_model 4096, eight where b_1 has no more) is done by one workgroup in one launch (4096: 8.8 -> 4.1 us,
// 12288: 8.9 -> 6.6, 16384: 9.1 / 8.0 where two launches take 7.8), and up to kMaxFolded workgroups every one of the update adds up
// the partial sums itself (65536: 9.5 -> 8.1).  Beyond that a single workgroup does; with fewer, looping workgroups and no third
// launch 2^26 elements take 490 us instead of 470.
#include <atomic>
#include <cmath>

#include "kernels.h"
#include "swarm_optim.h"

namespace swarm {
namespace {

constexpr int kThreads = 256;
constexpr int kPerThread = 16;                         // elements per thread in the first pass (4 x float4)
constexpr int kPerBlock = kThreads * kPerThread;

// Every element is touched once per pass, so all vector accesses are non-temporal: nothing is kept in the caches
// for a second use that never comes (5.2 -> 5.9 TB/s on the largest tensor).
typedef float f32x4n __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 ldg4(const float* p) {
  const f32x4n t = __builtin_nontemporal_load(reinterpret_cast<const f32x4n*>(p));
  return make_float4(t[0], t[1], t[2], t[3]);
}
__device__ __forceinline__ void stg4(float* p, const float4& v) {
  const f32x4n t = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(t, reinterpret_cast<f32x4n*>(p));
}

struct Hyper {
  float beta1, beta2, one_m_beta1, one_m_beta2, inv_bc1, inv_bc2, eps, wd, gscale, lr;
};

// Moments of one element in place, its update direction returned.  The fused operations are written out: which product of a sum
// of two keeps all its bits would be the compiler's choice, another one in every kernel, and the other way about v is a quarter further
// from 64 bits (3.7e-8 instead of 2.9e-8).
__device__ __forceinline__ float lamb_element(float w, float g, float& m, float& v, const Hyper& h) {
  const float gs = g * h.gscale;
  m = fmaf(h.beta1, m, h.one_m_beta1 * gs);
  v = fmaf(h.beta2, v, h.one_m_beta2 * gs * gs);
  return fmaf(h.wd, w, (m * h.inv_bc1) / (sqrtf(v * h.inv_bc2) + h.eps));
}
__device__ __forceinline__ float4 lamb_four(const float4& w, const float4& g, float4& m, float4& v, const Hyper& h, float& sw,
                                            float& su) {
  float4 u;
  u.x = lamb_element(w.x, g.x, m.x, v.x, h); sw += w.x * w.x; su += u.x * u.x;
  u.y = lamb_element(w.y, g.y, m.y, v.y, h); sw += w.y * w.y; su += u.y * u.y;
  u.z = lamb_element(w.z, g.z, m.z, v.z, h); sw += w.z * w.z; su += u.z * u.z;
  u.w = lamb_element(w.w, g.w, m.w, v.w, h); sw += w.w * w.w; su += u.w * u.w;
  return u;
}
// |w| / |u| (1 if either is zero)
__device__ __forceinline__ float trust_ratio_of(double w2, double u2) {
  const double nw = sqrt(w2), nu = sqrt(u2);
  return (nw > 0.0 && nu > 0.0) ? (float)(nw / nu) : 1.0f;
}
// Sums over a workgroup of THREADS, in every thread; s: [2][THREADS / 64] doubles of LDS.
template <int THREADS>
__device__ __forceinline__ void block_sums(double& sw, double& su, double (*s)[THREADS / 64]) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) { sw += __shfl_xor(sw, m, 64); su += __shfl_xor(su, m, 64); }
  if ((threadIdx.x & 63) == 0) { s[0][threadIdx.x >> 6] = sw; s[1][threadIdx.x >> 6] = su; }
  __syncthreads();
  sw = s[0][0]; su = s[1][0];
#pragma unroll
  for (int i = 1; i < THREADS / 64; ++i) { sw += s[0][i]; su += s[1][i]; }
}

__global__ __launch_bounds__(kThreads) void lamb_moments_kernel(const float* __restrict__ w, const float* __restrict__ g,
                                                                float* __restrict__ m, float* __restrict__ v,
                                                                float* __restrict__ u, float* __restrict__ partial,
                                                                size_t n, Hyper h) {
  __shared__ double s[2][kThreads / 64];
  const size_t base = (size_t)blockIdx.x * kPerBlock;
  float sw = 0.f, su = 0.f;
#pragma unroll
  for (int it = 0; it < kPerThread / 4; ++it) {
    const size_t i = base + ((size_t)it * kThreads + threadIdx.x) * 4;
    if (i + 4 <= n) {
      const float4 w4 = ldg4(w + i), g4 = ldg4(g + i);
      float4 m4 = ldg4(m + i), v4 = ldg4(v + i);
      const float4 u4 = lamb_four(w4, g4, m4, v4, h, sw, su);
      stg4(m + i, m4); stg4(v + i, v4);
      stg4(u + i, u4);
    } else {
      for (size_t j = i; j < n && j < i + 4; ++j) {          // ragged tail
        float mj = m[j], vj = v[j];
        const float uj = lamb_element(w[j], g[j], mj, vj, h);
        m[j] = mj; v[j] = vj; u[j] = uj;
        sw += w[j] * w[j];
        su += uj * uj;
      }
    }
  }
  double tw = sw, tu = su;
  block_sums<kThreads>(tw, tu, s);
  if (threadIdx.x == 0) { partial[2 * (size_t)blockIdx.x] = (float)tw; partial[2 * (size_t)blockIdx.x + 1] = (float)tu; }
}

// The ratio of many workgroups' sums; doubles keep the long fixed-order sum accurate.  One workgroup, bound by the latency of its
// loads (and, between two streaming passes, the whole chip's time): the full width of a unit and eight blocks' sums on
// their way per thread (32768 blocks, a 16384 x 8192 tensor: 33.6 -> 12.2 us with 256 threads before).
constexpr int kRatioThreads = 1024;
__global__ __launch_bounds__(kRatioThreads) void lamb_ratio_kernel(const float* __restrict__ partial, size_t nblocks,
                                                                   float* __restrict__ ratio_out,
                                                                   float* __restrict__ user) {
  __shared__ double s[2][kRatioThreads / 64];
  constexpr int U = 8;
  const float2* sums = reinterpret_cast<const float2*>(partial);   // a 256-byte aligned part of the workspace
  double sw = 0.0, su = 0.0;
  for (size_t b0 = threadIdx.x; b0 < nblocks; b0 += (size_t)U * kRatioThreads) {
    float2 x[U];
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const size_t b = b0 + (size_t)i * kRatioThreads;
      x[i] = b < nblocks ? sums[b] : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int i = 0; i < U; ++i) { sw += x[i].x; su += x[i].y; }
  }
  block_sums<kRatioThreads>(sw, su, s);
  if (threadIdx.x == 0) {
    const float r = trust_ratio_of(sw, su);
    *ratio_out = r;
    if (user) *user = r;
  }
}

template <typename T>
__device__ __forceinline__ void store_updated(float* w, T* param, size_t i, const float4& y) {
  stg4(w + i, y);
  if (!param) return;
  if constexpr (sizeof(T) == 4) {
    *reinterpret_cast<float4*>(param + i) = y;
  } else {
    T r[4];
    Elem<T>::store(r, y.x); Elem<T>::store(r + 1, y.y); Elem<T>::store(r + 2, y.z); Elem<T>::store(r + 3, y.w);
    *reinterpret_cast<uint2*>(param + i) = *reinterpret_cast<const uint2*>(r);
  }
}

// One workgroup per kPerBlock elements, as in the first pass.  ratio == nullptr: at most kMaxFolded of them, and each adds up the
// partial sums.
constexpr int kMaxFolded = 1024;
template <typename T>
__global__ __launch_bounds__(kThreads) void lamb_apply_kernel(float* __restrict__ w, const float* __restrict__ u,
                                                              T* __restrict__ param, const float* __restrict__ ratio,
                                                              const float* __restrict__ partial, float* __restrict__ user,
                                                              size_t n, float lr) {
  __shared__ double s[2][kThreads / 64];
  const size_t n4 = n / 4;
  constexpr int U = kPerThread / 4;
  const size_t i0 = (size_t)blockIdx.x * (kThreads * U) + threadIdx.x;
  float4 x[U], d[U];
#pragma unroll
  for (int it = 0; it < U; ++it) {
    const size_t i = i0 + (size_t)it * kThreads;
    if (i < n4) { x[it] = ldg4(w + 4 * i); d[it] = ldg4(u + 4 * i); }
  }
  float r;
  if (ratio) {
    r = *ratio;
  } else {
    const float2* sums = reinterpret_cast<const float2*>(partial);   // a 256-byte aligned part of the workspace
    float2 p[kMaxFolded / kThreads];
#pragma unroll
    for (int k = 0; k < kMaxFolded / kThreads; ++k) {
      const unsigned b = k * kThreads + threadIdx.x;
      p[k] = b < gridDim.x ? sums[b] : make_float2(0.f, 0.f);
    }
    double sw = 0.0, su = 0.0;
#pragma unroll
    for (int k = 0; k < kMaxFolded / kThreads; ++k) { sw += p[k].x; su += p[k].y; }
    block_sums<kThreads>(sw, su, s);
    r = trust_ratio_of(sw, su);
    if (user && blockIdx.x == 0 && threadIdx.x == 0) *user = r;
  }
  const float step = lr * r;
#pragma unroll
  for (int it = 0; it < U; ++it) {
    const size_t i = i0 + (size_t)it * kThreads;
    if (i >= n4) continue;
    float4 y = x[it];
    y.x -= step * d[it].x; y.y -= step * d[it].y; y.z -= step * d[it].z; y.w -= step * d[it].w;
    store_updated(w, param, 4 * i, y);
  }
  if (blockIdx.x == 0 && threadIdx.x < n - n4 * 4) {           // ragged tail
    const size_t i = n4 * 4 + threadIdx.x;
    const float x1 = w[i] - step * u[i];
    w[i] = x1;
    if (param) Elem<T>::store(param + i, x1);
  }
}

// One workgroup for a whole tensor, PT * 4 elements per thread, all of them loaded before the first is used and kept in
// registers between the two halves of the step.
constexpr int kSmallThreads = 1024, kSmall = kSmallThreads * 12;
template <typename T, int PT>
__global__ __launch_bounds__(kSmallThreads) void lamb_small_kernel(float* __restrict__ w, const float* __restrict__ g,
                                                                   float* __restrict__ m, float* __restrict__ v,
                                                                   T* __restrict__ param, float* __restrict__ user, int n,
                                                                   Hyper h) {
  __shared__ double s[2][kSmallThreads / 64];
  const int n4 = n / 4;
  float4 w4[PT], g4[PT], m4[PT], v4[PT];
#pragma unroll
  for (int it = 0; it < PT; ++it) {
    const int i = it * kSmallThreads + threadIdx.x;
    if (i < n4) { w4[it] = ldg4(w + 4 * i); g4[it] = ldg4(g + 4 * i); m4[it] = ldg4(m + 4 * i); v4[it] = ldg4(v + 4 * i); }
  }
  float sw = 0.f, su = 0.f;
#pragma unroll
  for (int it = 0; it < PT; ++it) {
    const int i = it * kSmallThreads + threadIdx.x;
    if (i >= n4) continue;
    g4[it] = lamb_four(w4[it], g4[it], m4[it], v4[it], h, sw, su);
    stg4(m + 4 * i, m4[it]);
    stg4(v + 4 * i, v4[it]);
  }
  const int j = 4 * n4 + (int)threadIdx.x;                     // ragged tail
  float wj = 0.f, uj = 0.f;
  if (j < n) {
    float mj = m[j], vj = v[j];
    wj = w[j];
    uj = lamb_element(wj, g[j], mj, vj, h);
    m[j] = mj; v[j] = vj;
    sw += wj * wj;
    su += uj * uj;
  }
  double tw = sw, tu = su;
  block_sums<kSmallThreads>(tw, tu, s);
  const float ratio = trust_ratio_of(tw, tu), step = h.lr * ratio;
  if (user && threadIdx.x == 0) *user = ratio;
#pragma unroll
  for (int it = 0; it < PT; ++it) {
    const int i = it * kSmallThreads + threadIdx.x;
    if (i >= n4) continue;
    float4 y = w4[it];
    y.x -= step * g4[it].x; y.y -= step * g4[it].y; y.z -= step * g4[it].z; y.w -= step * g4[it].w;
    store_updated(w, param, (size_t)4 * i, y);
  }
  if (j < n) {
    const float y = wj - step * uj;
    w[j] = y;
    if (param) Elem<T>::store(param + j, y);
  }
}

size_t n_blocks(size_t n) { return (n + kPerBlock - 1) / kPerBlock; }

}  // namespace
}  // namespace swarm

using namespace swarm;

// Scratch of swarm_lamb_step_static: the update direction of the largest tensor it accepts, the partial sums of
// its norms and the ratio.  One copy per GPU, at an address of its own, held until the process ends.
constexpr size_t kStaticU = SWARM_LAMB_STATIC_MAX_ELEMS * sizeof(float);
constexpr size_t kStaticPartial = (SWARM_LAMB_STATIC_MAX_ELEMS / kPerBlock) * 2 * sizeof(float);
static_assert(SWARM_LAMB_STATIC_MAX_ELEMS % kPerBlock == 0 && kStaticU % 256 == 0 && kStaticPartial % 256 == 0, "");
static __device__ __align__(256) unsigned char scratch[kStaticU + kStaticPartial + 256];

extern "C" size_t swarm_lamb_workspace_bytes(size_t n_elems) {
  if (n_elems < 1) return 0;
  const size_t u = (n_elems * 4 + 255) & ~(size_t)255;
  const size_t p = (n_blocks(n_elems) * 8 + 255) & ~(size_t)255;
  return u + p + 256;
}

namespace swarm {
namespace {

template <typename T>
swarm_status lamb_launch_as(const Hyper& h, size_t n, float* master, T* param, const float* grad, float* m, float* v,
                            float* trust_ratio, float* u, float* partial, float* ratio, hipStream_t st) {
  if (n <= kSmall) {
#define SMALL(PT)                                                                                                            \
  hipLaunchKernelGGL((lamb_small_kernel<T, PT>), dim3(1), dim3(kSmallThreads), 0, st, master, grad, m, v, param, trust_ratio, \
                     (int)n, h)
    if (n <= 4 * kSmallThreads) SMALL(1);
    else if (n <= 8 * kSmallThreads) SMALL(2);
    else SMALL(3);
#undef SMALL
    return launch_status();
  }
  const size_t nb = n_blocks(n);
  const bool folded = nb <= kMaxFolded;
  hipLaunchKernelGGL(lamb_moments_kernel, dim3((unsigned)nb), dim3(kThreads), 0, st, master, grad, m, v, u, partial, n, h);
  if (!folded)
    hipLaunchKernelGGL(lamb_ratio_kernel, dim3(1), dim3(kRatioThreads), 0, st, partial, nb, ratio, trust_ratio);
  hipLaunchKernelGGL(lamb_apply_kernel<T>, dim3((unsigned)nb), dim3(kThreads), 0, st, master, u, param,
                     folded ? nullptr : ratio, partial, trust_ratio, n, h.lr);
  return launch_status();
}

// The launches of one update; u [n] fp32, partial [2 * n_blocks(n)] fp32 and ratio [1] fp32 are scratch that the kernels
// overwrite before they read it (nothing has to be cleared between calls).
swarm_status lamb_launch(const swarm_lamb_config* cfg, size_t n, float* master, void* param, int32_t dtype,
                         const float* grad, float* m, float* v, float* trust_ratio, float* u, float* partial,
                         float* ratio, hipStream_t st) {
  Hyper h;
  h.beta1 = cfg->beta1; h.beta2 = cfg->beta2; h.one_m_beta1 = 1.0f - cfg->beta1; h.one_m_beta2 = 1.0f - cfg->beta2;
  h.inv_bc1 = (float)(1.0 / (1.0 - std::pow((double)cfg->beta1, (double)cfg->step)));
  h.inv_bc2 = (float)(1.0 / (1.0 - std::pow((double)cfg->beta2, (double)cfg->step)));
  h.eps = cfg->eps; h.wd = cfg->weight_decay; h.gscale = cfg->grad_scale; h.lr = cfg->lr;
  if (param && dtype == SWARM_BF16)
    return lamb_launch_as<bf16_raw>(h, n, master, (bf16_raw*)param, grad, m, v, trust_ratio, u, partial, ratio, st);
  return lamb_launch_as<float>(h, n, master, (float*)param, grad, m, v, trust_ratio, u, partial, ratio, st);
}

swarm_status lamb_check(const swarm_lamb_config* cfg, size_t n, const float* master, const void* param, int32_t dtype,
                        const float* grad, const float* m, const float* v) {
  if (!cfg || !master || !grad || !m || !v) return SWARM_ERR_NULL;
  if (param && dtype != SWARM_F32 && dtype != SWARM_BF16) return SWARM_ERR_DTYPE;
  if (n < 1 || cfg->step < 1 || !(cfg->beta1 >= 0.f && cfg->beta1 < 1.f) || !(cfg->beta2 >= 0.f && cfg->beta2 < 1.f) ||
      !(cfg->eps > 0.f) || !(cfg->lr >= 0.f) || !(cfg->weight_decay >= 0.f))
    return SWARM_ERR_SHAPE;
  auto al16 = [](const void* q) { return ((uintptr_t)q & 15) == 0; };
  if (!al16(master) || !al16(grad) || !al16(m) || !al16(v) || !al16(param)) return SWARM_ERR_SHAPE;
  return SWARM_OK;
}

// Device address of `scratch` on the current device (looked up once per device; the array's name is only a
// host-side handle and is never passed to a kernel).
std::atomic<unsigned char*> g_scratch_ptr[kMaxDevices];
unsigned char* static_scratch() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  unsigned char* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (!p) {
    void* q = nullptr;
    if (hipGetSymbolAddress(&q, HIP_SYMBOL(scratch)) != hipSuccess || !q) return nullptr;
    p = (unsigned char*)q;
    g_scratch_ptr[dev].store(p, std::memory_order_release);
  }
  return p;
}

}  // namespace
}  // namespace swarm

extern "C" swarm_status swarm_lamb_step(const swarm_lamb_config* cfg, size_t n, float* master, void* param,
                                        int32_t dtype, const float* grad, float* m, float* v, float* trust_ratio,
                                        void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!workspace) return SWARM_ERR_NULL;
  const swarm_status chk = lamb_check(cfg, n, master, param, dtype, grad, m, v);
  if (chk != SWARM_OK) return chk;
  if ((uintptr_t)workspace & 255) return SWARM_ERR_SHAPE;
  if (swarm_lamb_workspace_bytes(n) > workspace_bytes) return SWARM_ERR_WORKSPACE;
  float* u = (float*)workspace;
  float* partial = (float*)((char*)workspace + ((n * 4 + 255) & ~(size_t)255));
  const size_t nb = n_blocks(n);
  float* ratio = partial + 2 * nb + (64 - (2 * nb) % 64) % 64;   // behind the partial sums, inside the slack
  return lamb_launch(cfg, n, master, param, dtype, grad, m, v, trust_ratio, u, partial, ratio, (hipStream_t)hip_stream);
}

extern "C" swarm_status swarm_lamb_step_static(const swarm_lamb_config* cfg, size_t n, float* master, void* param,
                                               int32_t dtype, const float* grad, float* m, float* v,
                                               float* trust_ratio, void* hip_stream) {
  const swarm_status chk = lamb_check(cfg, n, master, param, dtype, grad, m, v);
  if (chk != SWARM_OK) return chk;
  if (n > SWARM_LAMB_STATIC_MAX_ELEMS) return SWARM_ERR_WORKSPACE;
  unsigned char* base = static_scratch();
  if (!base) return SWARM_ERR_LAUNCH;
  return lamb_launch(cfg, n, master, param, dtype, grad, m, v, trust_ratio, (float*)base, (float*)(base + kStaticU),
                     (float*)(base + kStaticU + kStaticPartial), (hipStream_t)hip_stream);
}
