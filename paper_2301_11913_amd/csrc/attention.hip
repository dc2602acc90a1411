// Attention dispatch: matrix-core kernels for d_head 64 and 128 (bf16 and fp32), direct kernels for other widths and for the
// smallest fp32 calls.
#include "kernels.h"

namespace swarm {

swarm_status attention_fwd_naive(const void*, void*, float*, int, int, int, int, bool, hipStream_t);
swarm_status attention_bwd_naive(const void*, const void*, const void*, const float*, float*, void*, int, int, int,
                                 int, bool, hipStream_t);

swarm_status attention_fwd_mfma(const void*, void*, float*, int, int, int, int, hipStream_t);
swarm_status attention_fwd_f32(const float*, float*, float*, int, int, int, int, hipStream_t);

// fp32 calls of so few short rows that the direct kernels, one workgroup per row and nothing to merge, are done before a
// 32-row tile has passed its chain of loads and products.  The line is where a round of the chip takes as long as the chain
// (either side of it, dk / dv / dq: d_head 64, 16 sequences x heads of 48 tokens 17.1 us against 19.7, 32 of 48 21.2 / 19.9;
// d_head 128, 16 of 64 31.1 / 33.5, 32 of 64 57 / 34; one token 11 / 17 and 12 / 26).
static bool direct_is_faster(int B, int S, int H, int dh) { return S <= dh && (long long)B * H * S * S <= 512ll * dh; }

swarm_status attention_fwd(const void* qkv, void* o, float* lse, int B, int S, int H, int dh, bool bf16,
                           hipStream_t st) {
  if (bf16 && (dh == 64 || dh == 128)) return attention_fwd_mfma(qkv, o, lse, B, S, H, dh, st);
  if (!bf16 && (dh == 64 || dh == 128) && !direct_is_faster(B, S, H, dh))
    return attention_fwd_f32((const float*)qkv, (float*)o, lse, B, S, H, dh, st);
  return attention_fwd_naive(qkv, o, lse, B, S, H, dh, bf16, st);
}

swarm_status attention_bwd_mfma(const void*, const void*, const void*, const float*, float*, void*, int, int, int,
                                int, hipStream_t);
swarm_status attention_bwd_f32(const float*, const float*, const float*, const float*, float*, float*, int, int, int,
                               int, hipStream_t);

swarm_status attention_bwd(const void* qkv, const void* o, const void* dout, const float* lse, float* delta,
                           void* dqkv, int B, int S, int H, int dh, bool bf16, hipStream_t st) {
  if (bf16 && (dh == 64 || dh == 128)) return attention_bwd_mfma(qkv, o, dout, lse, delta, dqkv, B, S, H, dh, st);
  if (!bf16 && (dh == 64 || dh == 128) && !direct_is_faster(B, S, H, dh))
    return attention_bwd_f32((const float*)qkv, (const float*)o, (const float*)dout, lse, delta, (float*)dqkv, B, S, H, dh,
                             st);
  return attention_bwd_naive(qkv, o, dout, lse, delta, dqkv, B, S, H, dh, bf16, st);
}

}  // namespace swarm
