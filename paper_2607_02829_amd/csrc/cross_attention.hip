// Asymmetric attention of the generative block's sparse middle stage (Sec. 3.4, "Integration
// with Generative Forecasting"; App. A.1 EDM table): queries from Sq tokens (the routed ones),
// keys and values from Skv tokens (all of the conditioning sequence); per sample and head
// O = softmax(q k^T / sqrt(hd)) v over the Skv keys, and its backward.
//
// Layouts: q, O, dO, dq [B*Sq, D] (head h at columns h*hd ..); kv, dkv [B*Skv, 2D] (k of head h
// at column h*hd, v at D + h*hd); lse, delta [B, H, Sq], lse the base-2 log-sum-exp of the scaled
// scores (P = exp2(s * log2(e)/sqrt(hd) - lse)), delta = rowsum(dO * O) per head.
//
// bf16 runs the MFMA attention kernels (attention.hip) and fp32 storage the fp32 ones
// (attention_f32.hip); both take the query and key/value buffers and their token counts separately.
#include "common.h"
#include "sr_internal.h"

namespace sr {

hipError_t launch_xattn_fwd(int dtype, const void* q, const void* kv, void* O, float* lse, int B, int Sq, int Skv,
                            int H, int D, hipStream_t st) {
  if (dtype == kBF16)
    return launch_attn_fwd_mfma((const bf16_t*)q, D, (const bf16_t*)kv, 2 * D, (uint32_t)((size_t)B * Skv * 2 * D),
                                (bf16_t*)O, lse, B, Sq, Skv, H, D, st);
  return launch_attn_fwd_f32((const float*)q, D, (uint32_t)((size_t)B * Sq * D), (const float*)kv, 2 * D,
                             (uint32_t)((size_t)B * Skv * 2 * D), (float*)O, lse, B, Sq, Skv, H, D, st);
}

hipError_t launch_xattn_bwd(int dtype, const void* q, const void* kv, const void* O, const void* dO, const float* lse,
                            float* delta, void* dq, void* dkv, int B, int Sq, int Skv, int H, int D, hipStream_t st) {
  hipError_t e = launch_attn_delta(dtype, dO, O, B, Sq, H, D / H, delta, st);
  if (e != hipSuccess) return e;
  if (dtype == kBF16) {
    const bf16_t *qb = (const bf16_t*)q, *kvb = (const bf16_t*)kv, *dOb = (const bf16_t*)dO;
    e = launch_attn_dkv_mfma(qb, D, (uint32_t)((size_t)B * Sq * D), kvb, 2 * D, dOb, lse, delta, (bf16_t*)dkv, 2 * D, B,
                             Sq, Skv, H, D, st);
    if (e != hipSuccess) return e;
    return launch_attn_dq_mfma(qb, D, kvb, 2 * D, (uint32_t)((size_t)B * Skv * 2 * D), dOb, lse, delta, (bf16_t*)dq, D,
                               B, Sq, Skv, H, D, st);
  }
  return launch_attn_bwd_f32((const float*)q, D, (uint32_t)((size_t)B * Sq * D), (const float*)kv, 2 * D,
                             (uint32_t)((size_t)B * Skv * 2 * D), (const float*)dO, lse, delta, (float*)dq, D,
                             (float*)dkv, 2 * D, B, Sq, Skv, H, D, st);
}

}  // namespace sr
