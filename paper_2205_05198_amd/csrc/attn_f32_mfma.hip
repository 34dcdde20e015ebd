// Attention core on fp32 matrix instructions: fp32 inputs, and the choice between the two input types.
#include "attn_f32_mfma.h"

namespace sar {

static hipError_t launch_attn_fwd_f32_of_f32(const AttnParams& P, const void* q, const void* k, const void* v, void* o, float* lse, hipStream_t st) {
  if (few(P)) return fwd_few<float>(P, q, k, v, o, lse, st);
  return by_shape(P, [&](auto m, auto dt) { return fwd_dt<decltype(m)::value, decltype(dt)::value, float>(P, q, k, v, o, lse, st); });
}
static hipError_t launch_attn_bwd_f32_of_f32(const AttnParams& P, const void* q, const void* k, const void* v, const void* o, const float* lse, const void* dO, void* dq,
                                      void* dk, void* dv, float* delta, int passes, hipStream_t st) {
  if (few(P)) return bwd_few<float>(P, q, k, v, o, lse, dO, dq, dk, dv, delta, passes, st);
  return by_shape(P, [&](auto m, auto dt) {
    return bwd_dt<decltype(m)::value, decltype(dt)::value, float>(P, q, k, v, o, lse, dO, dq, dk, dv, delta, passes, st);
  });
}

hipError_t launch_attn_fwd_f32_of_bf16(const AttnParams& P, const void* q, const void* k, const void* v, void* o, float* lse, hipStream_t st);  // attn_f32_mfma_bf16.hip
hipError_t launch_attn_bwd_f32_of_bf16(const AttnParams& P, const void* q, const void* k, const void* v, const void* o, const float* lse, const void* dO, void* dq,
                                       void* dk, void* dv, float* delta, int passes, hipStream_t st);

hipError_t launch_attn_fwd_f32(const AttnParams& P, bool bf16, const void* q, const void* k, const void* v, void* o, float* lse, hipStream_t st) {
  return bf16 ? launch_attn_fwd_f32_of_bf16(P, q, k, v, o, lse, st) : launch_attn_fwd_f32_of_f32(P, q, k, v, o, lse, st);
}
hipError_t launch_attn_bwd_f32(const AttnParams& P, bool bf16, const void* q, const void* k, const void* v, const void* o, const float* lse,
                               const void* dO, void* dq, void* dk, void* dv, float* delta, int passes, hipStream_t st) {
  return bf16 ? launch_attn_bwd_f32_of_bf16(P, q, k, v, o, lse, dO, dq, dk, dv, delta, passes, st)
              : launch_attn_bwd_f32_of_f32(P, q, k, v, o, lse, dO, dq, dk, dv, delta, passes, st);
}

}  // namespace sar
