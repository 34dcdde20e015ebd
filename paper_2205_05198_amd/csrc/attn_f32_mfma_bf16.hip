// Attention core on fp32 matrix instructions: bf16 inputs.
#include "attn_f32_mfma.h"

namespace sar {

hipError_t launch_attn_fwd_f32_of_bf16(const AttnParams& P, const void* q, const void* k, const void* v, void* o, float* lse, hipStream_t st) {
  if (few(P)) return fwd_few<uint16_t>(P, q, k, v, o, lse, st);
  return by_shape(P, [&](auto m, auto dt) { return fwd_dt<decltype(m)::value, decltype(dt)::value, uint16_t>(P, q, k, v, o, lse, st); });
}
hipError_t launch_attn_bwd_f32_of_bf16(const AttnParams& P, const void* q, const void* k, const void* v, const void* o, const float* lse, const void* dO, void* dq,
                                      void* dk, void* dv, float* delta, int passes, hipStream_t st) {
  if (few(P)) return bwd_few<uint16_t>(P, q, k, v, o, lse, dO, dq, dk, dv, delta, passes, st);
  return by_shape(P, [&](auto m, auto dt) {
    return bwd_dt<decltype(m)::value, decltype(dt)::value, uint16_t>(P, q, k, v, o, lse, dO, dq, dk, dv, delta, passes, st);
  });
}

}  // namespace sar
