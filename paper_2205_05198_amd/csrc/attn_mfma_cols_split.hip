// bf16 attention core, backward column pass (dK, dV) in its producer / consumer form (three waves per SIMD, each within
// 168 vector registers; compiled WITH -amdgpu-mfma-vgpr-form): every head dimension of the matrix-core path.
#include "attn_mfma_cols_split.h"

#include <type_traits>

namespace sar {

template <int D>
static hipError_t bwd_dkdv_split_d(const AttnParams& P, const void* q, const void* k, const void* v, const float* lse, const void* dO, const float* delta,
                                   void* dk, void* dv, uint16_t* ds_ws, int R, hipStream_t st) {
  const int N = P.b * P.A, nb = (P.s + 63) / 64;
  const bool use_pers = R > 0;  // R key blocks of every head at a time (attn_mfma_cols.hip decides)
  const unsigned grid = use_pers ? (unsigned)(R * N) : (unsigned)(nb * N);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(grid), dim3(768), 0, st, P, (const uint16_t*)q, (const uint16_t*)k, (const uint16_t*)v, lse,
                       (const uint16_t*)dO, delta, (uint16_t*)dk, (uint16_t*)dv, ds_ws);
  };
  auto with = [&](auto rag, auto persistent) {
    constexpr bool PERS = decltype(persistent)::value, RAG = decltype(rag)::value;
    if (ds_ws) {
      if (P.thresh != 0) go(attn_bwd_dkdv_split_kernel<D, true, true, PERS, RAG>);
      else go(attn_bwd_dkdv_split_kernel<D, false, true, PERS, RAG>);
    } else {
      if (P.thresh != 0) go(attn_bwd_dkdv_split_kernel<D, true, false, PERS, RAG>);
      else go(attn_bwd_dkdv_split_kernel<D, false, false, PERS, RAG>);
    }
  };
  if (P.s % 64 != 0) {
    if (use_pers) with(std::true_type(), std::true_type());
    else with(std::true_type(), std::false_type());
  } else if (use_pers) with(std::false_type(), std::true_type());
  else with(std::false_type(), std::false_type());
  return hipGetLastError();
}

hipError_t launch_attn_bwd_dkdv_mfma_split(const AttnParams& P, const void* q, const void* k, const void* v, const float* lse, const void* dO,
                                           const float* delta, void* dk, void* dv, uint16_t* ds_ws, int R, hipStream_t st) {
  switch (P.d) {
    case 64: return bwd_dkdv_split_d<64>(P, q, k, v, lse, dO, delta, dk, dv, ds_ws, R, st);
    case 96: return bwd_dkdv_split_d<96>(P, q, k, v, lse, dO, delta, dk, dv, ds_ws, R, st);
    case 128: return bwd_dkdv_split_d<128>(P, q, k, v, lse, dO, delta, dk, dv, ds_ws, R, st);
    case 160: return bwd_dkdv_split_d<160>(P, q, k, v, lse, dO, delta, dk, dv, ds_ws, R, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace sar
