// bf16 attention core, backward column pass (dK, dV) in its producer / consumer form (three waves per SIMD, each within
// 168 vector registers; compiled WITH -amdgpu-mfma-vgpr-form): every head dimension of the matrix-core path.
#include "attn_mfma_cols_split.h"

#include <algorithm>
#include <type_traits>

namespace sar {

template <int D>
static hipError_t bwd_dkdv_split_d(const AttnParams& P, const void* q, const void* k, const void* v, const float* lse, const void* dO, const float* delta,
                                   void* dk, void* dv, uint16_t* ds_ws, int pers, hipStream_t st) {
  const int N = P.b * P.A, nb = (P.s + 63) / 64;
  // Persistent workgroups (each takes several key blocks of its head, a heavy one then a light one, and overlaps a block's
  // start with the end of the one before): R key blocks of every head at a time, R x heads within the CU count.  Chosen where the longest
  // list does not exceed the rounds of single blocks (us, single / persistent: d = 160, 1024 x 48 heads, no mask, lists of 4 against 3 rounds
  // 83.8 / 94.8; 384 x 128, 3 against 3, 37.2 / 31.3).  Under the mask a list's blocks are not all heavy: every workgroup gets two or more
  // (2048 x 12, some with one, 42.0 / 42.4), and a list may be one longer (1000 x 48 55.1 / 52.0), two at d = 128 and 160 (whose single blocks have
  // a CU to themselves for longer); without it at d = 128, 160 one longer on heads of four blocks or less (256 x 192 35.3 / 30.6).  A short head a CU,
  // lists a third longer: single blocks spread a head over all dies, where the heads are no multiple of eight, and read its tiles into each one's L2
  // (d = 160 384 x 180, no mask, 133 / 124, but 512 x 192 116 / 127; d = 96 under the mask 384 x 180 69.3 / 63.6, 320 x 192 52.0 / 50.1).
  const int cus = attn_mfma_cu_count();
  const int R = N <= cus ? std::min(nb, cus / N) : 0;
  const int64_t rounds = ((int64_t)nb * N + cus - 1) / cus;
  bool use_pers = R > 0 && pers == 1;
  if (R > 0 && pers < 0 && rounds > 1) {
    const int64_t list = (nb + R - 1) / R;
    const bool head_a_cu = D >= 96 && R == 1 && nb <= 8 && 10 * N >= 7 * cus && 3 * list <= 4 * rounds;
    if (P.causal) use_pers = nb >= 2 * R && (list <= rounds + (D >= 128 ? 2 : 10 * R * N > 9 * cus ? 1 : 0) || (head_a_cu && (N % 8 != 0 || nb <= 6)));
    else use_pers = list <= rounds + (D >= 128 && nb <= 4 ? 1 : 0) || (head_a_cu && N % 8 != 0);
  }
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
                                           const float* delta, void* dk, void* dv, uint16_t* ds_ws, int pers, hipStream_t st) {
  switch (P.d) {
    case 64: return bwd_dkdv_split_d<64>(P, q, k, v, lse, dO, delta, dk, dv, ds_ws, pers, st);
    case 96: return bwd_dkdv_split_d<96>(P, q, k, v, lse, dO, delta, dk, dv, ds_ws, pers, st);
    case 128: return bwd_dkdv_split_d<128>(P, q, k, v, lse, dO, delta, dk, dv, ds_ws, pers, st);
    case 160: return bwd_dkdv_split_d<160>(P, q, k, v, lse, dO, delta, dk, dv, ds_ws, pers, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace sar
