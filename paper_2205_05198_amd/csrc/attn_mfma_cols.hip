// bf16 attention core, backward column pass (dK, dV): which of its forms runs.
#include "sar_internal.h"

#include <atomic>

namespace sar {

// form of the column pass: -1 = the library's choice; 0 plain (d = 64, 96), 2 producer / consumer waves, 3 the same with
// persistent workgroups (a forced form that does not exist falls back: 0 at d = 128, 160 to 2; 1 to 0; 3 to 2)
static std::atomic<int> g_force_form{-1};
void attn_mfma_force_dkdv_pipelined(int force) { g_force_form = force; }

hipError_t launch_attn_bwd_dkdv_mfma_small(const AttnParams& P, const void* q, const void* k, const void* v, const float* lse, const void* dO,
                                           const float* delta, void* dk, void* dv, uint16_t* ds_ws, hipStream_t st);  // attn_mfma_cols_small.hip
hipError_t launch_attn_bwd_dkdv_mfma_split(const AttnParams& P, const void* q, const void* k, const void* v, const float* lse, const void* dO,
                                           const float* delta, void* dk, void* dv, uint16_t* ds_ws, int pers, hipStream_t st);  // attn_mfma_cols_split.hip

// the producer / consumer form, rather than the plain one?
static bool dkdv_split(const AttnParams& P, const uint16_t* ds_ws) {
  const int force = g_force_form.load();
  // measured (once-form, us): 530B shard 78.6 / 80.2 / 69.6, 175B 70.4 / 60.5 / 48.1, 1T 98.3 / - / 90.0 for the plain, a software-
  // pipelined one-wave form and this one;
  // s = 1000, 24 heads, whole backward, plain / this: d = 128 54.6 / 40.2, d = 160 63.5 / 45.0 (without the tiles 54.0 / 45.2, 59.8 / 50.9)
  if (P.d >= 128) return true;
  if (force >= 0) return force >= 2;
  if (ds_ws && P.s % 64 == 0) return true;
  // Without dropout, or without the tiles to store, two plain workgroups on a CU are as good once the launch keeps both busy.
  // Whole backward at d = 64, plain / this, us: s = 2048, 12 heads, causal 58.5 / 47.5; no mask, s = 1000, 24 heads (384
  // workgroups) 42.4 / 44.2; s = 2048, 64 heads 301 / 302 and (p = 0.1, persistent) 376 / 366; s = 1000, 24 heads, causal,
  // p = 0.1, with tiles 37.9 / 30.5.  d = 96: 71.0 / 63.0, 52.1 / 55.6, 397 / 414, 481 / 474, 48.1 / 35.9.
  const int64_t blocks = (int64_t)((P.s + 63) / 64) * P.b * P.A;
  return P.thresh != 0 || blocks <= (P.causal ? 2 : 1) * attn_mfma_cu_count();
}

// persistent workgroups in the producer / consumer form: -1 the launcher decides by shape, 0 / 1 forced
static int split_pers() {
  const int force = g_force_form.load();
  return force == 2 ? 0 : force == 3 ? 1 : -1;
}

hipError_t launch_attn_bwd_dkdv_mfma(const AttnParams& P, const void* q, const void* k, const void* v, const float* lse, const void* dO,
                                     const float* delta, void* dk, void* dv, uint16_t* ds_ws, hipStream_t st) {
  if (dkdv_split(P, ds_ws)) return launch_attn_bwd_dkdv_mfma_split(P, q, k, v, lse, dO, delta, dk, dv, ds_ws, split_pers(), st);
  return launch_attn_bwd_dkdv_mfma_small(P, q, k, v, lse, dO, delta, dk, dv, ds_ws, st);
}

}  // namespace sar
