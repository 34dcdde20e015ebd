// bf16 attention core, backward column pass (dK, dV): which of its forms runs.
#include "sar_internal.h"

#include <algorithm>
#include <atomic>

namespace sar {

// form of the column pass: -1 = the library's choice; 0 plain (d = 64, 96), 2 producer / consumer waves, 3 the same with
// persistent workgroups (a forced form that does not exist falls back: 0 to 2 at d = 128, 160 and, with dropout and the tiles, at d = 96; 1 to 0; 3 to 2)
static std::atomic<int> g_force_form{-1};
void attn_mfma_force_dkdv_pipelined(int force) { g_force_form = force; }
// most key blocks of one launch of the producer / consumer form: <= 0 what a grid holds (tests force the division of a launch)
static std::atomic<int> g_force_grid_blocks{-1};
void attn_mfma_force_grid_blocks(int force) { g_force_grid_blocks = force; }

hipError_t launch_attn_bwd_dkdv_mfma_small(const AttnParams& P, const void* q, const void* k, const void* v, const float* lse, const void* dO,
                                           const float* delta, void* dk, void* dv, uint16_t* ds_ws, hipStream_t st);  // attn_mfma_cols_small.hip
hipError_t launch_attn_bwd_dkdv_mfma_split(const AttnParams& P, const void* q, const void* k, const void* v, const float* lse, const void* dO,
                                           const float* delta, void* dk, void* dv, uint16_t* ds_ws, int pers, hipStream_t st);  // attn_mfma_cols_split.hip

// The producer / consumer form, rather than the plain one?  From a sweep of both over 1140 shapes with and without the tiles (s = 64 .. 8192,
// 4 .. 256 heads); s x heads, us, plain / this, p = 0.1 under the mask unless said otherwise; blocks: workgroups of 64 keys.
//   d = 128, 160 have no plain form (s = 1000, 24 heads, whole backward: d = 128 54.6 / 40.2, d = 160 63.5 / 45.0).
//   Up to one block a CU always this one (2048 x 12 39.7 / 26.6).  Above, two plain workgroups share a CU and start sooner:
//   more than four blocks a CU: plain unless persistent workgroups come out even on full tiles (d = 64 512 x 192 36.0 / 40.7, but 384 x 256
//     32.5 / 30.7; 1000 x 128, no mask, 138 / 147; d = 96 with the tiles without dropout 512 x 192 46.7 / 54.4, with it 58.8 / 55.8; d = 96 without
//     the tiles always, 512 x 256 56.4 / 61.8, 3712 x 24 without dropout 148 / 157);
//   with the tiles to store also without mask and dropout on sequences that end inside a tile (d = 64 1000 x 24 29.0 / 30.1);
//   without them also heads of four blocks or less from one and a half a CU on (200 x 192 13.6 / 15.4; six blocks: 384 x 96 12.9 / 14.6), and without
//     dropout: no mask and more than one a CU (d = 96 1000 x 20 28.4 / 34.1), under the mask two (d = 64 1000 x 40 20.2 / 22.6);
//     with dropout only d = 96, no mask, up to one and a half a CU (1000 x 20 33.2 / 35.3);
//   heads of three to five blocks, one a CU: this one where persistent workgroups come out even, with dropout and no tiles (d = 96 256 x 210 48.9 / 45.6,
//     no mask 60.9 / 56.9) or with the tiles under the mask (200 x 210 40.4 / 38.3); without dropout, mask and tiles the plain one on single blocks (d = 64
//     64 x 320 12.5 / 14.0) and, where they do not come out even, up to eight (d = 64 320 x 180 37.6 / 41.8, but 2048 x 24 73.6 / 67.0).
static bool dkdv_split(const AttnParams& P, const uint16_t* ds_ws) {
  const int force = g_force_form.load();
  const bool drop = P.thresh != 0, causal = P.causal != 0, ragged = P.s % 64 != 0;
  if (P.d >= 128 || (P.d == 96 && ds_ws && drop)) return true;
  if (force >= 0) return force >= 2;
  const int64_t nb = (P.s + 63) / 64, N = (int64_t)P.b * P.A, blocks = nb * N, cus = attn_mfma_cu_count();
  const int64_t R = N <= cus ? std::min(nb, cus / N) : 0;  // key blocks of a head at a time, persistent
  const bool even = R > 0 && (nb + R - 1) / R <= (blocks + cus - 1) / cus;
  if (ds_ws && nb <= 4) return !(ragged && !drop && 2 * blocks > 5 * cus && !(causal && even));
  if (!ds_ws && drop && even && R == 1 && N < cus && nb >= 3 && nb <= 5) return true;
  if (nb <= 4) return 2 * blocks < 3 * cus && (nb > 1 || drop || causal || blocks <= cus);
  if (blocks > 4 * cus && (!even || ragged || (P.d == 96 && !ds_ws))) return false;
  if (ds_ws) return !(ragged && !drop && !causal && blocks > cus);
  if (nb <= 6 && blocks > 2 * cus && 2 * blocks <= 5 * cus) return false;
  if (drop) return !(P.d == 96 && ragged && !causal && blocks > cus && 2 * blocks <= 3 * cus);
  return causal ? blocks <= 2 * cus || (P.d == 96 && !ragged) : blocks <= cus || (P.d == 64 && !ragged && (even || nb > 8));
}

// persistent workgroups in the producer / consumer form: -1 the launcher decides by shape, 0 / 1 forced
static int split_pers() {
  const int force = g_force_form.load();
  return force == 2 ? 0 : force == 3 ? 1 : -1;
}

// A grid holds fewer than 2^32 threads, with 768 a workgroup 5.6 million key blocks: more of them (65535 heads of 86 blocks and up) go in
// two launches, each with half of the batches, or of one batch's heads.
static constexpr int64_t kGridBlocks = ((1ll << 32) - 1) / 768;
static hipError_t launch_split(const AttnParams& P, const void* q, const void* k, const void* v, const float* lse, const void* dO, const float* delta, void* dk,
                               void* dv, uint16_t* ds_ws, int pers, hipStream_t st) {
  const int64_t nb = (P.s + 63) / 64, N = (int64_t)P.b * P.A;
  const int force = g_force_grid_blocks.load();
  if (N == 1 || nb * N <= (force > 0 ? force : kGridBlocks)) return launch_attn_bwd_dkdv_mfma_split(P, q, k, v, lse, dO, delta, dk, dv, ds_ws, pers, st);
  AttnParams lo = P, hi = P;
  int64_t at, n;  // elements and heads before the upper half
  if (P.b > 1) {
    lo.b = P.b / 2;
    hi.b = P.b - lo.b;
    at = lo.b * P.stride_b;
    n = (int64_t)lo.b * P.A;
    hi.offset += (uint64_t)lo.b * (uint64_t)P.a_global * (uint64_t)P.s * (uint64_t)(P.s >> 3);
  } else {
    lo.A = P.A / 2;
    hi.A = P.A - lo.A;
    hi.head0 += lo.A;
    at = lo.A * P.stride_a;
    n = lo.A;
  }
  if (const hipError_t e = launch_split(lo, q, k, v, lse, dO, delta, dk, dv, ds_ws, pers, st); e != hipSuccess) return e;
  auto in = [&](const void* t) { return (const void*)((const uint16_t*)t + at); };
  auto out = [&](void* t) { return (void*)((uint16_t*)t + at); };
  return launch_split(hi, in(q), in(k), in(v), lse + n * P.s, in(dO), delta + n * P.s, out(dk), out(dv),
                      ds_ws ? ds_ws + n * ds_tiles_per_head(P) * kDsTileElems : nullptr, pers, st);
}

hipError_t launch_attn_bwd_dkdv_mfma(const AttnParams& P, const void* q, const void* k, const void* v, const float* lse, const void* dO,
                                     const float* delta, void* dk, void* dv, uint16_t* ds_ws, hipStream_t st) {
  if (dkdv_split(P, ds_ws)) return launch_split(P, q, k, v, lse, dO, delta, dk, dv, ds_ws, split_pers(), st);
  return launch_attn_bwd_dkdv_mfma_small(P, q, k, v, lse, dO, delta, dk, dv, ds_ws, st);
}

}  // namespace sar
