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
                                           const float* delta, void* dk, void* dv, uint16_t* ds_ws, int R, hipStream_t st);  // attn_mfma_cols_split.hip; R > 0: persistent, R key blocks of a head at a time

// The quantities that the choice of a form rests on: key blocks of a head, workgroups of one block, how many of them every CU gets one after the
// other, and the persistent grid: R key blocks of every head at a time, R x heads within the CU count, each workgroup with a list of `list` blocks.
struct ColShape {
  int64_t cus, N, nb, blocks, rounds, R, list;
  explicit ColShape(const AttnParams& P)
      : cus(attn_mfma_cu_count()), N((int64_t)P.b * P.A), nb((P.s + 63) / 64), blocks(nb * N), rounds((blocks + cus - 1) / cus),
        R(N <= cus ? std::min(nb, cus / N) : 0), list(R > 0 ? (nb + R - 1) / R : 0) {}
  bool even() const { return R > 0 && list <= rounds; }
  int64_t fill() const { return 100 * R * N / cus; }  // per cent of the CUs that a persistent grid occupies
};

// The producer / consumer form, rather than the plain one?  From a sweep of every form over 29571 shapes (s = 64 .. 8192, 1 .. 512 heads, with and without
// the tiles, mask, dropout), where this rule and the next take 1.003 times the best form's time in the
// geometric mean, no group of shapes above 1.006 (over 7087 other shapes 1.000, no head dimension above 1.003).
// Figures: s x heads, us, plain / producer / consumer as it then runs, p = 0.1 under the mask with the tiles unless said otherwise.
//   d = 128, 160, and d = 96 with dropout and tiles, have no plain form that keeps its registers.
//   Up to one workgroup a CU always this one (the plain one 1.05 to 1.37 of its time on heads of one to four blocks).  Above, two plain workgroups share a CU and start in half the time; this one makes up for it where persistent
//   workgroups hide the starts.  So:
//   lists no longer than the rounds of single blocks: this one (d = 64 512 x 128 27.6 / 24.1, 768 x 40 22.2 / 17.1; d = 96 without tiles 768 x 80 38.6 / 33.6),
//     but not heads of one or two blocks under the mask (d = 64 128 x 160 7.8 / 8.5; without the tiles also without mask 0.93), nor d = 96 with one list
//     a head of more than six blocks under it (512 x 256 without tiles 58.9 / 61.9; 0.88 to 0.98 without dropout);
//   lists longer: the plain one where the persistent grid would leave a quarter of the CUs empty, as it always does above one head a CU (d = 64 64 x 320
//     without tiles 6.1 / 8.0, 320 x 192 without tiles 17.3 / 19.9, 1024 x 192 131 / 137), under the mask on heads of more than twelve blocks also up to a seventh
//     with dropout (d = 64 0.97, d = 96 0.94) and a fourteenth without (d = 64 0.98, d = 96 0.96); not on long heads, where the starts weigh little: 37 blocks or more under
//     the mask with dropout (d = 64 2048 x 40 93.7 / 91.6 at 32 already), and without the mask, where every block is as long, 21 and 37 above one head a CU (d = 64 with dropout 13).
static bool dkdv_split(const AttnParams& P, const ColShape& c, bool tiles) {
  const int force = g_force_form.load();
  const bool drop = P.thresh != 0, causal = P.causal != 0;
  if (P.d >= 128 || (P.d == 96 && tiles && drop)) return true;
  if (force >= 0) return force >= 2;
  if (c.blocks <= c.cus) return true;
  if (c.even()) return !(c.nb <= 2 && (causal || (P.d == 64 && !tiles))) && !(causal && c.R == 1 && c.nb > 6 && P.d == 96);
  const int64_t fill = c.fill();
  if (!causal) return fill > 76 || c.nb > (drop && P.d == 64 ? 12 : c.R > 0 ? 20 : 36);
  return (drop && c.nb > 36) || fill > (c.nb <= 12 ? 76 : drop ? 85 : 93);
}

// Persistent workgroups in the producer / consumer form: each takes several key blocks of its head, a heavy one then a light one, and overlaps a
// block's start with the end of the one before.  From the same sweep; persistent workgroups' time over single blocks', or us single / persistent:
//   Lists no longer than the rounds of single blocks: yes (0.94 at every head dimension; d = 96 512 x 128 38.6 / 32.7; d = 160, no mask, 512 x 64 45.8 / 42.0, 248 x
//     128 29.3 / 27.2).  Under the mask, where some workgroups get one block and the others two, not below 1.15 blocks a CU on heads of seven or eight blocks, 1.3 up to
//     twelve, 1.5 up to twenty, 1.7 above (1.00 to 1.01 there, 0.92 to 0.98 above the lines); on heads of up to six always (0.90 to 0.99).
//   Lists one longer, one list a head: single blocks leave part of the CUs empty in their last round.  Heads no multiple of eight, which single blocks spread over all
//     dies so that each L2 reads all of their tiles: yes (0.92 to 0.97).  Otherwise d = 128, 160 (0.87 to 0.97) and 96 (0.88 to 0.99), except heads of three or four blocks
//     on less than two thirds of the CUs under the mask, and at d = 96 without it (1.04); d = 64 under the mask on three quarters and more (0.86 to 0.98), else 1.05.
//   Lists one longer, several a head: only under the mask, where a list's blocks are not all heavy, on heads of 7 to 20 blocks: d = 128 and 160 (0.90 to 0.99;
//     d = 160 from 5), d = 96 on more than three quarters of the CUs (0.94 to 1.00), d = 64 on more than 85 per cent (0.96).  Two longer: d = 128, 160 only (0.90 to 1.00).
static bool split_pers(const AttnParams& P, const ColShape& c) {
  const int force = g_force_form.load();
  if (c.R == 0) return false;
  if (force == 2 || force == 3) return force == 3;
  if (c.blocks <= c.cus) return false;
  const bool causal = P.causal != 0, wide = P.d >= 128;
  const int64_t over = c.list - c.rounds, fill = c.fill();
  if (over <= 0) return !causal || c.nb <= 6 || 100 * c.blocks >= (c.nb <= 8 ? 115 : c.nb <= 12 ? 130 : c.nb <= 20 ? 150 : 170) * c.cus;
  if (over == 1 && c.R == 1) return c.N % 8 != 0 || (P.d >= 96 ? c.nb >= 5 || fill > 68 || (wide && !causal) : causal && fill > 76);
  if (!causal || c.nb < (P.d == 160 ? 5 : 7) || c.nb > 20) return false;
  return wide ? over <= 2 : over == 1 && fill > (P.d == 96 ? 76 : 85);
}

// A grid holds fewer than 2^32 threads, with 768 a workgroup 5.6 million key blocks: more of them (65535 heads of 86 blocks and up) go in
// two launches, each with half of the batches, or of one batch's heads.
static constexpr int64_t kGridBlocks = ((1ll << 32) - 1) / 768;
static hipError_t launch_split(const AttnParams& P, const void* q, const void* k, const void* v, const float* lse, const void* dO, const float* delta, void* dk,
                               void* dv, uint16_t* ds_ws, int R, hipStream_t st) {
  const int64_t nb = (P.s + 63) / 64, N = (int64_t)P.b * P.A;
  const int force = g_force_grid_blocks.load();
  if (R > 0 || N == 1 || nb * N <= (force > 0 ? force : kGridBlocks)) return launch_attn_bwd_dkdv_mfma_split(P, q, k, v, lse, dO, delta, dk, dv, ds_ws, R, st);
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
  if (const hipError_t e = launch_split(lo, q, k, v, lse, dO, delta, dk, dv, ds_ws, 0, st); e != hipSuccess) return e;
  auto in = [&](const void* t) { return (const void*)((const uint16_t*)t + at); };
  auto out = [&](void* t) { return (void*)((uint16_t*)t + at); };
  return launch_split(hi, in(q), in(k), in(v), lse + n * P.s, in(dO), delta + n * P.s, out(dk), out(dv),
                      ds_ws ? ds_ws + n * ds_tiles_per_head(P) * kDsTileElems : nullptr, 0, st);
}

hipError_t launch_attn_bwd_dkdv_mfma(const AttnParams& P, const void* q, const void* k, const void* v, const float* lse, const void* dO,
                                     const float* delta, void* dk, void* dv, uint16_t* ds_ws, hipStream_t st) {
  const ColShape c(P);
  if (dkdv_split(P, c, ds_ws != nullptr)) return launch_split(P, q, k, v, lse, dO, delta, dk, dv, ds_ws, split_pers(P, c) ? (int)c.R : 0, st);
  return launch_attn_bwd_dkdv_mfma_small(P, q, k, v, lse, dO, delta, dk, dv, ds_ws, st);
}

int attn_mfma_cols_form(const AttnParams& P, bool tiles) {
  const ColShape c(P);
  return !dkdv_split(P, c, tiles) ? 0 : split_pers(P, c) ? 3 : 2;
}

}  // namespace sar
