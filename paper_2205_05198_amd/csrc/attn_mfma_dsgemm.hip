// bf16 attention core, the backward that recomputes the region of Section 5 once.
//
// The two-pass backward (attn_mfma_rows.hip row pass + column pass) regenerates softmax, the dropout mask and dO V^T in
// both passes, because dQ sums over keys and dK / dV over queries.  Here the column pass, which has every dS tile in
// registers anyway, also writes it out as bf16 (a backward-only scratch: nothing of it is kept from the forward), and dQ
// becomes a plain batched product over those tiles:
//   1. attn_bwd_delta_kernel      delta_i = sum_x dO_ix O_ix                      (reads dO, O once)
//   2. attn_bwd_dkdv_mfma_kernel  dK, dV, and dS tiles          (attn_mfma_cols_kernel.h, WDS = true)
//   3. attn_bwd_dq_gemm(128)_kernel dQ = alpha dS K                               (reads the tiles and K)
// 5 contractions are executed instead of 7, and Philox and the exponentials run once per backward instead of twice.
#include "attn_mfma_common.h"
#include <atomic>
#include <cmath>

namespace sar {

// sar_test_force_forms (tests, measurements) overrides the choices: -1 = by shape, 0 / 1 = off / on
static std::atomic<int> g_force_dq128{-1}, g_force_ds_stream{-1};
void attn_mfma_force_bwd_once(int dq128, int ds_stream) {
  g_force_dq128 = dq128;
  g_force_ds_stream = ds_stream;
}

// ---------------------------------------------------------------------------------------------------
// delta: one workgroup per 64 rows of one (batch, head).  Thread t takes the 16-byte chunks t, t + 256, ... of the
// block (chunk c = row c / CPR, piece c % CPR), the partial dot products meet in LDS and 64 threads add each row's
// CPR pieces in a fixed order (deterministic).
// ---------------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void attn_bwd_delta_kernel(AttnParams P, const uint16_t* __restrict__ o, const uint16_t* __restrict__ dO,
                                                            float* __restrict__ delta) {
  constexpr int CPR = D / 8, NCH = 64 * CPR;
  __shared__ float part[NCH];
  const int bn = blockIdx.y, beta = bn / P.A, n = bn % P.A;
  const int i0 = blockIdx.x * 64;
  const int64_t base = (int64_t)beta * P.stride_b + (int64_t)n * P.stride_a;
#pragma unroll
  for (int u = 0; u < (NCH + 255) / 256; ++u) {
    const int c = threadIdx.x + 256 * u;
    if (c < NCH) {
      const int r = c / CPR, cc = c - r * CPR;
      const int i = min(i0 + r, P.s - 1);
      const int64_t off = base + (int64_t)i * P.stride_s + 8 * cc;
      part[c] = dot8(ld_frag(dO + off), ld_frag(o + off));
    }
  }
  __syncthreads();
  if (threadIdx.x < 64 && i0 + (int)threadIdx.x < P.s) {
    float t = 0.f;
#pragma unroll
    for (int cc = 0; cc < CPR; ++cc) t += part[threadIdx.x * CPR + cc];
    delta[(size_t)bn * P.s + i0 + threadIdx.x] = t;
  }
}

// ---------------------------------------------------------------------------------------------------
// dQ = alpha dS K.  Workgroup = 64 query rows: 4 computing waves = 2 row groups x 2 key halves of each 64-key tile (summed
// through LDS at the end, as in the row pass of the two-pass backward) and 4 waves, one per SIMD, that only fetch the K
// tiles (rows swapped inside groups of 32, see attn_mfma_rows.hip) global -> LDS in pairs (one barrier per two tiles: the fixed cost of a barrier-to-barrier section, about 600 cycles
// beside 320 of matrix work per tile, is paid half as often), three stages of a pair each, two pairs ahead.
// The dS operand of a computing wave is 16 bytes per lane and 16-key group, read straight from the tile in the order
// the column pass wrote it, kDsAhead tiles ahead: the pass does little arithmetic per byte, so what bounds it is how many
// bytes a CU keeps in flight.  The computing waves issue no direct-to-LDS loads, so the compiler's own bookkeeping of
// their outstanding loads is exact and each step waits for its own operands only.
// ---------------------------------------------------------------------------------------------------
static constexpr int kDsAhead = 6;  // even: a round of the register ring is a whole number of tile pairs

template <int D>
__global__ __launch_bounds__(512, 1) void attn_bwd_dq_gemm_kernel(AttnParams P, const uint16_t* __restrict__ k, const uint16_t* __restrict__ ds_ws,
                                                                 uint16_t* __restrict__ dq) {
  constexpr int BM = 64, BN = 64, KP = D + 8, DT = D / 32, NS = 3;
  constexpr int TILE = BN * KP;
  // K stages of two tiles each (one barrier per pair of tiles); afterwards the exchange buffers, then the output tile
  __shared__ __attribute__((aligned(16))) uint16_t smem[NS * 2 * TILE];
  auto stage = [&](int jt) __attribute__((always_inline)) { return smem + (((jt >> 1) % NS) * 2 + (jt & 1)) * TILE; };

  const int N = P.b * P.A;
  const int nrb = (P.s + BM - 1) / BM;
  const int rb = nrb - 1 - (int)(blockIdx.x / N);  // heaviest row blocks first
  const int bn = blockIdx.x % N, beta = bn / P.A, n = bn % P.A;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, li = lane & 31, hh = lane >> 5;
  const int64_t base = (int64_t)beta * P.stride_b + (int64_t)n * P.stride_a;
  const int gstride = (int)P.stride_s;
  const int ntile = P.causal ? rb + 1 : nrb;
  if (wave >= 4) {  // a loader: same barriers as the computing waves
    const int lw = wave - 4;
    const uint16_t* kg = k + base;
    DmaMap<D> map;
    map.init(lw, lane, gstride, true);
    auto fetch = [&](int jt) __attribute__((always_inline)) {
      const int left = P.s - jt * BN;
      uint16_t* st2 = stage(jt);
      if (left >= BN) dma_tile<D>(map, kg + (int64_t)(jt * BN) * gstride, st2, lw);
      else dma_tile_ragged<D>(map, kg + (int64_t)(jt * BN) * gstride, st2, lw, lane, gstride, left);
    };
    for (int jt = 0; jt < 4 && jt < ntile; ++jt) fetch(jt);  // pairs 0 and 1
    for (int jt = 0; jt < ntile; jt += 2) {
      // the pair (jt, jt + 1) has landed; the loads of the next pair (at least DmaMap::PER - 1 per wave and tile) may
      // still be in flight
      const int later = ntile - (jt + 2);
      if (later >= 2) dma_wait_keep<2 * (DmaMap<D>::PER - 1)>();
      else if (later == 1) dma_wait_keep<DmaMap<D>::PER - 1>();
      else dma_wait();
      __syncthreads();  // top of the pair: its tiles are there, and nobody reads the pair before it (whose stage the pair after next takes) any more
      if (jt + 4 < ntile) fetch(jt + 4);
      if (jt + 5 < ntile) fetch(jt + 5);
    }
    __syncthreads();  // the four barriers of the others' epilogue
    __syncthreads();
    __syncthreads();
    __syncthreads();
    return;
  }
  const int rg = wave & 1, ks = wave >> 1;
  // this wave's 2 KB of tile (it = rb, kb = jt): key group c at + 512 c
  const uint16_t* dsw = ds_ws + (int64_t)bn * ds_tiles_per_head(P) * kDsTileElems + (2 * rg + ks) * 1024 + 8 * lane;
  auto ds_tile = [&](int jt) __attribute__((always_inline)) { return dsw + ds_tile_index(P, rb, jt) * kDsTileElems; };

  float16_t dqacc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) dqacc[dt][e] = 0.f;

  // One step: K tile jt against this wave's dS operands.  The operand reads run kAhead matrix instructions ahead, written
  // out (left to the compiler, every matrix instruction waits for a read issued just before it).
  auto step = [&](const int jt, bf16x8_t d0, bf16x8_t d1) __attribute__((always_inline)) {
    // the upper right quarter of the diagonal tile lies above the diagonal
    if (P.causal && jt == rb && rg == 0 && ks == 1) {
      const u32x4_t zero = {0u, 0u, 0u, 0u};
      d0 = __builtin_bit_cast(bf16x8_t, zero);
      d1 = __builtin_bit_cast(bf16x8_t, zero);
    }
    const uint16_t* Ks = stage(jt);
    constexpr int kAhead = 3, NF = 2 * DT;
    bf16x8_t fr[kAhead];
#pragma unroll
    for (int a = 0; a < kAhead; ++a) fr[a] = ld_frag_tr_perm(Ks, KP, 32 * ks + 16 * (a / DT), 32 * (a % DT), lane);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      dqacc[f % DT] = mfma32(fr[f % kAhead], f < DT ? d0 : d1, dqacc[f % DT]);
      if (f + kAhead < NF) fr[f % kAhead] = ld_frag_tr_perm(Ks, KP, 32 * ks + 16 * ((f + kAhead) / DT), 32 * ((f + kAhead) % DT), lane);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // dS operands kDsAhead tiles ahead, in a ring of registers with compile-time slots.  The main loop takes whole rounds of
  // the ring and has no condition inside (a load past the last tile re-reads the last tile); the remaining steps follow
  // without further loads.
  bf16x8_t ring[kDsAhead][2];
#pragma unroll
  for (int u = 0; u < kDsAhead; ++u) {
    const uint16_t* t = ds_tile(min(u, ntile - 1));
    ring[u][0] = ld_frag(t);
    ring[u][1] = ld_frag(t + 512);
  }
  int jt0 = 0;
  for (; jt0 + kDsAhead <= ntile; jt0 += kDsAhead) {
#pragma unroll
    for (int u = 0; u < kDsAhead; ++u) {
      if ((u & 1) == 0) __syncthreads();  // K tiles jt0 + u and jt0 + u + 1 are in their stage
      step(jt0 + u, ring[u][0], ring[u][1]);
      // refilled only now, when its last reader has been issued: the new load can then land in the same registers (loaded
      // at the top of the step it needs registers of its own, and the compiler moves every slot's value, load waited
      // for, around the back-edge)
      const uint16_t* t = ds_tile(min(jt0 + u + kDsAhead, ntile - 1));
      ring[u][0] = ld_frag(t);
      ring[u][1] = ld_frag(t + 512);
    }
  }
#pragma unroll
  for (int u = 0; u < kDsAhead - 1; ++u)
    if (jt0 + u < ntile) {
      if ((u & 1) == 0) __syncthreads();
      step(jt0 + u, ring[u][0], ring[u][1]);
    }
  // ---- sum the two key halves, scale, store ----
  __syncthreads();
  float* mg = reinterpret_cast<float*>(smem) + rg * (64 * 16 * DT);
  if (ks == 1) acc_put<DT>(mg, dqacc, lane);
  __syncthreads();
  if (ks == 0) acc_combine<DT>(mg, dqacc, 1.f, 1.f, lane);
  __syncthreads();  // the output tile overlaps both exchange buffers
  if (ks == 0) acc_to_lds_rows<DT>(smem, KP, 32 * rg + li, dqacc, P.scale, hh);
  __syncthreads();
  lds_rows_to_global<D>(smem, dq + base + (int64_t)(rb * BM) * P.stride_s, gstride, P.s - rb * BM, tid);
}

// The same product for 128 query rows: 4 computing waves, one per 32 rows, each over all 64 keys of a tile (no partial sums to
// merge), and 4 waves that fetch, now the dS tiles as well.  What bounds the 64-row form is the CU's path from the L2: loads into registers
// come at 32 B a cycle and direct loads into LDS at 62 (measured, hits in the L2), so a 64 x 64 step at d = 160 takes 8 KB / 32 + 21 KB / 62 =
// 600 cycles of it for 320 of matrix work.  Here dS goes through LDS and a K tile serves twice the rows: 300 cycles per 64 x 64.
template <int D>
__global__ __launch_bounds__(512, 1) void attn_bwd_dq_gemm128_kernel(AttnParams P, const uint16_t* __restrict__ k, const uint16_t* __restrict__ ds_ws,
                                                                    uint16_t* __restrict__ dq) {
  constexpr int BM = 128, BN = 64, KP = D + 8, DT = D / 32, NS = D == 64 ? 3 : 4, LA = NS - 1;
  constexpr int TILE = BN * KP, STAGE = TILE + 2 * kDsTileElems;
  __shared__ __attribute__((aligned(16))) uint16_t smem[NS * STAGE];  // stage: K tile, dS tiles of the upper and lower 64 rows; afterwards the output tiles
  const int N = P.b * P.A;
  const int nb = (P.s + 63) / 64, nrb = (P.s + BM - 1) / BM;
  const int rb = nrb - 1 - (int)(blockIdx.x / N);  // heaviest row blocks first
  const int bn = blockIdx.x % N, beta = bn / P.A, n = bn % P.A;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, li = lane & 31, hh = lane >> 5;
  const int64_t base = (int64_t)beta * P.stride_b + (int64_t)n * P.stride_a;
  const int gstride = (int)P.stride_s;
  const bool both = 2 * rb + 1 < nb;                          // the lower 64 rows exist
  const int ntile = P.causal ? 2 * rb + (both ? 2 : 1) : nb;  // tiles of the block; under the mask the upper rows have one less
  const int nt_up = P.causal ? 2 * rb + 1 : nb;
  if (wave >= 4) {  // a loader
    const int lw = wave - 4;
    constexpr int KMIN = DmaMap<D>::NL / 4;  // fewest loads of a K tile per wave; a dS tile is two
    const uint16_t* kg = k + base;
    const uint16_t* dsh = ds_ws + (int64_t)bn * ds_tiles_per_head(P) * kDsTileElems;
    DmaMap<D> map;
    map.init(lw, lane, gstride, true);
    auto fetch = [&](const int jt) __attribute__((always_inline)) {
      const int left = P.s - jt * BN;
      uint16_t* st = smem + (jt % NS) * STAGE;
      if (left >= BN) dma_tile<D>(map, kg + (int64_t)(jt * BN) * gstride, st, lw);
      else dma_tile_ragged<D>(map, kg + (int64_t)(jt * BN) * gstride, st, lw, lane, gstride, left);
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (h ? both : jt < nt_up) {
          const uint16_t* t = dsh + ds_tile_index(P, 2 * rb + h, jt) * kDsTileElems;
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const uint32_t dst = lds_addr(st + TILE + h * kDsTileElems) + 1024u * (uint32_t)(lw + 4 * u);
            if (P.ds_stream) dma16_nt(t + 512 * (lw + 4 * u), 16u * (uint32_t)lane, dst);
            else dma16(t + 512 * (lw + 4 * u), 16u * (uint32_t)lane, dst);
          }
        }
    };
    for (int jt = 0; jt < LA && jt < ntile; ++jt) fetch(jt);
    for (int jt = 0; jt < ntile; ++jt) {
      // tile jt has landed; the loads of the LA - 1 tiles after it may still be in flight (the last tile may hold one dS tile only)
      if (both && jt + LA < ntile) dma_wait_keep<(LA - 1) * (KMIN + 4)>();
      else if (LA > 2 && jt + 2 < ntile) dma_wait_keep<2 * (KMIN + 2)>();
      else if (jt + 1 < ntile) dma_wait_keep<KMIN + 2>();
      else dma_wait();
      __syncthreads();  // top of step jt: its tile is there, and nobody reads the one before it any more
      if (jt + LA < ntile) fetch(jt + LA);
    }
    __syncthreads();  // everybody is done with the last tile
    __syncthreads();  // the output tiles are complete
  } else {
    const int half = wave >> 1, rg = wave & 1;
    const bool mine = half == 0 || both;
    const int it = 2 * rb + half, nt_w = half == 0 ? nt_up : ntile;
    float16_t dqacc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int e = 0; e < 16; ++e) dqacc[dt][e] = 0.f;
    for (int jt = 0; jt < ntile; ++jt) {
      __syncthreads();
      if (!mine || jt >= nt_w) continue;
      const uint16_t* Ks = smem + (jt % NS) * STAGE;
      const uint16_t* Ds = Ks + TILE + half * kDsTileElems + 2048 * rg + 8 * lane;  // key group g (16 keys) at + 512 g
      constexpr int kAhead = 4, NF = 4 * DT;
      bf16x8_t d[4], fr[kAhead];
#pragma unroll
      for (int g = 0; g < 4; ++g) d[g] = ld_frag(Ds + 512 * g);
#pragma unroll
      for (int a = 0; a < kAhead; ++a) fr[a] = ld_frag_tr_perm(Ks, KP, 16 * (a / DT), 32 * (a % DT), lane);
      if (P.causal && jt == it && rg == 0) {  // the upper right quarter of the diagonal tile lies above the diagonal
        const u32x4_t zero = {0u, 0u, 0u, 0u};
        d[2] = __builtin_bit_cast(bf16x8_t, zero);
        d[3] = __builtin_bit_cast(bf16x8_t, zero);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        dqacc[f % DT] = mfma32(fr[f % kAhead], d[f / DT], dqacc[f % DT]);
        if (f + kAhead < NF) fr[f % kAhead] = ld_frag_tr_perm(Ks, KP, 16 * ((f + kAhead) / DT), 32 * ((f + kAhead) % DT), lane);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __syncthreads();
    if (mine) acc_to_lds_rows<DT>(smem + half * TILE, KP, 32 * rg + li, dqacc, P.scale, hh);
    __syncthreads();
  }
  const int half = tid >> 8;  // threads 0 .. 255 copy rows 0 .. 63 out, the loaders rows 64 .. 127
  lds_rows_to_global<D>(smem + half * TILE, dq + base + (int64_t)(rb * BM + 64 * half) * P.stride_s, gstride, P.s - rb * BM - 64 * half, tid & 255);
}

// The dQ product in blocks of 128 rows, rather than 64?  From both over 18317 shapes (s = 64 .. 8192, 1 .. 512 heads, more 64-row blocks than CUs), where this
// rule takes 1.001 times the faster one's time in the geometric mean, 1.002 in the worst group.  All blocks together take 0.6 to 0.85 of the 64-row form's time, as a K
// tile serves twice the rows; but one block is a chain one and a half times as long, and where the CUs get few of them the longest sets the pace.  s x heads, us, 64 / 128 rows:
//   Up to one 64-row block a CU: 64 (blocks of 128 would leave half of the CUs empty).
//   Without the mask, where all blocks are as long: 128 (d = 160 768 x 22, half a block a CU, 18.0 / 11.9; d = 128 768 x 24 13.8 / 11.2; d = 96 1024 x 80 48.1 /
//     41.1; d = 64 2048 x 64 124 / 100), but heads of three blocks, a quarter of whose rows is padding, where that costs a second round (d >= 96 1.02 to 1.11).
//   Under the mask the more tiles the heaviest block has, the more blocks a CU it takes to hide it: from a + b log2(nb / 8) hundredths of a 128-row block a CU
//     (nb tiles; d = 160 1024 x 20, 0.62 a CU, 11.3 / 12.0, 768 x 32, 0.75, 11.0 / 10.5, in the whole backward after the forward 56.6 / 55.0; d = 128 2048 x 12, 0.75, 15.5 / 21.8,
//     2048 x 16 18.6 / 22.4, 2048 x 20, 1.25, 25.7 / 23.4, 4096 x 24, 3, 122 / 93; d = 96 2048 x 16 16.7 / 17.7, 1024 x 32, 1.0, 11.6 / 11.2; d = 64 2048 x 16, 1.0, 14.2 / 16.9, 4096 x
//     20, 2.5, 74.7 / 68.4).  Where heads are a multiple of eight a die keeps their K in its L2, which helps the 64-row form: larger b (d = 160 2048 x 16, 1.0, 22.0 / 21.5 by itself but in the
//     whole layer's step 260.9 / 264.4; d = 64, two blocks a CU, 4096 x 16, 2.0, 51 / 60, but 17 heads 68 / 63).
template <int D>
static bool dq_rows128(const AttnParams& P) {
  if (const int force = g_force_dq128.load(); force >= 0) return force != 0;
  const int64_t cus = attn_mfma_cu_count(), N = (int64_t)P.b * P.A, nb = (P.s + 63) / 64, w128 = (nb + 1) / 2 * N;
  if (nb * N <= cus || (D >= 96 && nb == 3 && w128 > cus && 4 * w128 <= 5 * cus)) return false;
  if (!P.causal) return true;
  constexpr float a = D == 160 ? 49.f : D == 64 ? 70.f : 64.f, b_even[4] = {45.f, 20.f, 24.f, 26.f}, b_odd[4] = {28.f, 20.f, 20.f, 18.f};
  const float b = N % 8 == 0 ? b_even[D / 32 - 2] : b_odd[D / 32 - 2];
  return 100.f * (float)w128 >= (a + b * (std::log2((float)nb) - 3.f)) * (float)cus;
}

static bool ds_past_caches(const AttnParams& P) {  // the tiles do not fit the last-level cache: see ds_store2
  const int force = g_force_ds_stream.load();
  return force >= 0 ? force != 0 : (int64_t)P.b * P.A * ds_tiles_per_head(P) * kDsTileElems * 2 >= 256000000;
}

int attn_mfma_dq_form(const AttnParams& P0) {
  AttnParams P = P0;
  P.ds_stream = ds_past_caches(P);
  return (P.d == 64 ? dq_rows128<64>(P) : P.d == 96 ? dq_rows128<96>(P) : P.d == 128 ? dq_rows128<128>(P) : dq_rows128<160>(P)) + 2 * P.ds_stream;
}

template <int D>
static hipError_t bwd_once_d(const AttnParams& P0, const void* q, const void* k, const void* v, const void* o, const float* lse, const void* dO, void* dq,
                             void* dk, void* dv, float* delta, uint16_t* ds_ws, int stages, hipStream_t st) {
  const int N = P0.b * P0.A, nb = (P0.s + 63) / 64;
  AttnParams P = P0;
  P.ds_stream = ds_past_caches(P);
  hipError_t e = hipSuccess;
  if (stages & 1) {
    hipLaunchKernelGGL((attn_bwd_delta_kernel<D>), dim3((unsigned)nb, (unsigned)N), dim3(256), 0, st, P, (const uint16_t*)o, (const uint16_t*)dO, delta);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (stages & 2) {
    if ((e = launch_attn_bwd_dkdv_mfma(P, q, k, v, lse, dO, delta, dk, dv, ds_ws, st)) != hipSuccess) return e;
  }
  if (stages & 4) {
    auto go = [&](auto kern, int blocks) {
      hipLaunchKernelGGL(kern, dim3((unsigned)(blocks * N)), dim3(512), 0, st, P, (const uint16_t*)k, (const uint16_t*)ds_ws, (uint16_t*)dq);
    };
    if (dq_rows128<D>(P)) go(attn_bwd_dq_gemm128_kernel<D>, (nb + 1) / 2);
    else go(attn_bwd_dq_gemm_kernel<D>, nb);
    e = hipGetLastError();
  }
  return e;
}

hipError_t launch_attn_bwd_once_mfma(const AttnParams& P, const void* q, const void* k, const void* v, const void* o, const float* lse,
                                     const void* dO, void* dq, void* dk, void* dv, float* delta, uint16_t* ds_ws, int stages, hipStream_t st) {
  switch (P.d) {
    case 64: return bwd_once_d<64>(P, q, k, v, o, lse, dO, dq, dk, dv, delta, ds_ws, stages, st);
    case 96: return bwd_once_d<96>(P, q, k, v, o, lse, dO, dq, dk, dv, delta, ds_ws, stages, st);
    case 128: return bwd_once_d<128>(P, q, k, v, o, lse, dO, dq, dk, dv, delta, ds_ws, stages, st);
    case 160: return bwd_once_d<160>(P, q, k, v, o, lse, dO, dq, dk, dv, delta, ds_ws, stages, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace sar
