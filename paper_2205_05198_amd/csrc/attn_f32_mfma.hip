// Attention core with selective recomputation (Section 5) on the fp32 matrix instructions: the fp32 dtype, and bf16 inputs whose
// head dimension or score scale the bf16 kernels do not cover.  Any head dimension d % 4 == 0 up to 256.
//
// Every contraction is v_mfma_f32_32x32x2_f32: fp32 inputs, fp32 accumulation.  Lane = 32*hh + li:
//   A: lane holds row li, k = hh     B: lane holds column li, k = hh     D: lane holds column li, rows 8*g + 4*hh + r in acc[4*g + r]
// A result tile is directly the B operand of a second product whose k runs over its rows: register 4g + r supplies k = rows
// 8g + r (lanes hh = 0) and 8g + 4 + r (hh = 1), so neither the probabilities nor dS ever change layout, and which rows those
// are is only a matter of which rows of the other operand a lane reads.
//
// One matrix instruction takes 64 cycles of its SIMD for 256 bytes of either operand, so operands come straight from global
// memory (L1 / L2) without staging: rows as 16-byte pieces along the head dimension (4 consecutive k of one row per lane), and
// columns as coalesced reads along the head dimension.  A workgroup owns 32 query rows (forward, row pass) or 32 keys (column
// pass), keeps their operands in LDS, and its four waves take every fourth 32-wide tile of the other dimension; they meet once,
// at the end, to add their partial results in a fixed order.  No barrier inside the tile loop.  Bound: the fp32 matrix rate.
// Measured at s = 1024, 24 heads of 64, causal, against the plain one-wave-per-row kernels that these replace: forward
// 558 -> 52 us, row pass 928 -> 71, column pass 1043 -> 93 (62, 68 and 69 TFLOP/s of the 154 that a large product reaches).
#include "sar_device.h"
#include "sar_internal.h"

namespace sar {
namespace {

constexpr float kLog2eF = 1.4426950408889634f, kLn2F = 0.6931471805599453f;
constexpr float kLazyF = 60.0f;  // the running reference exponent moves only when a row maximum grew by > 2^60
constexpr int NWF = 4;           // waves of a workgroup

__device__ __forceinline__ float16_t mfma2(float a, float b, float16_t c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

__device__ __forceinline__ float4_t load4(const float* p) { return *reinterpret_cast<const float4_t*>(p); }
__device__ __forceinline__ float4_t load4(const uint16_t* p) {
  const uint2 u = *reinterpret_cast<const uint2*>(p);
  float4_t f = {__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xffff0000u)};
  return f;
}

__device__ __forceinline__ float xhalf_maxf(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// DT = columns of 32 that cover the head dimension.  Column m of a 32-wide operand or result stands for the DT consecutive
// elements col_start(m) .. + DT - 1 of a row (tile dt of the DT matrix products takes the dt-th of them), so that a lane reads
// and writes runs of DT elements.  Where 32 DT > d the last runs overlap: those elements are computed and written twice, equal.
template <int DT>
__device__ __forceinline__ int col_start(int m, int d) { return min(DT * m, d - DT); }

template <int DT>
__device__ __forceinline__ void load_cols(const float* p, float (&f)[DT]) {
  struct __attribute__((packed, aligned(4))) run { float v[DT]; };
  const run r = *reinterpret_cast<const run*>(p);
#pragma unroll
  for (int e = 0; e < DT; ++e) f[e] = r.v[e];
}
template <int DT>
__device__ __forceinline__ void load_cols(const uint16_t* p, float (&f)[DT]) {
#pragma unroll
  for (int e = 0; e < DT; ++e) f[e] = bf16_to_f32(p[e]);
}

// row of a 32-row operand tile -> key of the tile: bits 2 and 3 swapped, so that a lane's registers 8 c .. 8 c + 7 of a result
// whose rows are keys stand for the 8 consecutive keys 16 c + 8 hh .. + 7 (one Philox call)
__device__ __forceinline__ int swap23(int r) { return (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1); }

// LDS copy of 32 rows of a tensor, as fp32, zero beyond the head dimension; pitch 32 DT + 4
template <int DT, typename T>
__device__ __forceinline__ void rows_to_lds(float* dst, const T* g, int64_t gstride, int rows_valid, int d) {
  for (int c = threadIdx.x; c < 32 * 8 * DT; c += 64 * NWF) {
    const int r = c / (8 * DT), x = 4 * (c - r * 8 * DT);
    float4_t f = {0.f, 0.f, 0.f, 0.f};
    if (x < d) f = load4(g + (int64_t)min(r, rows_valid - 1) * gstride + x);
    *reinterpret_cast<float4_t*>(dst + r * (32 * DT + 4) + x) = f;
  }
}

// Operands that come from global memory are requested this far ahead of the matrix instruction that reads them (in floats per
// lane; a float is one 64-cycle instruction's worth, so 16 of them are a thousand cycles of one wave alone), in rings of registers.
constexpr int kAheadF = 16;

// Row operands: pieces of 4 consecutive elements (8 j + 4 hh) of one row per lane.  Pieces beyond the head dimension repeat the
// last one; the other operand is zero there.
constexpr int kRingF = kAheadF / 4;
template <int DT, typename T>
__device__ __forceinline__ float4_t load_piece(const T* row, int j, int hh, int d) {
  return load4(row + (j < 4 * (DT - 1) ? 8 * j + 4 * hh : min(8 * j + 4 * hh, d - 4)));  // d > 32 (DT - 1)
}
template <int DT, typename T>
__device__ __forceinline__ void ring_start(float4_t (&ring)[kRingF], const T* row, int hh, int d) {
#pragma unroll
  for (int j = 0; j < kRingF; ++j) ring[j] = load_piece<DT>(row, j, hh, d);
}
// 32 x 32 product over the head dimension of the row in `ring` / `row` and rows in LDS.  The ring is refilled with the rest of
// `row`, then (if `next` is not null) with the first pieces of `next`.  R0: ring slot of this row's piece 0.
template <int DT, int R0, typename T>
__device__ __forceinline__ float16_t dot_tile(float4_t (&ring)[kRingF], const T* row, const T* next, const float* lds_row, int hh, int d) {
  constexpr int NP = 4 * DT;
  float16_t acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  int off = 0;
  asm volatile("" : "+v"(off));  // the reads of LDS stay in the tile loop: hoisted out of it they would hold 16 DT registers
  lds_row += off;
  float4_t b = *reinterpret_cast<const float4_t*>(lds_row);
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    const float4_t a = ring[(R0 + j) % kRingF], bj = b;
    if (j + 1 < NP) b = *reinterpret_cast<const float4_t*>(lds_row + 8 * (j + 1));
#pragma unroll
    for (int u = 0; u < 4; ++u) acc = mfma2(a[u], bj[u], acc);
    asm volatile("" : "+v"(acc));  // in this place: left alone, the products sink below all of the loads
    ring[(R0 + j) % kRingF] = j + kRingF < NP ? load_piece<DT>(row, j + kRingF, hh, d) : load_piece<DT>(next, j + kRingF - NP, hh, d);
    __builtin_amdgcn_sched_barrier(0);
  }
  return acc;
}

// sum over the four waves of acc (one row of the output per lane li, columns 8 g + 4 hh + r), times mul, to rows 0 .. rows_valid-1
// of out.  buf: NWF * 32 * (8 DT + 4) floats; the waves' order is fixed.
template <int DT, typename T>
__device__ __forceinline__ void merge_store(const float16_t (&acc)[DT], float* buf, int wave, int li, int hh, float mul, T* out, int64_t gstride,
                                            int rows_valid, int d) {
  constexpr int PITCH = 8 * DT + 4;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    __syncthreads();
    float* w = buf + (wave * 32 + li) * PITCH + 4 * hh * DT;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) w[r * DT + dt] = acc[dt][4 * g + r];
    __syncthreads();
    const int row = threadIdx.x >> 3, m = threadIdx.x & 7;
    float s[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) s[dt] = buf[row * PITCH + m * DT + dt];
    for (int q = 1; q < NWF; ++q)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) s[dt] += buf[(q * 32 + row) * PITCH + m * DT + dt];
    if (row < rows_valid) {
      T* o = out + (int64_t)row * gstride + col_start<DT>(8 * g + m, d);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) Elem<T>::store(o + dt, s[dt] * mul);
    }
  }
}

// waves that share a SIMD: what the accumulators and the prefetched operands leave room for
constexpr int waves_rows(int DT) { return DT <= 2 ? 3 : 2; }
constexpr int waves_cols(int DT) { return DT <= 4 ? 2 : 1; }
constexpr int rows_ahead(int n) { return kAheadF / n < 2 ? 2 : kAheadF / n > 16 ? 16 : kAheadF / n; }  // n: floats of a row per lane

// ---------------------------------------------------------------------------------------------------
// forward: O, LSE of 32 query rows.  S^T = K Q^T (keys in rows), softmax along a lane's registers, O^T += V^T P^T.
// ---------------------------------------------------------------------------------------------------
template <int DT, bool DROP, typename T>
__global__ __launch_bounds__(64 * NWF, waves_rows(DT)) void attn_fwd_f32_kernel(AttnParams P, const T* __restrict__ q, const T* __restrict__ k,
                                                                              const T* __restrict__ v, T* __restrict__ o, float* __restrict__ lse) {
  constexpr int QP = 32 * DT + 4;
  __shared__ __attribute__((aligned(16))) float Qs[32 * QP];
  __shared__ __attribute__((aligned(16))) float buf[NWF * 32 * (8 * DT + 4)];
  __shared__ float ml[2][NWF][32];
  const int N = P.b * P.A, nrb = (P.s + 31) / 32;
  const int rb = nrb - 1 - (int)(blockIdx.x / N);  // heaviest row blocks first
  const int bn = blockIdx.x % N, beta = bn / P.A, n = bn % P.A;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, li = lane & 31, hh = lane >> 5;
  const int64_t base = (int64_t)beta * P.stride_b + (int64_t)n * P.stride_a;
  const int i0 = 32 * rb, i = i0 + li, i_ld = min(i, P.s - 1);
  const int jlim = P.causal ? i : P.s - 1;
  const int ntile = P.causal ? rb + 1 : nrb;
  rows_to_lds<DT>(Qs, q + base + (int64_t)i0 * P.stride_s, P.stride_s, P.s - i0, P.d);
  const uint64_t rowG = P.offset + (((uint64_t)beta * (uint64_t)P.a_global + (uint64_t)(P.head0 + n)) * (uint64_t)P.s + (uint64_t)i_ld) * (uint64_t)(P.s >> 3);
  const float sc2 = P.scale * kLog2eF;
  const T* kg = k + base;
  const T* vg = v + base + col_start<DT>(li, P.d);
  auto krow = [&](int jt) __attribute__((always_inline)) { return kg + (int64_t)min(32 * jt + swap23(li), P.s - 1) * P.stride_s; };
  float16_t oacc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) oacc[dt][e] = 0.f;
  float m_ref = -1.0e30f, l_run = 0.f;
  float4_t ring[kRingF];
  ring_start<DT>(ring, krow(wave), hh, P.d);
  __syncthreads();
  const float* qrow = Qs + li * QP + 4 * hh;
  constexpr int VA = rows_ahead(DT);
  for (int jt = wave; jt < ntile; jt += NWF) {
    const int j0 = 32 * jt;
    auto vrow = [&](int e) __attribute__((always_inline)) { return vg + (int64_t)min(j0 + 16 * (e >> 3) + 8 * hh + (e & 7), P.s - 1) * P.stride_s; };
    float vf[VA][DT];
#pragma unroll
    for (int e = 0; e < VA; ++e) load_cols<DT>(vrow(e), vf[e]);
    float16_t st = dot_tile<DT, 0>(ring, krow(jt), krow(jt + NWF), qrow, hh, P.d);
    float mt = -1.0e30f;
#pragma unroll
    for (int e = 0; e < 16; ++e) st[e] *= sc2;
    if (jt == ntile - 1) {  // keys beyond jlim (above the diagonal, or past the end) are masked
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (j0 + 16 * (e >> 3) + 8 * hh + (e & 7) > jlim) st[e] = -INFINITY;
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) mt = fmaxf(mt, st[e]);
    mt = xhalf_maxf(mt);
    if (__builtin_amdgcn_ballot_w64(mt > m_ref + kLazyF) != 0) {
      const float m_new = fmaxf(m_ref, mt), corr = __builtin_amdgcn_exp2f(m_ref - m_new);
      m_ref = m_new;
      l_run *= corr;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[dt][e] *= corr;
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      uint32_t keep = 0xffu;
      if (DROP) keep = keep_bits8(rowG + (uint64_t)((j0 + 16 * c + 8 * hh) >> 3), 0u, P.key0, P.key1, P.thresh);
#pragma unroll
      for (int x = 0; x < 8; ++x) {
        const int e = 8 * c + x;
        const float pe = __builtin_amdgcn_exp2f(st[e] - m_ref);
        l_run += pe;
        const float pd = !DROP || ((keep >> x) & 1u) ? pe : 0.f;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) oacc[dt] = mfma2(vf[e % VA][dt], pd, oacc[dt]);
        asm volatile("" : "+v"(oacc[0]));
        if (e + VA < 16) load_cols<DT>(vrow(e + VA), vf[e % VA]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  if (hh == 0) { ml[0][wave][li] = m_ref; ml[1][wave][li] = l_tot; }
  __syncthreads();
  float m = ml[0][0][li], l = 0.f;
  for (int w = 1; w < NWF; ++w) m = fmaxf(m, ml[0][w][li]);
  for (int w = 0; w < NWF; ++w) l = fmaf(ml[1][w][li], __builtin_amdgcn_exp2f(ml[0][w][li] - m), l);
  const float wgt = __builtin_amdgcn_exp2f(m_ref - m) * P.keep_scale / l;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) oacc[dt][e] *= wgt;
  if (wave == 0 && hh == 0 && i < P.s) lse[(size_t)bn * P.s + i] = (m + __builtin_amdgcn_logf(l)) * kLn2F;
  merge_store<DT>(oacc, buf, wave, li, hh, 1.f, o + base + (int64_t)i0 * P.stride_s, P.stride_s, P.s - i0, P.d);
}

// ---------------------------------------------------------------------------------------------------
// backward, row pass: delta_i = dO_i . O_i and dQ_i = alpha sum_j dS_ij K_j of 32 query rows.
// ---------------------------------------------------------------------------------------------------
template <int DT, bool DROP, typename T>
__global__ __launch_bounds__(64 * NWF, waves_rows(DT)) void attn_bwd_rows_f32_kernel(AttnParams P, const T* __restrict__ q, const T* __restrict__ k,
                                                                                   const T* __restrict__ v, const T* __restrict__ o,
                                                                                   const float* __restrict__ lse, const T* __restrict__ dO,
                                                                                   T* __restrict__ dq, float* __restrict__ delta) {
  constexpr int QP = 32 * DT + 4;
  __shared__ __attribute__((aligned(16))) float Qs[32 * QP], Gs[32 * QP];
  __shared__ __attribute__((aligned(16))) float buf[NWF * 32 * (8 * DT + 4)];
  __shared__ float part[32][8];
  const int N = P.b * P.A, nrb = (P.s + 31) / 32;
  const int rb = nrb - 1 - (int)(blockIdx.x / N);
  const int bn = blockIdx.x % N, beta = bn / P.A, n = bn % P.A;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, li = lane & 31, hh = lane >> 5;
  const int64_t base = (int64_t)beta * P.stride_b + (int64_t)n * P.stride_a;
  const int i0 = 32 * rb, i = i0 + li, i_ld = min(i, P.s - 1);
  const int jlim = P.causal ? i : P.s - 1;
  const int ntile = P.causal ? rb + 1 : nrb;
  rows_to_lds<DT>(Qs, q + base + (int64_t)i0 * P.stride_s, P.stride_s, P.s - i0, P.d);
  rows_to_lds<DT>(Gs, dO + base + (int64_t)i0 * P.stride_s, P.stride_s, P.s - i0, P.d);
  const T* kg = k + base;
  const T* vg = v + base;
  const T* kc = k + base + col_start<DT>(li, P.d);
  auto rowat = [&](int jt) __attribute__((always_inline)) { return (int64_t)min(32 * jt + swap23(li), P.s - 1) * P.stride_s; };
  float4_t ring[kRingF];
  ring_start<DT>(ring, kg + rowat(wave), hh, P.d);
  __syncthreads();
  {  // eight threads a row
    const int r = threadIdx.x >> 3, t8 = threadIdx.x & 7;
    const T* orow = o + base + (int64_t)min(i0 + r, P.s - 1) * P.stride_s;
    float a = 0.f;
    for (int x = 4 * t8; x < P.d; x += 32) {
      const float4_t f = load4(orow + x);
#pragma unroll
      for (int u = 0; u < 4; ++u) a = fmaf(f[u], Gs[r * QP + x + u], a);
    }
    part[r][t8] = a;
  }
  __syncthreads();
  float dl = 0.f;
#pragma unroll
  for (int t8 = 0; t8 < 8; ++t8) dl += part[li][t8];
  if (wave == 0 && hh == 0 && i < P.s) delta[(size_t)bn * P.s + i] = dl;
  const float lse2 = lse[(size_t)bn * P.s + i_ld] * kLog2eF;
  const uint64_t rowG = P.offset + (((uint64_t)beta * (uint64_t)P.a_global + (uint64_t)(P.head0 + n)) * (uint64_t)P.s + (uint64_t)i_ld) * (uint64_t)(P.s >> 3);
  const float sc2 = P.scale * kLog2eF;
  float16_t acc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[dt][e] = 0.f;
  constexpr int CA = rows_ahead(DT);
  for (int jt = wave; jt < ntile; jt += NWF) {
    const int j0 = 32 * jt;
    float16_t st = dot_tile<DT, 0>(ring, kg + rowat(jt), vg + rowat(jt), Qs + li * QP + 4 * hh, hh, P.d);
    auto crow = [&](int e) __attribute__((always_inline)) { return kc + (int64_t)min(j0 + 16 * (e >> 3) + 8 * hh + (e & 7), P.s - 1) * P.stride_s; };
    float cf[CA][DT];
#pragma unroll
    for (int e = 0; e < CA; ++e) load_cols<DT>(crow(e), cf[e]);
    const float16_t dd = dot_tile<DT, (4 * DT) % kRingF>(ring, vg + rowat(jt), kg + rowat(jt + NWF), Gs + li * QP + 4 * hh, hh, P.d);
#pragma unroll
    for (int e = 0; e < 16; ++e) st[e] = fmaf(st[e], sc2, -lse2);
    if (jt == ntile - 1) {
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (j0 + 16 * (e >> 3) + 8 * hh + (e & 7) > jlim) st[e] = -INFINITY;
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      uint32_t keep = 0xffu;
      if (DROP) keep = keep_bits8(rowG + (uint64_t)((j0 + 16 * c + 8 * hh) >> 3), 0u, P.key0, P.key1, P.thresh);
#pragma unroll
      for (int x = 0; x < 8; ++x) {
        const int e = 8 * c + x;
        const float pe = __builtin_amdgcn_exp2f(st[e]);
        const float dp = !DROP || ((keep >> x) & 1u) ? dd[e] * P.keep_scale : 0.f;
        const float ds = pe * (dp - dl);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) acc[dt] = mfma2(cf[e % CA][dt], ds, acc[dt]);
        asm volatile("" : "+v"(acc[0]));
        if (e + CA < 16) load_cols<DT>(crow(e + CA), cf[e % CA]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  merge_store<DT>(acc, buf, wave, li, hh, P.scale, dq + base + (int64_t)i0 * P.stride_s, P.stride_s, P.s - i0, P.d);
}

// ---------------------------------------------------------------------------------------------------
// backward, column pass: dK_j = alpha sum_i dS_ij q_i, dV_j = sum_i D_ij dO_i of 32 keys.  Scores the other way round, S = Q K^T:
// a lane owns one key, its registers are query rows, so D and dS are again B operands as they are.  One Philox call covers 8
// consecutive keys of a row = 8 lanes: each of the 8 lanes draws two of the 16 rows' calls and all read one another's bits.
// ---------------------------------------------------------------------------------------------------
template <int DT, bool DROP, typename T>
__global__ __launch_bounds__(64 * NWF, waves_cols(DT)) void attn_bwd_cols_f32_kernel(AttnParams P, const T* __restrict__ q, const T* __restrict__ k,
                                                                                   const T* __restrict__ v, const float* __restrict__ lse,
                                                                                   const T* __restrict__ dO, const float* __restrict__ delta,
                                                                                   T* __restrict__ dk, T* __restrict__ dv) {
  constexpr int QP = 32 * DT + 4;
  __shared__ __attribute__((aligned(16))) float Ks[32 * QP], Vs[32 * QP];
  __shared__ __attribute__((aligned(16))) float buf[NWF * 32 * (8 * DT + 4)];
  const int N = P.b * P.A, nb = (P.s + 31) / 32;
  const int kb = (int)(blockIdx.x / N);  // key block 0 sweeps the most rows: heaviest first
  const int bn = blockIdx.x % N, beta = bn / P.A, n = bn % P.A;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, li = lane & 31, hh = lane >> 5;
  const int64_t base = (int64_t)beta * P.stride_b + (int64_t)n * P.stride_a;
  const int j0 = 32 * kb, j = j0 + li;
  const int it0 = P.causal ? kb : 0;
  rows_to_lds<DT>(Ks, k + base + (int64_t)j0 * P.stride_s, P.stride_s, P.s - j0, P.d);
  rows_to_lds<DT>(Vs, v + base + (int64_t)j0 * P.stride_s, P.stride_s, P.s - j0, P.d);
  const T* qg = q + base;
  const T* gg = dO + base;
  const int cs = col_start<DT>(li, P.d);
  const float* lse_h = lse + (size_t)bn * P.s;
  const float* delta_h = delta + (size_t)bn * P.s;
  const uint64_t headG = P.offset + (((uint64_t)beta * (uint64_t)P.a_global + (uint64_t)(P.head0 + n)) * (uint64_t)P.s) * (uint64_t)(P.s >> 3) +
                         (uint64_t)((j0 + (li & 24)) >> 3);
  const float sc2 = P.scale * kLog2eF;
  float16_t ka[DT], va[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) { ka[dt][e] = 0.f; va[dt][e] = 0.f; }
  auto rowat = [&](int it) __attribute__((always_inline)) { return (int64_t)min(32 * it + li, P.s - 1) * P.stride_s; };
  float4_t ring[kRingF];
  ring_start<DT>(ring, qg + rowat(it0 + wave), hh, P.d);
  __syncthreads();
  constexpr int CA = rows_ahead(2 * DT);
  for (int it = it0 + wave; it < nb; it += NWF) {
    const int i0 = 32 * it;
    float16_t st = dot_tile<DT, 0>(ring, qg + rowat(it), gg + rowat(it), Ks + li * QP + 4 * hh, hh, P.d);
    // row e of this lane: i0 + 8 (e>>2) + 4 hh + (e&3); rows past the end get probability 0 (what they read is clamped)
    auto row_of = [&](int e) __attribute__((always_inline)) { return (int64_t)min(i0 + 8 * (e >> 2) + 4 * hh + (e & 3), P.s - 1) * P.stride_s + cs; };
    float gc[CA][DT], qc[CA][DT];
#pragma unroll
    for (int e = 0; e < CA; ++e) {
      load_cols<DT>(gg + row_of(e), gc[e]);
      load_cols<DT>(qg + row_of(e), qc[e]);
    }
    const float16_t dd = dot_tile<DT, (4 * DT) % kRingF>(ring, gg + rowat(it), qg + rowat(it + NWF), Vs + li * QP + 4 * hh, hh, P.d);
    float4_t dl[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int ib = min(i0 + 8 * g + 4 * hh, P.s - 4);  // s % 8 == 0: a group of four rows is inside or outside as a whole
      const float4_t ls = *reinterpret_cast<const float4_t*>(lse_h + ib);
      dl[g] = *reinterpret_cast<const float4_t*>(delta_h + ib);
#pragma unroll
      for (int r = 0; r < 4; ++r) st[4 * g + r] = fmaf(st[4 * g + r], sc2, -(ls[r] * kLog2eF));
    }
    if ((P.causal && it == kb) || i0 + 32 > P.s) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int i = i0 + 8 * (e >> 2) + 4 * hh + (e & 3);
        if ((P.causal && j > i) || i >= P.s) st[e] = -INFINITY;
      }
    }
    uint32_t mine = 0xffffu;
    if (DROP) {
      const int e0 = 2 * (li & 7);
      const uint64_t g0 = headG + (uint64_t)(i0 + 8 * (e0 >> 2) + 4 * hh + (e0 & 3)) * (uint64_t)(P.s >> 3);
      mine = keep_bits8(g0, 0u, P.key0, P.key1, P.thresh) | (keep_bits8(g0 + (uint64_t)(P.s >> 3), 0u, P.key0, P.key1, P.thresh) << 8);
    }
#define SAR_TWO_ROWS(X)                                                                                                     \
  {                                                                                                                         \
    uint32_t bits = mine;                                                                                                   \
    if (DROP) bits = (uint32_t)__builtin_amdgcn_ds_swizzle((int)mine, ((X) << 5) | 0x18) >> (li & 7);                       \
    _Pragma("unroll") for (int y = 0; y < 2; ++y) {                                                                         \
      constexpr int e_ = 2 * (X);                                                                                           \
      const int e = e_ + y;                                                                                                 \
      const bool keep = !DROP || ((bits >> (8 * y)) & 1u);                                                                  \
      const float pe = __builtin_amdgcn_exp2f(st[e]);                                                                       \
      const float pd = keep ? pe * P.keep_scale : 0.f, dp = keep ? dd[e] * P.keep_scale : 0.f;                              \
      const float ds = pe * (dp - dl[e >> 2][e & 3]);                                                                       \
      _Pragma("unroll") for (int dt = 0; dt < DT; ++dt) {                                                                   \
        va[dt] = mfma2(gc[e % CA][dt], pd, va[dt]);                                                                         \
        ka[dt] = mfma2(qc[e % CA][dt], ds, ka[dt]);                                                                         \
      }                                                                                                                     \
      asm volatile("" : "+v"(va[0]), "+v"(ka[0]));                                                                          \
      if (e + CA < 16) {                                                                                                    \
        load_cols<DT>(gg + row_of(e + CA), gc[e % CA]);                                                                     \
        load_cols<DT>(qg + row_of(e + CA), qc[e % CA]);                                                                     \
      }                                                                                                                     \
      __builtin_amdgcn_sched_barrier(0);                                                                                    \
    }                                                                                                                       \
  }
    SAR_TWO_ROWS(0) SAR_TWO_ROWS(1) SAR_TWO_ROWS(2) SAR_TWO_ROWS(3) SAR_TWO_ROWS(4) SAR_TWO_ROWS(5) SAR_TWO_ROWS(6) SAR_TWO_ROWS(7)
#undef SAR_TWO_ROWS
  }
  merge_store<DT>(va, buf, wave, li, hh, 1.f, dv + base + (int64_t)j0 * P.stride_s, P.stride_s, P.s - j0, P.d);
  merge_store<DT>(ka, buf, wave, li, hh, P.scale, dk + base + (int64_t)j0 * P.stride_s, P.stride_s, P.s - j0, P.d);
}

template <int DT, typename T>
hipError_t fwd_dt(const AttnParams& P, const void* q, const void* k, const void* v, void* o, float* lse, hipStream_t st) {
  const dim3 grid((unsigned)((P.s + 31) / 32 * P.b * P.A)), block(64 * NWF);
  auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, block, 0, st, P, (const T*)q, (const T*)k, (const T*)v, (T*)o, lse); };
  if (P.thresh != 0) go(attn_fwd_f32_kernel<DT, true, T>);
  else go(attn_fwd_f32_kernel<DT, false, T>);
  return hipGetLastError();
}

template <int DT, typename T>
hipError_t bwd_dt(const AttnParams& P, const void* q, const void* k, const void* v, const void* o, const float* lse, const void* dO, void* dq, void* dk,
                  void* dv, float* delta, int passes, hipStream_t st) {
  const dim3 grid((unsigned)((P.s + 31) / 32 * P.b * P.A)), block(64 * NWF);
  if (passes & 1) {
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, block, 0, st, P, (const T*)q, (const T*)k, (const T*)v, (const T*)o, lse, (const T*)dO, (T*)dq, delta); };
    if (P.thresh != 0) go(attn_bwd_rows_f32_kernel<DT, true, T>);
    else go(attn_bwd_rows_f32_kernel<DT, false, T>);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (passes & 2) {
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, block, 0, st, P, (const T*)q, (const T*)k, (const T*)v, lse, (const T*)dO, (const float*)delta, (T*)dk, (T*)dv); };
    if (P.thresh != 0) go(attn_bwd_cols_f32_kernel<DT, true, T>);
    else go(attn_bwd_cols_f32_kernel<DT, false, T>);
  }
  return hipGetLastError();
}

template <typename F>
hipError_t by_columns(int d, F&& f) {
  switch ((d + 31) / 32) {
    case 1: return f(std::integral_constant<int, 1>{});
    case 2: return f(std::integral_constant<int, 2>{});
    case 3: return f(std::integral_constant<int, 3>{});
    case 4: return f(std::integral_constant<int, 4>{});
    case 5: return f(std::integral_constant<int, 5>{});
    case 6: return f(std::integral_constant<int, 6>{});
    case 7: return f(std::integral_constant<int, 7>{});
    case 8: return f(std::integral_constant<int, 8>{});
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_attn_fwd_f32(const AttnParams& P, bool bf16, const void* q, const void* k, const void* v, void* o, float* lse, hipStream_t st) {
  return by_columns(P.d, [&](auto dt) {
    constexpr int DT = decltype(dt)::value;
    return bf16 ? fwd_dt<DT, uint16_t>(P, q, k, v, o, lse, st) : fwd_dt<DT, float>(P, q, k, v, o, lse, st);
  });
}

hipError_t launch_attn_bwd_f32(const AttnParams& P, bool bf16, const void* q, const void* k, const void* v, const void* o, const float* lse,
                               const void* dO, void* dq, void* dk, void* dv, float* delta, int passes, hipStream_t st) {
  return by_columns(P.d, [&](auto dt) {
    constexpr int DT = decltype(dt)::value;
    return bf16 ? bwd_dt<DT, uint16_t>(P, q, k, v, o, lse, dO, dq, dk, dv, delta, passes, st)
                : bwd_dt<DT, float>(P, q, k, v, o, lse, dO, dq, dk, dv, delta, passes, st);
  });
}

}  // namespace sar
