// Attention core with selective recomputation (Section 5) on the fp32 matrix instructions: the fp32 dtype, and bf16 inputs whose
// head dimension or score scale the bf16 kernels do not cover.  Any head dimension d % 4 == 0 up to 256.
//
// Every contraction is v_mfma_f32_{32x32x2,16x16x4}_f32: fp32 inputs, fp32 accumulation.  M = 32 or 16; lane = M*hh + li:
//   A: lane holds row li, k = hh     B: lane holds column li, k = hh
//   D: lane holds column li; M = 32: rows 8*g + 4*hh + r in acc[4*g + r]; M = 16: rows 4*hh + r in acc[r]
// A result tile is directly the B operand of a second product whose k runs over its rows: each register supplies one k for every
// hh, so neither the probabilities nor dS ever change layout, and which rows those are is only a matter of which rows of the
// other operand a lane reads.
//
// One M = 32 instruction takes 64 cycles of its SIMD for 256 bytes of either operand, so operands come straight from global
// memory (L1 / L2) without staging: rows as 16-byte pieces along the head dimension (4 consecutive k of one row per lane), and
// columns as coalesced reads along the head dimension.  A workgroup owns M query rows (forward, row pass) or M keys (column
// pass), keeps their operands in LDS, and its four waves take every fourth 32-wide tile of the other dimension; they meet once,
// at the end, to add their partial results in a fixed order.  No barrier inside the tile loop.  Bound: the fp32 matrix rate.
// Measured at s = 1024, 24 heads of 64, causal, against the plain one-wave-per-row kernels that these replace: forward and
// backward together 2538 -> 175 us (83 TFLOP/s of the nine contractions executed, of the 154 that a large product reaches).
#pragma once
#include <type_traits>
#include "sar_device.h"
#include "sar_internal.h"

namespace sar {
namespace {

constexpr float kLog2eF = 1.4426950408889634f, kLn2F = 0.6931471805599453f;
// The running reference of a row's exponentials moves only when its maximum grew by more than this (2^8): terms and their sums stay far
// from the end of the range.  It starts at the type's lowest value, which is below or equal to every score.
constexpr float kLazyF = 5.5f, kLowestF = -3.40282347e38f;
constexpr int NWF = 4;           // waves of a workgroup
constexpr int kTileF = 32;       // width of a step along the other dimension

template <int M> struct Geo;
template <> struct Geo<32> {
  typedef float16_t acc_t;
  static constexpr int HH = 2, SUB = 1, NV = 16;  // lanes along k, result tiles of a step, values of a step per lane
  static __device__ __forceinline__ acc_t mfma(float a, float b, acc_t c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
  // scores with keys in rows: the key of the tile that operand row m (of result tile t) stands for, and the key of value e of a lane:
  // a lane's values 8 c .. 8 c + 7 are 8 consecutive keys (one Philox call)
  static __device__ __forceinline__ int key_of_row(int, int m) { return (m & ~12) | ((m & 4) << 1) | ((m & 8) >> 1); }
  static __device__ __forceinline__ int key_of_value(int e, int hh) { return 16 * (e >> 3) + 8 * hh + (e & 7); }
  // scores with query rows in rows, in their natural order
  static __device__ __forceinline__ int row_of_row(int, int m) { return m; }
  static __device__ __forceinline__ int row_of_value(int e, int hh) { return 8 * (e >> 2) + 4 * hh + (e & 3); }
};
template <> struct Geo<16> {
  typedef float4_t acc_t;
  static constexpr int HH = 4, SUB = 2, NV = 8;
  static __device__ __forceinline__ acc_t mfma(float a, float b, acc_t c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  static __device__ __forceinline__ int key_of_row(int t, int m) { return 8 * (m >> 2) + 4 * t + (m & 3); }
  static __device__ __forceinline__ int key_of_value(int e, int hh) { return 8 * hh + e; }
  static __device__ __forceinline__ int row_of_row(int t, int m) { return 16 * t + m; }
  static __device__ __forceinline__ int row_of_value(int e, int hh) { return 16 * (e >> 2) + 4 * hh + (e & 3); }
};

// Operands in flight are held as they lie in memory and converted where they are used: a conversion next to the load waits for it.
__device__ __forceinline__ float lo_f32(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_f32(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
template <typename T> struct Raw4;  // 4 consecutive elements
template <> struct Raw4<float> { typedef float4_t type; };
template <> struct Raw4<uint16_t> { typedef uint2 type; };
__device__ __forceinline__ float4_t raw_load4(const float* p) { return *reinterpret_cast<const float4_t*>(p); }
__device__ __forceinline__ uint2 raw_load4(const uint16_t* p) { return *reinterpret_cast<const uint2*>(p); }
__device__ __forceinline__ float4_t get4(float4_t r) { return r; }
__device__ __forceinline__ float4_t get4(uint2 r) { return float4_t{lo_f32(r.x), hi_f32(r.x), lo_f32(r.y), hi_f32(r.y)}; }
template <typename T>
__device__ __forceinline__ float4_t load4(const T* p) { return get4(raw_load4(p)); }

__device__ __forceinline__ bool finite(float f) { return (__float_as_uint(f) & 0x7f800000u) != 0x7f800000u; }

// Scores stay in natural units until a difference of two is taken: score() rounds to the same value in the forward and in both
// backward passes, so that a score's distance from its row's log-sum-exp keeps the row's precision at any size of the scores.
__device__ __forceinline__ float score(float dot, float scale) {
#pragma clang fp contract(off)
  return dot * scale;
}
__device__ __forceinline__ float exp_diff(float a, float b) { return __builtin_amdgcn_exp2f((a - b) * kLog2eF); }

// over the lanes that hold one column
template <int M>
__device__ __forceinline__ float column_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  if (M == 16) v = fmaxf(v, __shfl_xor(v, 16, 64));
  return v;
}
template <int M>
__device__ __forceinline__ float column_sum(float v) {
  v += __shfl_xor(v, 32, 64);
  if (M == 16) v += __shfl_xor(v, 16, 64);
  return v;
}

// CT = column tiles of M that cover the head dimension.  Column m of an M-wide operand or result stands for the CT consecutive
// elements col_start(m) .. + CT - 1 of a row (tile ct of the CT matrix products takes the ct-th of them), so that a lane reads
// and writes runs of CT elements.  Where M CT > d the last runs overlap: those elements are computed and written twice, equal.
template <int CT>
__device__ __forceinline__ int col_start(int m, int d) { return min(CT * m, d - CT); }

template <typename T, int CT> struct Cols;  // such a run in flight
template <int CT> struct Cols<float, CT> {
  struct __attribute__((packed, aligned(4))) run { float v[CT]; } r;
  __device__ __forceinline__ void load(const float* p) { r = *reinterpret_cast<const run*>(p); }
  __device__ __forceinline__ float get(int e) const { return r.v[e]; }
};
template <int CT> struct Cols<uint16_t, CT> {  // d % 8 == 0: a run of even length starts at an even element
  struct __attribute__((packed, aligned(CT % 2 ? 2 : 4))) run { uint32_t v[CT / 2 ? CT / 2 : 1]; } r;
  uint16_t last;
  __device__ __forceinline__ void load(const uint16_t* p) {
    if (CT > 1) r = *reinterpret_cast<const run*>(p);
    if (CT % 2) last = p[CT - 1];
  }
  __device__ __forceinline__ float get(int e) const { return CT % 2 && e == CT - 1 ? bf16_to_f32(last) : e % 2 ? hi_f32(r.v[e / 2]) : lo_f32(r.v[e / 2]); }
};

template <int CT>
__device__ __forceinline__ void store_cols(float* p, const float (&f)[CT]) {
#pragma unroll
  for (int e = 0; e < CT; ++e) p[e] = f[e];
}
template <int CT>
__device__ __forceinline__ void store_cols(uint16_t* p, const float (&f)[CT]) {
  if constexpr (CT % 2 == 0) {
    struct __attribute__((packed, aligned(4))) run { uint32_t v[CT / 2]; } r;
#pragma unroll
    for (int e = 0; e < CT / 2; ++e) r.v[e] = pack_bf16x2(f[2 * e], f[2 * e + 1]);
    *reinterpret_cast<run*>(p) = r;
  } else {
#pragma unroll
    for (int e = 0; e < CT; ++e) p[e] = f32_to_bf16(f[e]);
  }
}

// Rows of a tensor in LDS, as fp32, zero beyond the head dimension; DT = 32-wide pieces that cover it, pitch 32 DT + 4
template <int M, int DT, typename T>
__device__ __forceinline__ void rows_to_lds(float* dst, const T* g, int64_t gstride, int rows_valid, int d) {
  constexpr int N = M * 8 * DT, U = (N + 64 * NWF - 1) / (64 * NWF);  // all loads of a thread in flight at once
  typename Raw4<T>::type f[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int c = threadIdx.x + 64 * NWF * u, r = c / (8 * DT), x = 4 * (c - r * 8 * DT);
    f[u] = raw_load4(g + (int64_t)min(r, rows_valid - 1) * gstride + min(x, d - 4));
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int c = threadIdx.x + 64 * NWF * u, r = c / (8 * DT), x = 4 * (c - r * 8 * DT);
    if (c < N) *reinterpret_cast<float4_t*>(dst + r * (32 * DT + 4) + x) = x < d ? get4(f[u]) : float4_t{0.f, 0.f, 0.f, 0.f};
  }
}

// Operands that come from global memory are requested this far ahead of the matrix instruction that reads them (in floats per
// lane; a float is one instruction's worth, 64 cycles at M = 32), in rings of registers.
constexpr int kAheadF = 16;
constexpr int rows_ahead(int n, int nv) { return kAheadF / n < 2 ? 2 : kAheadF / n > nv ? nv : kAheadF / n; }  // n: floats of a row per lane

// Row operands: pieces of 4 consecutive elements (4 (HH j + hh)) of one row per lane.  Pieces beyond the head dimension repeat the
// last one; the other operand is zero there (an infinity in the last piece makes a score NaN then, which the end of the kernels mends).
constexpr int kRingF = kAheadF / 4;
template <int M, int DT, typename T>
__device__ __forceinline__ typename Raw4<T>::type load_piece(const T* row, int j, int hh, int d) {
  constexpr int W = 4 * Geo<M>::HH;
  return raw_load4(row + (W * (j + 1) <= 32 * (DT - 1) ? W * j + 4 * hh : min(W * j + 4 * hh, d - 4)));  // d > 32 (DT - 1)
}
template <int M, int DT, typename T>
__device__ __forceinline__ void ring_start(typename Raw4<T>::type (&ring)[kRingF], const T* row, const T* next, int hh, int d) {
  constexpr int NP = 8 * DT / Geo<M>::HH;
#pragma unroll
  for (int j = 0; j < kRingF; ++j) ring[j] = j < NP ? load_piece<M, DT>(row, j, hh, d) : load_piece<M, DT>(next, j - NP, hh, d);
}
// M x M product over the head dimension of the row in `ring` / `row` and rows in LDS.  The ring is refilled with the rest of
// `row`, then with the first pieces of `next` (its pieces past the row after `next` with those of `after`).  R0: ring slot of this
// row's piece 0.
template <int M, int DT, int R0, typename T>
__device__ __forceinline__ typename Geo<M>::acc_t dot_tile(typename Raw4<T>::type (&ring)[kRingF], const T* row, const T* next, const T* after, const float* lds_row, int hh,
                                                           int d) {
  constexpr int NP = 8 * DT / Geo<M>::HH, W = 4 * Geo<M>::HH;
  typename Geo<M>::acc_t acc;
#pragma unroll
  for (int e = 0; e < Geo<M>::NV / Geo<M>::SUB; ++e) acc[e] = 0.f;
  int off = 0;
  asm volatile("" : "+v"(off));  // the reads of LDS stay in the tile loop: hoisted out of it they would hold 16 DT registers
  lds_row += off;
  float4_t b = *reinterpret_cast<const float4_t*>(lds_row);
  constexpr bool kConvert = sizeof(T) == 2;  // the next piece is converted beside this piece's products
  float4_t a_next;
  if (kConvert) a_next = get4(ring[R0 % kRingF]);
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    const float4_t a = kConvert ? a_next : get4(ring[(R0 + j) % kRingF]), bj = b;
    if (kConvert && j + 1 < NP) a_next = get4(ring[(R0 + j + 1) % kRingF]);
    if (j + 1 < NP) b = *reinterpret_cast<const float4_t*>(lds_row + W * (j + 1));
#pragma unroll
    for (int u = 0; u < 4; ++u) acc = Geo<M>::mfma(a[u], bj[u], acc);
    asm volatile("" : "+v"(acc));  // in this place: left alone, the products sink below all of the loads
    const int n = j + kRingF;  // piece that takes this slot
    ring[(R0 + j) % kRingF] = n < NP ? load_piece<M, DT>(row, n, hh, d) : n < 2 * NP ? load_piece<M, DT>(next, n - NP, hh, d) : load_piece<M, DT>(after, n - 2 * NP, hh, d);
    __builtin_amdgcn_sched_barrier(0);
  }
  return acc;
}

// sum over the four waves of acc (one row of the output per lane li), times mul, to rows 0 .. rows_valid - 1 of out.
// buf: NWF * M * (8 CT + 4) floats at M = 32 (eight columns m at a time), NWF * M * (16 CT + 4) at M = 16; the waves' order is fixed.
// A wave stores M / NWF consecutive rows, whole, from merge_row_of_wave on.  Returns whether this thread stored a value that is not finite.
template <int M, int CT>
constexpr int merge_pitch() { return (M == 32 ? 8 : 16) * CT + 4; }
template <int M, int CT, typename T>
__device__ __forceinline__ bool merge_store(const typename Geo<M>::acc_t (&acc)[CT], float* buf, int wave, int li, int hh, float mul, T* out, int64_t gstride,
                                            int rows_valid, int d) {
  constexpr int PITCH = merge_pitch<M, CT>(), NG = M == 32 ? 4 : 1, MM = M / NG;  // MM: columns m of a round
  bool odd = false;
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    __syncthreads();
    float* w = buf + (wave * M + li) * PITCH + 4 * hh * CT;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) w[r * CT + ct] = acc[ct][4 * g + r];
    __syncthreads();
    const int row = threadIdx.x / MM, m = threadIdx.x % MM;  // 256 threads = M x MM
    float s[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) s[ct] = buf[row * PITCH + m * CT + ct];
    for (int q = 1; q < NWF; ++q)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) s[ct] += buf[(q * M + row) * PITCH + m * CT + ct];
    if (row < rows_valid) {
      T* o = out + (int64_t)row * gstride + col_start<CT>(MM * g + m, d);
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        s[ct] *= mul;
        odd |= !finite(s[ct]);
      }
      store_cols<CT>(o, s);
    }
  }
  return odd;
}

// Pairs (i, j) that the mask excludes, and rows past the end, have probability 0 and take part in the matrix products of a tile all the
// same: 0 x infinity and 0 x NaN would reach outputs that the definition keeps them from.  A wave that has stored a value which is not
// finite therefore looks at the operands of its tiles with excluded pairs, and where one of those is not finite either, it computes
// the rows it stored again from the definition, over the allowed pairs only.  Where the head dimension is no multiple of 32 the products
// have excluded elements in every tile: there it computes them again whatever the operands are.  Finite results cost one compare each.
__device__ __forceinline__ bool wave_any(bool x) { return __builtin_amdgcn_ballot_w64(x) != 0; }
template <int M>
__device__ __forceinline__ int merge_row_of_wave(int wave) { return wave * (M / NWF); }  // the first; they are consecutive
template <typename T>
__device__ __forceinline__ bool any_odd(const T* g, int64_t gstride, int r0, int r1, int d) {  // this lane's share of rows r0 .. r1 - 1
  bool odd = false;
  for (int c = threadIdx.x & 63; c < (r1 - r0) * (d / 4); c += 64) {
    const float4_t f = load4(g + (int64_t)(r0 + c / (d / 4)) * gstride + 4 * (c % (d / 4)));
    odd |= !(finite(f[0]) && finite(f[1]) && finite(f[2]) && finite(f[3]));
  }
  return odd;
}
template <typename T>
__device__ __forceinline__ float dot_rows(const T* a, const T* b, int d) {
  float acc = 0.f;
  for (int x = 0; x < d; x += 4) {
    const float4_t fa = load4(a + x), fb = load4(b + x);
#pragma unroll
    for (int u = 0; u < 4; ++u) acc = fmaf(fa[u], fb[u], acc);
  }
  return acc;
}
// out = mul sum_{j = lo}^{hi - 1} weight(j) src_j; a lane draws the weight of every 64th j
template <typename T, typename W>
__device__ __forceinline__ void plain_row(W&& weight, int lo, int hi, const T* src, int64_t gstride, int d, float mul, T* out) {
  const int lane = threadIdx.x & 63;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int c0 = lo; c0 < hi; c0 += 64) {
    const float mine = c0 + lane < hi ? weight(c0 + lane) : 0.f;
    for (int y = 0; y < min(64, hi - c0); ++y) {
      const float w = __shfl(mine, y, 64);
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (lane + 64 * c < d) acc[c] = fmaf(w, Elem<T>::load(src + (int64_t)(c0 + y) * gstride + lane + 64 * c), acc[c]);
    }
  }
#pragma unroll
  for (int c = 0; c < 4; ++c)
    if (lane + 64 * c < d) Elem<T>::store(out + lane + 64 * c, acc[c] * mul);
}
// dropout decision of a single pair
template <bool DROP>
__device__ __forceinline__ bool kept_pair(const AttnParams& P, int beta, int n, int i, int j) {
  return !DROP || keep_bit1((((uint64_t)beta * (uint64_t)P.a_global + (uint64_t)(P.head0 + n)) * (uint64_t)P.s + (uint64_t)i) * (uint64_t)P.s + (uint64_t)j, P.offset,
                            0u, P.key0, P.key1, P.thresh);
}

// Work of workgroup blockIdx: heaviest first, every other round of 256 (one workgroup for each CU of the chip) the other way round, so that a CU that
// gets one of each round gets about the same work as the next (s = 1024, 24 heads, 768 workgroups: 196 -> 175 us for the whole
// forward and backward).
__device__ __forceinline__ int work_index() {
  const int b = blockIdx.x >> 8, c = blockIdx.x & 255, last = min(255, (int)gridDim.x - 1 - (b << 8));
  return (b << 8) + ((b & 1) ? last - c : c);
}

// Waves that share a SIMD: what the accumulators and the prefetched operands leave room for.  The column pass at M = 32, DT = 4 (head
// dimensions 100 to 128) spills 10 to 23 registers with two waves and none with one, and is the faster with two (whole backward,
// s = 1024, 24 heads of 128, causal: 257 us against 305; bf16, 104: 258 against 326).
constexpr int waves_rows(int M, int DT) { return M == 16 ? (DT <= 2 ? 4 : DT <= 4 ? 3 : 2) : DT <= 2 ? 3 : 2; }
constexpr int waves_cols(int M, int DT) { return M == 16 ? (DT <= 2 ? 3 : 2) : DT <= 4 ? 2 : 1; }

// ---------------------------------------------------------------------------------------------------
// forward: O, LSE of M query rows.  S^T = K Q^T (keys in rows), softmax along a lane's registers, O^T += V^T P^T.
// ---------------------------------------------------------------------------------------------------
template <int M, int DT, bool DROP, typename T>
__global__ __launch_bounds__(64 * NWF, waves_rows(M, DT)) void attn_fwd_f32_kernel(AttnParams P, const T* __restrict__ q, const T* __restrict__ k,
                                                                                 const T* __restrict__ v, T* __restrict__ o, float* __restrict__ lse) {
  typedef Geo<M> G;
  constexpr int QP = 32 * DT + 4, CT = 32 * DT / M, NV = G::NV;
  __shared__ __attribute__((aligned(16))) float Qs[M * QP];
  __shared__ __attribute__((aligned(16))) float buf[NWF * M * merge_pitch<M, CT>()];
  __shared__ float ml[2][NWF][M];
  const int N = P.b * P.A, nrb = (P.s + M - 1) / M, wi = work_index();
  const int rb = nrb - 1 - wi / N;  // heaviest row blocks first
  const int bn = wi % N, beta = bn / P.A, n = bn % P.A;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, li = lane & (M - 1), hh = lane / M;
  const int64_t base = (int64_t)beta * P.stride_b + (int64_t)n * P.stride_a;
  const int i0 = M * rb, i = i0 + li, i_ld = min(i, P.s - 1);
  const int jlim = P.causal ? i : P.s - 1;
  const int ntile = (P.causal ? min(i0 + M, P.s) : P.s) / kTileF + ((P.causal ? min(i0 + M, P.s) : P.s) % kTileF != 0);
  rows_to_lds<M, DT>(Qs, q + base + (int64_t)i0 * P.stride_s, P.stride_s, P.s - i0, P.d);
  const uint64_t rowG = P.offset + (((uint64_t)beta * (uint64_t)P.a_global + (uint64_t)(P.head0 + n)) * (uint64_t)P.s + (uint64_t)i_ld) * (uint64_t)(P.s >> 3);
  const T* kg = k + base;
  const T* vg = v + base + col_start<CT>(li, P.d);
  auto krow = [&](int jt, int t) __attribute__((always_inline)) { return kg + (int64_t)min(kTileF * jt + G::key_of_row(t, li), P.s - 1) * P.stride_s; };
  typename G::acc_t oacc[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int e = 0; e < NV / G::SUB; ++e) oacc[ct][e] = 0.f;
  float m_ref = kLowestF, l_run = 0.f;
  typename Raw4<T>::type ring[kRingF];
  ring_start<M, DT>(ring, krow(wave, 0), krow(wave, G::SUB - 1), hh, P.d);
  __syncthreads();
  const float* qrow = Qs + li * QP + 4 * hh;
  constexpr int VA = rows_ahead(CT, NV);
  for (int jt = wave; jt < ntile; jt += NWF) {
    const int j0 = kTileF * jt;
    auto vrow = [&](int e) __attribute__((always_inline)) { return vg + (int64_t)min(j0 + G::key_of_value(e, hh), P.s - 1) * P.stride_s; };
    Cols<T, CT> vf[VA];
#pragma unroll
    for (int e = 0; e < VA; ++e) vf[e].load(vrow(e));
    float st[NV];
    if constexpr (M == 32) {
      const float16_t s0 = dot_tile<M, DT, 0>(ring, krow(jt, 0), krow(jt + NWF, 0), krow(jt + NWF, 0), qrow, hh, P.d);
#pragma unroll
      for (int e = 0; e < NV; ++e) st[e] = score(s0[e], P.scale);
    } else {
      const float4_t s0 = dot_tile<M, DT, 0>(ring, krow(jt, 0), krow(jt, 1), krow(jt + NWF, 0), qrow, hh, P.d);
      const float4_t s1 = dot_tile<M, DT, (2 * DT) % kRingF>(ring, krow(jt, 1), krow(jt + NWF, 0), krow(jt + NWF, 1), qrow, hh, P.d);
#pragma unroll
      for (int e = 0; e < 4; ++e) { st[e] = score(s0[e], P.scale); st[4 + e] = score(s1[e], P.scale); }
    }
    float mt = kLowestF;
    if (jt == ntile - 1) {  // keys beyond jlim (above the diagonal, or past the end) are masked
#pragma unroll
      for (int e = 0; e < NV; ++e)
        if (j0 + G::key_of_value(e, hh) > jlim) st[e] = -INFINITY;
    }
#pragma unroll
    for (int e = 0; e < NV; ++e) mt = fmaxf(mt, st[e]);
    mt = column_max<M>(mt);
    if (__builtin_amdgcn_ballot_w64(mt > m_ref + kLazyF) != 0) {
      const float m_new = fmaxf(m_ref, mt), corr = exp_diff(m_ref, m_new);
      m_ref = m_new;
      l_run *= corr;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int e = 0; e < NV / G::SUB; ++e) oacc[ct][e] *= corr;
    }
#pragma unroll
    for (int c = 0; c < NV / 8; ++c) {
      uint32_t keep = 0xffu;
      if (DROP) keep = keep_bits8(rowG + (uint64_t)((j0 + G::key_of_value(8 * c, hh)) >> 3), 0u, P.key0, P.key1, P.thresh);
#pragma unroll
      for (int x = 0; x < 8; ++x) {
        const int e = 8 * c + x;
        const float pe = exp_diff(st[e], m_ref);
        l_run += pe;
        const float pd = !DROP || ((keep >> x) & 1u) ? pe : 0.f;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) oacc[ct] = G::mfma(vf[e % VA].get(ct), pd, oacc[ct]);
        asm volatile("" : "+v"(oacc[0]));
        if (e + VA < NV) vf[e % VA].load(vrow(e + VA));
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  const float l_tot = column_sum<M>(l_run);
  if (hh == 0) { ml[0][wave][li] = m_ref; ml[1][wave][li] = l_tot; }
  __syncthreads();
  float m = ml[0][0][li], l = 0.f;
  for (int w = 1; w < NWF; ++w) m = fmaxf(m, ml[0][w][li]);
  for (int w = 0; w < NWF; ++w) l = fmaf(ml[1][w][li], exp_diff(ml[0][w][li], m), l);
  const float wgt = exp_diff(m_ref, m) * P.keep_scale / l;
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int e = 0; e < NV / G::SUB; ++e) oacc[ct][e] *= wgt;
  const float lse_i = m + __builtin_amdgcn_logf(l) * kLn2F;
  if (wave == 0 && hh == 0 && i < P.s) lse[(size_t)bn * P.s + i] = lse_i;
  const bool odd = merge_store<M, CT>(oacc, buf, wave, li, hh, 1.f, o + base + (int64_t)i0 * P.stride_s, P.stride_s, P.s - i0, P.d);
  if (wave_any(odd)) {
    const int j0 = kTileF * (ntile - 1), r0 = i0 + merge_row_of_wave<M>(wave);
    if (P.d % 32 || ((P.causal || P.s % kTileF) && wave_any(any_odd(v + base, P.stride_s, j0, min(j0 + kTileF, P.s), P.d))))
      for (int r = r0; r < min(r0 + M / NWF, P.s); ++r) {
        const int end = P.causal ? r + 1 : P.s;
        auto scored = [&](int j) __attribute__((always_inline)) { return score(dot_rows(q + base + (int64_t)r * P.stride_s, k + base + (int64_t)j * P.stride_s, P.d), P.scale); };
        float mx = -INFINITY, sum = 0.f;
        for (int j = lane; j < end; j += 64) mx = fmaxf(mx, scored(j));
        mx = wave_max(mx);
        for (int j = lane; j < end; j += 64) sum += exp_diff(scored(j), mx);
        const float lse_r = mx + __builtin_amdgcn_logf(wave_sum(sum)) * kLn2F;
        if (lane == 0) lse[(size_t)bn * P.s + r] = lse_r;
        plain_row([&](int j) __attribute__((always_inline)) { return kept_pair<DROP>(P, beta, n, r, j) ? exp_diff(scored(j), lse_r) * P.keep_scale : 0.f; }, 0, end, v + base,
                  P.stride_s, P.d, 1.f, o + base + (int64_t)r * P.stride_s);
      }
  }
}

// ---------------------------------------------------------------------------------------------------
// backward, row pass: delta_i = dO_i . O_i and dQ_i = alpha sum_j dS_ij K_j of M query rows.
// ---------------------------------------------------------------------------------------------------
template <int M, int DT, bool DROP, typename T>
__global__ __launch_bounds__(64 * NWF, waves_rows(M, DT)) void attn_bwd_rows_f32_kernel(AttnParams P, const T* __restrict__ q, const T* __restrict__ k,
                                                                                      const T* __restrict__ v, const T* __restrict__ o,
                                                                                      const float* __restrict__ lse, const T* __restrict__ dO,
                                                                                      T* __restrict__ dq, float* __restrict__ delta) {
  typedef Geo<M> G;
  constexpr int QP = 32 * DT + 4, CT = 32 * DT / M, NV = G::NV, TPR = 64 * NWF / M;  // TPR: threads a row in the delta sums
  __shared__ __attribute__((aligned(16))) float Qs[M * QP], Gs[M * QP];
  __shared__ __attribute__((aligned(16))) float buf[NWF * M * merge_pitch<M, CT>()];
  __shared__ float part[M][TPR];
  const int N = P.b * P.A, nrb = (P.s + M - 1) / M, wi = work_index();
  const int rb = nrb - 1 - wi / N;
  const int bn = wi % N, beta = bn / P.A, n = bn % P.A;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, li = lane & (M - 1), hh = lane / M;
  const int64_t base = (int64_t)beta * P.stride_b + (int64_t)n * P.stride_a;
  const int i0 = M * rb, i = i0 + li, i_ld = min(i, P.s - 1);
  const int jlim = P.causal ? i : P.s - 1;
  const int ntile = ((P.causal ? min(i0 + M, P.s) : P.s) + kTileF - 1) / kTileF;
  rows_to_lds<M, DT>(Qs, q + base + (int64_t)i0 * P.stride_s, P.stride_s, P.s - i0, P.d);
  rows_to_lds<M, DT>(Gs, dO + base + (int64_t)i0 * P.stride_s, P.stride_s, P.s - i0, P.d);
  const T* kg = k + base;
  const T* vg = v + base;
  const T* kc = k + base + col_start<CT>(li, P.d);
  auto rowat = [&](int jt, int t) __attribute__((always_inline)) { return (int64_t)min(kTileF * jt + G::key_of_row(t, li), P.s - 1) * P.stride_s; };
  typename Raw4<T>::type ring[kRingF];
  ring_start<M, DT>(ring, kg + rowat(wave, 0), (M == 32 ? vg : kg) + rowat(wave, G::SUB - 1), hh, P.d);
  __syncthreads();
  {
    const int r = threadIdx.x / TPR, tr = threadIdx.x % TPR;
    const T* orow = o + base + (int64_t)min(i0 + r, P.s - 1) * P.stride_s;
    float a = 0.f;
    for (int x = 4 * tr; x < P.d; x += 4 * TPR) {
      const float4_t f = load4(orow + x);
#pragma unroll
      for (int u = 0; u < 4; ++u) a = fmaf(f[u], Gs[r * QP + x + u], a);
    }
    part[r][tr] = a;
  }
  __syncthreads();
  float dl = 0.f;
#pragma unroll
  for (int tr = 0; tr < TPR; ++tr) dl += part[li][tr];
  if (wave == 0 && hh == 0 && i < P.s) delta[(size_t)bn * P.s + i] = dl;
  const float lse_i = lse[(size_t)bn * P.s + i_ld];
  const uint64_t rowG = P.offset + (((uint64_t)beta * (uint64_t)P.a_global + (uint64_t)(P.head0 + n)) * (uint64_t)P.s + (uint64_t)i_ld) * (uint64_t)(P.s >> 3);
  typename G::acc_t acc[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int e = 0; e < NV / G::SUB; ++e) acc[ct][e] = 0.f;
  const float *qrow = Qs + li * QP + 4 * hh, *grow = Gs + li * QP + 4 * hh;
  constexpr int CA = rows_ahead(CT, NV);
  for (int jt = wave; jt < ntile; jt += NWF) {
    const int j0 = kTileF * jt;
    auto crow = [&](int e) __attribute__((always_inline)) { return kc + (int64_t)min(j0 + G::key_of_value(e, hh), P.s - 1) * P.stride_s; };
    Cols<T, CT> cf[CA];
    float st[NV], dd[NV];
    if constexpr (M == 32) {
      const float16_t s0 = dot_tile<M, DT, 0>(ring, kg + rowat(jt, 0), vg + rowat(jt, 0), vg + rowat(jt, 0), qrow, hh, P.d);
#pragma unroll
      for (int e = 0; e < CA; ++e) cf[e].load(crow(e));
      const float16_t d0 = dot_tile<M, DT, (4 * DT) % kRingF>(ring, vg + rowat(jt, 0), kg + rowat(jt + NWF, 0), kg + rowat(jt + NWF, 0), grow, hh, P.d);
#pragma unroll
      for (int e = 0; e < NV; ++e) { st[e] = s0[e]; dd[e] = d0[e]; }
    } else {
      const float4_t s0 = dot_tile<M, DT, 0>(ring, kg + rowat(jt, 0), kg + rowat(jt, 1), vg + rowat(jt, 0), qrow, hh, P.d);
      const float4_t s1 = dot_tile<M, DT, (2 * DT) % kRingF>(ring, kg + rowat(jt, 1), vg + rowat(jt, 0), vg + rowat(jt, 1), qrow, hh, P.d);
#pragma unroll
      for (int e = 0; e < CA; ++e) cf[e].load(crow(e));
      const float4_t d0 = dot_tile<M, DT, (4 * DT) % kRingF>(ring, vg + rowat(jt, 0), vg + rowat(jt, 1), kg + rowat(jt + NWF, 0), grow, hh, P.d);
      const float4_t d1 = dot_tile<M, DT, (6 * DT) % kRingF>(ring, vg + rowat(jt, 1), kg + rowat(jt + NWF, 0), kg + rowat(jt + NWF, 1), grow, hh, P.d);
#pragma unroll
      for (int e = 0; e < 4; ++e) { st[e] = s0[e]; st[4 + e] = s1[e]; dd[e] = d0[e]; dd[4 + e] = d1[e]; }
    }
#pragma unroll
    for (int e = 0; e < NV; ++e) st[e] = score(st[e], P.scale);
    if (jt == ntile - 1) {
#pragma unroll
      for (int e = 0; e < NV; ++e)
        if (j0 + G::key_of_value(e, hh) > jlim) st[e] = -INFINITY;
    }
#pragma unroll
    for (int c = 0; c < NV / 8; ++c) {
      uint32_t keep = 0xffu;
      if (DROP) keep = keep_bits8(rowG + (uint64_t)((j0 + G::key_of_value(8 * c, hh)) >> 3), 0u, P.key0, P.key1, P.thresh);
#pragma unroll
      for (int x = 0; x < 8; ++x) {
        const int e = 8 * c + x;
        const float pe = exp_diff(st[e], lse_i);
        const float dp = !DROP || ((keep >> x) & 1u) ? dd[e] * P.keep_scale : 0.f;
        const float ds = pe * (dp - dl);
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[ct] = G::mfma(cf[e % CA].get(ct), ds, acc[ct]);
        asm volatile("" : "+v"(acc[0]));
        if (e + CA < NV) cf[e % CA].load(crow(e + CA));
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  const bool odd = merge_store<M, CT>(acc, buf, wave, li, hh, P.scale, dq + base + (int64_t)i0 * P.stride_s, P.stride_s, P.s - i0, P.d);
  if (wave_any(odd)) {
    const int j0 = kTileF * (ntile - 1), j1 = min(j0 + kTileF, P.s), r0 = i0 + merge_row_of_wave<M>(wave);
    if (P.d % 32 || ((P.causal || P.s % kTileF) && wave_any(any_odd(kg, P.stride_s, j0, j1, P.d) || any_odd(vg, P.stride_s, j0, j1, P.d))))
      for (int r = r0; r < min(r0 + M / NWF, P.s); ++r) {
        const float dl_r = __shfl(dl, r - i0, 64), lse_r = __shfl(lse_i, r - i0, 64);
        plain_row([&](int j) __attribute__((always_inline)) {
          const float pe = exp_diff(score(dot_rows(q + base + (int64_t)r * P.stride_s, kg + (int64_t)j * P.stride_s, P.d), P.scale), lse_r);
          const float dp = dot_rows(dO + base + (int64_t)r * P.stride_s, vg + (int64_t)j * P.stride_s, P.d) * P.keep_scale;
          return pe * ((kept_pair<DROP>(P, beta, n, r, j) ? dp : 0.f) - dl_r);
        }, 0, P.causal ? r + 1 : P.s, kg, P.stride_s, P.d, P.scale, dq + base + (int64_t)r * P.stride_s);
      }
  }
}

// ---------------------------------------------------------------------------------------------------
// backward, column pass: dK_j = alpha sum_i dS_ij q_i, dV_j = sum_i D_ij dO_i of M keys.  Scores the other way round, S = Q K^T:
// a lane owns one key, its registers are query rows, so D and dS are again B operands as they are.  One Philox call covers 8
// consecutive keys of a row = 8 lanes: each of the 8 lanes draws an eighth of the calls of the lane's rows and all read one
// another's bits.
// ---------------------------------------------------------------------------------------------------
// keep decisions of value E from the lane of the group of eight that drew its row
template <int E, int CALLS>
__device__ __forceinline__ bool kept(uint32_t mine, int li) {
  return ((uint32_t)__builtin_amdgcn_ds_swizzle((int)mine, ((E / CALLS) << 5) | 0x18) >> (8 * (E % CALLS) + (li & 7))) & 1u;
}
template <int M, int DT, bool DROP, typename T>
__global__ __launch_bounds__(64 * NWF, waves_cols(M, DT)) void attn_bwd_cols_f32_kernel(AttnParams P, const T* __restrict__ q, const T* __restrict__ k,
                                                                                      const T* __restrict__ v, const float* __restrict__ lse,
                                                                                      const T* __restrict__ dO, const float* __restrict__ delta,
                                                                                      T* __restrict__ dk, T* __restrict__ dv) {
  typedef Geo<M> G;
  constexpr int QP = 32 * DT + 4, CT = 32 * DT / M, NV = G::NV, CALLS = NV / 8;
  __shared__ __attribute__((aligned(16))) float Ks[M * QP], Vs[M * QP];
  __shared__ __attribute__((aligned(16))) float buf[NWF * M * merge_pitch<M, CT>()];
  const int N = P.b * P.A, nt = (P.s + kTileF - 1) / kTileF, wi = work_index();
  const int kb = wi / N;  // key block 0 sweeps the most rows: heaviest first
  const int bn = wi % N, beta = bn / P.A, n = bn % P.A;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, li = lane & (M - 1), hh = lane / M;
  const int64_t base = (int64_t)beta * P.stride_b + (int64_t)n * P.stride_a;
  const int j0 = M * kb, j = j0 + li;
  const int it0 = P.causal ? j0 / kTileF : 0;
  rows_to_lds<M, DT>(Ks, k + base + (int64_t)j0 * P.stride_s, P.stride_s, P.s - j0, P.d);
  rows_to_lds<M, DT>(Vs, v + base + (int64_t)j0 * P.stride_s, P.stride_s, P.s - j0, P.d);
  const T* qg = q + base;
  const T* gg = dO + base;
  const int cs = col_start<CT>(li, P.d);
  const float* lse_h = lse + (size_t)bn * P.s;
  const float* delta_h = delta + (size_t)bn * P.s;
  const uint64_t headG = P.offset + (((uint64_t)beta * (uint64_t)P.a_global + (uint64_t)(P.head0 + n)) * (uint64_t)P.s) * (uint64_t)(P.s >> 3) +
                         (uint64_t)((j0 + (li & ~7)) >> 3);
  typename G::acc_t ka[CT], va[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int e = 0; e < NV / G::SUB; ++e) { ka[ct][e] = 0.f; va[ct][e] = 0.f; }
  auto rowat = [&](int it, int t) __attribute__((always_inline)) { return (int64_t)min(kTileF * it + G::row_of_row(t, li), P.s - 1) * P.stride_s; };
  typename Raw4<T>::type ring[kRingF];
  ring_start<M, DT>(ring, qg + rowat(it0 + wave, 0), (M == 32 ? gg : qg) + rowat(it0 + wave, G::SUB - 1), hh, P.d);
  __syncthreads();
  const float *krow = Ks + li * QP + 4 * hh, *vrow = Vs + li * QP + 4 * hh;
  constexpr int CA = rows_ahead(2 * CT, NV);
  for (int it = it0 + wave; it < nt; it += NWF) {
    const int i0 = kTileF * it;
    // rows past the end get probability 0 (what they read is clamped)
    auto row_of = [&](int e) __attribute__((always_inline)) { return (int64_t)min(i0 + G::row_of_value(e, hh), P.s - 1) * P.stride_s + cs; };
    Cols<T, CT> gc[CA], qc[CA];
    float st[NV], dd[NV];
    auto start_cols = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < CA; ++e) {
        gc[e].load(gg + row_of(e));
        qc[e].load(qg + row_of(e));
      }
    };
    float4_t dl[NV / 4], ls[NV / 4];
    auto start_stats = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int g = 0; g < NV / 4; ++g) {
        const int ib = min(i0 + G::row_of_value(4 * g, hh), P.s - 4);  // s % 8 == 0: a group of four rows is inside or outside as a whole
        ls[g] = *reinterpret_cast<const float4_t*>(lse_h + ib);
        dl[g] = *reinterpret_cast<const float4_t*>(delta_h + ib);
      }
    };
    if constexpr (M == 32) {
      const float16_t s0 = dot_tile<M, DT, 0>(ring, qg + rowat(it, 0), gg + rowat(it, 0), gg + rowat(it, 0), krow, hh, P.d);
      start_cols();
      const float16_t d0 = dot_tile<M, DT, (4 * DT) % kRingF>(ring, gg + rowat(it, 0), qg + rowat(it + NWF, 0), qg + rowat(it + NWF, 0), vrow, hh, P.d);
#pragma unroll
      for (int e = 0; e < NV; ++e) { st[e] = s0[e]; dd[e] = d0[e]; }
      start_stats();
    } else {
      start_stats();
      const float4_t s0 = dot_tile<M, DT, 0>(ring, qg + rowat(it, 0), qg + rowat(it, 1), gg + rowat(it, 0), krow, hh, P.d);
      const float4_t s1 = dot_tile<M, DT, (2 * DT) % kRingF>(ring, qg + rowat(it, 1), gg + rowat(it, 0), gg + rowat(it, 1), krow, hh, P.d);
      start_cols();
      const float4_t d0 = dot_tile<M, DT, (4 * DT) % kRingF>(ring, gg + rowat(it, 0), gg + rowat(it, 1), qg + rowat(it + NWF, 0), vrow, hh, P.d);
      const float4_t d1 = dot_tile<M, DT, (6 * DT) % kRingF>(ring, gg + rowat(it, 1), qg + rowat(it + NWF, 0), qg + rowat(it + NWF, 1), vrow, hh, P.d);
#pragma unroll
      for (int e = 0; e < 4; ++e) { st[e] = s0[e]; st[4 + e] = s1[e]; dd[e] = d0[e]; dd[4 + e] = d1[e]; }
    }
#pragma unroll
    for (int e = 0; e < NV; ++e) st[e] = score(st[e], P.scale) - ls[e >> 2][e & 3];
    if ((P.causal && i0 < j0 + M) || i0 + kTileF > P.s) {
#pragma unroll
      for (int e = 0; e < NV; ++e) {
        const int i = i0 + G::row_of_value(e, hh);
        if ((P.causal && j > i) || i >= P.s) st[e] = -INFINITY;
      }
    }
    uint32_t mine = 0;
    if (DROP) {
#pragma unroll
      for (int y = 0; y < CALLS; ++y) {
        const int i = i0 + G::row_of_value(CALLS * (li & 7) + y, hh);
        mine |= keep_bits8(headG + (uint64_t)i * (uint64_t)(P.s >> 3), 0u, P.key0, P.key1, P.thresh) << (8 * y);
      }
    }
#define SAR_ROW(E)                                                                                                          \
  if constexpr (E < NV) {                                                                                                   \
    const bool keep = !DROP || kept<E, CALLS>(mine, li);                                                                    \
    const float pe = __builtin_amdgcn_exp2f(st[E] * kLog2eF);                                                               \
    const float pd = keep ? pe * P.keep_scale : 0.f, dp = keep ? dd[E] * P.keep_scale : 0.f;                                \
    const float ds = pe * (dp - dl[(E) >> 2][(E) & 3]);                                                                     \
    _Pragma("unroll") for (int ct = 0; ct < CT; ++ct) {                                                                     \
      va[ct] = G::mfma(gc[(E) % CA].get(ct), pd, va[ct]);                                                                   \
      ka[ct] = G::mfma(qc[(E) % CA].get(ct), ds, ka[ct]);                                                                   \
    }                                                                                                                       \
    asm volatile("" : "+v"(va[0]), "+v"(ka[0]));                                                                            \
    if constexpr ((E) + CA < NV) {                                                                                          \
      gc[(E) % CA].load(gg + row_of((E) + CA));                                                                             \
      qc[(E) % CA].load(qg + row_of((E) + CA));                                                                             \
    }                                                                                                                       \
    __builtin_amdgcn_sched_barrier(0);                                                                                      \
  }
    SAR_ROW(0) SAR_ROW(1) SAR_ROW(2) SAR_ROW(3) SAR_ROW(4) SAR_ROW(5) SAR_ROW(6) SAR_ROW(7)
    SAR_ROW(8) SAR_ROW(9) SAR_ROW(10) SAR_ROW(11) SAR_ROW(12) SAR_ROW(13) SAR_ROW(14) SAR_ROW(15)
#undef SAR_ROW
  }
  bool odd = merge_store<M, CT>(va, buf, wave, li, hh, 1.f, dv + base + (int64_t)j0 * P.stride_s, P.stride_s, P.s - j0, P.d);
  odd |= merge_store<M, CT>(ka, buf, wave, li, hh, P.scale, dk + base + (int64_t)j0 * P.stride_s, P.stride_s, P.s - j0, P.d);
  if (wave_any(odd)) {
    auto odd_rows = [&](int it) {  // of a tile with excluded pairs
      const int r0 = kTileF * it, r1 = min(r0 + kTileF, P.s), r = r0 + lane;
      return any_odd(qg, P.stride_s, r0, r1, P.d) || any_odd(gg, P.stride_s, r0, r1, P.d) || (r < r1 && !(finite(lse_h[r]) && finite(delta_h[r])));
    };
    const int c0 = j0 + merge_row_of_wave<M>(wave);
    if (P.d % 32 || wave_any((P.causal && odd_rows(it0)) || (P.s % kTileF && odd_rows(nt - 1))))
      for (int c = c0; c < min(c0 + M / NWF, P.s); ++c) {
        const T *kc = k + base + (int64_t)c * P.stride_s, *vc = v + base + (int64_t)c * P.stride_s;
        auto prob = [&](int i) __attribute__((always_inline)) { return exp_diff(score(dot_rows(qg + (int64_t)i * P.stride_s, kc, P.d), P.scale), lse_h[i]); };
        plain_row([&](int i) __attribute__((always_inline)) { return kept_pair<DROP>(P, beta, n, i, c) ? prob(i) * P.keep_scale : 0.f; }, P.causal ? c : 0, P.s, gg, P.stride_s,
                  P.d, 1.f, dv + base + (int64_t)c * P.stride_s);
        plain_row([&](int i) __attribute__((always_inline)) {
          const float dp = dot_rows(gg + (int64_t)i * P.stride_s, vc, P.d) * P.keep_scale;
          return prob(i) * ((kept_pair<DROP>(P, beta, n, i, c) ? dp : 0.f) - delta_h[i]);
        }, P.causal ? c : 0, P.s, qg, P.stride_s, P.d, P.scale, dk + base + (int64_t)c * P.stride_s);
      }
  }
}

// ---------------------------------------------------------------------------------------------------
// Short sequences (s <= 64), one wave a row (forward, row pass) or a key (column pass): a lane holds the pair with the other index
// lane % KP, KP the power of two from s on, and every KP-th lane shares its products over the head dimension.  The kernels above spend
// themselves on the products of a 16 x 32 tile that is mostly padding, one matrix instruction after the other.
// ---------------------------------------------------------------------------------------------------
struct Few {
  int lane, kp, other;
  __device__ __forceinline__ explicit Few(int s) : lane(threadIdx.x & 63), kp(s <= 8 ? 8 : s <= 16 ? 16 : s <= 32 ? 32 : 64), other(lane & (kp - 1)) {}
  // a . b of this lane's pair; a: the wave's row, b: the lane's
  template <typename T>
  __device__ __forceinline__ float dot(const T* a, const T* b, int d) const {
    float acc = 0.f;
#pragma unroll 4
    for (int x = 4 * (lane / kp); x < d; x += 4 * (64 / kp)) {
      const float4_t fa = load4(a + x), fb = load4(b + x);
#pragma unroll
      for (int u = 0; u < 4; ++u) acc = fmaf(fa[u], fb[u], acc);
    }
    for (int o = kp; o < 64; o <<= 1) acc += __shfl_xor(acc, o, 64);
    return acc;
  }
  // out = mul sum_{y = lo}^{hi - 1} w(y) src_y, w in lane y
  template <typename T>
  __device__ __forceinline__ void sum(float w, int lo, int hi, const T* src, int64_t gstride, int d, float mul, T* out) const {
    const int x = 4 * lane, xl = min(x, d - 4);  // d <= 256; every lane stays active: its weight is read by the others
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int y = lo; y < hi; ++y) {
      const float wy = __shfl(w, y, 64);
      const float4_t f = load4(src + (int64_t)y * gstride + xl);
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] = fmaf(wy, f[u], acc[u]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[u] *= mul;
    if (x < d) store_cols<4>(out + x, acc);
  }
};
template <bool DROP, typename T>
__global__ __launch_bounds__(64 * NWF) void attn_fwd_few_kernel(AttnParams P, const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                                                               T* __restrict__ o, float* __restrict__ lse) {
  const int w = __builtin_amdgcn_readfirstlane(blockIdx.x * NWF + (threadIdx.x >> 6));
  if (w >= P.b * P.A * P.s) return;
  const int bn = w / P.s, i = w % P.s, beta = bn / P.A, n = bn % P.A, end = P.causal ? i + 1 : P.s;
  const int64_t base = (int64_t)beta * P.stride_b + (int64_t)n * P.stride_a, row = base + (int64_t)i * P.stride_s;
  const Few f(P.s);
  const float dot = f.dot(q + row, k + base + (int64_t)min(f.other, end - 1) * P.stride_s, P.d), st = f.other < end ? score(dot, P.scale) : -INFINITY;
  const float m = wave_max(st), pe = f.other < end ? exp_diff(st, m) : 0.f, l = wave_sum(f.lane < f.kp ? pe : 0.f);
  if (f.lane == 0) lse[w] = m + __builtin_amdgcn_logf(l) * kLn2F;
  f.sum(kept_pair<DROP>(P, beta, n, i, f.other) ? pe / l * P.keep_scale : 0.f, 0, end, v + base, P.stride_s, P.d, 1.f, o + row);
}
template <bool DROP, typename T>
__global__ __launch_bounds__(64 * NWF) void attn_bwd_rows_few_kernel(AttnParams P, const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                                                                    const T* __restrict__ o, const float* __restrict__ lse, const T* __restrict__ dO,
                                                                    T* __restrict__ dq, float* __restrict__ delta) {
  const int w = __builtin_amdgcn_readfirstlane(blockIdx.x * NWF + (threadIdx.x >> 6));
  if (w >= P.b * P.A * P.s) return;
  const int bn = w / P.s, i = w % P.s, beta = bn / P.A, n = bn % P.A, end = P.causal ? i + 1 : P.s;
  const int64_t base = (int64_t)beta * P.stride_b + (int64_t)n * P.stride_a, row = base + (int64_t)i * P.stride_s;
  const Few f(P.s);
  float dl = 0.f;
  for (int x = 4 * f.lane; x < P.d; x += 256) {
    const float4_t a = load4(o + row + x), b = load4(dO + row + x);
#pragma unroll
    for (int u = 0; u < 4; ++u) dl = fmaf(a[u], b[u], dl);
  }
  const int64_t other = base + (int64_t)min(f.other, end - 1) * P.stride_s;
  const float st = score(f.dot(q + row, k + other, P.d), P.scale), dd = f.dot(dO + row, v + other, P.d);
  dl = wave_sum(dl);
  if (f.lane == 0) delta[w] = dl;
  const float ds = exp_diff(st, lse[w]) * ((kept_pair<DROP>(P, beta, n, i, f.other) ? dd * P.keep_scale : 0.f) - dl);
  f.sum(ds, 0, end, k + base, P.stride_s, P.d, P.scale, dq + row);
}
template <bool DROP, typename T>
__global__ __launch_bounds__(64 * NWF) void attn_bwd_cols_few_kernel(AttnParams P, const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                                                                    const float* __restrict__ lse, const T* __restrict__ dO, const float* __restrict__ delta,
                                                                    T* __restrict__ dk, T* __restrict__ dv) {
  const int w = __builtin_amdgcn_readfirstlane(blockIdx.x * NWF + (threadIdx.x >> 6));
  if (w >= P.b * P.A * P.s) return;
  const int bn = w / P.s, j = w % P.s, beta = bn / P.A, n = bn % P.A, lo = P.causal ? j : 0;
  const int64_t base = (int64_t)beta * P.stride_b + (int64_t)n * P.stride_a, col = base + (int64_t)j * P.stride_s;
  const Few f(P.s);
  const int i = min(max(f.other, lo), P.s - 1);
  const int64_t other = base + (int64_t)i * P.stride_s;
  const float ls = lse[bn * P.s + i], dl = delta[bn * P.s + i];
  const float pe = exp_diff(score(f.dot(k + col, q + other, P.d), P.scale), ls), dd = f.dot(v + col, dO + other, P.d);
  const bool keep = kept_pair<DROP>(P, beta, n, i, j);
  f.sum(keep ? pe * P.keep_scale : 0.f, lo, P.s, dO + base, P.stride_s, P.d, 1.f, dv + col);
  f.sum(pe * ((keep ? dd * P.keep_scale : 0.f) - dl), lo, P.s, q + base, P.stride_s, P.d, P.scale, dk + col);
}

// M = 16 where M = 32 leaves less than two workgroups a CU: twice the workgroups with half the work each start sooner and spread a
// causal triangle better (us, forward and backward, M = 32 / 16: s = 128, 2 heads of 64 25.3 / 18.0; s = 1024, 8 heads of 128
// 189 / 136; from there on equal, 512 x 64 heads 134 / 136, or slower for twice the operand reads, 1024 x 24 heads 175 / 186), and
// where half of a block of 32 rows would be padding.
inline bool narrow(const AttnParams& P) { return P.s <= 16 || (int64_t)((P.s + 31) / 32) * P.b * P.A < 2 * (int64_t)attn_mfma_cu_count(); }

// One wave a row: s <= 8 (backward, us, before / here: fp32, 1 head of 256 27.9 / 12.4, 2048 heads of 256 449 / 88, 2048 of 4 44.8 / 25.7); up to
// s = 16 from head dimension 64 on, and 24 from 192 on, while there is at most one workgroup a CU (s = 16, 16 heads: d = 64
// 12.3 / 11.8, 128 16.8 / 13.7, 256 29.5 / 19.1; d = 32 10.5 / 10.5; s = 24, 16 heads of 256 29.3 / 28.5, of 128 16.7 / 19.9; s = 16, 256 heads of
// 64 12.6 / 20.9).
inline bool few(const AttnParams& P) {
  if (P.s <= 8) return true;
  return (int64_t)P.s * P.b * P.A <= NWF * (int64_t)attn_mfma_cu_count() && P.s <= (P.d >= 192 ? 24 : P.d >= 64 ? 16 : 8);
}

template <typename T>
hipError_t fwd_few(const AttnParams& P, const void* q, const void* k, const void* v, void* o, float* lse, hipStream_t st) {
  const dim3 grid((unsigned)((P.s * P.b * P.A + NWF - 1) / NWF)), block(64 * NWF);
  auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, block, 0, st, P, (const T*)q, (const T*)k, (const T*)v, (T*)o, lse); };
  if (P.thresh != 0) go(attn_fwd_few_kernel<true, T>);
  else go(attn_fwd_few_kernel<false, T>);
  return hipGetLastError();
}
template <typename T>
hipError_t bwd_few(const AttnParams& P, const void* q, const void* k, const void* v, const void* o, const float* lse, const void* dO, void* dq, void* dk,
                   void* dv, float* delta, int passes, hipStream_t st) {
  const dim3 grid((unsigned)((P.s * P.b * P.A + NWF - 1) / NWF)), block(64 * NWF);
  if (passes & 1) {
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, block, 0, st, P, (const T*)q, (const T*)k, (const T*)v, (const T*)o, lse, (const T*)dO, (T*)dq, delta); };
    if (P.thresh != 0) go(attn_bwd_rows_few_kernel<true, T>);
    else go(attn_bwd_rows_few_kernel<false, T>);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (passes & 2) {
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, block, 0, st, P, (const T*)q, (const T*)k, (const T*)v, lse, (const T*)dO, (const float*)delta, (T*)dk, (T*)dv); };
    if (P.thresh != 0) go(attn_bwd_cols_few_kernel<true, T>);
    else go(attn_bwd_cols_few_kernel<false, T>);
  }
  return hipGetLastError();
}

template <int M, int DT, typename T>
hipError_t fwd_dt(const AttnParams& P, const void* q, const void* k, const void* v, void* o, float* lse, hipStream_t st) {
  const dim3 grid((unsigned)((P.s + M - 1) / M * P.b * P.A)), block(64 * NWF);
  auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, block, 0, st, P, (const T*)q, (const T*)k, (const T*)v, (T*)o, lse); };
  if (P.thresh != 0) go(attn_fwd_f32_kernel<M, DT, true, T>);
  else go(attn_fwd_f32_kernel<M, DT, false, T>);
  return hipGetLastError();
}

template <int M, int DT, typename T>
hipError_t bwd_dt(const AttnParams& P, const void* q, const void* k, const void* v, const void* o, const float* lse, const void* dO, void* dq, void* dk,
                  void* dv, float* delta, int passes, hipStream_t st) {
  const dim3 grid((unsigned)((P.s + M - 1) / M * P.b * P.A)), block(64 * NWF);
  if (passes & 1) {
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, block, 0, st, P, (const T*)q, (const T*)k, (const T*)v, (const T*)o, lse, (const T*)dO, (T*)dq, delta); };
    if (P.thresh != 0) go(attn_bwd_rows_f32_kernel<M, DT, true, T>);
    else go(attn_bwd_rows_f32_kernel<M, DT, false, T>);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (passes & 2) {
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, block, 0, st, P, (const T*)q, (const T*)k, (const T*)v, lse, (const T*)dO, (const float*)delta, (T*)dk, (T*)dv); };
    if (P.thresh != 0) go(attn_bwd_cols_f32_kernel<M, DT, true, T>);
    else go(attn_bwd_cols_f32_kernel<M, DT, false, T>);
  }
  return hipGetLastError();
}

// f(M, DT) with the constants that the shape asks for
template <typename F>
hipError_t by_shape(const AttnParams& P, F&& f) {
#define SAR_DT(N) case N: return narrow(P) ? f(std::integral_constant<int, 16>{}, std::integral_constant<int, N>{}) : f(std::integral_constant<int, 32>{}, std::integral_constant<int, N>{});
  switch ((P.d + 31) / 32) {
    SAR_DT(1) SAR_DT(2) SAR_DT(3) SAR_DT(4) SAR_DT(5) SAR_DT(6) SAR_DT(7) SAR_DT(8)
    default: return hipErrorInvalidValue;
  }
#undef SAR_DT
}

}  // namespace
}  // namespace sar
