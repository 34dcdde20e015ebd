// Memory-bound operators of the sequence-parallel region (Section 4.2.2, Eq. 3) on one rank's rows:
// LayerNorm forward / backward and dropout(+bias)+residual.  One pass over HBM per tensor, 128-bit accesses.
#include "sar_device.h"
#include "sar_internal.h"

#include <atomic>

namespace sar {

// 16 bytes to memory; STREAM: nontemporal
template <bool STREAM, typename V>
__device__ __forceinline__ void store16(void* p, V v) {
  typedef __attribute__((__vector_size__(16))) uint32_t raw_t;
  const raw_t r = __builtin_bit_cast(raw_t, v);
  if (STREAM) __builtin_nontemporal_store(r, reinterpret_cast<raw_t*>(p));
  else *reinterpret_cast<raw_t*>(p) = r;
}

// 8 consecutive elements (one 16-byte access for bf16, two for fp32) <-> 8 floats
template <typename T> struct Vec8;
template <> struct Vec8<uint16_t> {
  static __device__ __forceinline__ void load(const uint16_t* p, float (&f)[8]) {
    uint4 u = *reinterpret_cast<const uint4*>(p);
    uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      f[2 * e] = __uint_as_float(w[e] << 16);
      f[2 * e + 1] = __uint_as_float(w[e] & 0xffff0000u);
    }
  }
  template <bool STREAM = false>
  static __device__ __forceinline__ void store(uint16_t* p, const float (&f)[8]) {
    uint4 u;
    u.x = pack_bf16x2(f[0], f[1]);
    u.y = pack_bf16x2(f[2], f[3]);
    u.z = pack_bf16x2(f[4], f[5]);
    u.w = pack_bf16x2(f[6], f[7]);
    store16<STREAM>(p, u);
  }
};
template <> struct Vec8<float> {
  static __device__ __forceinline__ void load(const float* p, float (&f)[8]) {
    float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
    f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w; f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
  }
  template <bool STREAM = false>
  static __device__ __forceinline__ void store(float* p, const float (&f)[8]) {
    store16<STREAM>(p, make_float4(f[0], f[1], f[2], f[3]));
    store16<STREAM>(p + 4, make_float4(f[4], f[5], f[6], f[7]));
  }
};

// 8 consecutive elements as they lie in memory: what a thread holds of a load in flight
template <typename T> struct Raw8;
template <> struct Raw8<uint16_t> {
  uint4 u;
  __device__ __forceinline__ void load(const uint16_t* p) { u = *reinterpret_cast<const uint4*>(p); }
  // converted afresh from here on: otherwise the compiler keeps the eight floats of an earlier get() in registers
  __device__ __forceinline__ void pin() { asm volatile("" : "+v"(u.x), "+v"(u.y), "+v"(u.z), "+v"(u.w)); }
  __device__ __forceinline__ void get(float (&f)[8]) const {
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      f[2 * e] = __uint_as_float(w[e] << 16);
      f[2 * e + 1] = __uint_as_float(w[e] & 0xffff0000u);
    }
  }
};
template <> struct Raw8<float> {
  float4 a, b;
  __device__ __forceinline__ void load(const float* p) { a = *reinterpret_cast<const float4*>(p); b = *reinterpret_cast<const float4*>(p + 4); }
  __device__ __forceinline__ void pin() { asm volatile("" : "+v"(a.x), "+v"(a.y), "+v"(a.z), "+v"(a.w), "+v"(b.x), "+v"(b.y), "+v"(b.z), "+v"(b.w)); }
  __device__ __forceinline__ void get(float (&f)[8]) const {
    f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w; f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
  }
};

// ---------------------------------------------------------------------------------------------------
// Elementwise passes that also sum every column (bias gradients).  A workgroup of 256 threads owns a block of 8 L columns, L =
// 2^lg lanes of 8 elements to a row segment, 256 / L segments; its rows are split, split + nsplit, ... in groups of 256 / L, so
// that all workgroups together walk through the tensor as one contiguous window.  Column sums: registers, then LDS across the
// segments, then (nsplit > 1) partial sums that colsum_finish_kernel adds.
//
// Bound: HBM.  One row of a thread at a time; the width of a segment is a template constant where the pass is a kernel of its own (as an
// argument it costs 0.2 us of the 5 that 256 rows take).
// ---------------------------------------------------------------------------------------------------
struct ColPlan {
  int lg, ncb, nsplit;  // lanes of a row segment (log2), column blocks, row splits
};
// one: lanes (log2) of a segment where a column block takes all of its rows, with no partial sums and no second launch (2.5 to 4 us); 0: rows
// split over about `groups` workgroups, in segments of 2^lg lanes: 16 (bias-dropout backward, us, 8 / 16 / 64 lanes: bf16 8192 x 3072 19.7 / 19.3 /
// 20.5, fp32 4096 x 8192 - / 43.5 / 50.3), 32 on the widest rows, and 64 where the pass's tensors together do not fit the last-level cache
// (bf16 4096 x 20480 - / 65.8 / 62.0; bias-GeLU backward of bf16 8192 x 8192 - / 87 / 80).
static inline ColPlan col_plan(int64_t rows, int64_t h, int64_t esz, int one, int groups, int lg, int tensors, int nt = 256) {
  const int64_t nchunk = h >> 3;
  ColPlan p{one, 0, 1};
  if (one) {
    p.ncb = (int)((nchunk + (1 << one) - 1) >> one);
    return p;
  }
  const bool large = rows * h * esz * tensors > 288000000;
  for (p.lg = large ? 6 : nchunk > 2560 ? 5 : lg; p.lg > 3; --p.lg) {  // the widest that leaves at most an eighth of the lanes without work
    const int64_t L = 1 << p.lg, used = (nchunk + L - 1) / L * L;
    if (used - nchunk <= nchunk / 8) break;
  }
  p.ncb = (int)((nchunk + (1 << p.lg) - 1) >> p.lg);
  const int64_t nseg = nt >> p.lg, most = (rows + nseg - 1) / nseg, want = (large ? 1024 : groups) / p.ncb;  // no more than are resident at once
  p.nsplit = (int)(want < 1 ? 1 : want < most ? want : most);
  return p;
}
// Rows up to which one split pays, given those measured on rows whose last block is full: in a block with idle lanes a trip can take twice as long
// (bias-dropout backward of 512 x 520 10.2 us in one split, 7.7 in several, of 512 x 1024 6.2, 7.6).
static inline int64_t one_split_rows(int64_t h, int64_t full) { return (h >> 3) % 8 == 0 ? full : 128; }

// op: In (what a row segment loads), column(col) (per column, before the rows), load(row, col), apply(in, row, col, sums)
template <int NT, typename Op>
__device__ __forceinline__ void colsum_block(Op& op, int64_t rows, int64_t h, const ColPlan& pl, int cb, int split, float (&acc)[Op::kSums][8]) {
  const int seg = threadIdx.x >> pl.lg, nseg = NT >> pl.lg;
  const int64_t chunk = (int64_t)cb << pl.lg | (threadIdx.x & ((1 << pl.lg) - 1));
#pragma unroll
  for (int s = 0; s < Op::kSums; ++s)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[s][e] = 0.f;
  if (chunk >= (h >> 3)) return;
  const int64_t col = chunk << 3, step = (int64_t)pl.nsplit * nseg;
  op.column(col);
  for (int64_t r = (int64_t)split * nseg + seg; r < rows; r += step) op.apply(op.load(r, col), r, col, acc);
}
// sums over the segments of a workgroup; the column block's sums go to out[s] + column (a split's partial sums or the result)
template <int NT, int S>
__device__ __forceinline__ void colsum_store(const float (&acc)[S][8], float* sb, int64_t h, const ColPlan& pl, int cb, float* const (&out)[S]) {
  const int nseg = NT >> pl.lg, width = 8 << pl.lg;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    if (s) __syncthreads();
#pragma unroll
    for (int e = 0; e < 8; ++e) sb[8 * threadIdx.x + e] = acc[s][e];
    __syncthreads();
    for (int c = threadIdx.x; c < width; c += NT) {
      float t[4] = {0.f, 0.f, 0.f, 0.f};  // nseg is a multiple of 4
#pragma unroll 2
      for (int q = 0; q < nseg; q += 4)
#pragma unroll
        for (int x = 0; x < 4; ++x) t[x] += sb[(q + x) * width + c];
      const int64_t cc = (int64_t)cb * width + c;
      if (cc < h) out[s][cc] = (t[0] + t[1]) + (t[2] + t[3]);
    }
  }
}
template <typename Op, int LG>
__global__ __launch_bounds__(256) void colsum_kernel(Op op, int64_t rows, int64_t h, float* __restrict__ out, ColPlan pl) {
  pl.lg = LG;
  __shared__ __attribute__((aligned(16))) float sb[8 * 256];
  float acc[1][8];
  colsum_block<256>(op, rows, h, pl, blockIdx.x, blockIdx.y, acc);
  float* const dst[1] = {out + (int64_t)blockIdx.y * h};
  colsum_store<256, 1>(acc, sb, h, pl, blockIdx.x, dst);
}

// part[nsplit][ncol] -> sums of columns 0 .. h-1 to out0, of the rest to out1.  32 columns a workgroup (8 lanes of 4), 32 groups
// of splits, four loads in flight each (one thread a column, one load after the other: 11.4 us for 43 splits of 3072 columns).
__global__ __launch_bounds__(256) void colsum_finish_kernel(const float* __restrict__ part, int nsplit, int64_t ncol, int64_t h, float* __restrict__ out0,
                                                           float* __restrict__ out1) {
  __shared__ __attribute__((aligned(16))) float4 sb[32][8];
  const int l = threadIdx.x & 7, g = threadIdx.x >> 3;
  const int64_t c = (int64_t)blockIdx.x * 32 + 4 * l;
  float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
  if (c < ncol)
#pragma unroll 4
    for (int q = g; q < nsplit; q += 32) {
      const float4 v = *reinterpret_cast<const float4*>(part + (int64_t)q * ncol + c);
      t.x += v.x; t.y += v.y; t.z += v.z; t.w += v.w;
    }
  sb[g][l] = t;
  __syncthreads();
  if (g == 0 && c < ncol) {
    for (int q = 1; q < 32; ++q) {
      const float4 v = sb[q][l];
      t.x += v.x; t.y += v.y; t.z += v.z; t.w += v.w;
    }
    float* o = c < h ? out0 + c : out1 + (c - h);  // the caller's array: aligned to a float only
    o[0] = t.x; o[1] = t.y; o[2] = t.z; o[3] = t.w;
  }
}
static hipError_t launch_colsum_finish(const float* part, int nsplit, int64_t ncol, int64_t h, float* out0, float* out1, hipStream_t st) {
  hipLaunchKernelGGL(colsum_finish_kernel, dim3((unsigned)((ncol + 31) / 32)), dim3(256), 0, st, part, nsplit, ncol, h, out0, out1);
  return hipGetLastError();
}
template <typename Op>
static hipError_t launch_colsum(const Op& op, int64_t rows, int64_t h, const ColPlan& pl, float* out, float* ws, hipStream_t st) {
  auto go = [&](auto kern) { hipLaunchKernelGGL(kern, dim3((unsigned)pl.ncb, (unsigned)pl.nsplit), dim3(256), 0, st, op, rows, h, pl.nsplit == 1 ? out : ws, pl); };
  switch (pl.lg) {
    case 3: go(colsum_kernel<Op, 3>); break;
    case 4: go(colsum_kernel<Op, 4>); break;
    case 5: go(colsum_kernel<Op, 5>); break;
    default: go(colsum_kernel<Op, 6>); break;
  }
  const hipError_t e = hipGetLastError();
  return e != hipSuccess || pl.nsplit == 1 ? e : launch_colsum_finish(ws, pl.nsplit, h, h, out, nullptr, st);
}
static inline size_t colsum_workspace_bytes(const ColPlan& pl, int64_t h) { return pl.nsplit > 1 ? (size_t)pl.nsplit * (size_t)h * sizeof(float) : 0; }

// block-wide sum of two values; every thread gets the totals.  red must hold 2 * 16 floats.
__device__ __forceinline__ void block_sum2(float& a, float& b, float* red) {
  a = wave_sum(a);
  b = wave_sum(b);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = (blockDim.x + 63) >> 6;
  if (lane == 0) { red[wave] = a; red[16 + wave] = b; }
  __syncthreads();
  float ta = 0.f, tb = 0.f;
  for (int w = 0; w < nw; ++w) { ta += red[w]; tb += red[16 + w]; }
  a = ta;
  b = tb;
  __syncthreads();
}

// ---------------------------------------------------------------------------------------------------
// LayerNorm forward: one workgroup per row, the row lives in registers (VPT chunks of 8 per thread).
// Statistics in fp32 with the row's first element as shift, so one reduction gives mean and variance.
// ---------------------------------------------------------------------------------------------------
template <typename T, int VPT>
__global__ __launch_bounds__(1024) void ln_fwd_kernel(RowsParams P, const T* __restrict__ x, const T* __restrict__ gamma, const T* __restrict__ beta,
                                                     T* __restrict__ y, float* __restrict__ mean, float* __restrict__ rstd) {
  __shared__ float red[32];
  const int64_t r = blockIdx.x;
  const int nchunk = (int)(P.h >> 3);
  const T* xr = x + r * P.h;
  float xv[VPT][8];
  const float shift = Elem<T>::load(xr);
  float s1 = 0.f, s2 = 0.f;
#pragma unroll
  for (int u = 0; u < VPT; ++u) {
    const int c = threadIdx.x + u * blockDim.x;
    if (c < nchunk) {
      Vec8<T>::load(xr + 8 * c, xv[u]);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float dlt = xv[u][e] - shift;
        s1 += dlt;
        s2 = fmaf(dlt, dlt, s2);
      }
    }
  }
  block_sum2(s1, s2, red);
  const float invh = 1.f / (float)P.h;
  const float m1 = s1 * invh;
  const float var = fmaxf(s2 * invh - m1 * m1, 0.f);
  const float mu = shift + m1;
  const float rs = rsqrtf(var + P.eps);
#pragma unroll
  for (int u = 0; u < VPT; ++u) {
    const int c = threadIdx.x + u * blockDim.x;
    if (c < nchunk) {
      float g[8], bt[8], out[8];
      Vec8<T>::load(gamma + 8 * c, g);
      Vec8<T>::load(beta + 8 * c, bt);
#pragma unroll
      for (int e = 0; e < 8; ++e) out[e] = fmaf((xv[u][e] - mu) * rs, g[e], bt[e]);
      Vec8<T>::store(y + r * P.h + 8 * c, out);
    }
  }
  if (threadIdx.x == 0) { mean[r] = mu; rstd[r] = rs; }
}

// ---------------------------------------------------------------------------------------------------
// LayerNorm backward: c1 = mean_c(g), c2 = mean_c(g xhat) of a row with g = dy*gamma, dx = rstd (g - c1 - xhat c2);
// dgamma = sum_r dy xhat, dbeta = sum_r dy.  Two forms:
//   few rows:  one launch with two kinds of workgroups (dgamma / dbeta do not depend on the row sums, so nothing orders them):
//              blockIdx <  rows: one row, kept in registers: dx;
//              blockIdx >= rows: a block of columns and a split of the rows, as in colsum_kernel: dgamma, dbeta.
//              x and dy are read twice, the second time mostly out of the caches;
//   many rows: G workgroups that walk through the rows together, each with the dgamma, dbeta sums of its rows in registers:
//              x and dy are read once, and 2 G rows of fp32 partial sums are written and read back.
// Bound: HBM and, below about 20 MB a tensor, the two or three memory round trips of a launch.  bf16, us, slabs of 64 columns beside 1024-thread row
// workgroups (always two reads) and now: 256 x 20480 14.8 -> 10.3, 512 x 4096 9.4 -> 7.8, 512 x 12288 17.2 -> 12.1, 1024 x 6144 17.4 -> 13.3,
// 2048 x 6144 26.4 -> 22.2, 8192 x 4096 58.1 -> 39.1, 4096 x 20480 190 -> 115 (4.4 TB/s of the three tensors).
// ---------------------------------------------------------------------------------------------------
template <typename T, int VPT>
struct LnRow {  // a thread's share of a row: chunks threadIdx + u * blockDim
  Raw8<T> x[VPT], dy[VPT];
  __device__ __forceinline__ void load(const T* xr, const T* dyr, int nchunk) {
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
      const int c = threadIdx.x + u * blockDim.x;
      if (c < nchunk) {
        x[u].load(xr + 8 * c);
        dy[u].load(dyr + 8 * c);
      }
    }
  }
};

template <typename T>
struct LnBwdCols {
  static constexpr int kSums = 2;
  struct In { Raw8<T> x, dy; float mu, rs; };
  int64_t h;
  const T *dy, *x;
  const float *mean, *rstd;
  __device__ __forceinline__ void column(int64_t) {}
  __device__ __forceinline__ In load(int64_t r, int64_t col) const {
    In in;
    in.x.load(x + r * h + col);
    in.dy.load(dy + r * h + col);
    in.mu = mean[r];
    in.rs = rstd[r];
    return in;
  }
  __device__ __forceinline__ void apply(const In& in, int64_t, int64_t, float (&acc)[2][8]) const {
    float xv[8], dv[8];
    in.x.get(xv);
    in.dy.get(dv);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      acc[0][e] = fmaf(dv[e], (xv[e] - in.mu) * in.rs, acc[0][e]);
      acc[1][e] += dv[e];
    }
  }
};

// dg_out, db_out: the results, or (pl.nsplit > 1) partial sums [nsplit][2][h]
template <typename T, int NT, int VPT>
__global__ __launch_bounds__(NT) void ln_bwd_kernel(RowsParams P, const T* __restrict__ dy, const T* __restrict__ x, const float* __restrict__ mean,
                                                   const float* __restrict__ rstd, const T* __restrict__ gamma, T* __restrict__ dx,
                                                   float* __restrict__ dg_out, float* __restrict__ db_out, ColPlan pl) {
  __shared__ __attribute__((aligned(16))) float sb[8 * NT];
  if ((int64_t)blockIdx.x >= P.rows) {
    const int block = (int)((int64_t)blockIdx.x - P.rows), cb = block % pl.ncb, split = block / pl.ncb;
    LnBwdCols<T> op{P.h, dy, x, mean, rstd};
    float acc[2][8];
    colsum_block<NT>(op, P.rows, P.h, pl, cb, split, acc);
    const int64_t at = (int64_t)split * 2 * P.h;
    float* const dst[2] = {dg_out + at, db_out + at};
    colsum_store<NT, 2>(acc, sb, P.h, pl, cb, dst);
    return;
  }
  const int64_t r = blockIdx.x;
  const int nchunk = (int)(P.h >> 3);
  const float mu = mean[r], rs = rstd[r];
  LnRow<T, VPT> row;
  row.load(x + r * P.h, dy + r * P.h, nchunk);
  Raw8<T> gr[VPT];
#pragma unroll
  for (int u = 0; u < VPT; ++u) {
    const int c = threadIdx.x + u * NT;
    if (c < nchunk) gr[u].load(gamma + 8 * c);
  }
  float s1 = 0.f, s2 = 0.f;
#pragma unroll
  for (int u = 0; u < VPT; ++u)
    if ((int)threadIdx.x + u * NT < nchunk) {
      float xv[8], dv[8], g[8];
      row.x[u].get(xv);
      row.dy[u].get(dv);
      gr[u].get(g);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float gg = dv[e] * g[e];
        s1 += gg;
        s2 = fmaf(gg, (xv[e] - mu) * rs, s2);
      }
    }
  block_sum2(s1, s2, sb);
  const float c1 = s1 / (float)P.h, c2 = s2 / (float)P.h;
#pragma unroll
  for (int u = 0; u < VPT; ++u) {
    const int c = threadIdx.x + u * NT;
    if (c < nchunk) {
      float xv[8], dv[8], g[8], out[8];
      row.x[u].pin();
      row.dy[u].pin();
      gr[u].pin();
      row.x[u].get(xv);
      row.dy[u].get(dv);
      gr[u].get(g);
#pragma unroll
      for (int e = 0; e < 8; ++e) out[e] = rs * (dv[e] * g[e] - c1 - (xv[e] - mu) * rs * c2);
      Vec8<T>::store(dx + r * P.h + 8 * c, out);
    }
  }
}

// many rows.  PF: the next row is requested before this one is worked on (where the registers allow it)
template <typename T, int NT, int VPT, bool PF>
__global__ __launch_bounds__(NT, 2) void ln_bwd_stream_kernel(RowsParams P, const T* __restrict__ dy, const T* __restrict__ x,
                                                                     const float* __restrict__ mean, const float* __restrict__ rstd,
                                                                     const T* __restrict__ gamma, T* __restrict__ dx, float* __restrict__ part) {
  __shared__ float red[2][2][NT / 64];
  const int nchunk = (int)(P.h >> 3);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  Raw8<T> gr[VPT];
  float ag[VPT][8], ab[VPT][8];
#pragma unroll
  for (int u = 0; u < VPT; ++u) {
    const int c = threadIdx.x + u * NT;
    if (c < nchunk) gr[u].load(gamma + 8 * c);
#pragma unroll
    for (int e = 0; e < 8; ++e) { ag[u][e] = 0.f; ab[u][e] = 0.f; }
  }
  LnRow<T, VPT> row, next;
  float mu = 0.f, rs = 0.f, mu_n = 0.f, rs_n = 0.f;
  int64_t r = blockIdx.x;
  if (PF) {
    next.load(x + r * P.h, dy + r * P.h, nchunk);
    mu_n = mean[r];
    rs_n = rstd[r];
  }
  for (int it = 0; r < P.rows; r += gridDim.x, it ^= 1) {
    if (PF) {
      row = next;
      mu = mu_n;
      rs = rs_n;
      if (r + gridDim.x < P.rows) {
        next.load(x + (r + gridDim.x) * P.h, dy + (r + gridDim.x) * P.h, nchunk);
        mu_n = mean[r + gridDim.x];
        rs_n = rstd[r + gridDim.x];
      }
    } else {
      row.load(x + r * P.h, dy + r * P.h, nchunk);
      mu = mean[r];
      rs = rstd[r];
    }
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int u = 0; u < VPT; ++u)
      if ((int)threadIdx.x + u * NT < nchunk) {
        float xv[8], dv[8], g[8];
        row.x[u].get(xv);
        row.dy[u].get(dv);
        gr[u].get(g);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float xh = (xv[e] - mu) * rs, gg = dv[e] * g[e];
          ag[u][e] = fmaf(dv[e], xh, ag[u][e]);
          ab[u][e] += dv[e];
          s1 += gg;
          s2 = fmaf(gg, xh, s2);
        }
      }
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
    if (lane == 0) { red[it][0][wave] = s1; red[it][1][wave] = s2; }
    __syncthreads();  // the other buffer is written next, after every wave has passed this point: one barrier a row
    s1 = 0.f;
    s2 = 0.f;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) { s1 += red[it][0][w]; s2 += red[it][1][w]; }
    const float c1 = s1 / (float)P.h, c2 = s2 / (float)P.h;
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
      const int c = threadIdx.x + u * NT;
      if (c < nchunk) {
        float xv[8], dv[8], g[8], out[8];
        row.x[u].pin();
        row.dy[u].pin();
        gr[u].pin();
        row.x[u].get(xv);
        row.dy[u].get(dv);
        gr[u].get(g);
#pragma unroll
        for (int e = 0; e < 8; ++e) out[e] = rs * (dv[e] * g[e] - c1 - (xv[e] - mu) * rs * c2);
        Vec8<T>::store(dx + r * P.h + 8 * c, out);
      }
    }
  }
  float* pg = part + (int64_t)blockIdx.x * 2 * P.h;
#pragma unroll
  for (int u = 0; u < VPT; ++u) {
    const int c = threadIdx.x + u * NT;
    if (c < nchunk) {
      Vec8<float>::store(pg + 8 * c, ag[u]);
      Vec8<float>::store(pg + P.h + 8 * c, ab[u]);
    }
  }
}

// ---------------------------------------------------------------------------------------------------
// bias-dropout-add: out = resid + M (x + bias) / (1-p); one thread per 8 elements = one Philox call.
// ---------------------------------------------------------------------------------------------------
template <typename T, bool HAS_BIAS, bool HAS_MASK>
__global__ __launch_bounds__(256) void bias_dropout_add_kernel(RowsParams P, const T* __restrict__ x, const T* __restrict__ bias, const T* resid,
                                                              T* out, uint8_t* __restrict__ mask) {
  const int64_t r = blockIdx.x, c = ((int64_t)blockIdx.y * 256 + threadIdx.x) << 3;  // grid = (rows, chunks of a row / 256): no index division
  if (c >= P.h) return;
  float xv[8], rv[8], bv[8], o[8];
  Vec8<T>::load(x + r * P.h + c, xv);
  Vec8<T>::load(resid + r * P.h + c, rv);
  if (HAS_BIAS) Vec8<T>::load(bias + c, bv);
  const uint64_t e = (uint64_t)(P.row_offset + r) * (uint64_t)P.h + (uint64_t)c;
  const uint32_t keep = keep_bits8(P.offset + (e >> 3), 1u, P.key0, P.key1, P.thresh);
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    float xb = HAS_BIAS ? xv[q] + bv[q] : xv[q];
    o[q] = ((keep >> q) & 1u) ? fmaf(xb, P.keep_scale, rv[q]) : rv[q];
  }
  Vec8<T>::store(out + r * P.h + c, o);
  if (HAS_MASK) {
    uint2 m;
    m.x = (keep & 1u) | ((keep & 2u) << 7) | ((keep & 4u) << 14) | ((keep & 8u) << 21);
    m.y = ((keep >> 4) & 1u) | ((keep & 32u) << 3) | ((keep & 64u) << 10) | ((keep & 128u) << 17);
    *reinterpret_cast<uint2*>(mask + r * P.h + c) = m;
  }
}

// ---------------------------------------------------------------------------------------------------
// Fused bias-dropout-add + LayerNorm forward (last line of Eq. 3 feeding the next layer's first line):
//   out = resid + M (x + bias)/(1-p),  y = LayerNorm(out).
// One workgroup per row, as ln_fwd: the row is read once instead of twice (8 instead of 10 bytes per element).
// The statistics are taken from `out` as it is stored (rounded to T), so that a later ln_bwd, which re-reads the
// stored row, sees exactly the values mean and rstd belong to.
// ---------------------------------------------------------------------------------------------------
template <typename T, int VPT, bool HAS_BIAS>
__global__ __launch_bounds__(1024) void bda_ln_fwd_kernel(RowsParams P, const T* __restrict__ x, const T* __restrict__ bias, const T* resid,
                                                         const T* __restrict__ gamma, const T* __restrict__ beta, T* out, T* __restrict__ y,
                                                         float* __restrict__ mean, float* __restrict__ rstd) {
  __shared__ float red[32];
  const int64_t r = blockIdx.x;
  const int nchunk = (int)(P.h >> 3);
  float ov[VPT][8];
  float s1 = 0.f, s2 = 0.f, shift = 0.f;
#pragma unroll
  for (int u = 0; u < VPT; ++u) {
    const int c = threadIdx.x + u * blockDim.x;
    if (c < nchunk) {
      float xv[8], rv[8], bv[8];
      Vec8<T>::load(x + r * P.h + 8 * c, xv);
      Vec8<T>::load(resid + r * P.h + 8 * c, rv);
      if (HAS_BIAS) Vec8<T>::load(bias + 8 * c, bv);
      const uint64_t e = (uint64_t)(P.row_offset + r) * (uint64_t)P.h + (uint64_t)(8 * c);
      const uint32_t keep = keep_bits8(P.offset + (e >> 3), 1u, P.key0, P.key1, P.thresh);
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const float xb = HAS_BIAS ? xv[q] + bv[q] : xv[q];
        ov[u][q] = Elem<T>::round(((keep >> q) & 1u) ? fmaf(xb, P.keep_scale, rv[q]) : rv[q]);
      }
      Vec8<T>::store(out + r * P.h + 8 * c, ov[u]);
    }
  }
  // shift = the row's first element, held by thread 0: broadcast through LDS
  if (threadIdx.x == 0) red[0] = ov[0][0];
  __syncthreads();
  shift = red[0];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < VPT; ++u) {
    const int c = threadIdx.x + u * blockDim.x;
    if (c < nchunk) {
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const float dlt = ov[u][q] - shift;
        s1 += dlt;
        s2 = fmaf(dlt, dlt, s2);
      }
    }
  }
  block_sum2(s1, s2, red);
  const float invh = 1.f / (float)P.h;
  const float m1 = s1 * invh;
  const float var = fmaxf(s2 * invh - m1 * m1, 0.f);
  const float mu = shift + m1;
  const float rs = rsqrtf(var + P.eps);
#pragma unroll
  for (int u = 0; u < VPT; ++u) {
    const int c = threadIdx.x + u * blockDim.x;
    if (c < nchunk) {
      float g[8], bt[8], o[8];
      Vec8<T>::load(gamma + 8 * c, g);
      Vec8<T>::load(beta + 8 * c, bt);
#pragma unroll
      for (int q = 0; q < 8; ++q) o[q] = fmaf((ov[u][q] - mu) * rs, g[q], bt[q]);
      Vec8<T>::store(y + r * P.h + 8 * c, o);
    }
  }
  if (threadIdx.x == 0) { mean[r] = mu; rstd[r] = rs; }
}

// ---------------------------------------------------------------------------------------------------
// bias-dropout-add backward: dx = M dout/(1-p) with M regenerated from Philox; the residual branch's gradient is
// dout itself and is not written.  Without dbias this is elementwise (one thread per 8 elements); with dbias a column-summing
// pass (bf16, us, slabs of 64 columns on one or two workgroups a CU and now: 300 x 6144 8.3 -> 5.0, 1024 x 6144 9.4 -> 8.2, 4096 x 8192 31.6 -> 23.4,
// 4096 x 20480 112 -> 63).
// ---------------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void bda_bwd_kernel(RowsParams P, const T* __restrict__ dout, T* __restrict__ dx) {
  const int64_t r = blockIdx.x, c = ((int64_t)blockIdx.y * 256 + threadIdx.x) << 3;  // grid = (rows, chunks of a row / 256): no index division
  if (c >= P.h) return;
  float dv[8], o[8];
  Vec8<T>::load(dout + r * P.h + c, dv);
  const uint64_t e = (uint64_t)(P.row_offset + r) * (uint64_t)P.h + (uint64_t)c;
  const uint32_t keep = keep_bits8(P.offset + (e >> 3), 1u, P.key0, P.key1, P.thresh);
#pragma unroll
  for (int q = 0; q < 8; ++q) o[q] = ((keep >> q) & 1u) ? dv[q] * P.keep_scale : 0.f;
  Vec8<T>::store(dx + r * P.h + c, o);
}

template <typename T, bool STREAM>
struct BdaBwdCols {
  static constexpr int kSums = 1;
  typedef Raw8<T> In;
  RowsParams P;
  const T* dout;
  T* dx;
  __device__ __forceinline__ void column(int64_t) {}
  __device__ __forceinline__ In load(int64_t r, int64_t col) const {
    In in;
    in.load(dout + r * P.h + col);
    return in;
  }
  __device__ __forceinline__ void apply(const In& in, int64_t r, int64_t col, float (&acc)[1][8]) const {
    float dv[8], o[8];
    in.get(dv);
    const uint64_t e = (uint64_t)(P.row_offset + r) * (uint64_t)P.h + (uint64_t)col;
    const uint32_t keep = keep_bits8(P.offset + (e >> 3), 1u, P.key0, P.key1, P.thresh);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      o[q] = ((keep >> q) & 1u) ? dv[q] * P.keep_scale : 0.f;
      acc[0][q] += o[q];
    }
    Vec8<T>::template store<STREAM>(dx + r * P.h + col, o);
  }
};

// ---------------------------------------------------------------------------------------------------
// bias + GeLU of the MLP block (Section 4.1): y = z Phi(z), z = x + bias, Phi the standard normal CDF (exact form,
// through erf).  Backward: dx = dy (Phi(z) + z phi(z)) from the stored input, dbias = column sums of dx.
// One thread per 8 elements; with dbias, a column-summing pass.
// ---------------------------------------------------------------------------------------------------
// Phi(z) and phi(z) from one exponential: erf by the rational approximation 7.1.26 of Abramowitz & Stegun,
// erf(x) = 1 - (a1 t + ... + a5 t^5) exp(-x^2), t = 1 / (1 + p x), x >= 0, |error| <= 1.5e-7, with x = |z| / sqrt 2,
// so that exp(-x^2) = exp(-z^2 / 2) also gives the density.  (The library erff costs about three times as many
// vector instructions and made both kernels ALU-bound.)
__device__ __forceinline__ void gelu_parts(float z, float& Phi, float& pdf) {
  const float x = fabsf(z) * 0.70710678118654752f;
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, x, 1.f));  // 1 ulp; a correctly rounded reciprocal costs ten more instructions
  const float e = __expf(-x * x);
  const float poly = t * fmaf(t, fmaf(t, fmaf(t, fmaf(t, 1.061405429f, -1.453152027f), 1.421413741f), -0.284496736f), 0.254829592f);
  const float erfa = fmaf(-poly, e, 1.f);
  Phi = 0.5f * (1.f + copysignf(erfa, z));
  pdf = 0.3989422804014327f * e;
}
__device__ __forceinline__ float gelu_phi_cdf(float z) {
  float Phi, pdf;
  gelu_parts(z, Phi, pdf);
  return Phi;
}
__device__ __forceinline__ float gelu_grad(float z) {
  float Phi, pdf;
  gelu_parts(z, Phi, pdf);
  return fmaf(z, pdf, Phi);
}

// One chunk of 8 elements per thread; grid = (rows, chunks of a row / 256): no index division in the kernel (it cost
// four instructions per element of a kernel that is bound by its vector arithmetic).  More chunks per thread were slower.
template <typename T, bool HAS_BIAS, bool STREAM>
__global__ __launch_bounds__(256) void bias_gelu_fwd_kernel(RowsParams P, const T* __restrict__ x, const T* __restrict__ bias, T* __restrict__ y) {
  const int64_t c = ((int64_t)blockIdx.y * 256 + threadIdx.x) << 3;
  if (c >= P.h) return;
  const int64_t at = (int64_t)blockIdx.x * P.h + c;
  float xv[8], bv[8], o[8];
  Vec8<T>::load(x + at, xv);
  if (HAS_BIAS) Vec8<T>::load(bias + c, bv);
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const float z = HAS_BIAS ? xv[q] + bv[q] : xv[q];
    o[q] = z * gelu_phi_cdf(z);
  }
  Vec8<T>::template store<STREAM>(y + at, o);
}

template <typename T, bool HAS_BIAS>
__global__ __launch_bounds__(256) void bias_gelu_bwd_kernel(RowsParams P, const T* __restrict__ dy, const T* __restrict__ x,
                                                           const T* __restrict__ bias, T* __restrict__ dx) {
  const int64_t c = ((int64_t)blockIdx.y * 256 + threadIdx.x) << 3;
  if (c >= P.h) return;
  const int64_t at = (int64_t)blockIdx.x * P.h + c;
  float xv[8], dv[8], bv[8], o[8];
  Vec8<T>::load(x + at, xv);
  Vec8<T>::load(dy + at, dv);
  if (HAS_BIAS) Vec8<T>::load(bias + c, bv);
#pragma unroll
  for (int q = 0; q < 8; ++q) o[q] = dv[q] * gelu_grad(HAS_BIAS ? xv[q] + bv[q] : xv[q]);
  Vec8<T>::store(dx + at, o);
}

template <typename T, bool HAS_BIAS>
struct GeluBwdCols {
  static constexpr int kSums = 1;
  struct In { Raw8<T> x, dy; };
  RowsParams P;
  const T *dy, *x, *bias;
  T* dx;
  float bv[8];
  __device__ __forceinline__ void column(int64_t col) {
#pragma unroll
    for (int e = 0; e < 8; ++e) bv[e] = 0.f;
    if (HAS_BIAS) Vec8<T>::load(bias + col, bv);
  }
  __device__ __forceinline__ In load(int64_t r, int64_t col) const {
    In in;
    in.x.load(x + r * P.h + col);
    in.dy.load(dy + r * P.h + col);
    return in;
  }
  __device__ __forceinline__ void apply(const In& in, int64_t r, int64_t col, float (&acc)[1][8]) const {
    float xv[8], dv[8], o[8];
    in.x.get(xv);
    in.dy.get(dv);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      o[q] = dv[q] * gelu_grad(xv[q] + bv[q]);
      acc[0][q] += o[q];
    }
    Vec8<T>::store(dx + r * P.h + col, o);
  }
};

// ------------------------------------------------------------------------------------------------ launchers
static inline int pick_vpt(int64_t h, int& threads) {
  const int nchunk = (int)(h >> 3);
  int vpt = (nchunk + 1023) / 1024;
  if (vpt < 1) vpt = 1;
  threads = (nchunk + vpt - 1) / vpt;
  threads = (threads + 63) / 64 * 64;
  return vpt;
}

template <typename T>
static hipError_t ln_fwd_t(const RowsParams& P, const void* x, const void* gamma, const void* beta, void* y, float* mean, float* rstd, hipStream_t st) {
  int threads;
  const int vpt = pick_vpt(P.h, threads);
  dim3 grid((unsigned)P.rows), block(threads);
#define SAR_LN_FWD(V) hipLaunchKernelGGL((ln_fwd_kernel<T, V>), grid, block, 0, st, P, (const T*)x, (const T*)gamma, (const T*)beta, (T*)y, mean, rstd)
  switch (vpt) {
    case 1: SAR_LN_FWD(1); break;
    case 2: SAR_LN_FWD(2); break;
    case 3: SAR_LN_FWD(3); break;
    default: SAR_LN_FWD(4); break;
  }
#undef SAR_LN_FWD
  return hipGetLastError();
}

hipError_t launch_ln_fwd(const RowsParams& P, bool bf16, const void* x, const void* gamma, const void* beta, void* y, float* mean, float* rstd,
                         hipStream_t st) {
  return bf16 ? ln_fwd_t<uint16_t>(P, x, gamma, beta, y, mean, rstd, st) : ln_fwd_t<float>(P, x, gamma, beta, y, mean, rstd, st);
}

// Workgroups of the form that reads x and dy once, 0 where the other one runs.  About 512 threads a CU; the narrower a row, the
// fewer threads work on it and the more rows' partial sums there are.  From eight rows a workgroup on they cost less than the
// second read (two reads / one, us, bf16: 8192 x 1024 20.8 / 20.5, 2048 x 6144 24.0 / 22.7, 8192 x 4096 54.1 / 38.9; fp32 2048 x 6144 41.0 / 30.8,
// 4096 x 2048 30.8 / 23.3).  Rows wider than 20480 leave no registers for a request ahead (bf16: from sixteen rows on, 2048 x 25600 90.9 /
// 99.8, 4096 x 25600 193 / 163; from 24576 on 13 registers spill, and it is the faster one all the same, 4096 x 28672 214 / 180), and beyond
// 28672 there is no room for the sums.
static inline int ln_bwd_stream_groups(int64_t rows, int64_t h, bool bf16) {
  const int64_t nchunk = h >> 3;
  const int groups = nchunk <= 128 ? 1024 : nchunk <= 512 ? 512 : 256;
  return nchunk <= (bf16 ? 3584 : 2560) && rows >= (nchunk <= 2560 ? 8 : 16) * groups ? groups : 0;
}
// x and dy read twice.  Rows wider than 28672: 1024 threads (four chunks a thread; eight of 512 threads: 1024 x 32768 61 / 70 us).
static inline int ln_bwd_threads(int64_t h) { return h <= 8192 ? 256 : h <= 28672 ? 512 : 1024; }
// Column sums in one split, us one / split: up to a few hundred rows (bf16 512 x 4096 7.7 / 8.9, fp32 300 x 6144 8.3 / 9.1; but fp32 512 x 3072 10.0 /
// 8.7, bf16 512 x 6144 11.2 / 9.9), and wide rows at any count, as there are blocks enough for every CU (bf16 1024 x 16384 28.7 / 30.9), in wider
// segments the wider they are (bf16 300 x 32768 by 8, 32 lanes 25.8 / 19.8); not beyond 85 MB, three of
// which do not fit the last-level cache (2048 x 32768 141 / 128), and not on rows of up to 12288 with many of them, where the blocks, 129 to 192, each
// have a long chain (bf16 2000 x 8208 38.3 / 32.4, in segments of 16 lanes 34.5; 1500 x 10240 30.1 / 28.1; 900 x 8208 20.3 / 18.4; fp32 1500 x 9216 53.1 / 48.7, 1200 x
// 8208 43.6 / 38.4, but 800 x 9216 26.5 / 29.3, bf16 900 x 9216 18.0 / 18.6).
static inline ColPlan ln_bwd_plan(int64_t rows, int64_t h, bool bf16) {
  const int64_t nchunk = h >> 3, esz = bf16 ? 2 : 4;
  int one = 0;
  if (nchunk > 1024) one = rows * h * esz > 85000000 || (nchunk <= 1536 && rows > (bf16 ? 800 : 1024)) ? 0 : nchunk > 3584 ? 5 : nchunk > 2048 ? 4 : 3;
  else if (rows <= one_split_rows(h, bf16 && nchunk <= 512 ? 512 : 384)) one = 3;
  return col_plan(rows, h, esz, one, bf16 ? 768 : 512, bf16 && nchunk > 1024 ? 5 : 4, 3, ln_bwd_threads(h));
}

size_t ln_bwd_workspace_bytes(int64_t rows, int64_t h, bool bf16) {
  const int groups = ln_bwd_stream_groups(rows, h, bf16), nsplit = groups ? groups : ln_bwd_plan(rows, h, bf16).nsplit;
  return nsplit > 1 ? (size_t)nsplit * 2 * (size_t)h * sizeof(float) : 256;
}

template <typename T>
static hipError_t ln_bwd_t(const RowsParams& P, const void* dy, const void* x, const float* mean, const float* rstd, const void* gamma, void* dx,
                           float* dgamma, float* dbeta, void* ws, hipStream_t st) {
  const int nchunk = (int)(P.h >> 3);
  float* part = (float*)ws;
  constexpr bool half = sizeof(T) == 2;
  if (const int groups = ln_bwd_stream_groups(P.rows, P.h, half)) {
    auto go = [&](auto kern, int nt) {
      hipLaunchKernelGGL(kern, dim3(groups), dim3(nt), 0, st, P, (const T*)dy, (const T*)x, mean, rstd, (const T*)gamma, (T*)dx, part);
    };
    if (nchunk <= 128) go(ln_bwd_stream_kernel<T, 128, 1, true>, 128);
    else if (nchunk <= 256) go(ln_bwd_stream_kernel<T, 256, 1, true>, 256);
    else if (nchunk <= 512) go(ln_bwd_stream_kernel<T, 256, 2, true>, 256);
    else switch ((nchunk + 511) / 512) {
      case 2: go(ln_bwd_stream_kernel<T, 512, 2, true>, 512); break;
      case 3: go(ln_bwd_stream_kernel<T, 512, 3, true>, 512); break;
      case 4: go(ln_bwd_stream_kernel<T, 512, 4, half>, 512); break;
      case 5: go(ln_bwd_stream_kernel<T, 512, 5, half>, 512); break;
      default:
        if constexpr (half) {
          if (nchunk <= 3072) go(ln_bwd_stream_kernel<T, 512, 6, false>, 512);
          else go(ln_bwd_stream_kernel<T, 512, 7, false>, 512);
        }
    }
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : launch_colsum_finish(part, groups, 2 * P.h, P.h, dgamma, dbeta, st);
  }
  const int nt = ln_bwd_threads(P.h);
  const ColPlan pl = ln_bwd_plan(P.rows, P.h, half);
  float* dg_out = pl.nsplit == 1 ? dgamma : part;
  float* db_out = pl.nsplit == 1 ? dbeta : part + P.h;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((unsigned)(P.rows + (int64_t)pl.ncb * pl.nsplit)), dim3(nt), 0, st, P, (const T*)dy, (const T*)x, mean, rstd,
                       (const T*)gamma, (T*)dx, dg_out, db_out, pl);
  };
  const int vpt = (nchunk + nt - 1) / nt;
  if (nt == 256) {
    switch (vpt) {
      case 1: go(ln_bwd_kernel<T, 256, 1>); break;
      case 2: go(ln_bwd_kernel<T, 256, 2>); break;
      case 3: go(ln_bwd_kernel<T, 256, 3>); break;
      default: go(ln_bwd_kernel<T, 256, 4>); break;
    }
  } else if (nt == 1024) {
    go(ln_bwd_kernel<T, 1024, 4>);
  } else {
    switch (vpt) {
      case 3: go(ln_bwd_kernel<T, 512, 3>); break;
      case 4: go(ln_bwd_kernel<T, 512, 4>); break;
      case 5: go(ln_bwd_kernel<T, 512, 5>); break;
      case 6: go(ln_bwd_kernel<T, 512, 6>); break;
      default: go(ln_bwd_kernel<T, 512, 7>); break;
    }
  }
  const hipError_t e = hipGetLastError();
  return e != hipSuccess || pl.nsplit == 1 ? e : launch_colsum_finish(part, pl.nsplit, 2 * P.h, P.h, dgamma, dbeta, st);
}

hipError_t launch_ln_bwd(const RowsParams& P, bool bf16, const void* dy, const void* x, const float* mean, const float* rstd, const void* gamma,
                         void* dx, float* dgamma, float* dbeta, void* ws, hipStream_t st) {
  return bf16 ? ln_bwd_t<uint16_t>(P, dy, x, mean, rstd, gamma, dx, dgamma, dbeta, ws, st)
              : ln_bwd_t<float>(P, dy, x, mean, rstd, gamma, dx, dgamma, dbeta, ws, st);
}

template <typename T>
static hipError_t bda_t(const RowsParams& P, const void* x, const void* bias, const void* resid, void* out, uint8_t* mask, hipStream_t st) {
  dim3 grid((unsigned)P.rows, (unsigned)(((P.h >> 3) + 255) / 256)), block(256);
#define SAR_BDA(B, M) hipLaunchKernelGGL((bias_dropout_add_kernel<T, B, M>), grid, block, 0, st, P, (const T*)x, (const T*)bias, (const T*)resid, (T*)out, mask)
  if (bias && mask) SAR_BDA(true, true);
  else if (bias) SAR_BDA(true, false);
  else if (mask) SAR_BDA(false, true);
  else SAR_BDA(false, false);
#undef SAR_BDA
  return hipGetLastError();
}

hipError_t launch_bias_dropout_add(const RowsParams& P, bool bf16, const void* x, const void* bias, const void* resid, void* out, uint8_t* mask,
                                   hipStream_t st) {
  return bf16 ? bda_t<uint16_t>(P, x, bias, resid, out, mask, st) : bda_t<float>(P, x, bias, resid, out, mask, st);
}

template <typename T>
static hipError_t bda_ln_t(const RowsParams& P, const void* x, const void* bias, const void* resid, const void* gamma, const void* beta, void* out,
                           void* y, float* mean, float* rstd, hipStream_t st) {
  int threads;
  const int vpt = pick_vpt(P.h, threads);
  dim3 grid((unsigned)P.rows), block(threads);
#define SAR_BDA_LN(V, B) hipLaunchKernelGGL((bda_ln_fwd_kernel<T, V, B>), grid, block, 0, st, P, (const T*)x, (const T*)bias, (const T*)resid, \
                                            (const T*)gamma, (const T*)beta, (T*)out, (T*)y, mean, rstd)
#define SAR_BDA_LN_V(V) do { if (bias) SAR_BDA_LN(V, true); else SAR_BDA_LN(V, false); } while (0)
  switch (vpt) {
    case 1: SAR_BDA_LN_V(1); break;
    case 2: SAR_BDA_LN_V(2); break;
    case 3: SAR_BDA_LN_V(3); break;
    default: SAR_BDA_LN_V(4); break;
  }
#undef SAR_BDA_LN_V
#undef SAR_BDA_LN
  return hipGetLastError();
}

hipError_t launch_bias_dropout_add_ln_fwd(const RowsParams& P, bool bf16, const void* x, const void* bias, const void* resid, const void* gamma,
                                          const void* beta, void* out, void* y, float* mean, float* rstd, hipStream_t st) {
  return bf16 ? bda_ln_t<uint16_t>(P, x, bias, resid, gamma, beta, out, y, mean, rstd, st)
              : bda_ln_t<float>(P, x, bias, resid, gamma, beta, out, y, mean, rstd, st);
}

// One split, us one / split: bias-dropout backward up to some hundred rows (bf16 512 x 6144 6.9 / 7.8, 700 x 6144 8.6 / 7.9; fp32 300 x 6144 7.0 / 8.3, 512 x
// 4096 8.7 / 7.3) and on rows of 48 KB or more, whose blocks fill the chip by themselves (bf16 1024 x 32768 22.0 / 24.5, fp32 1024 x 12288 18.0 / 18.9).
static ColPlan bda_bwd_plan(int64_t rows, int64_t h, bool bf16) {
  const int64_t esz = bf16 ? 2 : 4;
  const bool one = rows <= one_split_rows(h, bf16 ? 512 : 384) || (h * esz >= 49152 && rows * h * esz <= 144000000);
  return col_plan(rows, h, esz, one ? 3 : 0, bf16 ? 768 : 512, 4, 2);
}
// bias-GeLU backward, which does more on a row: up to 256 (300 x 4096 8.0 / 7.7), on wide rows a little further (fp32 512 x 16384 16.6 / 19.1, bf16 300 x 16384
// 8.0 / 10.1, but bf16 512 x 25600 19.2 / 17.0); in bf16, whose rows are half as long, twice the workgroups or more (bf16 2048 x 10240
// by 1040, 2080 workgroups 26.0 / 24.0; fp32 8192 x 4096 by 512, 2048 72.5 / 75.1), in segments of 32 lanes (16, 32: 4096 x 6144 28.7 / 27.9; fp32
// 8192 x 4096 72.5 / 77.8).
static ColPlan bias_gelu_bwd_plan(int64_t rows, int64_t h, bool bf16) {
  const int64_t few = h >= 12288 ? (bf16 ? 320 : 640) : 256;
  return col_plan(rows, h, bf16 ? 2 : 4, rows <= one_split_rows(h, few) ? 3 : 0, bf16 ? 2048 : 512, bf16 ? 5 : 4, 3);
}
// Where both passes need scratch, one size for both, so that a buffer sized for either serves the other; none where a pass needs none.
static inline size_t bias_bwd_workspace_bytes(const ColPlan& pl, const ColPlan& other, int64_t h) {
  return pl.nsplit > 1 ? std::max(colsum_workspace_bytes(pl, h), colsum_workspace_bytes(other, h)) : 0;
}
size_t bias_gelu_bwd_workspace_bytes(int64_t rows, int64_t h, bool bf16) {
  return bias_bwd_workspace_bytes(bias_gelu_bwd_plan(rows, h, bf16), bda_bwd_plan(rows, h, bf16), h);
}
size_t bda_bwd_workspace_bytes(int64_t rows, int64_t h, bool bf16) {
  return bias_bwd_workspace_bytes(bda_bwd_plan(rows, h, bf16), bias_gelu_bwd_plan(rows, h, bf16), h);
}

// Which results are written past the caches?  What the pair of a pass and the reader of its result takes decides, not the pass alone: in a loop over one set of buffers,
// where nobody reads the results, storing those of every pass past the caches from 32 or 48 MB on makes the passes up to 15 % faster (their inputs stay in the last-level cache for the next
// round), but a reader then finds them in memory.  us, kept / past, pass and reader together, inputs not in the cache unless said otherwise (bf16; 34 / 50 / 67 / 100 / 168 MB a tensor):
//   bias_gelu_fwd, x just written by a matrix product, y read by one of 2048 columns   148 / 148, 179 / 177, 242 / 238, 285 / 284, 472 / 465 (201 MB 492 / 481, but 268 MB 803 / 808), read by a copy
//     45 / 48, 62 / 66, 82 / 80, 122 / 120, 210 / 196 (268 MB 349 / 337)
//   bias_gelu_bwd, dx read by a matrix product   137 / 138, 163 / 166, 218 / 220, 256 / 262, 432 / 440, by a copy 34 / 37, 48 / 51, 67 / 67, 107 / 102, 162 / 167
//   bias_dropout_add_bwd with dbias, likewise   130 / 132, 152 / 154, 205 / 207, 234 / 235, 390 / 399; copy 27 / 30, 38 / 42, 48 / 53, 76 / 79, 127 / 129; dout just written (by a product) 67 / 100 /
//     134 / 168 / 200 MB: 247 / 244, 292 / 291, 429 / 419, 477 / 473, 498 / 488, copy 91 / 84, 126 / 124, 190 / 173, 217 / 202, 257 / 236 (268 MB 816 / 821, 355 / 355)
//   ln_bwd, dx read by a copy (as by the pass before it)   40 / 43, 59 / 62, 74 / 76, 115 / 109, 169 / 170
//   bias_dropout_add_ln_fwd, out and y, y read by a matrix product   141 / 142, 171 / 171, 228 / 230, 273 / 273, 461 / 459
// and a whole MLP block, forward and backward with its products, all of them past the caches, at nine shapes between 0.986 and 1.005 of the time kept.  So only below
// the cache's 256 MB, and where the input has just been written: the forward of the bias-GeLU from 40 MB, from where it gains with the product that reads its y in an MLP (42 MB 126 / 124, 116 / 114, 254 / 254, 50 MB
// above; with a copy from 64 MB), and bias_dropout_add_bwd, whose dout the pass before has written, from 64 MB, from where it gains with either reader (42 and 50 MB with a product 0.98 to 1.01).
static std::atomic<int> g_force_stream{-1};  // sar_test_force_forms (tests, measurements)
void rows_force_stream(int force) { g_force_stream = force; }
static inline bool result_stream(int64_t bytes, int64_t least) {
  const int force = g_force_stream.load(std::memory_order_relaxed);
  return force >= 0 ? force != 0 : bytes >= least && bytes < 256000000;
}

template <typename T>
static hipError_t bda_bwd_t(const RowsParams& P, const void* dout, void* dx, float* dbias, void* ws, hipStream_t st) {
  if (!dbias) {
    hipLaunchKernelGGL((bda_bwd_kernel<T>), dim3((unsigned)P.rows, (unsigned)(((P.h >> 3) + 255) / 256)), dim3(256), 0, st, P, (const T*)dout, (T*)dx);
    return hipGetLastError();
  }
  const ColPlan pl = bda_bwd_plan(P.rows, P.h, sizeof(T) == 2);
  if (result_stream(P.rows * P.h * (int64_t)sizeof(T), 64000000)) return launch_colsum(BdaBwdCols<T, true>{P, (const T*)dout, (T*)dx}, P.rows, P.h, pl, dbias, (float*)ws, st);
  return launch_colsum(BdaBwdCols<T, false>{P, (const T*)dout, (T*)dx}, P.rows, P.h, pl, dbias, (float*)ws, st);
}

hipError_t launch_bias_dropout_add_bwd(const RowsParams& P, bool bf16, const void* dout, void* dx, float* dbias, void* ws, hipStream_t st) {
  return bf16 ? bda_bwd_t<uint16_t>(P, dout, dx, dbias, ws, st) : bda_bwd_t<float>(P, dout, dx, dbias, ws, st);
}

template <typename T>
static hipError_t bias_gelu_fwd_t(const RowsParams& P, const void* x, const void* bias, void* y, hipStream_t st) {
  dim3 grid((unsigned)P.rows, (unsigned)(((P.h >> 3) + 255) / 256)), block(256);
  auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, block, 0, st, P, (const T*)x, (const T*)bias, (T*)y); };
  if (result_stream(P.rows * P.h * (int64_t)sizeof(T), 40000000)) bias ? go(bias_gelu_fwd_kernel<T, true, true>) : go(bias_gelu_fwd_kernel<T, false, true>);
  else bias ? go(bias_gelu_fwd_kernel<T, true, false>) : go(bias_gelu_fwd_kernel<T, false, false>);
  return hipGetLastError();
}

hipError_t launch_bias_gelu_fwd(const RowsParams& P, bool bf16, const void* x, const void* bias, void* y, hipStream_t st) {
  return bf16 ? bias_gelu_fwd_t<uint16_t>(P, x, bias, y, st) : bias_gelu_fwd_t<float>(P, x, bias, y, st);
}

template <typename T>
static hipError_t bias_gelu_bwd_t(const RowsParams& P, const void* dy, const void* x, const void* bias, void* dx, float* dbias, void* ws,
                                  hipStream_t st) {
  if (!dbias) {
    dim3 grid((unsigned)P.rows, (unsigned)(((P.h >> 3) + 255) / 256)), block(256);
    if (bias) hipLaunchKernelGGL((bias_gelu_bwd_kernel<T, true>), grid, block, 0, st, P, (const T*)dy, (const T*)x, (const T*)bias, (T*)dx);
    else hipLaunchKernelGGL((bias_gelu_bwd_kernel<T, false>), grid, block, 0, st, P, (const T*)dy, (const T*)x, (const T*)bias, (T*)dx);
    return hipGetLastError();
  }
  const ColPlan pl = bias_gelu_bwd_plan(P.rows, P.h, sizeof(T) == 2);
  if (bias) return launch_colsum(GeluBwdCols<T, true>{P, (const T*)dy, (const T*)x, (const T*)bias, (T*)dx, {}}, P.rows, P.h, pl, dbias, (float*)ws, st);
  return launch_colsum(GeluBwdCols<T, false>{P, (const T*)dy, (const T*)x, nullptr, (T*)dx, {}}, P.rows, P.h, pl, dbias, (float*)ws, st);
}

hipError_t launch_bias_gelu_bwd(const RowsParams& P, bool bf16, const void* dy, const void* x, const void* bias, void* dx, float* dbias, void* ws,
                                hipStream_t st) {
  return bf16 ? bias_gelu_bwd_t<uint16_t>(P, dy, x, bias, dx, dbias, ws, st) : bias_gelu_bwd_t<float>(P, dy, x, bias, dx, dbias, ws, st);
}

}  // namespace sar
