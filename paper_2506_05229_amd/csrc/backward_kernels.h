// Kernels of the ARMT backward pass (the paper's appendix states that a backward pass of the diagonal
// schedule exists; what it computes is the gradient of the forward of Section 2.1, Eq. 2-6).
// Everything that is a contraction goes through the grouped GEMM (with transposed operand copies made
// by transpose_kernel); this file holds the element-wise, row-wise and reduction parts, the
// attention backward and the backward of the delta rule.  Plain fp32 arithmetic throughout.
#pragma once

#include "attention_generic.h"
#include "common.h"
#include "rowwise_kernels.h"

namespace armt {

// dst[c * ldd + r] = src[r * lds + c] for r < R, c < C, per cell (cell strides in elements).
// Columns [R, ldd) of dst are never written: callers keep them zero (they pad the reduction dimension
// of the following GEMM).  grid: (ceil(C / 32), ceil(R / 32), g), block: (32, 8).
template <typename Tin, typename Tout>
__global__ __launch_bounds__(256) void transpose_kernel(const Tin* __restrict__ src, size_t src_cell, int lds,
                                                        Tout* __restrict__ dst, size_t dst_cell, int ldd, int R, int C) {
  __shared__ float tile[32][33];
  const Tin* s = src + (size_t)blockIdx.z * src_cell;
  Tout* o = dst + (size_t)blockIdx.z * dst_cell;
  const int c0 = blockIdx.x * 32, r0 = blockIdx.y * 32;
  for (int j = threadIdx.y; j < 32; j += 8) {
    const int r = r0 + j, c = c0 + threadIdx.x;
    tile[j][threadIdx.x] = (r < R && c < C) ? to_f32(s[(size_t)r * lds + c]) : 0.f;
  }
  __syncthreads();
  for (int j = threadIdx.y; j < 32; j += 8) {
    const int c = c0 + j, r = r0 + threadIdx.x;
    if (c < C && r < R) o[(size_t)c * ldd + r] = from_f32<Tout>(tile[threadIdx.x][j]);
  }
}

// Up to TRANSPOSE_JOBS transposes of that kind in one launch, each with its own number of cells.  A step of the fp32 configuration has a
// dozen of them of a few microseconds each, which were launches and little else.
// grid: (tiles of all jobs, 1, largest number of cells), block: (32, 8).
constexpr int TRANSPOSE_JOBS = 32;
struct TransposeJob { const void* src; void* dst; size_t src_cell, dst_cell; int lds, ldd, R, C, cells, tiles_c, end, pad_; };
struct TransposeJobs { TransposeJob job[TRANSPOSE_JOBS]; int n; };       // end: tiles of this job and those before it
static_assert(sizeof(TransposeJobs) <= 3600, "kernel arguments are limited to 4 KB");
__global__ __launch_bounds__(256) void transpose_many_kernel(TransposeJobs jobs) {
  __shared__ float tile[32][33];
  int w = 0;
  while (w < jobs.n - 1 && (int)blockIdx.x >= jobs.job[w].end) ++w;
  const TransposeJob j = jobs.job[w];
  if ((int)blockIdx.z >= j.cells) return;
  const int t = blockIdx.x - (w ? jobs.job[w - 1].end : 0), c0 = t % j.tiles_c * 32, r0 = t / j.tiles_c * 32;
  const float* s = (const float*)j.src + (size_t)blockIdx.z * j.src_cell;
  float* o = (float*)j.dst + (size_t)blockIdx.z * j.dst_cell;
  for (int y = threadIdx.y; y < 32; y += 8) {
    const int r = r0 + y, c = c0 + threadIdx.x;
    tile[y][threadIdx.x] = (r < j.R && c < j.C) ? s[(size_t)r * j.lds + c] : 0.f;
  }
  __syncthreads();
  for (int y = threadIdx.y; y < 32; y += 8) {
    const int c = c0 + y, r = r0 + threadIdx.x;
    if (c < j.C && r < j.R) o[(size_t)c * j.ldd + r] = tile[threadIdx.x][y];
  }
}

// The same for bf16 -> bf16 with 16-byte accesses on both sides: 64 x 64 tiles through LDS (row stride 66 keeps the
// column reads of the second phase on distinct banks).  Needs C, lds, ldd multiples of 8 and 16-byte aligned bases;
// rows [R, ldd) of a tile are written as zeros, which is what the padding columns of dst must hold anyway.
// grid: (ceil(C / 64), ceil(R / 64), g), block: 256.
__global__ __launch_bounds__(256) void transpose_bf16_kernel(const bf16* __restrict__ src, size_t src_cell, int lds,
                                                             bf16* __restrict__ dst, size_t dst_cell, int ldd, int R, int C) {
  __shared__ unsigned int tile[64 * 33];
  const bf16* s = src + (size_t)blockIdx.z * src_cell;
  bf16* o = dst + (size_t)blockIdx.z * dst_cell;
  const int c0 = blockIdx.x * 64, r0 = blockIdx.y * 64;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int idx = threadIdx.x + 256 * k, r = idx >> 3, ch = idx & 7;
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (r0 + r < R && c0 + 8 * ch < C) v = *(const uint4*)(s + (size_t)(r0 + r) * lds + c0 + 8 * ch);
    unsigned int* t = tile + r * 33 + 4 * ch;
    t[0] = v.x; t[1] = v.y; t[2] = v.z; t[3] = v.w;
  }
  __syncthreads();
  const unsigned short* th = (const unsigned short*)tile;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int idx = threadIdx.x + 256 * k, c = idx >> 3, rch = idx & 7;
    if (c0 + c >= C || r0 + 8 * rch + 7 >= ldd) continue;
    unsigned int w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const unsigned int lo = th[(8 * rch + 2 * e) * 66 + c], hi = th[(8 * rch + 2 * e + 1) * 66 + c];
      w[e] = lo | (hi << 16);
    }
    *(uint4*)(o + (size_t)(c0 + c) * ldd + r0 + 8 * rch) = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

// An fp32 gradient as the operands of the two products it enters, in one pass over it: dst [R][ldd] in bf16, columns [C, Cp) zero, and its
// transpose dst_t[c][r] (c < Cp, row stride ldt, rows [R, Rp) zero).  Cell z of the launch writes its transpose at layer z / batch and column
// offset (z % batch) * Rp, as the windows of the weight gradients want it.  Bound by memory; reading the bf16 copy back for a transpose of its
// own cost a third more traffic: 4096 x 128256 835 + 470 us -> 920, 1B shape (mean of 5.6 cells) 25 + 9 -> 19.
// wide: src and its rows start on 16 bytes; else it is read in 4-byte accesses, a row of the tile per wave.
// Cp, Rp, ldd, ldt multiples of 8 (Cp and Rp of 64); bases of the destinations on 16 bytes.
// grid: (Cp / 64, ceil(R / 64), cells), block: 256.
__global__ __launch_bounds__(256) void convert_transpose_kernel(const float* __restrict__ src, size_t src_cell, int lds, bool wide,
                                                                bf16* __restrict__ dst, size_t dst_cell, int ldd, bf16* __restrict__ dst_t,
                                                                size_t dst_t_layer, int ldt, int batch, int R, int C, int Rp) {
  __shared__ unsigned int tile[64 * 33];
  const float* s = src + (size_t)blockIdx.z * src_cell;
  bf16* o = dst + (size_t)blockIdx.z * dst_cell;
  bf16* ot = dst_t + (size_t)(blockIdx.z / batch) * dst_t_layer + (size_t)(blockIdx.z % batch) * Rp;
  const int c0 = blockIdx.x * 64, r0 = blockIdx.y * 64;
  unsigned short* th = (unsigned short*)tile;
  if (wide && c0 + 64 <= C) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int idx = threadIdx.x + 256 * k, r = idx >> 3, ch = idx & 7;
      bf16x8 v = {0, 0, 0, 0, 0, 0, 0, 0};
      if (r0 + r < R) {
        const float* p = s + (size_t)(r0 + r) * lds + c0 + 8 * ch;
        const f32x4 a = *(const f32x4*)p, b = *(const f32x4*)(p + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) { v[e] = (bf16)a[e]; v[4 + e] = (bf16)b[e]; }
      }
      const uint4 u = __builtin_bit_cast(uint4, v);
      unsigned int* t = tile + r * 33 + 4 * ch;
      t[0] = u.x; t[1] = u.y; t[2] = u.z; t[3] = u.w;
    }
  } else {
    const int c = c0 + (threadIdx.x & 63), rw = threadIdx.x >> 6;
    float v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int r = r0 + rw + 4 * k;
      v[k] = r < R && c < C ? s[(size_t)r * lds + c] : 0.f;
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) th[(rw + 4 * k) * 66 + (threadIdx.x & 63)] = __builtin_bit_cast(unsigned short, (bf16)v[k]);
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int idx = threadIdx.x + 256 * k, r = idx >> 3, ch = idx & 7;
    if (r0 + r < R) {
      const unsigned int* t = tile + r * 33 + 4 * ch;
      *(uint4*)(o + (size_t)(r0 + r) * ldd + c0 + 8 * ch) = make_uint4(t[0], t[1], t[2], t[3]);
    }
    if (r0 + 8 * ch + 7 < Rp) {                 // r counts columns here, ch eighths of the tile's rows
      unsigned int w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const unsigned int lo = th[(8 * ch + 2 * e) * 66 + r], hi = th[(8 * ch + 2 * e + 1) * 66 + r];
        w[e] = lo | (hi << 16);
      }
      *(uint4*)(ot + (size_t)(c0 + r) * ldt + r0 + 8 * ch) = make_uint4(w[0], w[1], w[2], w[3]);
    }
  }
}

// u[i] += u[n + i] + u[2 n + i] + ...: partial results of a product, added in order.
__global__ void sum_parts_kernel(float* __restrict__ u, size_t n, int parts) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    float s = u[i];
#pragma unroll 4
    for (int p = 1; p < parts; ++p) s += u[p * n + i];
    u[i] = s;
  }
}

template <typename Tin, typename Tout>
__global__ void convert_kernel(const Tin* __restrict__ src, Tout* __restrict__ dst, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    dst[i] = from_f32<Tout>(to_f32(src[i]));
}

// RMSNorm that keeps 1 / rms for the backward pass: out = x * rstd * gain.  grid: (T, g), block: 256.
template <typename T>
__global__ __launch_bounds__(256) void rmsnorm_train_kernel(const float* __restrict__ X, size_t x_cell,
                                                            const LayerAux* __restrict__ aux, int first, int which,
                                                            int Trows, int d, float eps, T* __restrict__ out,
                                                            float* __restrict__ rstd_out) {
  __shared__ float red[17];
  const int l = first + blockIdx.y;
  const float* x = X + (size_t)l * x_cell + (size_t)blockIdx.x * d;
  const size_t row = ((size_t)l * Trows + blockIdx.x) * d;
  const T* gain = (const T*)(which == 0 ? aux[l].rms1 : aux[l].rms2);
  float ss = 0.f;
  for (int c = threadIdx.x; c < d; c += blockDim.x) ss = fmaf(x[c], x[c], ss);
  ss = block_sum(ss, red);
  const float rstd = 1.0f / sqrtf(ss / (float)d + eps);
  for (int c = threadIdx.x; c < d; c += blockDim.x) out[row + c] = from_f32<T>(x[c] * rstd * to_f32(gain[c]));
  if (threadIdx.x == 0) rstd_out[(size_t)l * Trows + blockIdx.x] = rstd;
}

// Backward of n = x * rstd * gain for one row: dx = din + rstd * (g dn - x rstd^2 mean(g dn x)).
// dN, X, din, dout are [cells][T][d] with their own cell strides (din / dout may be slots of the gradient
// stream); doutb (optional) is an activation-typed copy of dout.  grid: (T, g), block: 256.
template <typename T>
__global__ __launch_bounds__(256) void rmsnorm_bwd_kernel(const T* __restrict__ dN, const float* __restrict__ X,
                                                          size_t x_cell, const LayerAux* __restrict__ aux, int first,
                                                          int which, const float* __restrict__ rstd_all,
                                                          const float* __restrict__ din, size_t din_cell,
                                                          float* __restrict__ dout, size_t dout_cell,
                                                          T* __restrict__ doutb, int Trows, int d) {
  __shared__ float red[17];
  const int l = first + blockIdx.y, i = blockIdx.x;
  const T* dn = dN + ((size_t)l * Trows + i) * d;
  const float* x = X + (size_t)l * x_cell + (size_t)i * d;
  const float* di = din + (size_t)l * din_cell + (size_t)i * d;
  float* dout_r = dout + (size_t)l * dout_cell + (size_t)i * d;
  const T* gain = (const T*)(which == 0 ? aux[l].rms1 : aux[l].rms2);
  const float rstd = rstd_all[(size_t)l * Trows + i];
  float s = 0.f;
  for (int c = threadIdx.x; c < d; c += blockDim.x) s = fmaf(to_f32(gain[c]) * to_f32(dn[c]), x[c], s);
  s = block_sum(s, red) / (float)d;
  const float k = rstd * rstd * s;
  for (int c = threadIdx.x; c < d; c += blockDim.x) {
    const float v = di[c] + rstd * (to_f32(gain[c]) * to_f32(dn[c]) - x[c] * k);
    dout_r[c] = v;
    if (doutb) doutb[((size_t)l * Trows + i) * d + c] = from_f32<T>(v);
  }
}

// rmsnorm_bwd_kernel and the gradient of the gain in one pass over dN and X (the pass is bound by memory, and the column sums over the rows
// read both of them again): part[cell][chunk][c] = sum_{i in chunk} rstd[i] dN[i, c] X[i, c], for colsum_finish_kernel.  A chunk is a block,
// whose threads share a row, R rows at a time: a thread holds the gain, the sums and R rows of its 4 NB columns only, so that 3 to 7 waves fit on a
// SIMD, and one barrier serves R rows.  (A wave per row held 4 d / 64 registers of each: one wave per SIMD from d 2048 on, and slower than two
// passes for few rows and at d 4096.)  us with the finish, 1040 rows, two passes / wave per row / here: d 768 1 cell 16.2 / 12.2 / 12.3,
// 5 cells 37.3 / 19.5 / 19.3; d 2048 1 cell 32.1 / 22.6 / 17.9, 5 cells 59.1 / 47.5 / 33.8, 16 cells 171 / 133 / 122; d 3072 1 cell 37.1 / 34.2 / 22.3,
// 5 cells 81.2 / 76.8 / 54.9; d 4096 1 cell 42.6 / 53.7 / 25.2, 5 cells 116 / 150 / 79; one cell of 272 rows, d 3072 13.3 / 18.4 / 12.4.
// d a multiple of 4, at most 1024 NB.  grid: (chunks, g), block: 256, or with d < 1024 the multiple of 64 that holds d / 4.
// 128 chunks of a cell's rows (9 rows of 1040), fewer below 512 and 128 rows, where empty chunks and the finish cost more than the blocks bring
// (us with 32 / 64 / 128: 1 cell of 1040 rows, d 2048 35.9 / 23.3 / 17.9; 8 cells of 272 rows, d 2048 18.8 / 17.9 / 20.1; 4 cells of 72 rows, d 128, fp32
// 5.7 / 6.3 / 7.3).  By the rows alone: a cell's sums may not depend on the cells beside it.
constexpr int NORM_CHUNKS = 128;
inline int norm_chunks(int Trows) { return Trows >= 512 ? NORM_CHUNKS : Trows >= 128 ? 64 : 32; }
template <typename T, int NB, int R>
__global__ __launch_bounds__(256) void rmsnorm_bwd_cols_kernel(const T* __restrict__ dN, const float* __restrict__ X, size_t x_cell,
                                                               const LayerAux* __restrict__ aux, int first, int which,
                                                               const float* __restrict__ rstd_all, const float* __restrict__ din,
                                                               size_t din_cell, float* __restrict__ dout, size_t dout_cell,
                                                               T* __restrict__ doutb, float* __restrict__ part, int Trows, int d) {
  typedef T T4 __attribute__((ext_vector_type(4)));
  __shared__ float red[2][R][4];             // the waves' sums of R rows; the other half while a wave may still read this one
  const int l = first + blockIdx.y, lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int c0 = 4 * threadIdx.x, step = 4 * blockDim.x;
  const T* gain = (const T*)(which == 0 ? aux[l].rms1 : aux[l].rms2);
  const int per = (Trows + gridDim.x - 1) / gridDim.x;
  const int i0 = blockIdx.x * per, i1 = min(Trows, i0 + per);
  f32x4 gn[NB], cs[NB];
#pragma unroll
  for (int k = 0; k < NB; ++k)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      gn[k][e] = c0 + k * step < d ? to_f32(gain[c0 + k * step + e]) : 0.f;     // (a caller's weight: may start anywhere)
      cs[k][e] = 0.f;
    }
  int half = 0;
  for (int i = i0; i < i1; i += R, half ^= 1) {
    f32x4 xv[R][NB], iv[R][NB];
    T4 t[R][NB];
    float rstd[R], s[R] = {};
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int row = min(i + r, i1 - 1);
      const size_t at_row = (size_t)row * d;
      rstd[r] = rstd_all[(size_t)l * Trows + row];
#pragma unroll
      for (int k = 0; k < NB; ++k) {
        const int at = min(c0 + k * step, d - 4);
        t[r][k] = *(const T4*)(dN + (size_t)l * Trows * d + at_row + at);
        xv[r][k] = *(const f32x4*)(X + (size_t)l * x_cell + at_row + at);
        iv[r][k] = *(const f32x4*)(din + (size_t)l * din_cell + at_row + at);
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (i + r >= i1) break;                // the last rows of a chunk: block-uniform
#pragma unroll
      for (int k = 0; k < NB; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float dn = c0 + k * step < d ? to_f32(t[r][k][e]) : 0.f;
          cs[k][e] = fmaf(dn * xv[r][k][e], rstd[r], cs[k][e]);
          s[r] = fmaf(dn * gn[k][e], xv[r][k][e], s[r]);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
      for (int r = 0; r < R; ++r) s[r] += __shfl_xor(s[r], o, kWave);
    if (lane == 0)
#pragma unroll
      for (int r = 0; r < R; ++r) red[half][r][w] = s[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (i + r >= i1) break;
      float sum = red[half][r][0];
      for (int v = 1; v < nw; ++v) sum += red[half][r][v];
      const float f = rstd[r] * rstd[r] * (sum / (float)d);
#pragma unroll
      for (int k = 0; k < NB; ++k) {
        const int c = c0 + k * step;
        if (c >= d) continue;
        f32x4 v;
        T4 b;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[e] = iv[r][k][e] + rstd[r] * (to_f32(t[r][k][e]) * gn[k][e] - xv[r][k][e] * f);
          b[e] = from_f32<T>(v[e]);
        }
        *(f32x4*)(dout + (size_t)l * dout_cell + (size_t)(i + r) * d + c) = v;
        if (doutb) *(T4*)(doutb + ((size_t)l * Trows + i + r) * d + c) = b;
      }
    }
  }
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    const int c = c0 + k * step;
    if (c < d) *(f32x4*)(part + ((size_t)l * gridDim.x + blockIdx.x) * d + c) = cs[k];
  }
}

// Column sums over the T rows of a cell, in two deterministic stages.  Stage 1: the rows are cut into gridDim.z
// chunks; a thread owns a column and adds its chunk's rows in order:
//   part[cell][chunk][c] = sum_{i in chunk} w[i] a[i, c] (b ? b[i, c] : 1).
// Stage 2 (colsum_finish_kernel) adds the chunks in order into the destination.
// a: [cells][T][C] activation type; b: fp32 with its own cell stride (or null); w: [cells][T].
// grid: (ceil(C / 256), g, chunks), block: 256.
// 64 chunks: the few columns of a feature map are a chain of row reads otherwise (1B shape, Phi 384, mean of 5.6 cells 27.5 us with 16 chunks, 10.1
// with 64; 4096 rows of the norm in front of the head 85 and 25).
constexpr int CS_CHUNKS = 64;
template <typename T>
__global__ __launch_bounds__(256) void colsum_partial_kernel(const T* __restrict__ a, const float* __restrict__ b, size_t b_cell,
                                                             const float* __restrict__ w, float* __restrict__ part, int first,
                                                             int Trows, int C) {
  const int l = first + blockIdx.y, c = blockIdx.x * 256 + threadIdx.x;
  if (c >= C) return;
  const int per = (Trows + gridDim.z - 1) / gridDim.z;
  const int i0 = blockIdx.z * per, i1 = min(Trows, i0 + per);
  const T* ap = a + (size_t)l * Trows * C;
  const float* bp = b ? b + (size_t)l * b_cell : nullptr;
  const float* wp = w + (size_t)l * Trows;
  float s = 0.f;
  for (int i = i0; i < i1; ++i) {
    const float v = to_f32(ap[(size_t)i * C + c]) * (bp ? bp[(size_t)i * C + c] : 1.f);
    s = fmaf(v, wp[i], s);
  }
  part[((size_t)l * gridDim.z + blockIdx.z) * C + c] = s;
}

// dst[c] += sum over nb consecutive cells and their chunks of part[cell][chunk][c]; dst = dst_tab[first cell] if a pointer
// table is given (the nb cells of a batch that share a layer's gradient), else dst_base + cell * C (nb = 1).
// grid: (ceil(C / 256), cells / nb), block: 256.
__global__ __launch_bounds__(256) void colsum_finish_kernel(const float* __restrict__ part, int chunks, float* const* __restrict__ dst_tab,
                                                            float* __restrict__ dst_base, int first, int C, int nb) {
  const int l = first + blockIdx.y * nb, c = blockIdx.x * 256 + threadIdx.x;      // destination of cells l .. l + nb - 1
  if (c >= C) return;
  float s = 0.f;
  for (int b = 0; b < nb; ++b)
#pragma unroll 16
    for (int k = 0; k < chunks; ++k) s += part[((size_t)(l + b) * chunks + k) * C + c];
  float* dst = dst_tab ? dst_tab[l] : dst_base + (size_t)l * C;
  dst[c] += s;
}

// u = silu(gate) * up from the stored [gate | up] rows.  GU: [cells][T][2F]; U: [cells][T][F].
template <typename T>
__global__ void swiglu_kernel(const T* __restrict__ GU, T* __restrict__ U, size_t rows, int F) {
  const size_t n = rows * F;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const size_t r = i / F, c = i % F;
    const float g = to_f32(GU[r * 2 * F + c]), u = to_f32(GU[r * 2 * F + F + c]);
    U[i] = from_f32<T>(g / (1.f + expf(-g)) * u);
  }
}

// In place on [gate | up]: dgate = dU up sig(g) (1 + g (1 - sig(g))), dup = dU silu(g).
template <typename T>
__global__ void swiglu_bwd_kernel(T* __restrict__ GU, const T* __restrict__ dU, size_t rows, int F) {
  const size_t n = rows * F;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const size_t r = i / F, c = i % F;
    const float g = to_f32(GU[r * 2 * F + c]), u = to_f32(GU[r * 2 * F + F + c]), du = to_f32(dU[i]);
    const float sg = 1.f / (1.f + expf(-g));
    GU[r * 2 * F + c] = from_f32<T>(du * u * sg * (1.f + g * (1.f - sg)));
    GU[r * 2 * F + F + c] = from_f32<T>(du * g * sg);
  }
}

// bf16 versions of the two SwiGLU kernels that also leave the transposed copy the weight-gradient GEMMs need, written
// straight into a layer's window rows (row stride ldd; the cell z of the launch belongs to layer z / batch and puts its
// T columns at column offset (z % batch) * Tp): 64 x 64 tiles, 16-byte accesses, the transposed half through LDS as in
// transpose_bf16_kernel (tile rows past T are written as zeros: the padding of the reduction dimension).
// Forward (BWD = false): u = silu(gate) up; U^T -> dst rows [c]; U itself only for rows >= first_row (the memory rows, all
//   the recomputed down projection reads).  GU: [cells][T][2F], U: [cells][T][F].
// Backward (BWD = true): [gate | up] <- [dgate | dup] in place from dU, and the same values transposed -> dst rows [c] (dgate)
//   and [F + c] (dup).
// grid: (F / 64, ceil(T / 64), cells), block: 256.  F a multiple of 64.
template <bool BWD>
__global__ __launch_bounds__(256) void swiglu_tiles_kernel(bf16* __restrict__ GU, bf16* __restrict__ U /* BWD: dU (read) */,
                                                           int Trows, int F, int first_row, bf16* __restrict__ dst,
                                                           size_t dst_layer, int ldd, int batch, int Tp) {
  __shared__ unsigned int tg[64 * 33], tu[64 * 33];
  const int z = blockIdx.z, c0 = blockIdx.x * 64, r0 = blockIdx.y * 64;
  bf16* gu = GU + (size_t)z * Trows * 2 * F;
  bf16* uu = U + (size_t)z * Trows * F;
  bf16* o = dst + (size_t)(z / batch) * dst_layer + (size_t)(z % batch) * Tp;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int idx = threadIdx.x + 256 * k, r = idx >> 3, ch = idx & 7, row = r0 + r, col = c0 + 8 * ch;
    bf16x8 a = {0, 0, 0, 0, 0, 0, 0, 0}, b = a;           // what goes to the transposed copy
    if (row < Trows) {
      const bf16x8 g = *(const bf16x8*)(gu + (size_t)row * 2 * F + col), up = *(const bf16x8*)(gu + (size_t)row * 2 * F + F + col);
      if (BWD) {
        const bf16x8 du = *(const bf16x8*)(uu + (size_t)row * F + col);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float gf = (float)g[e], sg = 1.f / (1.f + expf(-gf)), d = (float)du[e];
          a[e] = (bf16)(d * (float)up[e] * sg * (1.f + gf * (1.f - sg)));
          b[e] = (bf16)(d * gf * sg);
        }
        *(bf16x8*)(gu + (size_t)row * 2 * F + col) = a;
        *(bf16x8*)(gu + (size_t)row * 2 * F + F + col) = b;
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float gf = (float)g[e];
          a[e] = (bf16)(gf / (1.f + expf(-gf)) * (float)up[e]);
        }
        if (row >= first_row) *(bf16x8*)(uu + (size_t)row * F + col) = a;
      }
    }
    const uint4 av = __builtin_bit_cast(uint4, a), bv = __builtin_bit_cast(uint4, b);
    unsigned int* t = tg + r * 33 + 4 * ch;
    t[0] = av.x; t[1] = av.y; t[2] = av.z; t[3] = av.w;
    if (BWD) {
      unsigned int* t2 = tu + r * 33 + 4 * ch;
      t2[0] = bv.x; t2[1] = bv.y; t2[2] = bv.z; t2[3] = bv.w;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int idx = threadIdx.x + 256 * k, c = idx >> 3, rch = idx & 7;
    if (r0 + 8 * rch + 7 >= Tp) continue;                 // Tp is a multiple of 64: never true for a started tile row block
#pragma unroll
    for (int h = 0; h < (BWD ? 2 : 1); ++h) {
      const unsigned short* th = (const unsigned short*)(h ? tu : tg);
      unsigned int w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const unsigned int lo = th[(8 * rch + 2 * e) * 66 + c], hi = th[(8 * rch + 2 * e + 1) * 66 + c];
        w[e] = lo | (hi << 16);
      }
      *(uint4*)(o + (size_t)(h * F + c0 + c) * ldd + r0 + 8 * rch) = make_uint4(w[0], w[1], w[2], w[3]);
    }
  }
}

// Backward of the rotary embedding: rotate the gradient of q and k by the opposite angle, in place.
template <typename T>
__global__ __launch_bounds__(256) void rope_bwd_kernel(T* __restrict__ dQKV, const float* __restrict__ cs, int first,
                                                       int Trows, int n_rot_heads, int dh, int ldq) {
  const int l = first + blockIdx.y, p = blockIdx.x, half = dh >> 1;
  T* row = dQKV + ((size_t)l * Trows + p) * ldq;
  for (int i = threadIdx.x; i < n_rot_heads * half; i += blockDim.x) {
    const int h = i / half, j = i % half;
    const float c = cs[2 * (p * half + j)], s = cs[2 * (p * half + j) + 1];
    const float a = to_f32(row[h * dh + j]), b = to_f32(row[h * dh + j + half]);
    row[h * dh + j] = from_f32<T>(a * c + b * s);
    row[h * dh + j + half] = from_f32<T>(b * c - a * s);
  }
}

// ------------------------------------------------------------------------------------------------
// Attention backward, plain fp32 version, two passes.
// Pass 1, one wave per (query row i, head h): recomputes the softmax row, stores its log-sum-exp and
// D_i = dO_i . O_i, and writes dq_i = scale * sum_j p_ij (dO_i . v_j - D_i) k_j.
// QKV / dQKV: [cells][T][(H + 2 Hkv) dh]; O, dO: [cells][T][H dh]; LSE, Dv: [cells][H][T].
// grid: (T, H, g), block: 64; LDS: (2 dh + T) floats.
template <typename T>
__global__ __launch_bounds__(64) void attention_bwd_q_kernel(const T* __restrict__ QKV, const T* __restrict__ O,
                                                             const T* __restrict__ dO, T* __restrict__ dQKV,
                                                             float* __restrict__ LSE, float* __restrict__ Dv, int first,
                                                             int Trows, int H, int Hkv, int dh, float scale) {
  extern __shared__ __align__(16) float sm[];
  float* q = sm;
  float* go = sm + dh;
  float* p = sm + 2 * dh;
  const int i = blockIdx.x, h = blockIdx.y, l = first + blockIdx.z, lane = threadIdx.x;
  const int ldq = (H + 2 * Hkv) * dh, kvh = h / (H / Hkv);
  const T* base = QKV + (size_t)l * Trows * ldq;
  const T* kbase = base + H * dh + kvh * dh;
  const T* vbase = base + (H + Hkv) * dh + kvh * dh;
  const size_t orow = ((size_t)l * Trows + i) * (H * dh) + h * dh;
  const bool quads = quads_of_columns<T>(dh);
  float dsum = 0.f;
  for (int c = lane; c < dh; c += 64) {
    q[c] = to_f32(base[(size_t)i * ldq + h * dh + c]);
    go[c] = to_f32(dO[orow + c]);
    dsum = fmaf(go[c], to_f32(O[orow + c]), dsum);
  }
  dsum = wave_sum(dsum);
  __syncthreads();
  float mx = -INFINITY;
  for (int j = lane; j <= i; j += 64) {
    const float s = row_dot(q, kbase + (size_t)j * ldq, dh, quads) * scale;
    p[j] = s;
    mx = fmaxf(mx, s);
  }
  mx = wave_max(mx);
  float sum = 0.f;
  for (int j = lane; j <= i; j += 64) sum += expf(p[j] - mx);
  sum = wave_sum(sum);
  const float lse = mx + logf(sum);
  for (int j = lane; j <= i; j += 64) {
    const float dp = row_dot(go, vbase + (size_t)j * ldq, dh, quads);
    p[j] = expf(p[j] - lse) * (dp - dsum) * scale;      // dS_ij
  }
  __syncthreads();
  if (quads) {
    f32x4 a = {0.f, 0.f, 0.f, 0.f};
    add_rows(a, p, (const float*)kbase, ldq, i + 1, dh, lane);
    if (4 * lane < dh) *(f32x4*)((float*)dQKV + ((size_t)l * Trows + i) * ldq + h * dh + 4 * lane) = a;
  } else
  for (int c = lane; c < dh; c += 64) {
    float a = 0.f;
    for (int j = 0; j <= i; ++j) a = fmaf(p[j], to_f32(kbase[(size_t)j * ldq + c]), a);
    dQKV[((size_t)l * Trows + i) * ldq + h * dh + c] = from_f32<T>(a);
  }
  if (lane == 0) {
    LSE[((size_t)l * H + h) * Trows + i] = lse;
    Dv[((size_t)l * H + h) * Trows + i] = dsum;
  }
}

// Pass 2, one wave per (key row j, KV head): dk_j = scale * sum_{h in group} sum_{i >= j} p_ij (dO_i . v_j - D_i) q_i,
// dv_j = sum p_ij dO_i, with p_ij = exp(scale q_i . k_j - LSE_i).  Query rows are taken 64 at a time: every lane
// computes p and dS for one i, then the lanes turn to the head-dimension columns and add the 64 contributions.
// grid: (T, Hkv, g), block: 64; LDS: (2 dh + 128) floats.
template <typename T>
__global__ __launch_bounds__(64) void attention_bwd_kv_kernel(const T* __restrict__ QKV, const T* __restrict__ dO,
                                                              T* __restrict__ dQKV, const float* __restrict__ LSE,
                                                              const float* __restrict__ Dv, int first, int Trows, int H,
                                                              int Hkv, int dh, float scale) {
  extern __shared__ __align__(16) float sm[];
  float* kj = sm;
  float* vj = sm + dh;
  float* pp = sm + 2 * dh;       // p_ij of the current 64 query rows
  float* ds = pp + 64;           // dS_ij
  const int j = blockIdx.x, kvh = blockIdx.y, l = first + blockIdx.z, lane = threadIdx.x;
  const int ldq = (H + 2 * Hkv) * dh, rep = H / Hkv;
  const T* base = QKV + (size_t)l * Trows * ldq;
  for (int c = lane; c < dh; c += 64) {
    kj[c] = to_f32(base[(size_t)j * ldq + (H + kvh) * dh + c]);
    vj[c] = to_f32(base[(size_t)j * ldq + (H + Hkv + kvh) * dh + c]);
  }
  __syncthreads();
  const bool quads = quads_of_columns<T>(dh);
  f32x4 dk4 = {0.f, 0.f, 0.f, 0.f}, dv4 = dk4;
  float dk[2] = {0.f, 0.f}, dv[2] = {0.f, 0.f};          // columns lane and lane + 64 (dh <= 128)
  for (int h = kvh * rep; h < (kvh + 1) * rep; ++h) {
    const float* lse = LSE + ((size_t)l * H + h) * Trows;
    const float* dvec = Dv + ((size_t)l * H + h) * Trows;
    for (int i0 = j; i0 < Trows; i0 += 64) {
      const int i = i0 + lane;
      float pv = 0.f, dsv = 0.f;
      if (i < Trows) {
        const T* qr = base + (size_t)i * ldq + h * dh;
        const T* gr = dO + ((size_t)l * Trows + i) * (H * dh) + h * dh;
        const float s = row_dot(kj, qr, dh, quads), dp = row_dot(vj, gr, dh, quads);
        pv = expf(s * scale - lse[i]);
        dsv = pv * (dp - dvec[i]) * scale;
      }
      __syncthreads();
      pp[lane] = pv;
      ds[lane] = dsv;
      __syncthreads();
      const int n = min(64, Trows - i0);
      if (quads) {
        add_rows(dk4, ds, (const float*)base + (size_t)i0 * ldq + h * dh, ldq, n, dh, lane, false);
        add_rows(dv4, pp, (const float*)dO + ((size_t)l * Trows + i0) * (H * dh) + h * dh, H * dh, n, dh, lane, false);
        continue;
      }
      for (int t = 0; t < n; ++t) {
        const T* qr = base + (size_t)(i0 + t) * ldq + h * dh;
        const T* gr = dO + ((size_t)l * Trows + i0 + t) * (H * dh) + h * dh;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int c = lane + 64 * e;
          if (c < dh) {
            dk[e] = fmaf(ds[t], to_f32(qr[c]), dk[e]);
            dv[e] = fmaf(pp[t], to_f32(gr[c]), dv[e]);
          }
        }
      }
    }
  }
  if (quads) {
    add_groups(dk4, dh);
    add_groups(dv4, dh);
    if (4 * lane < dh) {
      float* out = (float*)dQKV + ((size_t)l * Trows + j) * ldq + 4 * lane;
      *(f32x4*)(out + (H + kvh) * dh) = dk4;
      *(f32x4*)(out + (H + Hkv + kvh) * dh) = dv4;
    }
    return;
  }
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int c = lane + 64 * e;
    if (c < dh) {
      dQKV[((size_t)l * Trows + j) * ldq + (H + kvh) * dh + c] = from_f32<T>(dk[e]);
      dQKV[((size_t)l * Trows + j) * ldq + (H + Hkv + kvh) * dh + c] = from_f32<T>(dv[e]);
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Backward of the DPFP feature map for one vector: k[dm] (LDS), df[Phi] (LDS) -> dk[c] for c = threadIdx.x ...
// r = [relu(k), relu(-k)], phi[(j-1) n + i] = r[i] r[(i - j) mod n]: r[i] appears as the first factor of entry
// (j, i) and as the second factor of entry (j, (i + j) mod n).
__device__ __forceinline__ float dpfp_dr(const float* k, const float* df, int dm, int nu, int i) {
  const int n = 2 * dm;
  float s = 0.f;
  for (int j = 1; j <= nu; ++j) {
    int a = i - j; if (a < 0) a += n;
    int b = i + j; if (b >= n) b -= n;
    s = fmaf(df[(j - 1) * n + i], dpfp_r(k, dm, a), s);
    s = fmaf(df[(j - 1) * n + b], dpfp_r(k, dm, b), s);
  }
  return s;
}
__device__ __forceinline__ float dpfp_dk(const float* k, const float* df, int dm, int nu, int c) {
  if (k[c] > 0.f) return dpfp_dr(k, df, dm, nu, c);
  if (k[c] < 0.f) return -dpfp_dr(k, df, dm, nu, c + dm);
  return 0.f;
}

// Read backward, row part 1 (Eq. 6: x1 = x + num / den): from dx1 (gradient of the read's output), x1 and x,
// dnum = dx1 / den (activation type, operand of the following GEMMs) and dden = -(dnum . (x1 - x)).
// grid: (T, g), block: 256.
template <typename T>
__global__ __launch_bounds__(256) void read_bwd_rows_kernel(const float* __restrict__ dX1, size_t dx_cell,
                                                            const float* __restrict__ X1, size_t x1_cell,
                                                            const float* __restrict__ Xin, size_t xin_cell,
                                                            const float* __restrict__ RDen, int first, int Trows, int d,
                                                            T* __restrict__ DNum, float* __restrict__ DDen) {
  __shared__ float red[17];
  const int l = first + blockIdx.y, i = blockIdx.x;
  const float* g = dX1 + (size_t)l * dx_cell + (size_t)i * d;
  const float* x1 = X1 + (size_t)l * x1_cell + (size_t)i * d;
  const float* x0 = Xin + (size_t)l * xin_cell + (size_t)i * d;
  const float rden = RDen[(size_t)l * Trows + i];
  // dden is formed from the ROUNDED dnum: df = A^T dnum + dden z removes from A^T dnum its component along the
  // read direction, and the two terms only cancel as they should if both see the same dnum
  float s = 0.f;
  for (int c = threadIdx.x; c < d; c += blockDim.x) {
    const T dn = from_f32<T>(g[c] * rden);
    s = fmaf(to_f32(dn), x1[c] - x0[c], s);
    DNum[((size_t)l * Trows + i) * d + c] = dn;
  }
  s = block_sum(s, red);
  if (threadIdx.x == 0) DDen[(size_t)l * Trows + i] = -s;
}

// Read backward, row part 2: df = dnum A (from the GEMM, fp32) + dden z, pushed through the feature map:
// dq = dphi(q)^T df, written in the activation type with row stride ldq (padding columns stay zero).
// grid: (T, g), block: 128; LDS: (dm + Phi) floats.
template <typename T>
__global__ __launch_bounds__(128) void read_bwd_dpfp_kernel(const float* __restrict__ Qm, const float* __restrict__ DF,
                                                            const float* __restrict__ DDen, const LayerAux* __restrict__ aux,
                                                            int first, int Trows, int dm, int nu, T* __restrict__ DQ, int ldq) {
  extern __shared__ float sm[];
  float* k = sm;
  float* df = sm + dm;
  const int l = first + blockIdx.y, Phi = 2 * nu * dm;
  const size_t r = (size_t)l * Trows + blockIdx.x;
  const float* z = aux[l].z;
  const float dden = DDen[r];
  for (int c = threadIdx.x; c < dm; c += blockDim.x) k[c] = Qm[r * dm + c];
  for (int c = threadIdx.x; c < Phi; c += blockDim.x) df[c] = fmaf(dden, z[c], DF[r * Phi + c]);
  __syncthreads();
  for (int c = threadIdx.x; c < dm; c += blockDim.x) DQ[r * ldq + c] = from_f32<T>(dpfp_dk(k, df, dm, nu, c));
}

// ------------------------------------------------------------------------------------------------
// Backward of the delta rule (Eq. 3-5), part 1: everything that is local to a row r of A.
// With G = dA' (gradient of the updated matrix), P_i[r] = G[r,:] . f_i, v_bar_i[r] = A[r,:] . f_i / den_i:
//   dv_i[r]      = beta_i P_i[r]                                   -> DV [cells][m][d]
//   w_i[r]       = -beta_i P_i[r] / den_i    (gradient of v_bar_i[r], divided by den_i)
//   G[r,:]      += sum_i w_i[r] f_i          (in place: becomes the gradient of the OLD matrix)
//   partial sums over the block's rows:  dbeta_i += (v_i[r] - v_bar_i[r]) P_i[r],
//        dden_i += beta_i v_bar_i[r] P_i[r] / den_i,   df_i[:] += beta_i (v_i[r] - v_bar_i[r]) G_old[r,:] + w_i[r] A[r,:]
// Part[cells][blocks][m][Phi + 2] holds the partial df_i, dbeta_i, dden_i of every block.
// Coef as written by memupd_prep_kernel ({beta, gamma, 1/den (0 = memory empty), z.f}).
// The memory tokens are taken in chunks of UB_M (their partial feature gradients live in registers); a wave re-reads
// its rows of A and G for every chunk, carries the running update of G between chunks in Upd and writes G with the last.
// The 16 dot products with either row are reduced by one transposing butterfly each (dr_sum16; 32 full wave reductions one after
// another were what bounded this kernel), after which a lane holds everything about one token and the two factors
// of the outer products are broadcast through scalar registers; the next row is requested before the current one is worked on.
// grid: (ceil(d / rows_per_block), g), block: 256; Phi <= 64 * NPL; LDS: UB_M * (64 NPL + Phi + 2) floats.
constexpr int UB_M = 16;
// rows per block: a wave takes a quarter of them one after another, so narrow models, whose launches are few blocks, take fewer.  A CU holds
// one block (256 registers and more at Phi = 384), so more than 256 blocks are a second round.  us for 8 / 32 rows, this kernel and
// update_bwd_tokens_kernel, which adds the blocks' parts: d 128: 42 / 54 (44 / 55 for 16 cells); d 256: 44 / 57, 76 / 58 from 12 cells
// on; d 512: 47 / 54 for one cell, 80 / 55 for 8; d 2048: 68 / 61 and 283 / 105
inline int update_bwd_rows_per_block(int d) { return d >= 512 ? 32 : 8; }
template <int NPL>
__global__ __launch_bounds__(256) void update_bwd_rows_kernel(const float* __restrict__ KV, const float* __restrict__ Fm,
                                                              const float* __restrict__ Coef,
                                                              const float* __restrict__ Aold, float* __restrict__ DA,
                                                              float* __restrict__ Upd, float* __restrict__ DV,
                                                              float* __restrict__ Part, int first, int m, int d, int dm, int Phi,
                                                              int rows_per_block) {
  extern __shared__ float sm[];
  constexpr int LF = 64 * NPL;
  float* F = sm;                               // [UB_M][LF]: the f_i of the current chunk of memory tokens, zeros behind
  float* acc = sm + UB_M * LF;                 // [UB_M][Phi + 2]
  const int l = first + blockIdx.y, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const float* Fl = Fm + (size_t)l * m * Phi;
  const float* cf = Coef + (size_t)l * m * 4;
  const float* A = Aold + (size_t)l * d * Phi;
  float* G = DA + (size_t)l * d * Phi;
  float* U = Upd + (size_t)l * d * Phi;        // sum_i w_i[r] f_i over the chunks so far (used only if m > UB_M)
  const float* V = KV + (size_t)l * m * (dm + d) + dm;
  const int r0 = blockIdx.x * rows_per_block, r1 = min(d, r0 + rows_per_block);
  const int stride = Phi + 2;
  float* out = Part + ((size_t)l * gridDim.x + blockIdx.x) * m * stride;

  for (int i0 = 0; i0 < m; i0 += UB_M) {       // memory tokens in chunks of UB_M; every chunk needs the ORIGINAL G
    const int n = min(UB_M, m - i0);
    __syncthreads();                           // the previous chunk's F and acc are no longer read
    for (int c = threadIdx.x; c < UB_M * LF; c += blockDim.x) {
      const int i = c / LF, x = c % LF;
      F[c] = i < n && x < Phi ? Fl[(size_t)(i0 + i) * Phi + x] : 0.f;
    }
    __syncthreads();
    const int mi = (lane >> 2) & 15, it = i0 + min(mi, n - 1);     // the token this lane ends up with
    const bool token = mi < n;
    const float beta = token ? cf[it * 4 + 0] : 0.f, rden = token ? cf[it * 4 + 2] : 0.f;
    const float* Vi = V + (size_t)it * (dm + d);
    float dfp[UB_M][NPL], db = 0.f, dd = 0.f;
#pragma unroll
    for (int i = 0; i < UB_M; ++i)
#pragma unroll
      for (int k = 0; k < NPL; ++k) dfp[i][k] = 0.f;
    float an[NPL], gn[NPL], vn = 0.f;
    auto request = [&](int r) {
#pragma unroll
      for (int k = 0; k < NPL; ++k) {
        const int c = lane + 64 * k;
        an[k] = c < Phi ? A[(size_t)r * Phi + c] : 0.f;
        gn[k] = c < Phi ? G[(size_t)r * Phi + c] : 0.f;
      }
      vn = Vi[r];
    };
    if (r0 + w < r1) request(r0 + w);
    for (int r = r0 + w; r < r1; r += 4) {
      float a[NPL], g[NPL], upd[NPL];
      const float v = vn;
#pragma unroll
      for (int k = 0; k < NPL; ++k) {
        const int c = lane + 64 * k;
        a[k] = an[k];
        g[k] = gn[k];
        upd[k] = (i0 > 0 && c < Phi) ? U[(size_t)r * Phi + c] : 0.f;
      }
      if (r + 4 < r1) request(r + 4);
      float p[UB_M], pq[UB_M];
#pragma unroll
      for (int i = 0; i < UB_M; ++i) {
        p[i] = pq[i] = 0.f;
#pragma unroll
        for (int k = 0; k < NPL; ++k) {
          const float f = F[i * LF + lane + 64 * k];
          p[i] = fmaf(a[k], f, p[i]);
          pq[i] = fmaf(g[k], f, pq[i]);
        }
      }
      const float pa = dr_sum16(p, lane), pg = dr_sum16(pq, lane);
      const float vbar = pa * rden, e = v - vbar;
      const float wi = token ? -beta * pg * rden : 0.f, be = token ? beta * e : 0.f;
      if (token && (lane & 3) == 0) DV[((size_t)l * m + it) * d + r] = beta * pg;
      db = fmaf(e, pg, db);
      dd = fmaf(beta * vbar * rden, pg, dd);
#pragma unroll
      for (int i = 0; i < UB_M; ++i) {
        const float bi = dr_lane(be, 4 * i), wl = dr_lane(wi, 4 * i);
#pragma unroll
        for (int k = 0; k < NPL; ++k) {
          dfp[i][k] = fmaf(bi, g[k], fmaf(wl, a[k], dfp[i][k]));
          upd[k] = fmaf(wl, F[i * LF + lane + 64 * k], upd[k]);
        }
      }
      const bool last = i0 + UB_M >= m;
#pragma unroll
      for (int k = 0; k < NPL; ++k) {
        const int c = lane + 64 * k;
        if (c < Phi) {
          if (last) G[(size_t)r * Phi + c] = g[k] + upd[k];      // rows are private to a wave: nobody reads this G again
          else U[(size_t)r * Phi + c] = upd[k];
        }
      }
    }
    // the four waves' partial sums -> one partial per block (the waves add into one LDS image in turn)
    for (int ww = 0; ww < 4; ++ww) {
      if (w == ww) {
#pragma unroll
        for (int i = 0; i < UB_M; ++i) {
          if (i >= n) continue;
#pragma unroll
          for (int k = 0; k < NPL; ++k) {
            const int c = lane + 64 * k;
            if (c < Phi) acc[(size_t)i * stride + c] = (ww ? acc[(size_t)i * stride + c] : 0.f) + dfp[i][k];
          }
        }
        if (token && (lane & 3) == 0) {
          acc[(size_t)mi * stride + Phi] = (ww ? acc[(size_t)mi * stride + Phi] : 0.f) + db;
          acc[(size_t)mi * stride + Phi + 1] = (ww ? acc[(size_t)mi * stride + Phi + 1] : 0.f) + dd;
        }
      }
      __syncthreads();
    }
    for (int c = threadIdx.x; c < n * stride; c += blockDim.x) out[(size_t)i0 * stride + c] = acc[c];
  }
}

// Part 2, one block per memory token i: sums the partials, adds the terms that come through z and gamma, pushes
// df_i through the feature map and writes the operands of the projection gradients:
//   dgamma_i = dz' . f_i,  dzf_i = dden_i - dgamma_i / (|f_i|^2 + eps),  dn_i = dgamma_i zf_i / (|f_i|^2 + eps)^2
//   df_i = partial + gamma_i dz' + 2 dn_i f_i + dzf_i z
//   DKV[i] = [dk_i | dv_i] (activation type, row stride ldkv, padding stays zero), DB[i] = dbeta_i beta_i (1 - beta_i),
//   DZF[i] = dzf_i (for update_bwd_z_kernel).
// grid: (m, g), block: 128; LDS: (dm + Phi + 17) floats.
template <typename T>
__global__ __launch_bounds__(128) void update_bwd_tokens_kernel(const float* __restrict__ KV, const float* __restrict__ Fm,
                                                                const float* __restrict__ Coef, const float* __restrict__ Part,
                                                                int nblocks, const float* __restrict__ DV,
                                                                const float* __restrict__ Zold, const float* __restrict__ DZ,
                                                                int first, int m, int d, int dm, int nu, float eps,
                                                                T* __restrict__ DKV, int ldkv, float* __restrict__ DB,
                                                                float* __restrict__ DZF) {
  extern __shared__ float sm[];
  float* k = sm;
  float* df = sm + dm;
  float* red = df + 2 * nu * dm;
  const int l = first + blockIdx.y, i = blockIdx.x, Phi = 2 * nu * dm, stride = Phi + 2;
  const size_t mi = (size_t)l * m + i;
  const float* f = Fm + mi * Phi;
  const float* z = Zold + (size_t)l * Phi;
  const float* dz = DZ + (size_t)l * Phi;
  const float* part = Part + (size_t)l * nblocks * m * stride + (size_t)i * stride;
  for (int c = threadIdx.x; c < dm; c += blockDim.x) k[c] = KV[mi * (dm + d) + c];
  float dg = 0.f, ff = 0.f;
  for (int c = threadIdx.x; c < Phi; c += blockDim.x) {
    float s = 0.f;
#pragma unroll 16
    for (int b = 0; b < nblocks; ++b) s += part[(size_t)b * m * stride + c];
    df[c] = s;
    dg = fmaf(dz[c], f[c], dg);
    ff = fmaf(f[c], f[c], ff);
  }
  dg = block_sum(dg, red);
  ff = block_sum(ff, red);
  // (read by all threads, added in block order by one: a chain of additions, not of memory latencies)
  __shared__ float pb[2][128];
  float dbeta = 0.f, dden = 0.f;
  for (int b0 = 0; b0 < nblocks; b0 += 128) {
    const int nb = min(128, nblocks - b0);
    __syncthreads();
    if ((int)threadIdx.x < nb) {
      pb[0][threadIdx.x] = part[(size_t)(b0 + threadIdx.x) * m * stride + Phi];
      pb[1][threadIdx.x] = part[(size_t)(b0 + threadIdx.x) * m * stride + Phi + 1];
    }
    __syncthreads();
    if (threadIdx.x == 0)
      for (int b = 0; b < nb; ++b) { dbeta += pb[0][b]; dden += pb[1][b]; }
  }
  const float beta = Coef[mi * 4 + 0], gamma = Coef[mi * 4 + 1], zf = Coef[mi * 4 + 3];
  const float inv = 1.0f / (ff + eps);
  __shared__ float dzf_s;
  if (threadIdx.x == 0) {
    dzf_s = dden - dg * inv;
    DZF[mi] = dzf_s;
    DB[mi] = dbeta * beta * (1.f - beta);
  }
  __syncthreads();
  const float dzf = dzf_s, dn = dg * zf * inv * inv;
  for (int c = threadIdx.x; c < Phi; c += blockDim.x) df[c] += gamma * dz[c] + 2.f * dn * f[c] + dzf * z[c];
  __syncthreads();
  for (int c = threadIdx.x; c < dm; c += blockDim.x) DKV[mi * ldkv + c] = from_f32<T>(dpfp_dk(k, df, dm, nu, c));
  for (int c = threadIdx.x; c < d; c += blockDim.x) DKV[mi * ldkv + dm + c] = from_f32<T>(DV[mi * d + c]);
}

// Part 3: dz (in place: gradient of the OLD z) += sum_i dzf_i f_i.  grid: (ceil(Phi / 256), g), block: 256.
__global__ __launch_bounds__(256) void update_bwd_z_kernel(const float* __restrict__ Fm, const float* __restrict__ DZF,
                                                           float* __restrict__ DZ, int first, int m, int Phi) {
  const int l = first + blockIdx.y, c = blockIdx.x * 256 + threadIdx.x;
  if (c >= Phi) return;
  float s = 0.f;
  for (int i = 0; i < m; ++i) s = fmaf(DZF[(size_t)l * m + i], Fm[((size_t)l * m + i) * Phi + c], s);
  DZ[(size_t)l * Phi + c] += s;
}

// beta_i = sigmoid(w_b . y_i): the memory rows of the output gradient get db_i w_b, and part[cell] = sum_i db_i y_i.
// dY: gradient slots (row 0 of the memory rows of cell l at dY + l * dy_cell); Ym: [cells][m][d] memory rows of the output.
// grid: (ceil(d / 256), g), block: 256.
template <typename T>
__global__ __launch_bounds__(256) void beta_bwd_kernel(const float* __restrict__ DB, const T* __restrict__ Ym, size_t ym_cell,
                                                       const LayerAux* __restrict__ aux, float* __restrict__ dY,
                                                       size_t dy_cell, float* __restrict__ part, int first, int m, int d) {
  const int l = first + blockIdx.y, c = blockIdx.x * 256 + threadIdx.x;
  if (c >= d) return;
  const float wb = to_f32(((const T*)aux[l].wm_b)[c]);
  float s = 0.f;
  for (int i = 0; i < m; ++i) {
    const float db = DB[(size_t)l * m + i];
    dY[(size_t)l * dy_cell + (size_t)i * d + c] += db * wb;
    s = fmaf(db, to_f32(Ym[(size_t)l * ym_cell + (size_t)i * d + c]), s);
  }
  part[(size_t)l * d + c] = s;       // per cell; colsum_finish_kernel adds the cells of a layer into dw_b
}

// ------------------------------------------------------------------------------------------------
// Tape of the training forward: inputs of a cell that the backward pass cannot recompute from its neighbours.
// Per cell (segment s, layer l, sequence b), record index s * n_cells + l * batch + b: the cell input [T][d] fp32, the layer's A [d][Phi] and
// z [Phi] from BEFORE the cell's update.  Cell l of a launch belongs to layer l / batch and to segment t - l / batch.
// Saving and restoring are copies and nothing else, bound by memory if enough of it is asked for: 16 bytes at a time, four of them in flight
// per thread (1B shape, mean of 5.6 cells: save 57 -> 24 us).
__device__ __forceinline__ float* tape_record(float* tape, size_t rec_floats, int t, int l, int n_cells, int batch) {
  return tape + ((size_t)(t - l / batch) * n_cells + l) * rec_floats;
}
// put(i, v, n): v holds n = 4 or 1 floats from src + i on.
template <typename Put>
__device__ __forceinline__ void tape_span(const float* __restrict__ src, size_t n, bool quads, Put put) {
  const size_t step = (size_t)gridDim.x * blockDim.x, at = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (quads) {
    const size_t nq = n >> 2;
    size_t i = at;
    for (; i + 3 * step < nq; i += 4 * step) {
      f32x4 v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = *(const f32x4*)(src + 4 * (i + k * step));
#pragma unroll
      for (int k = 0; k < 4; ++k) put(4 * (i + k * step), v[k], 4);
    }
    for (; i < nq; i += step) put(4 * i, *(const f32x4*)(src + 4 * i), 4);
  } else {
    for (size_t i = at; i < n; i += step) put(i, f32x4{src[i], 0.f, 0.f, 0.f}, 1);
  }
}
__device__ __forceinline__ void tape_put(float* dst, size_t i, f32x4 v, int n) {
  if (n == 4) *(f32x4*)(dst + i) = v; else dst[i] = v[0];
}
__device__ __forceinline__ void tape_put(bf16* dst, size_t i, f32x4 v, int n) {
  if (n == 4) *(bf16x4*)(dst + i) = bf16x4{(bf16)v[0], (bf16)v[1], (bf16)v[2], (bf16)v[3]}; else dst[i] = (bf16)v[0];
}

// Slots and memory state -> tape.  The state is the caller's and may start anywhere.  grid: (blocks, g), block: 256.
__global__ __launch_bounds__(256) void tape_save_kernel(float* __restrict__ tape, size_t rec_floats, const float* __restrict__ X,
                                                        const LayerAux* __restrict__ aux, int first, int t, int n_cells, int batch,
                                                        size_t nx, size_t nA, size_t nz) {
  const int l = first + blockIdx.y;
  float* rec = tape_record(tape, rec_floats, t, l, n_cells, batch);
  const float *A = aux[l].A, *z = aux[l].z;
  const bool x4 = (nx & 3) == 0;           // slots and records then start on 16 bytes
  tape_span(X + (size_t)l * nx, nx, x4, [&](size_t i, f32x4 v, int n) { tape_put(rec, i, v, n); });
  tape_span(A, nA, x4 && (nA & 3) == 0 && ((uintptr_t)A & 15) == 0, [&](size_t i, f32x4 v, int n) { tape_put(rec + nx, i, v, n); });
  tape_span(z, nz, false, [&](size_t i, f32x4 v, int n) { tape_put(rec + nx + nA, i, v, n); });
}

// Tape -> what the recomputation of a cell starts from, in one pass: the input in fp32 (Xin) and as the GEMM operand (Xop; T = float: Xin
// itself), A likewise, z; for the cells from `no_read` on, which have no read in front of the block, also X1 (elsewhere the read writes it).
// 1B shape, mean of 5.6 cells: 31 us; a restoring copy, a copy and two conversions took 57 + 21 + 28.
// grid: (blocks, g), block: 256.
template <typename T>
__global__ __launch_bounds__(256) void tape_restore_kernel(float* __restrict__ tape, size_t rec_floats, float* __restrict__ Xin,
                                                           T* __restrict__ Xop, float* __restrict__ X1, float* __restrict__ Aw,
                                                           T* __restrict__ Aop, float* __restrict__ zw, int first, int t, int n_cells,
                                                           int batch, int no_read, size_t nx, size_t nA, size_t nz) {
  constexpr bool OPERANDS = sizeof(T) != 4;      // T = float: the fp32 copies are the operands
  const int l = first + blockIdx.y;
  const float* rec = tape_record(tape, rec_floats, t, l, n_cells, batch);
  const size_t x = (size_t)l * nx, a = (size_t)l * nA;
  const bool x4 = (nx & 3) == 0, has_x1 = l >= no_read;
  tape_span(rec, nx, x4, [&](size_t i, f32x4 v, int n) {
    tape_put(Xin + x, i, v, n);
    if (OPERANDS) tape_put(Xop + x, i, v, n);
    if (has_x1) tape_put(X1 + x, i, v, n);
  });
  tape_span(rec + nx, nA, x4 && (nA & 3) == 0, [&](size_t i, f32x4 v, int n) {
    tape_put(Aw + a, i, v, n);
    if (OPERANDS) tape_put(Aop + a, i, v, n);
  });
  tape_span(rec + nx + nA, nz, false, [&](size_t i, f32x4 v, int n) { tape_put(zw + (size_t)l * nz, i, v, n); });
}

// Memory-state gradients between the caller's order [batch][layers][n] and the cell order [layers][batch][n] of a step.
// to_cells = 1: cells <- caller; 0: caller <- cells.  grid: (blocks, layers * batch), block: 256.
__global__ __launch_bounds__(256) void state_permute_kernel(float* __restrict__ dst, const float* __restrict__ src, int n_layers,
                                                            int batch, size_t n, int to_cells) {
  const int v = blockIdx.y, l = v / batch, b = v % batch;
  const size_t cell = (size_t)v * n, user = ((size_t)b * n_layers + l) * n;
  float* d = dst + (to_cells ? cell : user);
  const float* s = src + (to_cells ? user : cell);
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) d[i] = s[i];
}

// Gradient of the top layer's output: token rows from the caller's d_hidden, memory rows zero.
template <typename T>
__global__ __launch_bounds__(256) void load_dhidden_kernel(const T* __restrict__ dh, int S, int d, float* __restrict__ slot) {
  const int r = blockIdx.x;
  for (int c = threadIdx.x; c < d; c += blockDim.x) slot[(size_t)r * d + c] = r < S ? to_f32(dh[(size_t)r * d + c]) : 0.f;
}

// Gradient of a layer-0 cell's input: token rows -> dx of the segment (if asked for), memory rows += d_mem_emb.
__global__ __launch_bounds__(256) void store_dx_kernel(const float* __restrict__ slot, int S, int d, float* __restrict__ dx,
                                                       float* __restrict__ dmem) {
  const int r = blockIdx.x;
  for (int c = threadIdx.x; c < d; c += blockDim.x) {
    const float v = slot[(size_t)r * d + c];
    if (r < S) { if (dx) dx[(size_t)r * d + c] = v; }
    else dmem[(size_t)(r - S) * d + c] += v;
  }
}

}  // namespace armt
