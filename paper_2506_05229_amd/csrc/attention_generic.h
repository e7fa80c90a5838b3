// Causal grouped-query attention over the T rows of each cell, plain fp32 version (any head_dim,
// any T).  Used by fp32 configurations; the bf16 path uses the MFMA kernel in attention_mfma.h.
#pragma once

#include "common.h"

namespace armt {

// The fp32 kernels (this one and the backward in backward_kernels.h) run one wave per row and head, so what bounds them is the chain of
// memory latencies of that wave.  Where a head is 4, 8, ... 256 columns, rows are read 16 bytes at a time: a lane takes whole rows for the dot
// products and, for weighted sums of rows, four columns of every (64 / (dh / 4))-th row.  The rows must then start on 16 bytes: the buffers of
// the workspace do, a caller's need not.
template <typename T>
__device__ __forceinline__ bool quads_of_columns(int dh) {
  return sizeof(T) == 4 && (dh & 3) == 0 && dh <= 256 && 64 % (dh >> 2) == 0;
}

// x (LDS, 16-byte aligned) . row, dh columns
template <typename T>
__device__ __forceinline__ float row_dot(const float* x, const T* row, int dh, bool quads) {
  float s = 0.f;
  if (quads) {
#pragma unroll 8
    for (int c = 0; c < dh; c += 4) {
      const f32x4 a = *(const f32x4*)(x + c), b = *(const f32x4*)((const float*)row + c);
#pragma unroll
      for (int e = 0; e < 4; ++e) s = fmaf(a[e], b[e], s);
    }
  } else {
    for (int c = 0; c < dh; ++c) s = fmaf(x[c], to_f32(row[c]), s);
  }
  return s;
}

// Sum over the groups of dh / 4 lanes; every group gets it.
__device__ __forceinline__ void add_groups(f32x4& a, int dh) {
  for (int off = dh >> 2; off < 64; off <<= 1)
#pragma unroll
    for (int e = 0; e < 4; ++e) a[e] += __shfl_xor(a[e], off, kWave);
}

// a += sum_t w[t] rows[t][4 c .. 4 c + 3], c = lane mod dh / 4; of rows t = lane / (dh / 4), ... only, unless `all`.
__device__ __forceinline__ void add_rows(f32x4& a, const float* w, const float* rows, int ld, int n, int dh, int lane, bool all = true) {
  const int per = dh >> 2, c = lane % per * 4, step = 64 / per;
#pragma unroll 4
  for (int t = lane / per; t < n; t += step) {
    const f32x4 v = *(const f32x4*)(rows + (size_t)t * ld + c);
    const float f = w[t];
#pragma unroll
    for (int e = 0; e < 4; ++e) a[e] = fmaf(f, v[e], a[e]);
  }
  if (all) add_groups(a, dh);
}

// QKV: [L][T][(H + 2 Hkv) dh], rows laid out [q heads | k heads | v heads], q and k already rotated.
// Out: [L][T][H dh].  aligned: both start on 16 bytes.  grid: (T, H, g), block: 64 (one wave per query row and head).
template <typename T>
__global__ __launch_bounds__(64) void attention_generic_kernel(const T* __restrict__ QKV, T* __restrict__ Out,
                                                               int first, int Trows, int H, int Hkv, int dh,
                                                               float scale, bool aligned) {
  extern __shared__ __align__(16) float sm[];      // q: dh floats, p: Trows floats
  float* q = sm;
  float* p = sm + dh;
  const int i = blockIdx.x, h = blockIdx.y, l = first + blockIdx.z, lane = threadIdx.x;
  const int ldq = (H + 2 * Hkv) * dh, kvh = h / (H / Hkv);
  const T* base = QKV + (size_t)l * Trows * ldq;
  const T* kbase = base + H * dh + kvh * dh;
  const T* vbase = base + (H + Hkv) * dh + kvh * dh;
  for (int c = lane; c < dh; c += 64) q[c] = to_f32(base[(size_t)i * ldq + h * dh + c]);
  __syncthreads();
  const bool quads = aligned && quads_of_columns<T>(dh);
  float mx = -INFINITY;
  for (int j = lane; j <= i; j += 64) {
    const float s = row_dot(q, kbase + (size_t)j * ldq, dh, quads) * scale;
    p[j] = s;
    mx = fmaxf(mx, s);
  }
  mx = wave_max(mx);
  float sum = 0.f;
  for (int j = lane; j <= i; j += 64) {
    const float e = expf(p[j] - mx);
    p[j] = e;
    sum += e;
  }
  sum = wave_sum(sum);
  __syncthreads();
  const float inv = 1.0f / sum;
  if (quads) {
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
    add_rows(o, p, (const float*)vbase, ldq, i + 1, dh, lane);
    if (4 * lane < dh) *(f32x4*)((float*)Out + ((size_t)l * Trows + i) * (H * dh) + h * dh + 4 * lane) = o * inv;
    return;
  }
  for (int c = lane; c < dh; c += 64) {
    float o = 0.f;
    for (int j = 0; j <= i; ++j) o = fmaf(p[j], to_f32(vbase[(size_t)j * ldq + c]), o);
    Out[((size_t)l * Trows + i) * (H * dh) + h * dh + c] = from_f32<T>(o * inv);
  }
}

}  // namespace armt
