// Grouped GEMM of the fp32 configurations on the matrix cores: v_mfma_f32_16x16x4_f32 multiplies and adds in fp32.
//
// These problems are small (a cell of the fp32 configuration is 72 x 128 ... 512 with K = 128 ... 512) and what bounds a launch is one
// chain of memory latencies, not arithmetic: with 64 x 64 tiles staged through LDS in k-steps of 16 the down projection (K = 512)
// went through 32 of them.  Here a workgroup owns a 32 x 32 tile (16 x 32 for at most 16 rows), its four waves a quarter of K each,
// and a wave loads its operands straight into registers, CH chunks of 16 k ahead: a lane holds four consecutive k of one row, and
// the i-th of four MFMAs takes element i of either operand (the products of a chunk are summed in that order on both sides).  The four
// partial tiles are added in wave order through LDS, so a result depends on K alone.
//
// Against the plain FMA kernel, us per launch: 4 x (72 x 256, K 128) 19.9 -> 13.9, 4 x (72 x 128, K 512) 61.3 -> 14.4, 4 x (512 x 128,
// K 2560) 313 -> 51, 1040 x 2048 x 2048 561 -> 226, 4096 x 4096 x 1024 1350 -> 824; error against 64 bits half as large (sums of
// a quarter of the length).  Rows that cannot be read 16 bytes at a time are read element by element, in the same order: 4 x (1000 x
// 1000, K 333) 127 -> 108 us, 4 x (4096 x 4096, K 1023) 6.56 -> 4.80 ms, 1 x (1032 x 512, K 1002) 139 -> 60.  One kernel for
// all launches: which kernel runs may not depend on the number of groups, or a cell would have other bits alone, on a diagonal and
// in a batch.
//
// What is left of a step is its chain of launches of 2 to 8 us, so the small kernels around the products are part of them (F32With):
// the norm in front of QKV and gate/up, the rotation of q and k, the feature map and denominator of the read behind W_Q, features and
// coefficients of the update behind W_K | W_V.  A step of the 4-layer configuration is 9 launches instead of 14: 8 segments of 64 in 587 us, 683 before.
#pragma once

#include "common.h"
#include "gemm_generic.h"
#include "rowwise_kernels.h"

namespace armt {

enum F32With {
  F32_PLAIN,
  F32_NORM,       // GemmShape::norm; with EPI_QKV_ROPE also the rotation of heads of 8, 16 or 32 columns, which lie inside a tile
  F32_DPFP,       // EPI_DPFP_READ, N <= 32: one tile column
  F32_UPDATE      // EPI_UPDATE_F32
};

// grid: (ceil(N / 32), ceil(M / (16 TM)), g); block: 256.
// CH: chunks of 16 k per batch of loads; a wave's share should be a batch (K <= 128: 2) or several (4; 32-row tiles with the norm: 2).
template <int TM, bool SWIGLU, int CH, F32With WITH>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const GemmGroup* __restrict__ table, int first, GemmShape s) {
  constexpr int TN = 2, NB = SWIGLU ? 2 : 1, BM = 16 * TM, BN = 16 * TN, LD = BN + 4;
  constexpr bool ROWSUM = WITH == F32_NORM || WITH == F32_UPDATE;      // a sum over each row of A: squares, or products with W_beta
  __shared__ __align__(16) float part[NB][4][BM][LD];
  __shared__ float rowsum[4][BM];
  GemmGroup g = table[first + blockIdx.z];
  if (!restrict_k<float>(g, s)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, q = lane >> 4;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  // 16-byte loads need 16-byte aligned rows and a K that ends with one; anything else is read element by element
  const float* along = (const float*)g.gain;               // ROWSUM: gain or W_beta
  const bool wide = (((uintptr_t)g.A | (uintptr_t)g.B0 | (uintptr_t)g.B1 | (uintptr_t)g.B2 | (ROWSUM ? (uintptr_t)along : 0)) & 15) == 0 &&
                    ((s.K | s.lda | s.ldb) & 3) == 0;
  const float* a[TM];
  const float* b[NB][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) a[i] = (const float*)g.A + (size_t)min(m0 + 16 * i + r16, s.M - 1) * s.lda;
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int n = min(n0 + 16 * j + r16, s.N - 1);       // rows past the edges repeat the last one; masked on store
    if (SWIGLU) {
      b[0][j] = (const float*)g.B0 + (size_t)n * s.ldb;
      b[NB - 1][j] = (const float*)g.B1 + (size_t)n * s.ldb;
    } else {
      b[0][j] = weight_row<float>(g, s, n);
    }
  }
  // this thread's four results, and what their epilogue reads: requested together with the operands
  const int row = tid >> 3, col = (tid & 7) * 4, m = m0 + row, n = n0 + col;
  const bool mine = row < BM && m < s.M && n < s.N;
  const bool wide_out = n + 3 < s.N && ((s.ldc | s.ldr | s.ldc2) & 3) == 0 &&
                        (((uintptr_t)g.C | (uintptr_t)g.C2 | (uintptr_t)g.R) & 15) == 0;
  f32x4 res = {0.f, 0.f, 0.f, 0.f};
  float rs = 1.f;
  const bool rotate = WITH == F32_NORM && !SWIGLU && s.epi == EPI_QKV_ROPE && n < s.n0 + s.n1;
  const int half = s.ldr >> 1, in_head = rotate ? n & (s.ldr - 1) : 0;      // (rotate: ldr = 8, 16 or 32)
  f32x4 cs0 = {0.f, 0.f, 0.f, 0.f}, cs1 = cs0;                               // cos and sin of this thread's four columns
  if (rotate && mine) {
    const float* cs = g.R + ((size_t)m * half + (in_head & (half - 1))) * 2;
    cs0 = *(const f32x4*)cs;
    cs1 = *(const f32x4*)(cs + 4);
  }
  if (mine) {
    if (g.rowscale) rs = g.rowscale[m];
    if (s.epi == EPI_RESID_F32 && g.R) {
      const float* r = g.R + (size_t)m * s.ldr + n;
      if (wide_out) {
        res = *(const f32x4*)r;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (n + e < s.N) res[e] = r[e];
      }
    }
  }
  // features lane, lane + 64, ...: z there, and the two factors of feature c as columns of the row and their signs (see dpfp_at)
  const int Phi = 2 * (WITH == F32_DPFP ? s.ldr : s.nu) * s.n0;
  float zv[8], sign_a[8], sign_b[8];
  int col_a[8], col_b[8];
  if (WITH == F32_DPFP || WITH == F32_UPDATE) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (64 * k >= Phi) break;
      const int c = lane + 64 * k, dm = s.n0, j = c / (2 * dm) + 1, i = c % (2 * dm), i2 = i >= j ? i - j : i - j + 2 * dm;
      zv[k] = c < Phi ? g.R[c] : 0.f;
      sign_a[k] = i < dm ? 1.f : -1.f;
      sign_b[k] = i2 < dm ? 1.f : -1.f;
      col_a[k] = c < Phi ? (i < dm ? i : i - dm) : 0;
      col_b[k] = c < Phi ? (i2 < dm ? i2 : i2 - dm) : 0;
    }
  }
  f32x4 acc[NB][TM][TN];
#pragma unroll
  for (int u = 0; u < NB; ++u)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[u][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int chunks = (s.K + 15) >> 4, per = (chunks + 3) >> 2;
  const int c0 = min(wave * per, chunks), c1 = min(c0 + per, chunks);
  struct Batch { f32x4 a[CH][TM], b[CH][NB][TN], along[ROWSUM ? CH : 1]; };
  float sum[TM] = {};
  auto multiply = [&](Batch& t, int h) __attribute__((always_inline)) {
    if (ROWSUM) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (WITH == F32_NORM) {
            sum[i] = fmaf(t.a[h][i][e], t.a[h][i][e], sum[i]);
            t.a[h][i][e] *= t.along[h][e];
          } else {
            sum[i] = fmaf(t.a[h][i][e], t.along[h][e], sum[i]);
          }
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int u = 0; u < NB; ++u)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[u][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(t.a[h][i][e], t.b[h][u][j][e], acc[u][i][j], 0, 0, 0);
  };
  if (wide) {
    // branch-free: past the row's end its last 16 bytes are read again
    auto fetch = [&](Batch& t, int c) __attribute__((always_inline)) {
#pragma unroll
      for (int h = 0; h < CH; ++h) {
        const int at = min(16 * (c + h) + 4 * q, s.K - 4);
#pragma unroll
        for (int i = 0; i < TM; ++i) t.a[h][i] = *(const f32x4*)(a[i] + at);
        if (ROWSUM) t.along[h] = *(const f32x4*)(along + at);
#pragma unroll
        for (int u = 0; u < NB; ++u)
#pragma unroll
          for (int j = 0; j < TN; ++j) t.b[h][u][j] = *(const f32x4*)(b[u][j] + at);
      }
    };
    // a batch that reaches past this wave's share of K: what lies there becomes zero in both operands (an infinity or NaN there
    // times a zero would be a NaN in the sum).  Done in front of the products, where the batch has landed anyway.
    auto trim = [&](Batch& t, int c) __attribute__((always_inline)) {
#pragma unroll
      for (int h = 0; h < CH; ++h) {
        const bool in = c + h < c1 && 16 * (c + h) + 4 * q < s.K;
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < TM; ++i) t.a[h][i] = in ? t.a[h][i] : zero;
        if (ROWSUM) t.along[h] = in ? t.along[h] : zero;
#pragma unroll
        for (int u = 0; u < NB; ++u)
#pragma unroll
          for (int j = 0; j < TN; ++j) t.b[h][u][j] = in ? t.b[h][u][j] : zero;
      }
    };
    const int whole = min(16 * c1, s.K);
    Batch t, next;
    fetch(t, c0);
#pragma unroll 1
    for (int c = c0; c < c1; c += CH) {
      const bool more = c + CH < c1;
      if (more) fetch(next, c + CH);
      if (16 * (c + CH) > whole) trim(t, c);
#pragma unroll
      for (int h = 0; h < CH; ++h) multiply(t, h);
      if (more) t = next;
    }
  } else {
#pragma unroll 1
    for (int c = c0; c < c1; ++c) {
      Batch t;
      auto load = [&](const float* row) __attribute__((always_inline)) {
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (16 * c + 4 * q + e < s.K) v[e] = row[16 * c + 4 * q + e];
        return v;
      };
#pragma unroll
      for (int i = 0; i < TM; ++i) t.a[0][i] = load(a[i]);
      if (ROWSUM) t.along[0] = load(along);
#pragma unroll
      for (int u = 0; u < NB; ++u)
#pragma unroll
        for (int j = 0; j < TN; ++j) t.b[0][u][j] = load(b[u][j]);
      multiply(t, 0);
    }
  }
  // a 16 x 16 result block has lane = column lane % 16 and registers = rows 4 * (lane / 16) + r
#pragma unroll
  for (int u = 0; u < NB; ++u)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) part[u][wave][16 * i + 4 * q + r][16 * j + r16] = acc[u][i][j][r];
  if (ROWSUM) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      sum[i] += __shfl_xor(sum[i], 16, kWave);
      sum[i] += __shfl_xor(sum[i], 32, kWave);
      if (q == 0) rowsum[wave][16 * i + r16] = sum[i];
    }
  }
  __syncthreads();
  auto row_total = [&](int r) { return (rowsum[0][r] + rowsum[1][r]) + (rowsum[2][r] + rowsum[3][r]); };
  if (WITH == F32_DPFP || (WITH == F32_UPDATE && blockIdx.x == 0)) {
    // The N = d_mem (F32_UPDATE: n0) columns of a row lie in this tile: they go back to LDS, and a wave expands whole rows.
    float(&x)[BM][LD] = part[0][0];
    if (row < BM) {
      f32x4 v = *(const f32x4*)&x[row][col];
#pragma unroll
      for (int w = 1; w < 4; ++w) v += *(const f32x4*)&part[0][w][row][col];
      *(f32x4*)&x[row][col] = v;           // read and written by this thread only
      if (WITH == F32_UPDATE && mine) {
        float* out = (float*)g.C + (size_t)m * s.ldc + n;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (n + e < s.N) out[e] = v[e];
      }
    }
    __syncthreads();
    constexpr int ROWS = BM / 4;           // of this wave: their reductions go side by side
    float zf[ROWS], ff[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      const int r = wave + 4 * i;
      zf[i] = ff[i] = 0.f;
      float* out = (float*)(WITH == F32_DPFP ? g.C : g.C2) + (size_t)(m0 + r) * (WITH == F32_DPFP ? s.ldc : Phi);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (64 * k >= Phi) break;
        const float f = fmaxf(sign_a[k] * x[r][col_a[k]], 0.f) * fmaxf(sign_b[k] * x[r][col_b[k]], 0.f);
        if (lane + 64 * k < Phi) {
          zf[i] = fmaf(f, zv[k], zf[i]);
          ff[i] = fmaf(f, f, ff[i]);
          if (m0 + r < s.M) out[lane + 64 * k] = f;
        }
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
      for (int i = 0; i < ROWS; ++i) {
        zf[i] += __shfl_xor(zf[i], o, kWave);
        if (WITH == F32_UPDATE) ff[i] += __shfl_xor(ff[i], o, kWave);
      }
    const int l = first + blockIdx.z;
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      const int r = wave + 4 * i;
      if (lane != i || m0 + r >= s.M) continue;
      if (WITH == F32_DPFP) {
        ((float*)g.C2)[m0 + r] = 1.0f / (zf[i] + s.fparam);
      } else {
        float* cf = g.ssq_out + 4 * (m0 + r);
        cf[0] = 1.0f / (1.0f + expf(-row_total(r)));
        cf[1] = 1.0f - zf[i] / (ff[i] + s.fparam);
        cf[2] = l >= s.empty_lo && l < s.empty_hi ? 0.f : 1.0f / (zf[i] + s.fparam);
        cf[3] = zf[i];
      }
    }
    return;
  }
  if (!mine) return;
  if (WITH == F32_NORM) rs = 1.0f / sqrtf(row_total(row) / (float)s.K + s.fparam);
  auto total = [&](int u) {
    f32x4 v = *(const f32x4*)&part[u][0][row][col];
#pragma unroll
    for (int w = 1; w < 4; ++w) v += *(const f32x4*)&part[u][w][row][col];
    return v;
  };
  f32x4 v = total(0), v2;
  if (SWIGLU) {
    const f32x4 up = total(NB - 1);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float gv = v[e] * rs;
      v[e] = gv / (1.f + expf(-gv)) * (up[e] * rs);
    }
  } else if (rotate) {      // rotate-half pairing: column j of a head with j + half
    const bool low = in_head < half;
    f32x4 w = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i) w += *(const f32x4*)&part[0][i][row][low ? col + half : col - half];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float c = e < 2 ? cs0[2 * e] : cs1[2 * e - 4], sn = e < 2 ? cs0[2 * e + 1] : cs1[2 * e - 3];
      v[e] = v[e] * rs * c + (low ? -w[e] : w[e]) * rs * sn;
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = res[e] + v[e] * rs;      // res: zeros without a residual
  }
  const bool copy = s.epi == EPI_RESID_F32 && g.C2;
  if (copy) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v2[e] = g.gain ? v[e] * ((const float*)g.gain)[min(n + e, s.N - 1)] : v[e];
  }
  float* out = (float*)g.C + (size_t)m * s.ldc + n;
  float* out2 = (float*)g.C2 + (size_t)m * s.ldc2 + n;
  if (wide_out) {
    *(f32x4*)out = v;
    if (copy) *(f32x4*)out2 = v2;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (n + e >= s.N) break;
      out[e] = v[e];
      if (copy) out2[e] = v2[e];
    }
  }
}

inline hipError_t launch_gemm_f32(const GemmGroup* table, int first, int g, const GemmShape& s, hipStream_t st) {
  if (g <= 0 || s.M <= 0 || s.N <= 0) return hipSuccess;
  // The feature map is a chain of its own behind the product: the fewer rows per wave the better (4 cells of 72 rows, K 128: 32-row tiles 7.6 us
  // per launch, 16-row tiles with the reductions of a wave's rows side by side 4.9), until a long product on more 16-row tiles than CUs costs more.
  // us per launch of 4 cells, 16 / 32 rows: 1040 rows, K 512 11.3 / 13.1, 1024 18.0 / 18.6, 2048 29.9 / 25.7, 3072 41.8 / 32.7;
  // 4112 rows, K 2048 68.5 / 65.7; one cell of 1040 rows, K 2048 (65 tiles) 16.6 / 24.6.  Either tile gives the same bits.
  const bool read16 = s.epi == EPI_DPFP_READ && !(s.K > 1024 && (int64_t)g * ((s.M + 15) / 16) > 256);
  const bool narrow = s.M <= 16 || read16, brief = s.K <= 128;
  const dim3 grid((s.N + 31) / 32, (s.M + (narrow ? 15 : 31)) / (narrow ? 16 : 32), g);
#define ARMT_F32(SW)                                                                                                  \
  (narrow ? (brief ? gemm_f32_kernel<1, SW, 2, F32_PLAIN> : gemm_f32_kernel<1, SW, 4, F32_PLAIN>)                      \
          : (brief ? gemm_f32_kernel<2, SW, 2, F32_PLAIN> : gemm_f32_kernel<2, SW, 4, F32_PLAIN>))
  auto kern = ARMT_F32(false);
  if (s.epi == EPI_DPFP_READ) {
    if (s.N != s.n0 || s.N > 32 || s.ldr < 1 || 2 * s.ldr * s.n0 > 512 || s.ldc < 2 * s.ldr * s.n0) return hipErrorInvalidValue;
    kern = !narrow ? gemm_f32_kernel<2, false, 4, F32_DPFP> : brief ? gemm_f32_kernel<1, false, 2, F32_DPFP> : gemm_f32_kernel<1, false, 4, F32_DPFP>;
  } else if (s.epi == EPI_UPDATE_F32) {
    if (!narrow || s.n0 > 32 || s.nu < 1 || 2 * s.nu * s.n0 > 512) return hipErrorInvalidValue;
    kern = brief ? gemm_f32_kernel<1, false, 2, F32_UPDATE> : gemm_f32_kernel<1, false, 4, F32_UPDATE>;
  } else if (s.norm) {
    if (s.epi == EPI_QKV_ROPE && s.ldr != 8 && s.ldr != 16 && s.ldr != 32) return hipErrorInvalidValue;
    // Batches of two chunks also for a long K in 32-row tiles: with four, the gain's registers leave gate/up one wave per SIMD (280 registers; 167
    // here) and QKV two (240; 144 and three).  Same order of every sum.  us per launch, d_ff 4 d, four / two (norm in a launch of its own):
    // gate/up 4 x (1040 x 512) 359 / 211 (304), 1 x (272 x 512) 33.7 / 24.7 (31.0), 4 x (72 x 1024) 118 / 78 (128), 4 x (1040 x 2048) 4327 / 3082 (4746);
    // QKV 4 x (1040 x 512) 93.8 / 78.6 (99.7), 4 x (1040 x 2048) 1285 / 1198 (1497)
    if (s.epi == EPI_SWIGLU)
      kern = !narrow ? gemm_f32_kernel<2, true, 2, F32_NORM> : brief ? gemm_f32_kernel<1, true, 2, F32_NORM> : gemm_f32_kernel<1, true, 4, F32_NORM>;
    else
      kern = !narrow ? gemm_f32_kernel<2, false, 2, F32_NORM> : brief ? gemm_f32_kernel<1, false, 2, F32_NORM> : gemm_f32_kernel<1, false, 4, F32_NORM>;
  } else if (s.epi == EPI_SWIGLU) {
    kern = ARMT_F32(true);
  } else if (s.epi == EPI_QKV_ROPE) {
    return hipErrorInvalidValue;         // only the kernel with the norm rotates
  }
#undef ARMT_F32
  kern<<<grid, 256, 0, st>>>(table, first, s);
  return hipGetLastError();
}

}  // namespace armt
