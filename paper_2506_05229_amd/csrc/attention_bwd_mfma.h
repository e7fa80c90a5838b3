// Backward of the segment attention on the CDNA4 matrix cores (bf16, head_dim 64 or 128).
//
// With P = softmax(scale Q K^T) (causal), O = P V and upstream gradient dO:
//   D_i = dO_i . O_i,   dP = dO V^T,   dS = P (dP - D),   dQ = scale dS K,   dK = scale dS^T Q,   dV = P^T dO.
// P is recomputed from the log-sum-exp the forward kernel leaves behind (log2 domain), so no T x T matrix is stored.
// Two kernels, both built like the forward one (v_mfma_f32_32x32x16_bf16, a lane owns ONE column of every 32 x 32
// result, so the result of one product is directly the B operand of the next):
//   dq kernel:  a lane owns a query.  S^T = K Q^T and dP^T = V dO^T (keys along the rows), dS^T in registers,
//               dQ^T += K^T dS^T.  K, V and K^T tiles of a KV head are shared in LDS by the waves of its query heads.
//   dkv kernel: a lane owns a key.  S = Q K^T and dP = dO V^T (queries along the rows), P and dS in registers,
//               dV^T += dO^T P, dK^T += Q^T dS.  A wave keeps its 32 keys for the whole kernel and adds up all query
//               heads of the KV group; the waves of a workgroup share the Q, dO, Q^T, dO^T tiles of the current head in LDS.
// Operands with the sequence index contiguous (K^T, Q^T, dO^T) come from head_transpose_kernel.
#pragma once

#include "attention_mfma.h"
#include "common.h"

namespace armt {

// The three transposed operands of a cell in one launch: Xt[l][h][c][j] = X[l][j][h * dh + c], j padded with zeros to Tp, for the heads of Q and K
// (columns of QKV) and of dO.  64 x 64 tiles through LDS with 16-byte accesses on both sides, as in transpose_bf16_kernel: the pass is bound by
// memory, and 2-byte accesses in three launches took three times as long (1B shape, mean of 5.6 cells: 63 -> 19 us).
// grid: (Tp / 64, (2 H + Hkv) dh / 64, g), block: 256.
__global__ __launch_bounds__(256) void head_transpose_kernel(const bf16* __restrict__ QKV, const bf16* __restrict__ dO, bf16* __restrict__ Kt,
                                                             bf16* __restrict__ Qt, bf16* __restrict__ Gt, int first, int Trows, int Tp,
                                                             int H, int Hkv, int dh) {
  __shared__ unsigned int tile[64 * 33];
  const int l = first + blockIdx.z, j0 = blockIdx.x * 64;
  const int q_tiles = H * dh / 64, qk_tiles = q_tiles + Hkv * dh / 64;      // tiles of 64 columns: Q, K, then dO
  const int ct = blockIdx.y;
  const bool grad = ct >= qk_tiles;
  const int ldx = grad ? H * dh : (H + 2 * Hkv) * dh, c0 = (grad ? ct - qk_tiles : ct) * 64;
  const bf16* src = (grad ? dO : QKV) + (size_t)l * Trows * ldx + c0;
  // row c of a cell's Xt is its column c: heads are dh rows each
  bf16* dst = grad ? Gt + ((size_t)l * H * dh + c0) * Tp
                   : ct < q_tiles ? Qt + ((size_t)l * H * dh + c0) * Tp : Kt + ((size_t)l * Hkv * dh + c0 - H * dh) * Tp;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int idx = threadIdx.x + 256 * k, r = idx >> 3, ch = idx & 7;
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (j0 + r < Trows) v = *(const uint4*)(src + (size_t)(j0 + r) * ldx + 8 * ch);
    unsigned int* t = tile + r * 33 + 4 * ch;
    t[0] = v.x; t[1] = v.y; t[2] = v.z; t[3] = v.w;
  }
  __syncthreads();
  const unsigned short* th = (const unsigned short*)tile;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int idx = threadIdx.x + 256 * k, c = idx >> 3, rch = idx & 7;
    unsigned int w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const unsigned int lo = th[(8 * rch + 2 * e) * 66 + c], hi = th[(8 * rch + 2 * e + 1) * 66 + c];
      w[e] = lo | (hi << 16);
    }
    *(uint4*)(dst + (size_t)c * Tp + j0 + 8 * rch) = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

// D[l][h][i] = dO[l][i][h*dh : (h+1)*dh] . O[same]: 16 bytes of either per lane, DH / 8 lanes a head (1B shape, mean of 5.6 cells:
// 28.8 -> 9.8 us; one head at a time, two bytes per lane, was a chain of H reductions).
// grid: (ceil(T / 4), g), block: 256 (a wave per row, all heads).
template <int DH>
__global__ __launch_bounds__(256) void attention_dvec_kernel(const bf16* __restrict__ O, const bf16* __restrict__ dO,
                                                             float* __restrict__ Dv, int first, int Trows, int H) {
  const int l = first + blockIdx.y, i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (i >= Trows) return;
  const size_t row = ((size_t)l * Trows + i) * (H * DH);
#pragma unroll 4
  for (int c0 = 0; c0 < H * DH; c0 += 512) {
    const int c = c0 + 8 * lane, at = min(c, H * DH - 8);
    const bf16x8 a = *(const bf16x8*)(dO + row + at), b = *(const bf16x8*)(O + row + at);
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) s = fmaf((float)a[e], (float)b[e], s);
#pragma unroll
    for (int o = 1; o < DH / 8; o <<= 1) s += __shfl_xor(s, o, kWave);
    if (c < H * DH && c % DH == 0) Dv[((size_t)l * H + c / DH) * Trows + i] = s;
  }
}

// dQ.  QKV: [cells][T][(H + 2 Hkv) dh] (q, k rotated); Kt: [cells][Hkv][dh][Tp]; dO: [cells][T][H dh];
// LSE2 (log2 domain), Dv: [cells][H][T]; dQKV: gradient rows, q columns written here.
// (68 us per launch with 8-byte reads of K^T and a copy addressed per lane, 60 as it is; 1B shape, mean of 5.6 cells.)
// As in the forward kernel a workgroup takes NQ consecutive 32-row tiles (NQ > 1 when a KV head has fewer than four
// query heads): wave w handles query head kv * GROUP + w % GROUP and row tile w / GROUP.
// grid: 1-D, 8 * ceil(Hkv g / 8) * ceil(T / (32 NQ)) workgroups, block: NQ * GROUP * 64; LDS: 2 stages of K, V, K^T tiles.
template <int DH>
__global__ __launch_bounds__(512) void attention_bwd_dq_kernel(const bf16* __restrict__ QKV, const bf16* __restrict__ Kt,
                                                               const bf16* __restrict__ dO, const float* __restrict__ LSE2,
                                                               const float* __restrict__ Dv, bf16* __restrict__ dQKV,
                                                               int first, int Trows, int Tp, int H, int Hkv, int nq, float scale,
                                                               int nqt, int npairs) {
  constexpr int K_BYTES = AT_KT * DH * 2;          // K and V tiles: DH / 64 sub-tiles [64 keys][64 dims], 128-byte rows
  constexpr int T_BYTES = DH * AT_KT * 2;          // K^T tile: [DH dims][64 keys]
  constexpr int STAGE = 2 * K_BYTES + T_BYTES;
  constexpr int K_SLABS = K_BYTES / 1024, T_SLABS = T_BYTES / 1024;
  constexpr int KS = DH / 16, OT = DH / 32;
  extern __shared__ __align__(16) unsigned char smem[];   // [2][STAGE]

  // work order of the forward kernel: a (cell, KV head) pair stays on one XCD, longest row tiles first over all pairs
  const int ppx = (npairs + 7) >> 3, xj = blockIdx.x >> 3;
  const int qt = nqt - 1 - xj / ppx;
  const int pair = (xj % ppx) * 8 + (blockIdx.x & 7);
  if (pair >= npairs) return;
  const int kvh = pair % Hkv, l = first + pair / Hkv;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = blockDim.x >> 6, group = H / Hkv;
  const int head = kvh * group + wave % group;
  const int ldq = (H + 2 * Hkv) * DH;
  const int q0 = (qt * nq + wave / group) * AT_QT;   // may lie past the cell in the last workgroup
  const bool live = q0 < Trows;
  const int qcol = lane & 31, half = lane >> 5;
  const float scale_log2e = scale * 1.4426950408889634f;

  const bf16* cell = QKV + (size_t)l * Trows * ldq;
  const char* kbase = (const char*)(cell + H * DH + kvh * DH);
  const char* vbase = (const char*)(cell + (H + Hkv) * DH + kvh * DH);
  const char* tbase = (const char*)(Kt + (size_t)(l * Hkv + kvh) * DH * Tp);

  const int qrow = min(q0 + qcol, Trows - 1);
  bf16x8 qf[KS], gf[KS];       // B operands: this lane's query row of Q and of dO
  {
    const bf16* qp = cell + (size_t)qrow * ldq + head * DH + half * 8;
    const bf16* gp = dO + ((size_t)l * Trows + qrow) * (H * DH) + head * DH + half * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      qf[ks] = *(const bf16x8*)(qp + ks * 16);
      gf[ks] = *(const bf16x8*)(gp + ks * 16);
    }
  }
  const float lse = LSE2[((size_t)l * H + head) * Trows + qrow];
  const float dvec = Dv[((size_t)l * H + head) * Trows + qrow];

  // tile copies as in the forward kernel: scalar base + one lane offset per operand, the K and V rows permuted (at_key_of_row)
  const int R = lane >> 3, pc = lane & 7;
  const unsigned chunk0 = (unsigned)((pc ^ mf_swz(R)) << 4);
  const unsigned voffK = (unsigned)((R & 3) + ((R >> 2) << 3)) * (unsigned)ldq * 2u + chunk0;
  const unsigned voffT = (unsigned)R * (unsigned)Tp * 2u + chunk0;
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)smem;
  auto issue_tile = [&](int kt, int buf) {
    typedef const __attribute__((address_space(1))) void* gptr_t;
    typedef __attribute__((address_space(3))) void* lptr_t;
    unsigned char* Ks = smem + buf * STAGE;
    const unsigned lds = lds0 + buf * STAGE;
    const int k0 = kt * AT_KT;
    const bool whole = k0 + AT_KT <= Trows;            // wave-uniform: every key of the tile exists
    for (int sl = wave; sl < 2 * K_SLABS + T_SLABS; sl += nw) {
      if (sl < 2 * K_SLABS) {
        const bool isv = sl >= K_SLABS;
        const int s2 = isv ? sl - K_SLABS : sl, sub = s2 >> 3, a = s2 & 7;
        const char* base = isv ? vbase : kbase;
        if (whole) {
          const int keyS = k0 + ((a & 1) << 2) + ((a >> 1) << 4);
          lds_copy16(base + ((size_t)keyS * ldq + sub * 64) * 2, voffK ^ ((unsigned)(a & 1) << 6), lds + sl * 1024);
        } else {
          const int row = a * 8 + R, key = min(k0 + at_key_of_row(row), Trows - 1);
          const char* src = base + ((size_t)key * ldq + sub * 64 + ((pc ^ mf_swz(row)) << 3)) * 2;
          __builtin_amdgcn_global_load_lds((gptr_t)src, (lptr_t)(Ks + sl * 1024), 16, 0, 0);
        }
      } else {
        const int ts = sl - 2 * K_SLABS;
        lds_copy16(tbase + ((size_t)ts * 8 * Tp + k0) * 2, voffT ^ ((unsigned)(ts & 1) << 6), lds + sl * 1024);
      }
    }
  };

  const int fl = mf_swz(lane & 31);
  f32x16 o[OT];
#pragma unroll
  for (int t = 0; t < OT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[t][r] = 0.f;

  const int qi = q0 + qcol;
  const int nkt = (min((qt + 1) * nq * AT_QT, Trows) + AT_KT - 1) / AT_KT;   // key tiles of the workgroup's last rows
  issue_tile(0, 0);
  __builtin_amdgcn_s_waitcnt(0x0F70);
  __syncthreads();

  for (int kt = 0; kt < nkt; ++kt) {
    const int cur = kt & 1, k0 = kt * AT_KT;
    if (kt + 1 < nkt) issue_tile(kt + 1, cur ^ 1);
    const unsigned char* Ks = smem + cur * STAGE;
    const unsigned char* Vs = Ks + K_BYTES;
    const unsigned char* Ts = Ks + 2 * K_BYTES;
    if (live && k0 < q0 + AT_QT) {                 // wave-uniform: the tile holds keys this wave's rows may see
    bf16x8 dsf[2][2];
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) {
      f32x16 s, dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = dp[r] = 0.f;
      const int roff = (jj * 32 + (lane & 31)) * MF_ROW_BYTES;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int off = roff + (ks >> 2) * (AT_KT * MF_ROW_BYTES) + (((2 * (ks & 3) + half) ^ fl) << 4);
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8*)(Ks + off), qf[ks], s, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8*)(Vs + off), gf[ks], dp, 0, 0, 0);
      }
      if (k0 + jj * 32 + 31 > q0) {              // this half crosses the diagonal: keys after the query contribute nothing
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = k0 + jj * 32 + 16 * (r >> 3) + 8 * half + (r & 7);   // see at_key_of_row
          const float p = key > qi ? 0.f : __builtin_amdgcn_exp2f(fmaf(s[r], scale_log2e, -lse));
          dsf[jj][r >> 3][r & 7] = (bf16)(p * (dp[r] - dvec));
        }
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float p = __builtin_amdgcn_exp2f(fmaf(s[r], scale_log2e, -lse));
          dsf[jj][r >> 3][r & 7] = (bf16)(p * (dp[r] - dvec));
        }
      }
    }
    // dQ^T[dim][query] += K^T[dim][key] dS^T[key][query]
#pragma unroll
    for (int t = 0; t < OT; ++t) {
      const unsigned char* trow = Ts + (t * 32 + (lane & 31)) * MF_ROW_BYTES;
#pragma unroll
      for (int jj = 0; jj < 2; ++jj)
#pragma unroll
        for (int ss = 0; ss < 2; ++ss) {
          const bf16x8 tf = *(const bf16x8*)(trow + (((jj * 4 + 2 * ss + half) ^ fl) << 4));
          o[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tf, dsf[jj][ss], o[t], 0, 0, 0);
        }
    }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
  }

  if (qi < Trows) {
    bf16* dst = dQKV + ((size_t)l * Trows + qi) * ldq + head * DH;
#pragma unroll
    for (int t = 0; t < OT; ++t)
#pragma unroll
      for (int rg = 0; rg < 4; ++rg) {
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (bf16)(o[t][4 * rg + e] * scale);
        *(bf16x4*)(dst + t * 32 + 8 * rg + 4 * half) = v;
      }
  }
}

// dK, dV.  Qt, dOt: [cells][H][dh][Tp] (sequence index contiguous, zero padded); dQKV: k and v columns written here.
// One workgroup = one KV head of one cell x 256 keys; wave w (of 8) owns keys [32 w, 32 w + 32) of them (K, V rows in registers
// as B operands) for the whole kernel and adds the contributions of all query heads of the KV group, one after the
// other, in its registers: no reduction between waves or workgroups.  The eight waves share the tiles of the current
// (query head, 64 query rows): Q and dO rows, Q^T and dO^T columns, the rows' log-sum-exp and D, double buffered in LDS.
// What bounds it: the longest workgroup (key block 0 meets every query of every head) and, inside an iteration, two waves per SIMD that take
// turns with products and exponentials.  head_dim 64, 1B shape, us per launch (mean of 5.6 cells): 237 with
// the transposed operands read 8 bytes at a time (bank conflicts) and a branch around every exponential, 206 with permuted rows
// (at_key_of_row: a fragment is one 16-byte read), 153 with the mask in a loop of its own.  Four or two waves (128 or 64 keys) per workgroup
// copy more and gain no balance: 193, 261 (205 with eight).
// head_dim 128: K, V, dK and dV of a wave are 192 of its 256 registers, and what does not fit is loaded again behind the prefetch of the next
// tile.  So it takes the products one by one (P, dV, dP, dK: one 32 x 32 result and P at a time), half a tile at a time, which spills nothing:
// 3B shape (mean of 2.8 cells) 348 us with 8-byte reads, 375 with the steps of head_dim 64 (49 registers spilled), 230 as it is; d 4096 498 -> 304.
// In that order head_dim 64 takes 174.
// grid: 1-D, 8 * ceil(Hkv g / 8) * ceil(T / 256) workgroups, block: 512; LDS: 2 stages of 4 tiles + 512 bytes.
constexpr int DKV_WAVES = 8;
template <int DH>
__global__ __launch_bounds__(64 * DKV_WAVES) void attention_bwd_dkv_kernel(const bf16* __restrict__ QKV, const bf16* __restrict__ Qt,
                                                                const bf16* __restrict__ dO, const bf16* __restrict__ dOt,
                                                                const float* __restrict__ LSE2, const float* __restrict__ Dv,
                                                                bf16* __restrict__ dQKV, int first, int Trows, int Tp, int H,
                                                                int Hkv, float scale, int npairs) {
  constexpr int Q_BYTES = 64 * DH * 2;             // one tile: 64 x DH or DH x 64 bf16
  constexpr int STAGE = 4 * Q_BYTES + 512;         // Q, dO, Q^T, dO^T, then lse[64], D[64]
  constexpr int Q_SLABS = Q_BYTES / 1024;
  constexpr int KS = DH / 16, OT = DH / 32;
  constexpr bool ONE_BY_ONE = DH == 128;           // one product at a time (see above)
  constexpr int HALVES = ONE_BY_ONE ? 1 : 2;       // of a tile, unrolled
  extern __shared__ __align__(16) unsigned char smem[];   // [2][STAGE]

  // key block 0 meets every query row, the last one a few: longest first over all (cell, KV head) pairs, a pair on one XCD
  const int ppx = (npairs + 7) >> 3, xj = blockIdx.x >> 3;
  const int kb = xj / ppx;
  const int pair = (xj % ppx) * 8 + (blockIdx.x & 7);
  if (pair >= npairs) return;
  const int kvh = pair % Hkv, l = first + pair / Hkv;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int group = H / Hkv;
  const int ldq = (H + 2 * Hkv) * DH, ldo = H * DH;
  const int k0 = kb * (32 * DKV_WAVES) + wave * 32;
  const int half = lane >> 5;
  const float scale_log2e = scale * 1.4426950408889634f;
  const int ki = k0 + (lane & 31);

  const bf16* cell = QKV + (size_t)l * Trows * ldq;
  const bf16* gcell = dO + (size_t)l * Trows * ldo;
  bf16x8 kf[KS], vf[KS];       // B operands: this lane's key row of K and of V
  {
    const int krow = min(ki, Trows - 1);
    const bf16* kp = cell + (size_t)krow * ldq + (H + kvh) * DH + half * 8;
    const bf16* vp = cell + (size_t)krow * ldq + (H + Hkv + kvh) * DH + half * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      kf[ks] = *(const bf16x8*)(kp + ks * 16);
      vf[ks] = *(const bf16x8*)(vp + ks * 16);
    }
  }

  const int qt_first = kb * (DKV_WAVES / 2);       // first 64-row query tile that can see these keys
  const int nq = Tp / 64 - qt_first;               // query tiles per head
  const int iters = group * nq;
  // tile copies as in the forward kernel: scalar base + one lane offset per operand, the Q and dO rows permuted (at_key_of_row)
  const unsigned chunk0 = (unsigned)(((lane & 7) ^ mf_swz(lane >> 3)) << 4);
  const unsigned rowR = (unsigned)(((lane >> 3) & 3) + ((lane >> 5) << 3));
  const unsigned voffQ = rowR * (unsigned)ldq * 2u + chunk0, voffG = rowR * (unsigned)ldo * 2u + chunk0;
  const unsigned voffT = (unsigned)(lane >> 3) * (unsigned)Tp * 2u + chunk0;
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)smem;
  auto issue_tile = [&](int head, int q0, int buf) {
    int at = lane;               // (DH 128: no register is left to keep the lane in)
    if constexpr (ONE_BY_ONE) asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(at));
    const int R = at >> 3, pc = at & 7;
    typedef const __attribute__((address_space(1))) void* gptr_t;
    typedef __attribute__((address_space(3))) void* lptr_t;
    unsigned char* base = smem + buf * STAGE;
    const unsigned lds = lds0 + buf * STAGE;
    const char* qrows = (const char*)(cell + head * DH);
    const char* grows = (const char*)(gcell + head * DH);
    const char* qcols = (const char*)(Qt + (size_t)(l * H + head) * DH * Tp + q0);
    const char* gcols = (const char*)(dOt + (size_t)(l * H + head) * DH * Tp + q0);
    const bool whole = q0 + 64 <= Trows;             // wave-uniform: every query of the tile exists
    for (int sl = wave; sl < 4 * Q_SLABS; sl += DKV_WAVES) {
      const int which = sl / Q_SLABS, s2 = sl - which * Q_SLABS;
      if (which < 2) {           // rows of Q / dO: DH / 64 sub-tiles [64 rows][64 dims]
        const int sub = s2 >> 3, a = s2 & 7;
        const char* rows = which == 0 ? qrows : grows;
        const size_t ld = which == 0 ? ldq : ldo;
        if (whole) {
          const int qS = q0 + ((a & 1) << 2) + ((a >> 1) << 4);
          lds_copy16(rows + (qS * ld + sub * 64) * 2, (which == 0 ? voffQ : voffG) ^ ((unsigned)(a & 1) << 6), lds + sl * 1024);
        } else {
          const int row = a * 8 + R, q = min(q0 + at_key_of_row(row), Trows - 1);
          const char* src = rows + (q * ld + sub * 64 + ((pc ^ mf_swz(row)) << 3)) * 2;
          __builtin_amdgcn_global_load_lds((gptr_t)src, (lptr_t)(base + sl * 1024), 16, 0, 0);
        }
      } else {                   // columns: [DH dims][64 rows of the sequence]
        lds_copy16((which == 2 ? qcols : gcols) + (size_t)s2 * 8 * Tp * 2, voffT ^ ((unsigned)(s2 & 1) << 6), lds + sl * 1024);
      }
    }
    if (wave < 2) {              // lse (wave 0) and D (wave 1) of the 64 rows, also as direct loads: a load through
      const float* srcf = (wave == 0 ? LSE2 : Dv) + ((size_t)l * H + head) * Trows + min(q0 + at, Trows - 1);     // registers
      __builtin_amdgcn_global_load_lds((gptr_t)srcf, (lptr_t)(base + 4 * Q_BYTES + wave * 256), 4, 0, 0);         // would make the
    }                            // wave wait for the whole prefetch before it starts on the current tile
  };

  const int fl = mf_swz(lane & 31);
  f32x16 dk[OT], dv[OT];
#pragma unroll
  for (int t = 0; t < OT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) dk[t][r] = dv[t][r] = 0.f;

  int head = kvh * group, q0 = qt_first * 64;        // of the current tile
  issue_tile(head, q0, 0);
  __builtin_amdgcn_s_waitcnt(0x0F70);
  __syncthreads();

  for (int it = 0; it < iters; ++it) {
    const int cur = it & 1;
    const bool wrap = q0 + 64 >= Tp;                 // last tile of the head
    const int next_head = wrap ? head + 1 : head, next_q0 = wrap ? qt_first * 64 : q0 + 64;
    if (it + 1 < iters) issue_tile(next_head, next_q0, cur ^ 1);
    const unsigned char* Qs = smem + cur * STAGE;
    const unsigned char* Gs = Qs + Q_BYTES;
    const unsigned char* QTs = Qs + 2 * Q_BYTES;
    const unsigned char* GTs = Qs + 3 * Q_BYTES;
    const float* sL = (const float*)(Qs + 4 * Q_BYTES);
    const float* sD = sL + 64;
    if (k0 <= q0 + 63 && k0 < Trows) {             // wave-uniform: some query of the tile can see some key of this wave
#pragma unroll HALVES
      for (int jj = 0; jj < 2; ++jj) {
        if (q0 + jj * 32 + 31 < k0) continue;      // this half of the tile lies before the keys
        const int roff = (jj * 32 + (lane & 31)) * MF_ROW_BYTES;
        auto row_at = [&](int ks) { return roff + (ks >> 2) * (64 * MF_ROW_BYTES) + (((2 * (ks & 3) + half) ^ fl) << 4); };
        auto col_at = [&](int t, int ss) { return (t * 32 + (lane & 31)) * MF_ROW_BYTES + (((jj * 4 + 2 * ss + half) ^ fl) << 4); };
        auto row_of = [&](int rg) { return jj * 32 + 16 * (rg >> 1) + 8 * half + 4 * (rg & 1); };   // rows of registers 4 rg .. 4 rg + 3
        f32x16 s, dp;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = dp[r] = 0.f;
        auto add_dp = [&](int ks) { dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8*)(Gs + row_at(ks)), vf[ks], dp, 0, 0, 0); };
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8*)(Qs + row_at(ks)), kf[ks], s, 0, 0, 0);
          if constexpr (!ONE_BY_ONE) add_dp(ks);
        }
        // all 32 queries of this half exist and lie at or after all 32 keys of the wave: nothing to mask
        const bool interior = q0 + jj * 32 >= k0 + 31 && q0 + jj * 32 + 31 < Trows;
        f32x4 l4[4], d4[4];
        auto lse_of = [&](int rg) { l4[rg] = *(const f32x4*)(sL + row_of(rg)); };
        auto d_of = [&](int rg) { d4[rg] = *(const f32x4*)(sD + row_of(rg)); };
        if constexpr (!ONE_BY_ONE) {
#pragma unroll
          for (int rg = 0; rg < 4; ++rg) { lse_of(rg); d_of(rg); }
        }
        float p[16];
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
          if constexpr (ONE_BY_ONE) lse_of(rg);
#pragma unroll
          for (int e = 0; e < 4; ++e) p[4 * rg + e] = __builtin_amdgcn_exp2f(fmaf(s[4 * rg + e], scale_log2e, -l4[rg][e]));
        }
        // (the mask is a loop of its own: with its condition inside the common one the compiler branched around every exponential)
        if (!interior) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int q = q0 + jj * 32 + 16 * (r >> 3) + 8 * half + (r & 7);
            p[r] = q < Trows && ki <= q ? p[r] : 0.f;
          }
        }
        bf16x8 pf[2], dsf[2];
#pragma unroll
        for (int r = 0; r < 16; ++r) pf[r >> 3][r & 7] = (bf16)p[r];
        // dV^T[dim][key] += dO^T[dim][query] P[query][key],  dK^T[dim][key] += Q^T[dim][query] dS[query][key]
        auto add_dv = [&](int t, int ss) {
          dv[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8*)(GTs + col_at(t, ss)), pf[ss], dv[t], 0, 0, 0);
        };
        if constexpr (ONE_BY_ONE) {
#pragma unroll
          for (int t = 0; t < OT; ++t)
#pragma unroll
            for (int ss = 0; ss < 2; ++ss) add_dv(t, ss);
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) add_dp(ks);
        }
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
          if constexpr (ONE_BY_ONE) d_of(rg);
#pragma unroll
          for (int e = 0; e < 4; ++e) dsf[rg >> 1][4 * (rg & 1) + e] = (bf16)(p[4 * rg + e] * (dp[4 * rg + e] - d4[rg][e]));
        }
#pragma unroll
        for (int t = 0; t < OT; ++t)
#pragma unroll
          for (int ss = 0; ss < 2; ++ss) {
            if constexpr (!ONE_BY_ONE) add_dv(t, ss);
            dk[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8*)(QTs + col_at(t, ss)), dsf[ss], dk[t], 0, 0, 0);
          }
      }
    }
    head = next_head;
    q0 = next_q0;
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
  }

  if (ki < Trows) {
    bf16* dkp = dQKV + ((size_t)l * Trows + ki) * ldq + (H + kvh) * DH;
    bf16* dvp = dQKV + ((size_t)l * Trows + ki) * ldq + (H + Hkv + kvh) * DH;
#pragma unroll
    for (int t = 0; t < OT; ++t)
#pragma unroll
      for (int rg = 0; rg < 4; ++rg) {
        bf16x4 a, b;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          a[e] = (bf16)(dk[t][4 * rg + e] * scale);
          b[e] = (bf16)dv[t][4 * rg + e];
        }
        *(bf16x4*)(dkp + t * 32 + 8 * rg + 4 * half) = a;
        *(bf16x4*)(dvp + t * 32 + 8 * rg + 4 * half) = b;
      }
  }
}

// bytes of the transposed operands for g cells: K^T [Hkv], Q^T [H], dO^T [H], each [dh][Tp]
inline size_t attention_bwd_scratch_bytes(int g, int Trows, int H, int Hkv, int dh) {
  return (size_t)g * (2 * H + Hkv) * dh * attention_tp(Trows) * 2;
}

// QKV (rotated q, k; v), O, dO as in the kernels above; LSE2 from the forward kernel; scratch as sized above.
inline hipError_t launch_attention_bwd_mfma(const bf16* QKV, const bf16* O, const bf16* dO, const float* LSE2, float* Dv,
                                            bf16* scratch, bf16* dQKV, int first, int g, int Lcells, int Trows, int H, int Hkv,
                                            int dh, hipStream_t st) {
  const int Tp = attention_tp(Trows), group = H / Hkv, ldq = (H + 2 * Hkv) * dh;
  bf16* Kt = scratch;
  bf16* Qt = Kt + (size_t)Lcells * Hkv * dh * Tp;
  bf16* Gt = Qt + (size_t)Lcells * H * dh * Tp;
  head_transpose_kernel<<<dim3(Tp / 64, (2 * H + Hkv) * dh / 64, g), 256, 0, st>>>(QKV, dO, Kt, Qt, Gt, first, Trows, Tp, H, Hkv, dh);
  (dh == 64 ? attention_dvec_kernel<64> : attention_dvec_kernel<128>)<<<dim3((Trows + 3) / 4, g), 256, 0, st>>>(O, dO, Dv, first, Trows, H);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const float scale = 1.0f / sqrtf((float)dh);
  const int nq = group == 1 ? 4 : (group == 2 ? 2 : 1);       // row tiles per dQ workgroup, as in the forward kernel
  const int nqt = (Trows + 32 * nq - 1) / (32 * nq), npairs = Hkv * g;
  const int nkb = (Trows + 32 * DKV_WAVES - 1) / (32 * DKV_WAVES);
  const dim3 grid(8 * ((npairs + 7) / 8) * nqt), gkv(8 * ((npairs + 7) / 8) * nkb);
  const int lds_q = 2 * 3 * (64 * dh * 2), lds_kv = 2 * (4 * 64 * dh * 2 + 512);
  auto dq = dh == 64 ? attention_bwd_dq_kernel<64> : attention_bwd_dq_kernel<128>;
  auto dkv = dh == 64 ? attention_bwd_dkv_kernel<64> : attention_bwd_dkv_kernel<128>;
  static std::atomic<uint64_t> dq_raised[2], dkv_raised[2];      // head_dim 64, 128
  e = raise_lds_limit((const void*)dq, lds_q, dq_raised[dh != 64]);
  if (e == hipSuccess) e = raise_lds_limit((const void*)dkv, lds_kv, dkv_raised[dh != 64]);
  if (e != hipSuccess) return e;
  dq<<<grid, nq * group * 64, lds_q, st>>>(QKV, Kt, dO, LSE2, Dv, dQKV, first, Trows, Tp, H, Hkv, nq, scale, nqt, npairs);
  dkv<<<gkv, 64 * DKV_WAVES, lds_kv, st>>>(QKV, Qt, dO, Gt, LSE2, Dv, dQKV, first, Trows, Tp, H, Hkv, scale, npairs);
  return hipGetLastError();
}

}  // namespace armt
