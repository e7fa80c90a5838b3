// Grouped bf16 GEMM on the CDNA4 matrix cores (paper Section 3.3 item 1, Section 4.1).
//
//   C_g = A_g B_g^T for every group g of the launch; A_g [M, K] activations, B_g [N, K] the
//   weights of the group's own layer (taken from a pointer table, never stacked), fp32
//   accumulation in v_mfma_f32_16x16x32_bf16, epilogue fused (residual add, row scale,
//   SwiGLU, bf16 copy and sums of squares for the next RMSNorm, rotary embedding and transposed
//   V for the QKV projection).
//
// Tiling: one workgroup per BM x BN output tile, BK = 64.  Both operands are K-contiguous, so a
// tile row is 128 bytes = eight 16-byte chunks; chunks are XOR-swizzled inside a row so that the
// MFMA fragment reads (one row per lane, 16 bytes) spread over all LDS banks.  Tiles are double
// buffered in LDS (NS = 2 stages; more are possible for small tiles) and filled by direct
// global-to-LDS loads (no staging registers): the copies of k-tile i+1 are in flight while k-tile i
// is multiplied.  For regular shapes (template flag REG) the copies are addressed by a scalar base
// and one lane offset per operand, so that issuing them needs no vector-ALU instruction.
// The 256 x 256 tile of regular shapes is a kernel of its own (gemm_tile256.h).
// The 1-D grid is laid out so that each XCD (workgroup id mod 8) owns a contiguous run of the
// group-major tile sequence: with 16 groups every XCD streams the weights of 2 layers through its
// own L2, and the M-tiles sharing a weight panel run back to back.
// Template parameters of the kernel: BM x BN tile, WGM x WGN waves, REG (see above), EPI (GemmEpilogue),
// TAIL (see below), NS (LDS stages).  The launcher picks the configuration from the shape and the number of tiles of
// the launch (mfma_pick_config).
#pragma once

#include <atomic>
#include <type_traits>

#include "common.h"
#include "gemm_generic.h"

namespace armt {

constexpr int MF_BK = 64;                 // k-tile (bf16 elements): 128 bytes per tile row
constexpr int MF_ROW_BYTES = MF_BK * 2;
constexpr int MF_CUS = 256;            // compute units of the chip: a round of one tile per unit
constexpr int MF_NUM_CONFIGS = 9;         // tile configuration numbers of launch_gemm_mfma_epi lie below this

// swizzle of the 16-byte chunk index inside a 128-byte tile row; depends on row bits 0..3 only
__device__ __forceinline__ int mf_swz(int row) { return ((row >> 1) & 7) ^ ((row & 1) << 2); }

template <int N>
__device__ __forceinline__ void mf_wait_vmcnt() {      // s_waitcnt vmcnt(N) only (N <= 63)
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
}
// vmcnt(N) if left >= 0, else vmcnt(0); left is wave-uniform.  The branch is inside the asm: one that the compiler sees ends its block, and
// then the barrier behind the wait is not moved in front of a k-tile's last MFMAs, which need nothing but registers.  64 x 128 tiles with
// four stages, us, branch in the source / here: 16 x 2048, K 5632 36.1 / 32.9 (operands from the L2; two stages: 32.9)
template <int N>
__device__ __forceinline__ void mf_wait_vmcnt_if(int left) {
  static_assert(N <= 63, "vmcnt has six bits");
  asm volatile("s_cmp_ge_i32 %0, 0\n\ts_cbranch_scc1 .Lmf_wait_%=\n\ts_waitcnt vmcnt(0)\n.Lmf_wait_%=:\n\ts_waitcnt vmcnt(%1)"
               : : "s"(__builtin_amdgcn_readfirstlane(left)), "n"(N) : "memory", "scc");
}

#ifdef ARMT_GEMM_TIMELINE
// Probe build (build(timeline=True) of paper_2506_05229_amd.build, never the product library): one armed launch records, per
// tile, where its time goes: [0] hardware id, [1] / [6] wall clock (100 MHz) at start / end, [2] .. [5] shader
// clock at start, after the first k-tile has landed, after the main loop, after the epilogue.  A workgroup of the persistent tile (gemm_tile256.h) writes a
// record for each of its tiles: [2] and [3] are the same there (a tile starts on what the one before it fetched), and the products of a tile's
// first k-step that run under the epilogue of the one before count in that epilogue.
__device__ unsigned long long armt_timeline[8 * 65536];
inline int g_tl_kind = -2, g_tl_countdown = -1;      // host: the n-th next launch of this kind is the armed one
#define TL_STAMP(i)                                                     \
  do {                                                                  \
    if (tl_on && threadIdx.x == 0) tl[i] = __builtin_readcyclecounter(); \
  } while (0)
#else
#define TL_STAMP(i) do {} while (0)
#endif

}  // namespace armt

#include "gemm_tile256.h"

namespace armt {

// LDS bytes of the tile buffers of a configuration: NS buffers of a k-tile (A rows, B rows), and at least the two fp32
// staging tiles [staged rows][tile columns + 4] of the epilogue, which reuse them.
template <int BM, int BN, int WGM, int WGN, int EPI, bool TAIL, int NS>
constexpr int mfma_tile_lds_bytes() {
  const int tiles = NS * ((TAIL ? BM + 16 : BM) + BN) * MF_ROW_BYTES;
  const int stg = 2 * WGM * 16 * (((EPI == EPI_SWIGLU) ? BN / 2 : BN) + 4) * 4;
  return ((tiles > stg ? tiles : stg) + 255) / 256 * 256;
}

// TAIL: the last M-tile of every group also owns the 16 rows that follow it (M = tiles_m * BM + 16).  With
// T = seg_len + 16 memory rows and seg_len a multiple of BM this removes the nearly empty fifth tile a
// 1040-row cell would otherwise need: the 16 memory rows ride along as one extra strip of 16x16x32 MFMAs.
template <int BM, int BN, int WGM, int WGN, bool REG, int EPI, bool TAIL, int NS>
__global__ __launch_bounds__(WGM* WGN * 64) void gemm_mfma_kernel(const GemmGroup* __restrict__ table, int first,
                                                                  GemmShape s, int tiles_m, int tiles_n, int m_group,
                                                                  int total_tiles, int tile_begin) {
  constexpr int NW = WGM * WGN, BK = MF_BK;
  constexpr int WROWS = BM / WGM, WCOLS = BN / WGN;       // wave tile
  constexpr int TM = WROWS / 16, TN = WCOLS / 16;         // 16x16 MFMA tiles per wave
  constexpr int ROWB = BK * 2;                            // bytes of a tile row
  constexpr int RPS = 1024 / ROWB;                        // rows of a 1 KB slab (one copy instruction)
  constexpr int A_DMA = BM / RPS / NW, B_DMA = BN / RPS / NW;   // slabs each wave copies per k-tile
  constexpr int TAIL_SLABS = 16 / RPS;                    // slabs of the 16 tail rows, copied by the first waves
  constexpr int A_ROWS = TAIL ? BM + 16 : BM;
  constexpr int A_BYTES = A_ROWS * ROWB, B_BYTES = BN * ROWB;
  constexpr int BN_OUT = (EPI == EPI_SWIGLU) ? BN / 2 : BN;   // output columns per tile
  static_assert(BM % (WGM * 16) == 0 && BN % (WGN * 16) == 0, "wave tile must be a multiple of 16x16");
  static_assert(EPI != EPI_SWIGLU || WCOLS % 64 == 0, "SwiGLU: a wave owns whole gate/up pairs of 32-row weight blocks");
  static_assert(BM % (RPS * NW) == 0 && BN % (RPS * NW) == 0, "tile rows must divide into slabs per wave");
  static_assert(!TAIL || (BN <= NW * 32 && NW >= 2), "the tail strip gives each of the first BN / 32 waves two 16-column tiles");

  extern __shared__ __align__(16) unsigned char smem[];   // [NS][A_BYTES], [NS][B_BYTES], then A_ROWS row scales

#ifdef ARMT_GEMM_TIMELINE
  const bool tl_on = (s.dbg >> 20) & 1;
  unsigned long long* tl = armt_timeline + 8 * (size_t)(blockIdx.x & 65535);
  if (tl_on && threadIdx.x == 0) {
    unsigned hw, xcc;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_HW_ID)" : "=s"(hw));
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
    tl[0] = ((unsigned long long)xcc << 32) | hw;
    tl[1] = __builtin_amdgcn_s_memrealtime();
    tl[2] = __builtin_readcyclecounter();
  }
#endif
  // XCD-aware tile order: workgroup b runs on XCD b % 8; give each XCD a contiguous range.  The launch covers the
  // total_tiles tiles from tile_begin on of the order (group, M-group, N-tile, M-tile of the M-group).
  const int per_xcd = (total_tiles + 7) >> 3;
  const int lid0 = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (lid0 >= total_tiles) return;
  const int per_group = tiles_m * tiles_n;
  int lid = tile_begin + lid0;
  if (s.spread) {                          // (whole launches, groups of a multiple of 8 tiles)
    const int share = per_group >> 3, i = blockIdx.x >> 3;
    lid = i / share * per_group + (blockIdx.x & 7) * share + i % share;
  }
  const int grp = lid / per_group, rem = lid - grp * per_group;
  // M-tiles of one weight panel are adjacent; tall problems are cut into M-groups of m_group tiles (mfma_m_group).  (A division is a
  // few hundred cycles in front of the first copy of every tile: none for groups that a problem does not have.)
  int mg0 = 0, rem_mg = rem, mg_tiles = tiles_m;      // first M-tile and M-tiles of the group
  if (m_group < tiles_m) {
    const int mg = rem / (m_group * tiles_n);
    mg0 = mg * m_group;
    rem_mg = rem - mg0 * tiles_n;
    mg_tiles = min(m_group, tiles_m - mg0);
  }
  const int tn = rem_mg / mg_tiles, tm = mg0 + rem_mg - tn * mg_tiles;
  GemmGroup g = table[first + grp];
  if (!restrict_k<bf16>(g, s)) return;
  const int m0 = tm * BM, n0 = tn * BN_OUT;
  const int m0_strip = tiles_m * BM;                        // first row of the strip (TAIL)
  const bool tail_blk = TAIL && tm == tiles_m - 1;             // block-uniform: the last M-tile computes the strip behind it

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // per-row scale of the result (1 / rms of a fused RMSNorm, or 1 / denominator of the associative read),
  // fetched once; visible to everybody after the first barrier of the main loop
  float* rs_lds = (float*)(smem + mfma_tile_lds_bytes<BM, BN, WGM, WGN, EPI, TAIL, NS>());
  auto row_scale_of = [&](int r) {
    const int m = r < BM ? m0 + r : m0_strip + r - BM;
    return (g.rowscale && m < s.M) ? g.rowscale[m] : 1.f;
  };
  for (int r = tid; r < A_ROWS; r += NW * 64) rs_lds[r] = row_scale_of(r);
  const int wm = wave / WGN, wn = wave % WGN;
  const bool tail = tail_blk && wave < (TAIL ? BN / 32 : 0);   // wave-uniform: this wave computes part of the strip
  // first row / column of the 16 x 16 result blocks of a wave
  auto blk_row = [&](int i) { return wm * WROWS + i * 16; };
  auto blk_col = [&](int j) { return wn * WCOLS + j * 16; };

  // ---- global -> LDS copies go straight to LDS (global_load_lds_dwordx4): one instruction moves 64 x 16
  // bytes into 1 KB of consecutive LDS = 8 tile rows.  Lane i fills row i / 8, physical chunk i % 8 of the
  // slab, so it fetches the logical chunk (i % 8) ^ swz(row) of that row from global memory.
  // first element of row `row` of this block's weight tile
  // row n of the logical [N, K] weight, which comes in up to three blocks (selected by value: the table entry must not
  // be indexed dynamically, or it ends up in scratch memory instead of scalar registers)
  const bf16 *wB0 = (const bf16*)g.B0, *wB1 = (const bf16*)g.B1, *wB2 = (const bf16*)g.B2;
  auto w_row = [&](int n) -> const bf16* {
    if (n < s.n0) return wB0 + (size_t)n * s.ldb;
    n -= s.n0;
    if (n < s.n1) return wB1 + (size_t)n * s.ldb;
    return wB2 + (size_t)(n - s.n1) * s.ldb;
  };
  auto b_row = [&](int row) -> const bf16* {
    if (EPI == EPI_SWIGLU) {
      // tile rows come in 32-row blocks: even blocks from the gate weight, odd from the up weight,
      // both for output columns n0 + (block / 2) * 32 ...
      const int blk = row >> 5;
      const int n = min(n0 + (blk >> 1) * 32 + (row & 31), s.N - 1);
      return (const bf16*)((blk & 1) ? g.B1 : g.B0) + (size_t)n * s.ldb;
    }
    return w_row(min(n0 + row, s.N - 1));
  };
  const int dR = lane >> 3, dpc = lane & 7;
  // source of this lane for A slab j / the tail slab / B slab j, at k = 0
  auto a_src = [&](int j) -> const char* {
    const int row = (wave + j * NW) * 8 + dR;
    const int m = min(m0 + row, s.M - 1);                  // rows past M re-read the last row; masked on store
    return (const char*)g.A + ((size_t)m * s.lda + ((dpc ^ mf_swz(row)) << 3)) * 2;
  };
  auto t_src = [&]() -> const char* {                      // tail rows: copying waves 0 and 1 move one extra slab each
    const int row = BM + (wave & 1) * 8 + dR;
    const int m = min(m0 + row, s.M - 1);
    return (const char*)g.A + ((size_t)m * s.lda + ((dpc ^ mf_swz(row)) << 3)) * 2;
  };
  auto b_src = [&](int j) -> const char* {
    const int row = (wave + j * NW) * 8 + dR;
    return (const char*)(b_row(row) + ((dpc ^ mf_swz(row)) << 3));
  };
  // Two ways to address the sources.
  // General shapes: every lane keeps one 64-bit pointer per slab (rows past M or N are clamped per lane).
  // Regular shapes (REG: no ragged M or N, weight blocks that end on tile boundaries): all sources of a lane
  // differ by wave-uniform amounts, because the swizzle of row 8 * slab + lane / 8 depends on the slab's parity
  // only and a wave's slabs wave + NW * j all have the parity of the wave.  One 32-bit lane offset per operand
  // plus a scalar base per slab then address everything, and issuing a copy takes scalar instructions only.
  // That matters: a wave's vector-ALU instructions are not issued while other waves keep the SIMD's
  // matrix core busy with back-to-back MFMAs, scalar and memory instructions are.  Address arithmetic in the
  // vector ALU would hold the copies back until the multiplying waves pause.
  constexpr bool KEEP_PTRS = !REG;
  static_assert(!REG || NW % 2 == 0, "slabs of a wave must share their parity");
  const char* ap[KEEP_PTRS ? A_DMA : 1];
  const char* bp[KEEP_PTRS ? B_DMA : 1];
  const char* tp = nullptr;
  unsigned a_off0 = 0, b_off0 = 0;
  if (KEEP_PTRS) {
#pragma unroll
    for (int j = 0; j < (KEEP_PTRS ? A_DMA : 0); ++j) ap[j] = a_src(j);
    if (TAIL) tp = t_src();
#pragma unroll
    for (int j = 0; j < (KEEP_PTRS ? B_DMA : 0); ++j) bp[j] = b_src(j);
  } else {
    // lane i fills row i / 8, physical chunk i % 8 of its slab
    const int chunk = (dpc ^ mf_swz((wave & 1) * 8 + dR)) << 4;
    a_off0 = (unsigned)dR * (unsigned)s.lda * 2u + chunk;
    b_off0 = (unsigned)dR * (unsigned)s.ldb * 2u + chunk;
  }
  // scalar source of the first row of slab `slab` (REG only)
  auto a_base = [&](int slab) -> const char* { return (const char*)g.A + (size_t)(m0 + RPS * slab) * s.lda * 2; };
  auto b_base = [&](int slab) -> const char* {
    if (EPI == EPI_SWIGLU) {   // tile rows 32 * blk ..: blk even from the gate, odd from the up weight, columns n0 + 32 * (blk / 2) ..
      const int row = slab * RPS, blk = row >> 5;
      const int n = n0 + (blk >> 1) * 32 + (row & 31);
      return (const char*)((blk & 1) ? g.B1 : g.B0) + (size_t)n * s.ldb * 2;
    }
    return (const char*)w_row(n0 + RPS * slab);
  };
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)smem;
  // A copy from one 64-bit pointer per lane is an instruction like the ones with a scalar base (lds_copy16) and no builtin, too: the fence
  // of a barrier then does not wait for the copies of the younger k-tiles that are meant to stay in flight (the waits for the copies are
  // explicit, below).
  auto issue_tile = [&](int kt, int buf) {
    const size_t ka = (size_t)kt * ROWB, kb = ka;
    if (KEEP_PTRS) {
      const unsigned ldsA = lds0 + buf * A_BYTES, ldsB = lds0 + NS * A_BYTES + buf * B_BYTES;
#pragma unroll
      for (int j = 0; j < A_DMA; ++j)
        lds_copy16(ap[KEEP_PTRS ? j : 0] + ka, ldsA + (wave + j * NW) * 1024);
      if (TAIL && tail_blk && wave < 2)
        lds_copy16(tp + ka, ldsA + BM * MF_ROW_BYTES + wave * 1024);
#pragma unroll
      for (int j = 0; j < B_DMA; ++j)
        lds_copy16(bp[KEEP_PTRS ? j : 0] + kb, ldsB + (wave + j * NW) * 1024);
    } else {
      const unsigned As = lds0 + buf * A_BYTES, Bs = lds0 + NS * A_BYTES + buf * B_BYTES;
#pragma unroll
      for (int j = 0; j < A_DMA; ++j) lds_copy16(a_base(wave + j * NW) + ka, a_off0, As + (wave + j * NW) * 1024);
      if (TAIL && tail_blk && wave < TAIL_SLABS) lds_copy16(a_base(BM / RPS + wave) + ka, a_off0, As + BM * ROWB + wave * 1024);
#pragma unroll
      for (int j = 0; j < B_DMA; ++j) lds_copy16(b_base(wave + j * NW) + kb, b_off0, Bs + (wave + j * NW) * 1024);
    }
  };

  // ---- MFMA fragment addresses (v_mfma_f32_16x16x32_bf16: under random operands this instruction sustains
  // 1.9 PFLOP/s on the chip against 1.35 for the 32x32x16 form, which draws more power per flop; measured with
  // register-only loops): lane reads tile row (lane % 16) of each 16-row block, 16-byte chunk 4 * ks2 + lane / 16
  // of the 128-byte row; a 16x16 result tile has lane = column lane % 16 and registers = rows 4 * (lane / 16) + r.
  constexpr int KS2 = BK / 32;                 // MFMA k-steps per k-tile
  const int t_sw = mf_swz(lane & 15), t_q = lane >> 4;
  int koff[KS2];
#pragma unroll
  for (int ks2 = 0; ks2 < KS2; ++ks2) koff[ks2] = ((4 * ks2 + t_q) ^ t_sw) << 4;
  const int a_frag = (blk_row(0) + (lane & 15)) * ROWB;
  const int b_frag = (blk_col(0) + (lane & 15)) * ROWB;
  // tail strip: the same instruction on the 16 extra rows.  Wave w owns two 16-column
  // tiles whose B rows lie 32 apart, so that for SwiGLU tile 0 is the gate and tile 1 the up projection of the
  // same 16 output columns: B tile rows ((w / 2) * 2 + t) * 32 + (w % 2) * 16 + lane % 16.
  const int t_a = (BM + (lane & 15)) * ROWB;
  const int t_brow = ((wave >> 1) * 2) * 32 + (wave & 1) * 16 + (lane & 15);
  constexpr int T_STEP = 32;                               // columns between the wave's two blocks of the strip
  const int t_b = t_brow * ROWB;

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 tacc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};

  {
    // main loop: NS tile buffers; the copies of k-tiles kt+1 .. kt+NS-1 are in flight while k-tile kt is
    // multiplied (copies complete in issue order, so waiting for tile kt+1 leaves the younger ones outstanding);
    // one barrier per k-tile
    constexpr int CNT = A_DMA + B_DMA;                 // copy instructions per wave and tile (+1 on the tail waves)
    const bool extra = TAIL && tail_blk && wave < TAIL_SLABS;
    const int nk = s.K / BK;
#pragma unroll
    for (int p = 0; p < NS - 1; ++p)
      if (p < nk) issue_tile(p, p);
    if (NS > 2 && nk > NS - 2) {
      if (extra) mf_wait_vmcnt<(NS - 2) * (CNT + 1)>(); else mf_wait_vmcnt<(NS - 2) * CNT>();
    } else {
      mf_wait_vmcnt<0>();
    }
    __syncthreads();
    TL_STAMP(3);
    int cur = 0, nxt = NS - 1;                           // buffers of tile kt and of tile kt + NS - 1
    for (int kt = 0; kt < nk; ++kt) {
      // buffer nxt was last read in iteration kt - 1, which ended with a barrier
      if (kt + NS - 1 < nk) issue_tile(kt + NS - 1, nxt);
      const unsigned char* As = smem + cur * A_BYTES;
      const unsigned char* Bs = smem + NS * A_BYTES + cur * B_BYTES;
      // (the strip first: behind the others, its branch would stand between the last products and the barrier; 80 x 64, K 5632: 51.1 -> 47.9 us)
      if (TAIL && tail) {
#pragma unroll
        for (int ks2 = 0; ks2 < KS2; ++ks2) {
          const int ko = koff[ks2];
          const bf16x8 ta = *(const bf16x8*)(As + t_a + ko);
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const bf16x8 tb = *(const bf16x8*)(Bs + t_b + t * 32 * ROWB + ko);
            tacc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ta, tb, tacc[t], 0, 0, 0);
          }
        }
      }
#pragma unroll
      for (int ks2 = 0; ks2 < KS2; ++ks2) {
        bf16x8 af[TM], bfr[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) af[i] = *(const bf16x8*)(As + a_frag + i * 16 * ROWB + koff[ks2]);
#pragma unroll
        for (int j = 0; j < TN; ++j) bfr[j] = *(const bf16x8*)(Bs + b_frag + j * 16 * ROWB + koff[ks2]);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
      }
      // tile kt+1 must have landed; tiles kt+2 .. kt+NS-1 (if they were issued) may stay in flight (waves that also copy the strip
      // wait for a little more than they need)
      if constexpr (NS > 2) mf_wait_vmcnt_if<(NS - 2) * CNT>(nk - kt - NS);
      else mf_wait_vmcnt<0>();
      __syncthreads();
      cur = (cur + 1 == NS) ? 0 : cur + 1;
      nxt = (nxt + 1 == NS) ? 0 : nxt + 1;
    }
  }

  TL_STAMP(4);
  // ---- epilogue, staged through LDS so that global memory sees whole rows: a 16x16 result tile has lane =
  // column (lane % 16) and registers = rows 4 * (lane / 16) + r, which written directly would touch global
  // memory in 32- or 64-byte pieces.  Instead, in TM passes every wave drops one 16-row block of its tile into
  // a fp32 staging tile [WGM * 16][BN_OUT + 4] (the +4 puts the four row groups of a wave on different banks),
  // and all threads then walk the staging tile row-major, C4 = BN_OUT / 4 lanes per row: 16-byte accesses, full rows
  // of R, C, C2.  The tail strip goes through the same path as one more pass of 16 rows.
  // There are two staging tiles (the tile buffers are free: the main loop ended with a barrier): pass p + 1 is staged
  // while pass p is still being drained, so a pass costs one barrier, and nothing of it waits for global memory
  // between the barriers: what a pass reads from global memory (residual rows, rotary table) is requested before its
  // staging writes, and the barriers wait for LDS traffic only.
  constexpr int SLD = BN_OUT + 4, SR = WGM * 16, C4 = BN_OUT / 4, NT = NW * 64;
  constexpr int STG_FLOATS = SR * SLD;
  static_assert(2 * STG_FLOATS * 4 <= mfma_tile_lds_bytes<BM, BN, WGM, WGN, EPI, TAIL, NS>(), "two staging tiles must fit in the tile buffers");
  static_assert(C4 == 16 || C4 == 32 || C4 == 64, "a staged row is handled by 16, 32 or 64 consecutive lanes");
  static_assert(NT % C4 == 0, "a thread keeps its columns from one row of the walk to the next");
  const bool vec_ok = ((s.N | s.ldc | s.ldr | s.ldc2) & 3) == 0;
  // silu(gate) * up; the reciprocal is the hardware's (1 ulp), the result is rounded to bf16 afterwards
  auto silu_mul = [](float gt, float up) { return gt * __builtin_amdgcn_rcpf(1.f + __expf(-gt)) * up; };
  auto row_scale = [&](int m) { return rs_lds[m - m0]; };      // scale of output row m
  // EPI_DPFP_READ: feature idx = lane + 64 k of phi(q) = r[i] r[(i - j) mod 2 d_mem], r = [relu(q), relu(-q)], j = 1..nu
  // (the untrained feature map of Section 2.1) is max(sa q[ia], 0) max(sb q[ib], 0); which columns and signs, and the
  // lane's entries of z, are the same for every row: set up once per thread
  constexpr int DP_MAXK = (EPI == EPI_DPFP_READ) ? 8 : 1;      // 2 nu d_mem <= 512 features
  int dp_ia[DP_MAXK], dp_ib[DP_MAXK], dp_phi = 0;
  float dp_sa[DP_MAXK], dp_sb[DP_MAXK], dp_z[DP_MAXK];
  if constexpr (EPI == EPI_DPFP_READ) {
    const int dm = s.n0, n2 = 2 * dm;
    dp_phi = s.ldr * n2;
#pragma unroll
    for (int k = 0; k < DP_MAXK; ++k) {
      const int idx = min(k * 64 + lane, dp_phi - 1);
      const int j = idx / n2 + 1, i = idx - (j - 1) * n2;
      int i2 = i - j;
      if (i2 < 0) i2 += n2;
      dp_ia[k] = i < dm ? i : i - dm;   dp_sa[k] = i < dm ? 1.f : -1.f;
      dp_ib[k] = i2 < dm ? i2 : i2 - dm; dp_sb[k] = i2 < dm ? 1.f : -1.f;
      dp_z[k] = g.R[idx];
    }
  }
  // The walk: thread tid takes column group c4 = tid % C4 (4 columns) of the staged rows tid / C4 + it * (NT / C4).
  const int c4 = tid % C4, sr_first = tid / C4;
  const int n = n0 + c4 * 4;
  // per-thread constants of the walk: the gain of its four columns (EPI_RESID_F32 with a normalised copy)
  f32x4 gq = {1.f, 1.f, 1.f, 1.f};
  if (EPI == EPI_RESID_F32 && g.C2 && g.gain) {
#pragma unroll
    for (int e = 0; e < 4; ++e) gq[e] = (float)((const bf16*)g.gain)[min(n + e, s.N - 1)];
  }
  // sum over the 32 lanes that hold 128 consecutive columns of a row: four steps inside a row of 16 lanes with
  // data-parallel moves (no LDS), one exchange between the two rows
  auto sum32 = [](float v) __attribute__((always_inline)) {
    auto dpp = [](float x, auto ctrl) {
      return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value, 0xF, 0xF, true));
    };
    v += dpp(v, std::integral_constant<int, 0xB1>{});      // quad_perm [1, 0, 3, 2]
    v += dpp(v, std::integral_constant<int, 0x4E>{});      // quad_perm [2, 3, 0, 1]
    v += dpp(v, std::integral_constant<int, 0x141>{});     // row_half_mirror
    v += dpp(v, std::integral_constant<int, 0x140>{});     // row_mirror
    v += __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), 0x401F));   // lane ^ 16
    return v;
  };
  // What one pass of the walk reads from global memory, requested ahead of the pass.
  constexpr int MAX_ITER = (SR * C4 + NT - 1) / NT;
  struct Pre { f32x4 r[MAX_ITER]; };
  auto prefetch = [&](auto nrows_c, auto m_of, Pre& pre) __attribute__((always_inline)) {
    constexpr int NROWS = decltype(nrows_c)::value, ITER = (NROWS * C4 + NT - 1) / NT;
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
      const int sr = sr_first + it * (NT / C4);
      const int m = m_of(min(sr, NROWS - 1));
      const bool valid = sr < NROWS && m < s.M && n < s.N;
      pre.r[it] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (EPI == EPI_RESID_F32 && g.R && valid) {
        if (vec_ok) {
          pre.r[it] = *(const f32x4*)(g.R + (size_t)m * s.ldr + n);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (n + e < s.N) pre.r[it][e] = g.R[(size_t)m * s.ldr + n + e];
        }
      }
    }
  };
  // walk NROWS staged rows of staging tile stg; staged row sr is output row m_of(sr)
  auto drain = [&](const float* stg, auto nrows_c, auto m_of, const Pre& pre) __attribute__((always_inline)) {
    constexpr int NROWS = decltype(nrows_c)::value, ITER = (NROWS * C4 + NT - 1) / NT;
    if constexpr (EPI == EPI_DPFP_READ) {
      // One wave per staged row: the row's d_mem values q sit in the staging tile; lane L computes the features
      // L, L + 64, ... of phi(q) (dp_* above), stores them in the activation type and adds up its share of z . phi(q).
      // The summation order (lane-strided partial sums, then the wave reduction) does not depend on the tile
      // configuration, so every configuration produces the same bits.
      // A wave takes the staged rows wave, wave + NW, ...: all of them side by side (features of every row first, then the
      // row sums, then the stores), so that the LDS reads and the wave reductions of different rows overlap.
      constexpr int RW = (NROWS + NW - 1) / NW;           // rows per wave
      float f[RW][DP_MAXK], den[RW];
      int mrow[RW];
#pragma unroll
      for (int j = 0; j < RW; ++j) {
        const int sr = min(wave + j * NW, NROWS - 1);
        mrow[j] = (wave + j * NW < NROWS) ? m_of(sr) : s.M;      // rows past the tile or past M are skipped below
        const float* q = stg + sr * SLD;
        den[j] = 0.f;
#pragma unroll
        for (int k = 0; k < DP_MAXK; ++k) {
          f[j][k] = fmaxf(dp_sa[k] * q[dp_ia[k]], 0.f) * fmaxf(dp_sb[k] * q[dp_ib[k]], 0.f);
          if (k * 64 + lane < dp_phi) den[j] = fmaf(f[j][k], dp_z[k], den[j]);
        }
      }
#pragma unroll
      for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int j = 0; j < RW; ++j) den[j] += __shfl_xor(den[j], off, kWave);
#pragma unroll
      for (int j = 0; j < RW; ++j) {
        if (mrow[j] >= s.M) continue;                    // wave-uniform
        bf16* frow = (bf16*)g.C + (size_t)mrow[j] * s.ldc + lane;
#pragma unroll
        for (int k = 0; k < DP_MAXK; ++k)
          if (k * 64 + lane < dp_phi) frow[k * 64] = (bf16)f[j][k];
        if (lane == 0) ((float*)g.C2)[mrow[j]] = 1.0f / (den[j] + s.fparam);
      }
      return;
    }
    // EPI_QKV_ROPE: the cos / sin pairs of all rows of the walk first (stores to C could alias the table as far as
    // the compiler knows, so loads placed between the stores would wait for one another)
    f32x4 rc0[EPI == EPI_QKV_ROPE ? ITER : 1], rc1[EPI == EPI_QKV_ROPE ? ITER : 1];
    if constexpr (EPI == EPI_QKV_ROPE) {
      const int hd = s.ldr >> 1, j = n % s.ldr;
#pragma unroll
      for (int it = 0; it < ITER; ++it) {
        const int sr = sr_first + it * (NT / C4);
        const int m = m_of(min(sr, NROWS - 1));
        rc0[it] = rc1[it] = f32x4{1.f, 0.f, 1.f, 0.f};
        if (sr < NROWS && m < s.M && n < s.n0 + s.n1 && n < s.N) {
          const float* cs = g.R + 2 * ((size_t)m * hd + (j - (j < hd ? 0 : hd)));
          rc0[it] = *(const f32x4*)cs;                   // c0 s0 c1 s1 | c2 s2 c3 s3
          rc1[it] = *(const f32x4*)(cs + 4);
        }
      }
    }
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
      const int sr = sr_first + it * (NT / C4);
      const int m = m_of(min(sr, NROWS - 1));
      const bool valid = sr < NROWS && m < s.M && n < s.N;
      f32x4 o = {0.f, 0.f, 0.f, 0.f};
      if (valid) {
        o = *(const f32x4*)(stg + sr * SLD + c4 * 4);
        if (EPI != EPI_SWIGLU) o *= row_scale(m);        // SwiGLU applied it before the nonlinearity
        if constexpr (EPI == EPI_QKV_ROPE) {
          if (n < s.n0 + s.n1) {
            // rotary embedding (rotate-half): column j of a head pairs with j +- dh/2, which lies in the same
            // staged row; out_j = x_j cos_j' - x_{j+h} sin_j' (j < h), x_j cos_j' + x_{j-h} sin_j' (j >= h), j' = j mod h
            const int dh = s.ldr, hd = dh >> 1, j = n % dh, lo = j < hd;
            const f32x4 p = *(const f32x4*)(stg + sr * SLD + c4 * 4 + (lo ? hd : -hd)) * row_scale(m);
            const f32x4 cs0 = rc0[it], cs1 = rc1[it];
            const float sg = lo ? -1.f : 1.f;
            o[0] = o[0] * cs0[0] + sg * p[0] * cs0[1];
            o[1] = o[1] * cs0[2] + sg * p[1] * cs0[3];
            o[2] = o[2] * cs1[0] + sg * p[2] * cs1[1];
            o[3] = o[3] * cs1[2] + sg * p[3] * cs1[3];
          }
        }
        if (EPI == EPI_RESID_F32) o += pre.r[it];        // zeros without a residual
        if (!vec_ok) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (n + e >= s.N) o[e] = 0.f;
        }
        bf16x4 ob, og;
#pragma unroll
        for (int e = 0; e < 4; ++e) ob[e] = (bf16)o[e];
        if (EPI == EPI_RESID_F32 && g.C2) {
          // with a gain the copy is the un-normalised input of the next RMSNorm: x * gain
#pragma unroll
          for (int e = 0; e < 4; ++e) og[e] = g.gain ? (bf16)(o[e] * gq[e]) : ob[e];
        }
        if (vec_ok) {
          if (EPI == EPI_STORE_ACT || EPI == EPI_SWIGLU || EPI == EPI_QKV_ROPE) {
            *(bf16x4*)((bf16*)g.C + (size_t)m * s.ldc + n) = ob;
          } else {
            *(f32x4*)((float*)g.C + (size_t)m * s.ldc + n) = o;
            if (EPI == EPI_RESID_F32 && g.C2) *(bf16x4*)((bf16*)g.C2 + (size_t)m * s.ldc2 + n) = og;
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (n + e >= s.N) continue;
            if (EPI == EPI_STORE_ACT || EPI == EPI_SWIGLU || EPI == EPI_QKV_ROPE) {
              ((bf16*)g.C)[(size_t)m * s.ldc + n + e] = ob[e];
            } else {
              ((float*)g.C)[(size_t)m * s.ldc + n + e] = o[e];
              if (EPI == EPI_RESID_F32 && g.C2) ((bf16*)g.C2)[(size_t)m * s.ldc2 + n + e] = og[e];
            }
          }
        }
      }
      if (EPI == EPI_RESID_F32 && g.ssq_out) {
        // sum of squares of this row for the RMSNorm that consumes the row: one partial per (row, 128 columns),
        // summed later in column order (deterministic, no atomics).  The granularity and the order of the additions
        // are fixed, not tied to the tile width, so that every tile configuration produces the same partials bit for bit.
        static_assert(EPI != EPI_RESID_F32 || BN_OUT % 128 == 0, "partials cover 128 columns = 32 lanes");
        const float part = sum32(o[0] * o[0] + o[1] * o[1] + o[2] * o[2] + o[3] * o[3]);
        if ((c4 & 31) == 0 && sr < NROWS && m < s.M && n < s.N)      // (a wide tile's columns past N: the next row's partial stands there)
          g.ssq_out[(size_t)m * ((s.N + 127) >> 7) + tn * (BN_OUT / 128) + (c4 >> 5)] = part;
      }
    }
  };
  // EPI_QKV_ROPE, tiles of the v columns: the attention kernel wants V transposed ([column][row], row stride ldc2),
  // so these tiles are drained column-wise: a thread takes 8 consecutive rows of one column, 16 bytes per store.
  const bool vt_tile = EPI == EPI_QKV_ROPE && s.ldc2 > 0 && n0 >= s.n0 + s.n1;      // block-uniform
  auto drain_vt = [&](const float* stg, int nrows, auto m_of) __attribute__((always_inline)) {
    bf16* vt = (bf16*)g.C2 + (size_t)(n0 - (s.n0 + s.n1)) * s.ldc2;
    for (int u = tid; u < (nrows >> 3) * BN_OUT; u += NT) {
      const int rg = u / BN_OUT, col = u - rg * BN_OUT;
      const int m = m_of(rg * 8);          // rows rg * 8 .. + 7 of the staging tile are consecutive output rows
      if (m >= s.M || n0 + col >= s.N) continue;
      bf16x8 v;
#pragma unroll
      for (int i = 0; i < 8; ++i)
        v[i] = (m + i < s.M) ? (bf16)(stg[(rg * 8 + i) * SLD + col] * row_scale(m + i)) : (bf16)0.f;
      *(bf16x8*)(vt + (size_t)col * s.ldc2 + m) = v;
    }
  };
  const int col_in = lane & 15;
  auto row_of_pass = [&](int pass) { return [=](int sr) { return m0 + (sr >> 4) * WROWS + pass * 16 + (sr & 15); }; };
  using AllRows = std::integral_constant<int, SR>;
  Pre pre;
#pragma unroll
  for (int pass = 0; pass < TM; ++pass) {        // a pass stages one 16-row block of every wave row
    float* stg = (float*)smem + (pass & 1) * STG_FLOATS;
    const auto pass_row = row_of_pass(pass);
    if (EPI == EPI_RESID_F32) prefetch(AllRows{}, pass_row, pre);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row16 = 4 * t_q + r;
      float* dst = stg + (wm * 16 + row16) * SLD + col_in;
      if (EPI == EPI_SWIGLU) {
        // the wave's weight rows come in 32-row blocks, gate / up alternating: tiles 4q + h (gate) and 4q + 2 + h
        // (up), h = 0, 1, give output columns (wn * WCOLS / 64 + q) * 32 + h * 16 + lane % 16
        const float rs = rs_lds[blk_row(pass) + row16];
#pragma unroll
        for (int j = 0; j < TN; ++j)
          if ((j & 2) == 0)
            dst[(wn * (WCOLS / 64) + (j >> 2)) * 32 + (j & 1) * 16] = silu_mul(rs * acc[pass][j][r], rs * acc[pass][j + 2][r]);
      } else {
#pragma unroll
        for (int j = 0; j < TN; ++j) dst[blk_col(j)] = acc[pass][j][r];
      }
    }
    __syncthreads();         // pass p is staged; everybody has left the walk of pass p - 1, whose tile pass p + 1 reuses
    if (vt_tile) drain_vt(stg, SR, pass_row);
    else drain(stg, AllRows{}, pass_row, pre);
  }
  if (TAIL && tail_blk) {     // 16x16 result tile: lane holds column lane % 16, rows 4*(lane/16) + r
    float* stg = (float*)smem + (TM & 1) * STG_FLOATS;
    auto tail_row = [&](int sr) { return m0_strip + sr; };
    if (EPI == EPI_RESID_F32) prefetch(std::integral_constant<int, 16>{}, tail_row, pre);
    if (tail) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float* dst = stg + (4 * t_q + r) * SLD;
        if (EPI == EPI_SWIGLU) {
          const float rs = rs_lds[BM + 4 * t_q + r];
          dst[(wave >> 1) * 32 + (wave & 1) * 16 + (lane & 15)] = silu_mul(rs * tacc[0][r], rs * tacc[1][r]);
        } else {
          dst[t_brow] = tacc[0][r];
          dst[t_brow + T_STEP] = tacc[1][r];
        }
      }
    }
    __syncthreads();
    if (vt_tile) drain_vt(stg, 16, tail_row);
    else drain(stg, std::integral_constant<int, 16>{}, tail_row, pre);
  }
#ifdef ARMT_GEMM_TIMELINE
  if (tl_on && threadIdx.x == 0) { tl[5] = __builtin_readcyclecounter(); tl[6] = __builtin_amdgcn_s_memrealtime(); }
#endif
}

// M-tiles of 256 rows, of which the last takes a strip of 16 rows behind it along (not with switch 32, as in the launches: a cut launch counts by both)
constexpr int mfma_m_tiles(const GemmShape& s) { return (s.M > 256 && s.M % 256 == 16 && !(s.dbg & 32)) ? s.M / 256 : (s.M + 255) / 256; }

// M-tiles (of 256 rows) that follow one another on a weight panel.  The 32 compute units of an XCD work on 32 consecutive
// tiles of the order: with 4 to 8 M-tiles side by side these touch 11 to 12 operand panels, with 32 of one weight panel
// 33 (a weight gradient of 8192 x 2048, or the head's).  Tall problems are cut into equal groups of at most 8: one product of
// 8192^3 1.24 -> 1.38 PFLOP/s, 8 weight gradients of 8192 x 2048 x 8704 1.13 -> 1.31.
constexpr int mfma_m_group(const GemmShape& s) {
  const int tm = mfma_m_tiles(s), n = (tm + 7) / 8;
  return (tm + n - 1) / n;
}

// Part of a launch's work, so that two tile sizes can share it: units [begin, end), a unit being the tiles of one M-group
// on one panel of unit_cols output columns, in the order of the tiles.  unit_cols = 0: everything.
struct TileRange { int unit_cols = 0, begin = 0, end = 0; };
constexpr int mfma_units(const GemmShape& s, int g, int panels) { return g * ((mfma_m_tiles(s) + mfma_m_group(s) - 1) / mfma_m_group(s)) * panels; }

// First tile of unit u (counted over the groups) for tiles of BM rows of which `tiles_m` cover M, m_group (of BM rows) and
// tiles_n N-tiles per group, cols_per_unit of them in a unit.
constexpr int mfma_unit_tile(int u, int tiles_m, int m_group, int tiles_n, int cols_per_unit) {
  const int panels = tiles_n / cols_per_unit, n_mg = (tiles_m + m_group - 1) / m_group;
  const int grp = u / (n_mg * panels), r = u % (n_mg * panels), mg = r / panels, p = r % panels;
  const int rows = tiles_m - mg * m_group < m_group ? tiles_m - mg * m_group : m_group;
  return grp * tiles_m * tiles_n + mg * m_group * tiles_n + p * cols_per_unit * rows;
}

template <int BM, int BN, int WGM, int WGN, bool REG, int EPI, bool TAIL, int NS>
inline hipError_t launch_mfma_tail(const GemmGroup* table, int first, int g, GemmShape s, hipStream_t st,
                                   const TileRange& rng) {
  constexpr int BN_OUT = (EPI == EPI_SWIGLU) ? BN / 2 : BN;
  constexpr int LDS = mfma_tile_lds_bytes<BM, BN, WGM, WGN, EPI, TAIL, NS>() + (BM + 16) * 4;
  const int tiles_m = TAIL ? s.M / BM : (s.M + BM - 1) / BM, tiles_n = (s.N + BN_OUT - 1) / BN_OUT;
  const int m_group = mfma_m_group(s) * 256 / BM;
  // the whole launch or, for a part of it, whole units
  int begin = 0, total = g * tiles_m * tiles_n;
  if (rng.unit_cols > 0) {
    begin = mfma_unit_tile(rng.begin, tiles_m, m_group, tiles_n, rng.unit_cols / BN_OUT);
    total = mfma_unit_tile(rng.end, tiles_m, m_group, tiles_n, rng.unit_cols / BN_OUT) - begin;
  }
  if (total <= 0) return hipSuccess;
  // Groups of unequal length (ranges of a reduction): a contiguous run of tiles per XCD would give some of them the long groups
  // only, so every XCD takes an eighth of each group.  (Groups of equal length keep an XCD's weights to themselves.)
  s.spread = s.spread && rng.unit_cols == 0 && tiles_m * tiles_n % 8 == 0;
  const int grid = ((total + 7) / 8) * 8;
  auto kern = gemm_mfma_kernel<BM, BN, WGM, WGN, REG, EPI, TAIL, NS>;
  static std::atomic<uint64_t> lds_raised{0};
  const hipError_t e = raise_lds_limit((const void*)kern, LDS, lds_raised);
  if (e != hipSuccess) return e;
#ifdef ARMT_GEMM_TIMELINE
  if (s.tag == g_tl_kind && g_tl_countdown >= 0 && g_tl_countdown-- == 0) {
    GemmShape s_tl = s;
    s_tl.dbg |= 1 << 20;
    kern<<<grid, WGM * WGN * 64, LDS, st>>>(table, first, s_tl, tiles_m, tiles_n, m_group, total, begin);
    return hipGetLastError();
  }
#endif
  kern<<<grid, WGM * WGN * 64, LDS, st>>>(table, first, s, tiles_m, tiles_n, m_group, total, begin);
  return hipGetLastError();
}

// Groups of one or two k-tiles, or some of them
constexpr bool tile256_short(const GemmShape& s) { return s.K < 3 * MF_BK || (s.k_slot > 0 && (s.k_min > 0 ? s.k_min : s.k_slot) < 3); }

// Shapes that the persistent 256 x 256 tile takes, of the regular ones: rows that can be stored in 16-byte pieces and reached by 32-bit offsets from a tile's
// first row, heads of 64 or 128 columns (a wave's columns hold whole ones).
template <int EPI>
constexpr bool tile256_shape(const GemmShape& s) {
  constexpr int LD = 1 << 21;
  if (s.K < MF_BK) return false;                            // a group without products is not stored
  if (((s.N | s.ldc | s.ldr | s.ldc2) & 3) != 0 || s.lda > LD || s.ldb > LD || s.ldc > LD || s.ldr > LD || s.ldc2 > LD) return false;
  if (EPI == EPI_QKV_ROPE && tile256_short(s)) return false;      // (none is regular: its first weight block has K columns)
  if (EPI == EPI_QKV_ROPE && s.ldc2 > 0 && s.M % 8 != 0) return false;      // V^T leaves in pieces of eight rows, of which it looks at the first
  return EPI != EPI_QKV_ROPE || s.ldr == 64 || s.ldr == 128;
}

template <int EPI>
inline hipError_t launch_tile256(const GemmGroup* table, int first, int g, GemmShape s, hipStream_t st, const TileRange& rng = TileRange()) {
  constexpr int BN_OUT = EPI == EPI_SWIGLU ? 128 : 256;
  const bool strip = s.M > 256 && s.M % 256 == 16 && !(s.dbg & 32);
  TileWalk w;
  w.tiles_m = strip ? s.M / 256 : (s.M + 255) / 256;
  w.tiles_n = s.N / BN_OUT;
  w.m_group = mfma_m_group(s);
  w.begin = 0;
  w.total = g * w.tiles_m * w.tiles_n;
  if (rng.unit_cols > 0) {
    w.begin = mfma_unit_tile(rng.begin, w.tiles_m, w.m_group, w.tiles_n, rng.unit_cols / BN_OUT);
    w.total = mfma_unit_tile(rng.end, w.tiles_m, w.m_group, w.tiles_n, rng.unit_cols / BN_OUT) - w.begin;
  }
  if (w.total <= 0) return hipSuccess;
  s.spread = s.spread && rng.unit_cols == 0 && w.tiles_m * w.tiles_n % 8 == 0;
  w.r_group = t256_recip(w.tiles_m * w.tiles_n);
  w.r_mgroup = t256_recip(w.m_group * w.tiles_n);
  w.r_full = t256_recip(w.m_group < w.tiles_m ? w.m_group : w.tiles_m);
  const int last_group = w.tiles_m - (w.tiles_m - 1) / w.m_group * w.m_group;      // M-tiles of the last M-group: two share the strip, where there are
  w.r_last = t256_recip(last_group);
  w.r_share = t256_recip(w.tiles_m * w.tiles_n / 8);
  const int grid = w.total < MF_CUS ? (w.total + 7) / 8 * 8 : MF_CUS;
  constexpr int HB = EPI == EPI_QKV_ROPE ? 2 : 0;
  const int tail = !strip ? 0 : last_group > 1 ? 1 : 2;
  typedef decltype(&gemm_tile256_kernel<EPI, false, HB>) Kernel;
  static const Kernel plain[3] = {gemm_tile256_kernel<EPI, false, HB>, gemm_tile256_kernel<EPI, true, HB>, gemm_tile272_kernel<EPI, HB>};
  Kernel kern = plain[tail];
  bool other = false;                                       // heads of 128 columns, or fewer than three k-tiles
  if constexpr (EPI == EPI_QKV_ROPE) {
    static const Kernel wide[3] = {gemm_tile256_kernel<EPI, false, 2 * HB>, gemm_tile256_kernel<EPI, true, 2 * HB>, gemm_tile272_kernel<EPI, 2 * HB>};
    if ((other = s.ldr == 128)) kern = wide[tail];
  } else {
    static const Kernel brief[3] = {gemm_short256_kernel<EPI, 0>, gemm_short256_kernel<EPI, 1>, gemm_short256_kernel<EPI, 2>};
    if ((other = tile256_short(s))) kern = brief[tail];
  }
  static std::atomic<uint64_t> lds_raised[2][3];
  const hipError_t e = raise_lds_limit((const void*)kern, T256_LDS, lds_raised[other][tail]);
  if (e != hipSuccess) return e;
#ifdef ARMT_GEMM_TIMELINE
  if (s.tag == g_tl_kind && g_tl_countdown >= 0 && g_tl_countdown-- == 0) s.dbg |= 1 << 20;
#endif
  kern<<<grid, 256, T256_LDS, st>>>(table, first, s, w);
  return hipGetLastError();
}

// M = tiles * BM + 16 (a cell: seg_len rows + 16 memory rows) takes the tail variant.
// shapes the copy-wave variant addresses with one lane offset per operand
template <int BM, int BN, int EPI>
constexpr bool mfma_regular_shape(const GemmShape& s) {
  constexpr int BN_OUT = (EPI == EPI_SWIGLU) ? BN / 2 : BN;
  const bool m_ok = s.M % BM == 0 || (s.M > BM && s.M % BM == 16 && !(s.dbg & 32)) || s.a_rows >= (s.M + BM - 1) / BM * BM;
  const int e0 = s.n0, e1 = s.n0 + s.n1;      // ends of weight blocks 0 and 1
  const bool w_ok = EPI == EPI_SWIGLU || ((e0 >= s.N || e0 % BN == 0) && (e1 >= s.N || e1 % BN == 0));
  return m_ok && s.N % BN_OUT == 0 && w_ok && s.K % MF_BK == 0;
}

template <int BM, int BN, int WGM, int WGN, int EPI, bool REG = false, int NS = 2>
inline hipError_t launch_mfma_cfg(const GemmGroup* table, int first, int g, const GemmShape& s, hipStream_t st,
                                  const TileRange& rng = TileRange()) {
  if constexpr (BN <= WGM * WGN * 32) {
    if (s.M > BM && s.M % BM == 16 && !(s.dbg & 32))
      return launch_mfma_tail<BM, BN, WGM, WGN, REG, EPI, true, NS>(table, first, g, s, st, rng);
  }
  return launch_mfma_tail<BM, BN, WGM, WGN, REG, EPI, false, NS>(table, first, g, s, st, rng);
}

// Big tiles move the fewest bytes per flop, but a launch needs about one tile per CU to use the chip: a single
// cell (sequential order, or the first and last steps of the diagonal order) has too few 256x256 tiles.
constexpr int mfma_pick_config(const GemmShape& s, int g, int force_cfg) {
  if (force_cfg >= 0 && force_cfg < MF_NUM_CONFIGS) return force_cfg;
  // a few rows against wide weights (W_K | W_V on the memory rows): the launch streams the weights once and is bound
  // by how many bytes a CU has in flight, so narrow tiles that give every CU two workgroups
  if (s.M <= 64 && s.epi == EPI_STORE_F32 && (long)g * ((s.N + 127) / 128) < 512) return 3;
  // W_Q of the read with the feature map as its epilogue: one d_mem-wide tile column, so the workgroups are the M-tiles;
  // 32-row tiles put two or more workgroups on a CU, whose waves then fill each other's waits
  if (s.epi == EPI_DPFP_READ && s.M >= 64 && (long)g * ((s.M + 63) / 64) < 1024) return 4;
  // Launches that leave a CU at most one workgroup wait for the latency of its copies: small tiles with a deep ring.
  // us per launch, two stages of 128 x 128 -> here (1040 rows): attention output (N = K = 2048) of one cell 30.4 -> 24.8, two cells
  // 36.4 -> 28.2; down (K = 8192) 108 -> 75, 112 -> 87; with more tiles than CUs the rings of four cost occupancy and
  // lose (down, three cells: 138 against 154 and 210)
  const auto tiles_of = [&](int bm) {
    const long tm = (s.M > bm && s.M % bm == 16) ? s.M / bm : (s.M + bm - 1) / bm, cols = s.epi == EPI_SWIGLU ? 64 : 128;
    return g * tm * ((s.N + cols - 1) / cols);
  };
  // (one or two k-tiles do not fill a ring: 64 x 1536, K 128 6.3 us with two stages, 6.7 with four, K 192 7.1 and 7.0, K 1024 14.6 and 11.7)
  if (s.epi != EPI_DPFP_READ && tiles_of(64) <= MF_CUS) return s.K > 2 * MF_BK ? 7 : 2;
  if (s.M < 96 || s.N < 96) return 2;
  if (s.epi != EPI_DPFP_READ && tiles_of(128) <= MF_CUS) return 8;
  // 128x128 tiles as long as all of them are on the chip at once, two workgroups per CU; us per launch, 256 x 256 / 128 x 128 (N = 256 ... 3072, K = 768 ...
  // 8192): 512 of them (4 x (1040 x 2048, K 2048)) 48.3 / 39.4, 486 ragged ones (135 of 256 x 256: 3 x (1100 x 2300, K 2048)) 47.6 / 41.6, 510 (5 x (2100 x 768),
  // K 768) 23.9 / 22.0, K 4096 78 / 71; 528 (11 x (1040 x 768), K 768) 24.4 / 28.6, K 3072 66.8 / 81.1, ragged (13 x (500 x 1280), K 1024) 28.0 / 35.6
  return (s.M >= 192 && s.N >= 192 && tiles_of(128) > 2 * MF_CUS) ? 5 : 6;
}

// Whole rounds of the chip with 256 x 256 tiles; if what is left fills at most half of another round, it runs as 128 x 128 tiles (four
// times as many, two workgroups per CU: one short round instead of a long one that leaves most CUs idle).  The units (TileRange) that keep
// 256 x 256 tiles, 0: all of them.  Both tile sizes give the same bits (same order of the k-steps, row sums of squares at a fixed
// granularity), so where the cut falls does not show in the result.  The kernel that takes the whole rounds has no say in it.  us per launch, one launch / cut:
// 9 x (1040 x 2048, K 8192) 360 / 318, K 2048 96 / 81, 12 x (1040 x 2048, K 8192) 386 / 362, 4352^3 173 / 150, 9 x (272 x 8192, K 2048) 120 / 107, 32 x (272 x
// 3072, K 2048) 135 / 133; with one or two k-tiles, where the second launch is most of the difference, 17.9 / 18.7 and (12 x (1040 x 3072)) 28.7 / 29.8.
template <int EPI>
constexpr int mfma_round_cut(const GemmShape& s, int g, int force_cfg) {
  if (EPI == EPI_SWIGLU || EPI == EPI_DPFP_READ || force_cfg >= 0 || s.spread || !mfma_regular_shape<256, 256, EPI>(s) ||
      !mfma_regular_shape<128, 128, EPI>(s))
    return 0;
  const int tm = mfma_m_tiles(s), mg = mfma_m_group(s), panels = s.N / 256, tiles = g * tm * panels, rem = tiles % MF_CUS;
  if (tiles <= MF_CUS || rem == 0 || rem > MF_CUS / 2) return 0;
  int cut = mfma_units(s, g, panels);                 // the last units that hold at least the tiles of the partial round
  while (cut > 0 && tiles - mfma_unit_tile(cut, tm, mg, panels, 1) < rem) --cut;
  return cut;
}

// Tile configuration by problem shape: big square tiles for the block's linears, small tiles for
// the skinny associative-memory projections (N = d_mem columns, or M = n_mem rows).
template <int EPI>
inline hipError_t launch_gemm_mfma_epi(const GemmGroup* table, int first, int g, const GemmShape& s, hipStream_t st,
                                       int force_cfg) {
  const int cfg = mfma_pick_config(s, g, force_cfg);
  switch (cfg) {
    case 1: return launch_mfma_cfg<128, 128, 2, 2, EPI>(table, first, g, s, st);
    case 3:   // 64 x 64: only instantiated for the plain fp32 store
      // four k-tiles in LDS: the loop of these small tiles is bound by the latency of a copy, not by its arithmetic
      // (eight do not pay, also not for at most one workgroup per CU: 12.0 us against 12.4 for one cell of d 2048, 20.6 / 19.4 for four of
      // 3072, 7.9 / 8.9 for twelve of 768)
      if constexpr (EPI == EPI_STORE_F32) return launch_mfma_cfg<64, 64, 2, 2, EPI, false, 4>(table, first, g, s, st);
      break;
    case 4:   // only instantiated for the feature-map epilogue of the W_Q projection
      // 32 x 64 where that holds all columns (d_mem 64): half of a 128-wide tile's copies and products would be of columns past d_mem.  Four waves of
      // 16 x 32, four k-tiles in LDS (two workgroups still fit on a CU; three lose what the tile gains, six 0 - 25 %); two waves of 32 x 32
      // and 64 x 64 tiles wait longer in the epilogue.  us per launch, 32 x 128 / 32 x 64 (means of a pass): 1B model, one cell 23.5 / 21.3,
      // 1 - 8 cells 29.7 / 23.5, 16 cells of 528 rows 31.7 / 25.4, twelve of width 768 18.6 / 17.4
      if constexpr (EPI == EPI_DPFP_READ) {
        // (narrower d_mem are not regular: these copies would read rows that the weight does not have)
        if (mfma_regular_shape<32, 64, EPI>(s) && s.N == 64) return launch_mfma_cfg<32, 64, 2, 2, EPI, true, 4>(table, first, g, s, st);
        // else 32 x 128, waves side by side, three k-tiles in LDS (two workgroups still fit on a CU)
        // (six do not pay, also not for at most one workgroup per CU: 25.7 us with either for one cell of d 2048)
        return launch_mfma_cfg<32, 128, 1, 4, EPI, false, 3>(table, first, g, s, st);
      }
      break;
    case 5:   // 256 x 256: the persistent tile of four waves (gemm_tile256.h), for other shapes 16 waves and one barrier per k-tile.  us per
              // launch of bf16 results, 16 waves / persistent: 12 x (1040 x 768, K 768) 27.8 / 25.6, K 3072 68.3 / 67.4 (at most one tile per CU), 12 x (1040 x
              // 6144, K 768) 140 / 114, 16 x (1040 x 3072, K 2048) 191 / 166, 16 x (1040 x 2048, K 8192) 453 / 437, 16 x (1040 x 16384, K 2048) 996 / 884,
              // 8192^3 831 / 713
      if constexpr (EPI != EPI_DPFP_READ) if (mfma_regular_shape<256, 256, EPI>(s)) {
        auto tiles_256 = [&](const TileRange& rng) {
          return tile256_shape<EPI>(s) ? launch_tile256<EPI>(table, first, g, s, st, rng) : launch_mfma_cfg<256, 256, 4, 4, EPI>(table, first, g, s, st, rng);
        };
        if constexpr (EPI != EPI_SWIGLU) {
          const int cut = mfma_round_cut<EPI>(s, g, force_cfg);
          if (cut > 0) {
            TileRange big, rest;
            big.unit_cols = rest.unit_cols = 256;
            big.begin = 0; big.end = rest.begin = cut; rest.end = mfma_units(s, g, s.N / 256);
            hipError_t e = tiles_256(big);
            if (e != hipSuccess) return e;
            return launch_mfma_cfg<128, 128, 4, 2, EPI, true>(table, first, g, s, st, rest);
          }
        }
        return tiles_256(TileRange());
      }
      return launch_mfma_cfg<256, 256, 4, 4, EPI>(table, first, g, s, st);
    case 6:   // as 1, copies addressed by scalar base + lane offset where the shape allows
      // Eight waves of 32 x 64 instead of four of 64 x 64: two workgroups of four waves leave a SIMD two waves, which wait for their
      // fragments together.  us per launch, four / eight: attention output and down of the 768-wide model (mean of its launches)
      // 49.5 / 44.3, QKV 25.0 / 21.6, gate/up of one cell 20.3 / 18.7; down of two and three cells of d 2048 109.6 / 104.0.
      // The feature map of d_mem 128 too, though eight waves keep 31 registers of it in scratch memory (3 without the strip): 64 cells of 1040 rows,
      // K 2048 130.3 / 117.0, 84 of K 3072 222.8 / 205.7, 16 of 4224 rows 157.1 / 143.2, 96 of K 768 106.5 / 104.3.
      // Irregular shapes keep four waves: only few launches of a model come here (timed: feature map of d_mem 96, 64 cells, K 2048 125.5 / 114.4).
      if (mfma_regular_shape<128, 128, EPI>(s)) return launch_mfma_cfg<128, 128, 4, 2, EPI, true>(table, first, g, s, st);
      return launch_mfma_cfg<128, 128, 2, 2, EPI>(table, first, g, s, st);
    case 7:   // at most one workgroup per CU: nobody else fills the waits for a copy, so four k-tiles in LDS
      // Nor for a fragment: eight waves of 32 x 32, two per SIMD, instead of four of 32 x 64 (SwiGLU needs these: whole gate/up pairs of
      // blocks).  One cell of 1040 rows, us per launch (read, attention output and down together): 39.2 -> 31.1; six k-tiles
      // 40.5 and 31.4, so it was the SIMD's one wave that waited and not the copies.
      if constexpr (EPI != EPI_DPFP_READ) {
        constexpr int WGN = EPI == EPI_SWIGLU ? 2 : 4;
        if (mfma_regular_shape<64, 128, EPI>(s)) return launch_mfma_cfg<64, 128, 2, WGN, EPI, true, 4>(table, first, g, s, st);
        return launch_mfma_cfg<64, 128, 2, WGN, EPI, false, 4>(table, first, g, s, st);
      }
      break;
    case 8:   // the same for 128 x 128 tiles: sixteen waves of 32 x 32 (SwiGLU eight of 32 x 64); sixteen against eight: QKV of one cell of d 2048
              // 27.2 -> 26.1 us, attention output of two 27.3 -> 25.9, of the 768-wide model 23.4 -> 22.2.  Over 226 shapes of 144 to 4224 rows, K 768 to 16384: residual
              // epilogue 0.95 of the time of eight with the strip, 0.91 without; plain store 1.00 (0.96 to 1.04: slower where the tiles fill the chip) and 0.96
      if constexpr (EPI != EPI_DPFP_READ) {
        constexpr int WGN = EPI == EPI_SWIGLU ? 2 : 4;
        if (mfma_regular_shape<128, 128, EPI>(s)) return launch_mfma_cfg<128, 128, 4, WGN, EPI, true, 4>(table, first, g, s, st);
        return launch_mfma_cfg<128, 128, 4, 2, EPI, false, 4>(table, first, g, s, st);
      }
      break;
    default: break;
  }
  return launch_mfma_cfg<64, 128, 2, 2, EPI>(table, first, g, s, st);
}

inline hipError_t launch_gemm_mfma(const GemmGroup* table, int first, int g, const GemmShape& s, hipStream_t st,
                                   int force_cfg = -1) {
  if (g <= 0 || s.M <= 0 || s.N <= 0) return hipSuccess;
  switch (s.epi) {
    case EPI_STORE_ACT: return launch_gemm_mfma_epi<EPI_STORE_ACT>(table, first, g, s, st, force_cfg);
    case EPI_STORE_F32: return launch_gemm_mfma_epi<EPI_STORE_F32>(table, first, g, s, st, force_cfg);
    case EPI_RESID_F32: return launch_gemm_mfma_epi<EPI_RESID_F32>(table, first, g, s, st, force_cfg);
    case EPI_SWIGLU: return launch_gemm_mfma_epi<EPI_SWIGLU>(table, first, g, s, st, force_cfg);
    case EPI_DPFP_READ:
      // all d_mem columns of a row in one output tile (the narrowest tile is 128 wide)
      if (s.N != s.n0 || s.N > 128 || s.ldr < 1 || s.ldc < 2 * s.ldr * s.n0 || 2 * s.ldr * s.n0 > 512) return hipErrorInvalidValue;
      return launch_gemm_mfma_epi<EPI_DPFP_READ>(table, first, g, s, st, force_cfg);
    case EPI_QKV_ROPE:
      // the rotation reads its partner column from the staged tile: heads must not straddle tiles (128 or 256 wide)
      if (s.ldr <= 0 || 128 % s.ldr != 0 || (s.N & 3) || (s.ldc & 3)) return hipErrorInvalidValue;
      return launch_gemm_mfma_epi<EPI_QKV_ROPE>(table, first, g, s, st, force_cfg);
  }
  return hipErrorInvalidValue;
}

}  // namespace armt
