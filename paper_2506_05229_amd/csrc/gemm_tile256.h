// The 256 x 256 tile of the grouped bf16 GEMM for regular shapes: four waves of 128 x 128, one per SIMD, one persistent workgroup per
// compute unit.  Included by gemm_mfma.h, whose configurations cover everything else.
//
// Loop.  A k-tile of 64 is two k-steps of 64 MFMAs per wave; while a step is multiplied, the 16 fragments of the next one are read
// into the other half of the fragment registers.  The fragments of a k-tile's second step are in registers a third into its first step: a barrier
// there frees the k-tile's LDS buffer, and the copies of the k-tile after next go out from then on, spread over the MFMAs.  (Packed more
// closely they hold the wave up, which has no second one beside it: 8192^3 1.01 PFLOP/s with a copy every third MFMA, 1.48 with
// every sixth.)  Four waves read 128 KB of LDS per k-tile where eight of 128 x 64 read 192.
// Tiles.  The copies run two k-tiles ahead through ALL tiles of the workgroup: the last two k-tiles of a tile fetch the first two of the next, whose
// start costs no latency, and the epilogue runs while they land: the LDS that it uses (T256_SSQ, T256_OUT) is none of theirs.
// Epilogue.  A 16 x 16 block is multiplied with the weights as first operand: a lane then holds four consecutive columns of one row.  Whole rows of
// 64 columns leave through LDS of the wave's own.  Buffer stores drop what lies past M.
#pragma once

#include "common.h"

namespace armt {

typedef float f32x4t __attribute__((ext_vector_type(4)));
typedef unsigned u32x2t __attribute__((ext_vector_type(2)));
typedef unsigned u32x4t __attribute__((ext_vector_type(4)));

// Order of the tiles of a launch (see gemm_mfma.h), with what the divisions by its constants need.
struct TileWalk {
  int total, begin, tiles_m, tiles_n, m_group;
  unsigned r_group, r_mgroup, r_full, r_last, r_share;      // t256_recip of tiles per group, per M-group, M-tiles of a full and of the last M-group, an XCD's share of a group
};

inline unsigned t256_recip(int d) { return d <= 1 ? 0xffffffffu : (unsigned)((1ull << 32) / (unsigned)d); }
// n / d for 0 <= n, r = t256_recip(d): the estimate is exact or one too small
__device__ __forceinline__ int t256_div(int n, int d, unsigned r) {
  const int q = (int)__umulhi((unsigned)n, r);
  return n - q * d >= d ? q + 1 : q;
}

// The pointer table and a group's range through the scalar cache, wherever in the kernel they are read (written by earlier launches only).
typedef const __attribute__((address_space(4))) GemmGroup* ConstGroups;
typedef const __attribute__((address_space(4))) int* ConstInts;

// Row scales and gains of products that have none: the epilogues read them without a branch (a load that the compiler sees in flight on one of two
// paths makes it wait for everything in the next tile's loop).
struct T256Ones {
  float f[256];
  bf16 h[256];
};
constexpr T256Ones t256_ones_value() {
  T256Ones o{};
  for (int i = 0; i < 256; ++i) { o.f[i] = 1.f; o.h[i] = (bf16)1.f; }
  return o;
}
static __device__ const T256Ones t256_ones = t256_ones_value();

// Cache policy of the result stores: nt, not kept in the L2.  A round of tiles writes as much as the L2 holds, and what it displaces are the
// operands of the next one.  us per launch, kept / not: gate/up of the 3B model 837 / 824, of twelve cells of width 768 96.8 / 94.3, fp32 results
// of 16 x (1024 x 2048, K 2048) 132 / 118, 8192^3 754 / 736
constexpr int T256_NT = 2;

constexpr int T256_STAGE = 65536;                             // a k-tile: 256 rows of A, 256 of B
constexpr int T256_STRIP = 2 * T256_STAGE;                    // two buffers of the 16 strip rows
constexpr int T256_SSQ = T256_STRIP + 2 * 2048;               // sums of squares: [half][wave column][256], strip [half][wave][16]
constexpr int T256_OUT = T256_SSQ + 4 * 256 * 4 + 2 * 4 * 16 * 4;      // results on their way out: 4 KB per wave
constexpr int T256_LDS = T256_OUT + 4 * 4096;

// TAIL: 16 rows behind the last M-tile, the strip.  1: the last M-tile and the one in front of it compute it, half of the columns each.  2: the
// last M-group has one M-tile only (cells of 256 + 16 rows), which computes both halves: 8 of 136 products a wave and k-tile.  us per launch, 16 waves / so:
// 16 x (272 x 8192, K 2048) 157 / 145, 24 x (272 x 2048, K 2048) 61.9 / 53.8, 32 x (272 x 2048, K 8192) 291 / 276, 1 x (14608 x 2048, K 2048)
// 102.5 / 97.3, gate/up of four cells of the 1B model 79.0 / 76.6; its pass over 48 segments 40.1 / 38.6 ms.
// HB: EPI_QKV_ROPE, blocks of 16 columns in half a head (2 or 4), otherwise 0
// SHORT: tiles of any number of k-tiles.  Otherwise they have three at least, and the copies, two k-tiles ahead, never more than one tile; what it takes to follow
// them over more costs long products 0.2 - 0.5 % (their registers for scalars are all in use).  us per launch, 16 waves / so: the read of 16 cells of 1040 x 2048 with 64
// features 58.5 / 52, with 128 60.4 / 54.5, 16 x (1024 x 8192, K 64) 76.5 / 59, K 128 93 / 66, the head's weight gradient over 124 rows (46027 x 768) 56 / 53.5.
template <int EPI, int TAIL, int HB, bool SHORT>
__device__ __forceinline__ void tile256(const GemmGroup* __restrict__ table_g, int first, const GemmShape& s, const TileWalk& w) {
  constexpr bool ROPE = EPI == EPI_QKV_ROPE, GLU = EPI == EPI_SWIGLU, RESID = EPI == EPI_RESID_F32;
  constexpr int ROWB = 128, BN_OUT = GLU ? 128 : 256;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, t_q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int xcd = blockIdx.x & 7, stride = gridDim.x >> 3, per_xcd = (w.total + 7) >> 3, per_group = w.tiles_m * w.tiles_n;
  const int m0_strip = w.tiles_m * 256;
  const ConstGroups table = (ConstGroups)table_g + first;

  struct Tile { int r, grp, m0, n0, nk, half; };               // half: first of the strip's halves that it computes; -1 none
  // first tile of this workgroup's sequence from number r on that has something to do; r = -1: none
  auto tile_from = [&](int r) __attribute__((always_inline)) {
    Tile t{-1, 0, 0, 0, 0, -1};
    for (;; r += stride) {
      int lid = xcd * per_xcd + r;
      if (r >= per_xcd || lid >= w.total) return t;
      if (s.spread) {                                          // every group spread over all XCDs
        const int share = per_group >> 3, i = t256_div(r, share, w.r_share);
        lid = i * per_group + xcd * share + (r - i * share);
      } else {
        lid += w.begin;
      }
      t.grp = t256_div(lid, per_group, w.r_group);
      int rem = lid - t.grp * per_group, mg0 = 0, mg_tiles = w.tiles_m;
      unsigned recip = w.r_full;
      if (w.m_group < w.tiles_m) {
        const int mg = t256_div(rem, w.m_group * w.tiles_n, w.r_mgroup);
        mg0 = mg * w.m_group;
        rem -= mg0 * w.tiles_n;
        if (w.tiles_m - mg0 < w.m_group) { mg_tiles = w.tiles_m - mg0; recip = w.r_last; } else mg_tiles = w.m_group;
      }
      const int tn = t256_div(rem, mg_tiles, recip), tm = mg0 + rem - tn * mg_tiles, from_end = w.tiles_m - 1 - tm;
      const ConstInts range = (ConstInts)table[t.grp].krange;
      t.nk = (range ? range[1] * s.k_slot : s.K / MF_BK);
      if (t.nk <= 0) continue;
      t.m0 = tm * 256; t.n0 = tn * BN_OUT; t.r = r;
      t.half = from_end < (TAIL == 1 ? 2 : TAIL == 2) ? from_end : -1;
      return t;
    }
  };

  // ---- copies: cursor over the k-tiles of all tiles.  Slab wave + 4 j (8 rows) of an operand: base of its half, lane offset j & 3
  const char *cA0, *cA1, *cB0, *cB1, *cT;
  int c_left = 1, c_step = ROWB;
  int before_ct = -1;                                          // SHORT: number of the tile in front of the cursor's
  Tile ct{(int)(blockIdx.x >> 3) - stride, 0, 0, 0, 0, -1};
  auto advance = [&]() __attribute__((always_inline)) {
    if (--c_left > 0) {
      cA0 += c_step; cA1 += c_step; cB0 += c_step; cB1 += c_step; cT += c_step;
      return;
    }
    const Tile t = tile_from(ct.r + stride);
    if (SHORT) before_ct = ct.r;
    if (t.r < 0) { c_left = 0x7fffffff; c_step = 0; ct.r = -1; return; }      // behind the last k-tile: that one again (nobody reads it)
    ct = t;
    c_left = t.nk;
    const auto& g = table[t.grp];
    const size_t skip = g.krange ? (size_t)((ConstInts)g.krange)[0] * s.k_slot * ROWB : 0;
    const char* a = (const char*)g.A + skip;
    cA0 = a + (size_t)t.m0 * s.lda * 2;
    cA1 = cA0 + (size_t)128 * s.lda * 2;
    cT = a + (size_t)m0_strip * s.lda * 2;
    const char* b = (const char*)g.B0 + skip;
    if (GLU) {                                                 // lower half of the rows from the gate, upper half from the up weight
      cB0 = b + (size_t)t.n0 * s.ldb * 2;
      cB1 = (const char*)g.B1 + (size_t)t.n0 * s.ldb * 2;
    } else {                                                   // weight blocks end on tiles
      int n = t.n0;
      if (n >= s.n0) { n -= s.n0; b = (const char*)g.B1; if (n >= s.n1) { n -= s.n1; b = (const char*)g.B2; } }
      cB0 = b + (size_t)n * s.ldb * 2;
      cB1 = cB0 + (size_t)128 * s.ldb * 2;
    }
  };
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)smem;
  unsigned vA[4], vB[4];
  {
    const int row = 8 * wave + (lane >> 3), chunk = ((lane & 7) ^ mf_swz(row & 15)) << 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      vA[j] = (unsigned)(row + 32 * j) * (unsigned)s.lda * 2u + chunk;
      vB[j] = (unsigned)(row + 32 * j) * (unsigned)s.ldb * 2u + chunk;
    }
  }
  auto copy = [&](int buf, int c) __attribute__((always_inline)) {
    const int j = c >> 1;
    const unsigned at = lds0 + buf * T256_STAGE + (wave + 4 * j) * 1024;
    if ((c & 1) == 0) lds_copy16(j < 4 ? cA0 : cA1, vA[j & 3], at);
    else lds_copy16(j < 4 ? cB0 : cB1, vB[j & 3], at + 32768);
  };
  auto copy_strip = [&](int buf) __attribute__((always_inline)) {
    if (TAIL && ct.half >= 0 && wave < 2) lds_copy16(cT, vA[0], lds0 + T256_STRIP + buf * 2048 + wave * 1024);
  };

  // ---- fragments.  x: operand whose index goes into the registers of a result block (the weights), y: into its lanes (rows of A); V
  // tiles of the QKV projection the other way round.  Blocks of 16 of a wave: x in column wave & 1, y in row wave >> 1.
  const int wy = wave >> 1, wx = wave & 1;
  auto at16 = [&](int wv, int i) { return ROPE ? wv * 128 + i * 16 : (i >> 2) * 128 + wv * 64 + (i & 3) * 16; };
  int koff[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) koff[ks] = ((4 * ks + t_q) ^ mf_swz(l16)) << 4;
  bf16x8 fx[2][8], fy[2][8];
  f32x4t acc[8][8], tacc[TAIL == 2 ? 2 : 1][2];
  auto transposed = [&](const Tile& t) { return ROPE && s.ldc2 > 0 && t.n0 >= s.n0 + s.n1; };      // V tile
  Tile tile{-1, 0, 0, 0, 0, -1};                               // the one that is multiplied
  int x_base, y_base;
  auto orient = [&](bool vt) {
    x_base = (vt ? 0 : 32768) + (at16(wx, 0) + l16) * ROWB;
    y_base = (vt ? 32768 : 0) + (at16(wy, 0) + l16) * ROWB;
  };
  auto read = [&](int buf, int ks, int q, int xb, int yb) __attribute__((always_inline)) {
    const unsigned char* p = smem + buf * T256_STAGE + koff[ks];
    const int i = q >> 1, at = (at16(0, i) - at16(0, 0)) * ROWB;
    if (q < 16 && (q & 1) == 0) fx[ks][i] = *(const bf16x8*)(p + xb + at);
    else fy[ks][i] = *(const bf16x8*)(p + yb + at);
  };
  // Strip: a wave computes two blocks of a half, 16 rows x 16 columns at tile rows (of the weights) strip_row(h, 0) and (h, 1): 32
  // neighbouring columns, the two that a rotation mixes, or the gate and the up projection of the same columns.  The fragments are read again
  // (an address costs nothing, a choice of registers a branch), the products written as instructions: the accumulators fill one half of the register
  // file, and the compiler does not mix the halves.  It does not look into the text for hazards either: two wait states behind a vector
  // write of an operand, eleven in front of a vector read of a result.
  auto strip_row = [&](const Tile& t, int b) {
    if (GLU) return b * 128 + t.half * 64 + wave * 16;
    if (ROPE && !transposed(t)) return t.half * 128 + (HB == 2 ? (wave >> 1) * 64 + (wave & 1) * 16 + b * 32 : wave * 16 + b * 64);
    return t.half * 128 + wave * 32 + b * 16;
  };
  constexpr int HALF = GLU ? 64 : 128;                        // rows of the weights between the halves
  auto strip_half = [&](int buf, int r0, int r1, bool vt, f32x4t (&tacc)[2]) __attribute__((always_inline)) {
    const unsigned char* pt = smem + T256_STRIP + buf * 2048 + l16 * ROWB;
    const unsigned char* pb = smem + buf * T256_STAGE + 32768 + l16 * ROWB;
    const bf16x8 a0 = *(const bf16x8*)(pt + koff[0]), a1 = *(const bf16x8*)(pt + koff[1]);
    const bf16x8 b0 = *(const bf16x8*)(pb + r0 * ROWB + koff[0]), c0 = *(const bf16x8*)(pb + r1 * ROWB + koff[0]);
    const bf16x8 b1 = *(const bf16x8*)(pb + r0 * ROWB + koff[1]), c1 = *(const bf16x8*)(pb + r1 * ROWB + koff[1]);
    if (ROPE && vt)
      asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %2, %4, %0\n\tv_mfma_f32_16x16x32_bf16 %1, %2, %5, %1\n\t"
                   "v_mfma_f32_16x16x32_bf16 %0, %3, %6, %0\n\tv_mfma_f32_16x16x32_bf16 %1, %3, %7, %1\n\ts_nop 10"
                   : "+v"(tacc[0]), "+v"(tacc[1]) : "v"(a0), "v"(a1), "v"(b0), "v"(c0), "v"(b1), "v"(c1));
    else
      asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %4, %2, %0\n\tv_mfma_f32_16x16x32_bf16 %1, %5, %2, %1\n\t"
                   "v_mfma_f32_16x16x32_bf16 %0, %6, %3, %0\n\tv_mfma_f32_16x16x32_bf16 %1, %7, %3, %1\n\ts_nop 10"
                   : "+v"(tacc[0]), "+v"(tacc[1]) : "v"(a0), "v"(a1), "v"(b0), "v"(c0), "v"(b1), "v"(c1));
  };
  auto strip = [&](int buf, int r0, int r1, bool vt) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < TAIL; ++h) strip_half(buf, r0 + h * HALF, r1 + h * HALF, vt, tacc[h]);
  };
  // A product, its accumulator held in the accumulation half of the register file: left to choose, the compiler moves accumulators and fragments
  // between the halves in the middle of the loop.  (The fragments are LDS reads, which it waits for; the accumulators are written and read by others only
  // in the epilogue, behind the wait states in front of it.)
  auto mul = [&](f32x4t& c, const bf16x8& a, const bf16x8& b) __attribute__((always_inline)) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
  };
  // ... the first one of a tile
  auto mul0 = [&](f32x4t& c, const bf16x8& a, const bf16x8& b) __attribute__((always_inline)) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(c) : "v"(a), "v"(b));
  };
  auto barrier = [&]() __attribute__((always_inline)) {
    asm volatile("s_barrier" : : : "memory");
    __builtin_amdgcn_sched_barrier(0);
  };

  constexpr int NC = 16;
  constexpr int QB = 16 + 4, CS = 7, C0 = (63 - QB) / CS, CS1 = 64 / (NC - C0);     // copies: C0 in the first step, the others in the second
  static_assert(C0 < NC && 64 / CS1 + C0 >= NC, "every copy has its MFMA");
  // memory instructions that every wave issues in an epilogue, at least: the copies in front of it may be that many further down the queue
  constexpr int E = GLU ? 16 : RESID || EPI == EPI_STORE_F32 ? 63 : 32;
  // ---- first two k-tiles
#pragma unroll 1
  for (int p = -1; p < 2; ++p) {
    if (p >= 0) {
#pragma unroll
      for (int c = 0; c < NC; ++c) copy(p, c);
      copy_strip(p);
    }
    advance();
    if (p < 0) {
      if (ct.r < 0) return;
      tile = ct;
    }
  }
  orient(transposed(tile));
  mf_wait_vmcnt<NC>();
  barrier();
#pragma unroll
  for (int q = 0; q < 16; ++q) read(0, 0, q, x_base, y_base);
  int buf = 0;
#pragma unroll
  for (int q = 0; q < 64; ++q) mul0(acc[q >> 3][q & 7], fx[0][q & 7], fy[0][q >> 3]);
  int behind_epilogue = 0;

  for (;;) {
    const bool vt = transposed(tile);
#ifdef ARMT_GEMM_TIMELINE
    const bool tl_on = (s.dbg >> 20) & 1;
    unsigned long long* tl = armt_timeline + 8 * (size_t)((xcd * per_xcd + tile.r) & 65535);
    if (tl_on && tid == 0) {
      unsigned hw, xcc;
      asm volatile("s_getreg_b32 %0, hwreg(HW_REG_HW_ID)" : "=s"(hw));
      asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
      tl[0] = ((unsigned long long)xcc << 32) | hw;
      tl[1] = __builtin_amdgcn_s_memrealtime();
      tl[2] = tl[3] = __builtin_readcyclecounter();
    }
#endif
#pragma unroll
    for (int t = 0; t < 2 * TAIL; ++t) tacc[t >> 1][t & 1] = f32x4t{0.f, 0.f, 0.f, 0.f};
    const int r0 = strip_row(tile, 0), r1 = strip_row(tile, 1);
    int left = tile.nk;
    int next = -1;                                             // SHORT: number of the tile behind this one, -1 none
    // second step of a k-tile, with the last N copies of the one after next
    auto second_step = [&](auto n_c) __attribute__((always_inline)) {
      constexpr int N = decltype(n_c)::value, GAP = 64 / N;
      if (ROPE && left == 1) orient(transposed(ct));             // the cursor stands in the next tile
      if (SHORT && left == 1) next = before_ct == tile.r ? ct.r : before_ct;      // ... or, if that has one k-tile, in the one behind it
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < 64; ++q) {
        mul(acc[q >> 3][q & 7], fx[1][q & 7], fy[1][q >> 3]);
        if (q < 16) read(buf ^ 1, 0, q, x_base, y_base);
        if (q % GAP == GAP - 1 && q / GAP < N) copy(buf, q / GAP + NC - N);
        __builtin_amdgcn_sched_barrier(0);
      }
      copy_strip(buf);
      advance();
      buf ^= 1;
    };
    // First k-tile: the products of its first step are done (in the prologue, or under the epilogue of the tile before).
#pragma unroll
    for (int q = 0; q < 16; ++q) read(buf, 1, q, x_base, y_base);
    if (TAIL && tile.half >= 0) strip(buf, r0, r1, vt);
    __builtin_amdgcn_s_waitcnt(0xC07F);                        // lgkmcnt(0): the buffer has been read
    // the next k-tile has landed (its copies were issued in front of the epilogue)
    asm volatile("s_cmp_lg_u32 %0, 0\n\ts_cbranch_scc1 .Lt256_%=\n\ts_waitcnt vmcnt(0)\n.Lt256_%=:\n\ts_waitcnt vmcnt(%1)\n\ts_barrier"
                 : : "s"(behind_epilogue), "n"(E) : "memory", "scc");
    __builtin_amdgcn_sched_barrier(0);
    second_step(std::integral_constant<int, NC>{});
    while (--left > 0) {
#pragma unroll
      for (int q = 0; q < 64; ++q) {
        mul(acc[q >> 3][q & 7], fx[0][q & 7], fy[0][q >> 3]);
        if (q < 16) read(buf, 1, q, x_base, y_base);
        if (TAIL && q == 16 && tile.half >= 0) strip(buf, r0, r1, vt);
        if (q == QB) {                                         // the buffer has been read
          __builtin_amdgcn_s_waitcnt(0xC07F);                  // lgkmcnt(0)
          asm volatile("s_barrier" : : : "memory");
        } else if (q > QB && (q - QB) % CS == 0) {
          copy(buf, (q - QB) / CS - 1);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" : : "n"(C0) : "memory");       // the next k-tile has landed
      __builtin_amdgcn_sched_barrier(0);
      second_step(std::integral_constant<int, NC - C0>{});
    }
    asm volatile("s_nop 15" : : : "memory");
    __builtin_amdgcn_sched_barrier(0);

    // ---- epilogue of `tile`
    TL_STAMP(4);
    // (opaque copies: what the epilogue derives from them is not kept in registers through the loop)
    int lane_e = lane, ldc = s.ldc, ldc2 = s.ldc2, ldr = s.ldr;
    asm volatile("" : "+v"(lane_e));
    asm volatile("" : "+s"(ldc));
    asm volatile("" : "+s"(ldc2));
    asm volatile("" : "+s"(ldr));
    const int l16 = lane_e & 15, t_q = lane_e >> 4;
    const auto& g = table[tile.grp];
    const int rows = min(256, s.M - tile.m0);                  // rows of the tile that exist
    auto rsrc = [&](const void* p, size_t bytes) __attribute__((always_inline)) {
      return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)(unsigned)(bytes > 0xfffffffcu ? 0xfffffffcu : bytes), 0x00027000);
    };
    auto pack = [](float a, float b) __attribute__((always_inline)) {
      typedef bf16 bf16x2 __attribute__((ext_vector_type(2)));
      const bf16x2 v = {(bf16)a, (bf16)b};
      return __builtin_bit_cast(unsigned, v);
    };
    // Results leave through 4 KB of LDS per wave (no barrier: a wave's LDS accesses run in order).  A result block has neighbouring lanes in different
    // rows, and the memory pipe takes four neighbouring lanes at a time, at a quarter of its rate if their 16 bytes are not neighbours.  us per launch, straight
    // from the registers / this way: attention output, down and read 275 / 267 (3B model), 60.8 / 57.0 (768-wide), QKV 50.0 / 48.5,
    // the head on 4096 rows 1817 / 1751, its weight gradient 1955 / 1890; gate/up 0.5 % slower.  The 16-byte chunks of a row are exchanged (XOR) so that neither side meets a bank twice.
    unsigned char* out_lds = smem + T256_OUT + wave * 4096;
    const int r8 = lane_e >> 3, c8 = lane_e & 7, r4 = t_q, c4 = l16;       // row and 16-byte column of a lane in rows of 128, of 256 bytes
    // 16 rows x 64 columns in bf16; back: rows 8 k + r8, columns 8 c8 .. + 7
    auto put16 = [&](int half, const f32x4t (&v)[4]) __attribute__((always_inline)) {
#pragma unroll
      for (int x = 0; x < 4; ++x)
        *(u32x2t*)(out_lds + half * 2048 + l16 * 128 + (((2 * x + (t_q >> 1)) ^ (l16 >> 1)) << 4) + (t_q & 1) * 8) = u32x2t{pack(v[x][0], v[x][1]), pack(v[x][2], v[x][3])};
    };
    auto get16 = [&](int half, u32x4t (&r)[2]) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < 2; ++k) r[k] = *(const u32x4t*)(out_lds + half * 2048 + (8 * k + r8) * 128 + ((c8 ^ (((8 * k + r8) >> 1) & 7)) << 4));
    };
    // 16 rows x 64 columns in fp32; back: rows 4 k + r4, columns 4 c4 .. + 3
    auto put32 = [&](const f32x4t (&v)[4]) __attribute__((always_inline)) {
#pragma unroll
      for (int x = 0; x < 4; ++x) *(f32x4t*)(out_lds + l16 * 256 + (((4 * x + t_q) ^ l16) << 4)) = v[x];
    };
    auto get32 = [&](f32x4t (&r)[4]) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < 4; ++k) r[k] = *(const f32x4t*)(out_lds + (4 * k + r4) * 256 + ((c4 ^ (4 * k + r4)) << 4));
    };
    // N pieces of 16 x 64: piece i + 1 is made while piece i comes back from LDS
    auto out16 = [&](auto n_c, auto make, auto store) __attribute__((always_inline)) {
      constexpr int N = decltype(n_c)::value;
      u32x4t r[2][2];
#pragma unroll
      for (int i = 0; i <= N; ++i) {
        if (i < N) {
          f32x4t v[4];
          make(i, v);
          put16(i & 1, v);
        }
        if (i > 0) store(i - 1, r[(i - 1) & 1]);
        if (i < N) get16(i & 1, r[i & 1]);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    auto out32 = [&](auto n_c, auto make, auto store) __attribute__((always_inline)) {
      constexpr int N = decltype(n_c)::value;
      f32x4t r[2][4];
#pragma unroll
      for (int i = 0; i <= N; ++i) {
        if (i < N) {
          f32x4t v[4];
          make(i, v);
          put32(v);
        }
        if (i > 0) store(i - 1, r[(i - 1) & 1]);
        if (i < N) get32(r[i & 1]);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // First products of the next tile, whose first fragments are in registers, on accumulators that have been taken (behind the last tile nobody reads
    // them): the matrix pipe has nothing else to do here, and the accumulators need no zeros.  us per launch, without / with: attention output, down
    // and read 258.7 / 255.7 (3B model), 117.5 / 115.2 (1B), gate/up 805 / 794, 311 / 304.
    auto next_products = [&](int y, int x0, int n) __attribute__((always_inline)) {
#pragma unroll
      for (int x = 0; x < 8; ++x)
        if (x >= x0 && x < x0 + n) mul0(acc[y][x], fx[0][x], fy[0][y]);
    };
    using N8 = std::integral_constant<int, 8>;
    using N16 = std::integral_constant<int, 16>;
    auto take = [&](int y, int x) __attribute__((always_inline)) {       // a result block; next_products overwrites its accumulators
      f32x4t v;
      // (where it is needed: the compiler would copy them all out at the end of the loop)
      asm volatile("v_accvgpr_read_b32 %0, %4\n\tv_accvgpr_read_b32 %1, %5\n\tv_accvgpr_read_b32 %2, %6\n\tv_accvgpr_read_b32 %3, %7"
                   : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
                   : "a"(acc[y][x][0]), "a"(acc[y][x][1]), "a"(acc[y][x][2]), "a"(acc[y][x][3]));
      return v;
    };
    const float* scales = g.rowscale ? g.rowscale + tile.m0 : t256_ones.f;
    auto scale_rsrc = rsrc(scales, (size_t)rows * 4);
    // (requested one row block ahead: more than 63 memory instructions between a load and its use, and the compiler waits for it in the loop)
    auto scale_of = [&](int y) __attribute__((always_inline)) {
      return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(scale_rsrc, (at16(wy, y) + l16) * 4, 0, 0));
    };
    auto strip_scale = [&]() { return g.rowscale ? g.rowscale[m0_strip + l16] : 1.f; };
    auto silu_mul = [](float gt, float up) { return gt * __builtin_amdgcn_rcpf(1.f + __expf(-gt)) * up; };

    if (vt) {
      // columns n0 + .. of the V block transposed: C2[column][row], eight rows of a column per lane (M is a multiple of 8: tile256_shape)
      bf16* out = (bf16*)g.C2 + (size_t)(tile.n0 - (s.n0 + s.n1)) * ldc2 + tile.m0;
      auto o = rsrc(out, (size_t)256 * ldc2 * 2);
      f32x4t rs[8];
#pragma unroll
      for (int x = 0; x < 8; ++x) {
        rs[x] = __builtin_bit_cast(f32x4t, __builtin_amdgcn_raw_buffer_load_b128(scale_rsrc, (at16(wx, x) + 4 * t_q) * 4, 0, 0));
      }
      out16(N16{}, [&](int i, f32x4t (&v)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < 4; ++x) v[x] = take(i >> 1, 4 * (i & 1) + x) * rs[4 * (i & 1) + x];
      }, [&](int i, const u32x4t (&r)[2]) __attribute__((always_inline)) {
        const int m = at16(wx, 4 * (i & 1)) + 8 * c8;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const unsigned off = ((unsigned)(at16(wy, i >> 1) + 8 * k + r8) * (unsigned)ldc2 + m) * 2u;
          __builtin_amdgcn_raw_buffer_store_b128(r[k], o, m < rows ? off : 0xfffffff0u, 0, T256_NT);
        }
      });
      if (TAIL && tile.half >= 0) {
        bf16* ts = (bf16*)g.C2 + (size_t)(tile.n0 - (s.n0 + s.n1) + r0 + l16) * ldc2 + m0_strip + 4 * t_q;
        f32x4t r = {1.f, 1.f, 1.f, 1.f};
        if (g.rowscale) r = *(const f32x4t*)(g.rowscale + m0_strip + 4 * t_q);
#pragma unroll
        for (int t = 0; t < 2 * TAIL; ++t) {
          const f32x4t v = tacc[t >> 1][t & 1] * r;
          *(u32x2t*)(ts + (size_t)((t >> 1) * HALF + (t & 1) * 16) * ldc2) = u32x2t{pack(v[0], v[1]), pack(v[2], v[3])};
        }
      }
    } else if constexpr (GLU) {
      auto o = rsrc((bf16*)g.C + (size_t)tile.m0 * ldc, (size_t)rows * ldc * 2);
      float rs[8];
      rs[0] = scale_of(0);
      out16(N8{}, [&](int y, f32x4t (&v)[4]) __attribute__((always_inline)) {
        if (y < 7) rs[y + 1] = scale_of(y + 1);
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const f32x4t gt = take(y, x), up = take(y, x + 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[x][e] = silu_mul(rs[y] * gt[e], rs[y] * up[e]);
        }
        next_products(y, 0, 8);
      }, [&](int y, const u32x4t (&r)[2]) __attribute__((always_inline)) {
        const unsigned at = (unsigned)(at16(wy, y) + r8) * (unsigned)ldc + tile.n0 + wx * 64 + 8 * c8;
        __builtin_amdgcn_raw_buffer_store_b128(r[0], o, at * 2u, 0, T256_NT);
        __builtin_amdgcn_raw_buffer_store_b128(r[1], o, (at + 8 * ldc) * 2u, 0, T256_NT);
      });
      if (TAIL && tile.half >= 0) {
        const float r = strip_scale();
#pragma unroll
        for (int h = 0; h < TAIL; ++h) {
          f32x4t v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = silu_mul(r * tacc[h][0][e], r * tacc[h][1][e]);
          *(u32x2t*)((bf16*)g.C + (size_t)(m0_strip + l16) * ldc + tile.n0 + r0 + h * HALF + 4 * t_q) = u32x2t{pack(v[0], v[1]), pack(v[2], v[3])};
        }
      }
    } else {
      float rs[8];
      if constexpr (!ROPE && !RESID) rs[0] = scale_of(0);
      auto scaled = [&](int i, f32x4t (&v)[4]) __attribute__((always_inline)) {       // half h = i & 1 of row block y = i >> 1
        const int y = i >> 1, h = i & 1;
        if (h == 0 && y < 7) rs[y + 1] = scale_of(y + 1);
#pragma unroll
        for (int x = 0; x < 4; ++x) v[x] = take(y, 4 * h + x) * rs[y];
        next_products(y, 4 * h, 4);
      };
      if constexpr (EPI == EPI_STORE_ACT) {
        auto o = rsrc((bf16*)g.C + (size_t)tile.m0 * ldc, (size_t)rows * ldc * 2);
        out16(N16{}, scaled, [&](int i, const u32x4t (&r)[2]) __attribute__((always_inline)) {
          const unsigned at = (unsigned)(at16(wy, i >> 1) + r8) * (unsigned)ldc + tile.n0 + at16(wx, 4 * (i & 1)) + 8 * c8;
          __builtin_amdgcn_raw_buffer_store_b128(r[0], o, at * 2u, 0, T256_NT);
          __builtin_amdgcn_raw_buffer_store_b128(r[1], o, (at + 8 * ldc) * 2u, 0, T256_NT);
        });
        if (TAIL && tile.half >= 0) {
          const float r = strip_scale();
          bf16* out = (bf16*)g.C + (size_t)(m0_strip + l16) * ldc + tile.n0 + r0 + 4 * t_q;
#pragma unroll
          for (int t = 0; t < 2 * TAIL; ++t) {
            const f32x4t v = tacc[t >> 1][t & 1] * r;
            *(u32x2t*)(out + (t >> 1) * HALF + (t & 1) * 16) = u32x2t{pack(v[0], v[1]), pack(v[2], v[3])};
          }
        }
      } else if constexpr (EPI == EPI_STORE_F32) {
        auto o = rsrc((float*)g.C + (size_t)tile.m0 * ldc, (size_t)rows * ldc * 4);
        out32(N16{}, scaled, [&](int i, const f32x4t (&r)[4]) __attribute__((always_inline)) {
          const unsigned at = (unsigned)(at16(wy, i >> 1) + r4) * (unsigned)ldc + tile.n0 + at16(wx, 4 * (i & 1)) + 4 * c4;
#pragma unroll
          for (int k = 0; k < 4; ++k) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4t, r[k]), o, (at + 4 * k * ldc) * 4u, 0, T256_NT);
        });
        if (TAIL && tile.half >= 0) {
          const float r = strip_scale();
          float* out = (float*)g.C + (size_t)(m0_strip + l16) * ldc + tile.n0 + r0 + 4 * t_q;
#pragma unroll
          for (int t = 0; t < 2 * TAIL; ++t) *(f32x4t*)(out + (t >> 1) * HALF + (t & 1) * 16) = tacc[t >> 1][t & 1] * r;
        }
      } else if constexpr (RESID) {
        float* part = (float*)(smem + T256_SSQ);
        auto o = rsrc((float*)g.C + (size_t)tile.m0 * ldc, (size_t)rows * ldc * 4);
        auto res = rsrc(g.R ? g.R + (size_t)tile.m0 * ldr : nullptr, g.R ? (size_t)rows * ldr * 4 : 0);      // none: reads zeros
        auto o2 = rsrc(g.C2 ? (bf16*)g.C2 + (size_t)tile.m0 * ldc2 : nullptr, g.C2 ? (size_t)rows * ldc2 * 2 : 0);
        const int nc = tile.n0 + 4 * t_q;
        const bool copied = g.C2 != nullptr, summed = g.ssq_out != nullptr;
        const bf16* gains = copied && g.gain ? (const bf16*)g.gain + tile.n0 : t256_ones.h;
        auto gain_rsrc = rsrc(gains, 512);
        bf16x4 gq[2];                                          // gains of the copy, columns of half h
#pragma unroll
        for (int h = 0; h < 2; ++h) gq[h] = __builtin_bit_cast(bf16x4, __builtin_amdgcn_raw_buffer_load_b64(gain_rsrc, (at16(wx, 4 * h) + 4 * c4) * 2, 0, 0));
        // residual rows, requested AHEAD pieces in front of the one that is made, which is one in front of the one that uses them, and their scales
        constexpr int AHEAD = 2, RING = AHEAD + 2;
        f32x4t pre[RING][4];
        float rr[3][4];
        auto request = [&](int i) __attribute__((always_inline)) {
          const unsigned at = (unsigned)(at16(wy, i >> 1) + r4) * (unsigned)ldr + tile.n0 + at16(wx, 4 * (i & 1)) + 4 * c4;
#pragma unroll
          for (int k = 0; k < 4; ++k) pre[i % RING][k] = __builtin_bit_cast(f32x4t, __builtin_amdgcn_raw_buffer_load_b128(res, (at + 4 * k * ldr) * 4u, 0, 0));
        };
        auto row_scales = [&](int y) __attribute__((always_inline)) {
#pragma unroll
          for (int k = 0; k < 4; ++k)
            rr[y % 3][k] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(scale_rsrc, (at16(wy, y) + 4 * k + r4) * 4, 0, 0));
        };
        // sum over the 16 lanes of a row: the columns of its half in the order of the tiles' other sums (gemm_mfma.h)
        auto sum16 = [](float v) __attribute__((always_inline)) {
          auto dpp = [](float x, auto ctrl) {
            return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value, 0xF, 0xF, true));
          };
          v += dpp(v, std::integral_constant<int, 0xB1>{});
          v += dpp(v, std::integral_constant<int, 0x4E>{});
          v += dpp(v, std::integral_constant<int, 0x141>{});
          v += dpp(v, std::integral_constant<int, 0x140>{});
          return v;
        };
        // sums over the four lane rows of 16 columns, over the blocks in column order: lane row t_q first holds the sum of block t_q
        auto sum64 = [&](const float (&p)[4]) __attribute__((always_inline)) {
          auto fold16 = [](float a, float b) __attribute__((always_inline)) {
            const u32x2t r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
            return __uint_as_float(r[0]) + __uint_as_float(r[1]);
          };
          auto fold32 = [](float a, float b) __attribute__((always_inline)) {
            const u32x2t r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
            return __uint_as_float(r[0]) + __uint_as_float(r[1]);
          };
          const float q = fold32(fold16(p[0], p[1]), fold16(p[2], p[3]));
          const float h = fold16(q, q);
          return fold32(h, h);
        };
        auto ssq4 = [](f32x4t v) { return v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3]; };
        row_scales(0);
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) request(i);
        out32(N16{}, [&](int i, f32x4t (&v)[4]) __attribute__((always_inline)) {
          if ((i & 1) == 0 && i < 14) row_scales((i >> 1) + 1);
          if (i + AHEAD < 16) request(i + AHEAD);
#pragma unroll
          for (int x = 0; x < 4; ++x) v[x] = take(i >> 1, 4 * (i & 1) + x);
          next_products(i >> 1, 4 * (i & 1), 4);
        }, [&](int i, const f32x4t (&r)[4]) __attribute__((always_inline)) {
          const int y = i >> 1, h = i & 1;
          const unsigned row = (unsigned)(at16(wy, y) + r4), col = tile.n0 + at16(wx, 4 * h) + 4 * c4;
          f32x4t v[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[k][e] = fmaf(r[k][e], rr[y % 3][k], pre[i % RING][k][e]);
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4t, v[k]), o, ((row + 4 * k) * (unsigned)ldc + col) * 4u, 0, T256_NT);
          }
          if (copied) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              f32x4t c = v[k];
#pragma unroll
              for (int e = 0; e < 4; ++e) c[e] *= (float)gq[h][e];
              __builtin_amdgcn_raw_buffer_store_b64(u32x2t{pack(c[0], c[1]), pack(c[2], c[3])}, o2, ((row + 4 * k) * (unsigned)ldc2 + col) * 2u, 0, T256_NT);
            }
          }
          if (summed) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const float sum = sum16(ssq4(v[k]));
              if (c4 == 0) part[(h * 2 + wx) * 256 + row + 4 * k] = sum;
            }
          }
        });
        float* tpart = part + 4 * 256;
        if (TAIL && tile.half >= 0) {
          const float r = strip_scale();
          const size_t m = m0_strip + l16;
#pragma unroll
          for (int h = 0; h < TAIL; ++h) {
            float q[2];
#pragma unroll
            for (int b = 0; b < 2; ++b) {
              const int n = nc + r0 + h * HALF + 16 * b;
              f32x4t v = {0.f, 0.f, 0.f, 0.f};
              if (g.R) v = *(const f32x4t*)(g.R + m * ldr + n);
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] = fmaf(tacc[h][b][e], r, v[e]);
              *(f32x4t*)((float*)g.C + m * ldc + n) = v;
              if (copied) {
                f32x4t c = v;
                if (g.gain) {
                  const bf16x4 gb = *(const bf16x4*)((const bf16*)g.gain + n);
#pragma unroll
                  for (int e = 0; e < 4; ++e) c[e] = v[e] * (float)gb[e];
                }
                *(u32x2t*)((bf16*)g.C2 + m * ldc2 + n) = u32x2t{pack(c[0], c[1]), pack(c[2], c[3])};
              }
              q[b] = ssq4(v);
            }
            if (summed) {
              const float z4[4] = {q[0], q[1], 0.f, 0.f};        // (+ 0 leaves the bits of a sum of squares)
              const float sum = sum64(z4);
              if (t_q == 0) tpart[h * 64 + wave * 16 + l16] = sum;
            }
          }
        }
        if (summed) {
          __builtin_amdgcn_s_waitcnt(0xC07F);
          barrier();
          const int parts = (s.N + 127) >> 7;
          if (tid < rows) {
#pragma unroll
            for (int h = 0; h < 2; ++h) g.ssq_out[(size_t)(tile.m0 + tid) * parts + (tile.n0 >> 7) + h] = part[h * 2 * 256 + tid] + part[(h * 2 + 1) * 256 + tid];
          }
          if (TAIL && tid < 16 && tile.half >= 0) {
#pragma unroll
            for (int h = 0; h < TAIL; ++h) {
              const float* p = tpart + h * 64 + tid;
              g.ssq_out[(size_t)(m0_strip + tid) * parts + (tile.n0 >> 7) + tile.half + h] = (p[0] + p[16]) + (p[32] + p[48]);
            }
          }
        }
      } else if constexpr (ROPE) {
        auto o = rsrc((bf16*)g.C + (size_t)tile.m0 * ldc, (size_t)rows * ldc * 2);
        const int col = tile.n0 + at16(wx, 0);                 // a wave's 128 columns hold whole heads
        // blocks x and x + HB of a head of 32 HB columns: out_j = x_j cos - x_{j+h} sin, out_{j+h} = x_{j+h} cos + x_j sin
        auto rotate = [&](f32x4t& a, f32x4t& b, f32x4t c0, f32x4t c1) __attribute__((always_inline)) {
          const f32x4t p = a, q = b;
          const f32x4t c = {c0[0], c0[2], c1[0], c1[2]}, n = {c0[1], c0[3], c1[1], c1[3]};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            a[e] = fmaf(p[e], c[e], -(q[e] * n[e]));           // (contracted as in the walk of gemm_mfma.h: the same bits)
            b[e] = fmaf(q[e], c[e], p[e] * n[e]);
          }
        };
        constexpr int DH = 32 * HB;
        const bool turn = tile.n0 < s.n0 + s.n1;               // q or k columns (weight blocks end on tiles)
        {
          auto cs = rsrc(g.R + (size_t)tile.m0 * DH, (size_t)rows * DH * 4);
          rs[0] = scale_of(0);
          f32x4t c[2][HB][2];                                  // table entries of a row block, requested one ahead
          auto entries = [&](int y) __attribute__((always_inline)) {
            const unsigned at = ((unsigned)(at16(wy, y) + l16) * (DH / 2) + 4 * t_q) * 8u;
#pragma unroll
            for (int k = 0; k < HB; ++k)
#pragma unroll
              for (int e = 0; e < 2; ++e) c[y & 1][k][e] = __builtin_bit_cast(f32x4t, __builtin_amdgcn_raw_buffer_load_b128(cs, at + 128 * k + 16 * e, 0, 0));
          };
          entries(0);
          f32x4t v[8];
          out16(N16{}, [&](int i, f32x4t (&out)[4]) __attribute__((always_inline)) {
            const int y = i >> 1, h = i & 1;
            if (h == 0) {
              if (y < 7) { rs[y + 1] = scale_of(y + 1); entries(y + 1); }
#pragma unroll
              for (int x = 0; x < 8; ++x) v[x] = take(y, x) * rs[y];
              if (turn) {
#pragma unroll
                for (int k = 0; k < HB; ++k)
#pragma unroll
                  for (int x = k; x < 8; x += 2 * HB) rotate(v[x], v[x + HB], c[y & 1][k][0], c[y & 1][k][1]);
              }
            }
#pragma unroll
            for (int x = 0; x < 4; ++x) out[x] = v[4 * h + x];
          }, [&](int i, const u32x4t (&r)[2]) __attribute__((always_inline)) {
            const unsigned at = (unsigned)(at16(wy, i >> 1) + r8) * (unsigned)ldc + col + 64 * (i & 1) + 8 * c8;
            __builtin_amdgcn_raw_buffer_store_b128(r[0], o, at * 2u, 0, T256_NT);
            __builtin_amdgcn_raw_buffer_store_b128(r[1], o, (at + 8 * ldc) * 2u, 0, T256_NT);
          });
          if (TAIL && tile.half >= 0) {
            const float r = strip_scale();
            const size_t m = m0_strip + l16;
#pragma unroll
            for (int h = 0; h < TAIL; ++h) {
              f32x4t a = tacc[h][0] * r, b = tacc[h][1] * r;
              if (turn) {
                const float* t = g.R + 2 * (m * (DH / 2) + r0 % DH + 4 * t_q);      // (a half holds whole heads)
                rotate(a, b, *(const f32x4t*)t, *(const f32x4t*)(t + 4));
              }
              bf16* out = (bf16*)g.C + m * ldc + tile.n0 + r0 + h * HALF + 4 * t_q;
              *(u32x2t*)out = u32x2t{pack(a[0], a[1]), pack(a[2], a[3])};
              *(u32x2t*)(out + HB * 16) = u32x2t{pack(b[0], b[1]), pack(b[2], b[3])};
            }
          }
        }
      }
    }
    if constexpr (ROPE) {                                      // behind both kinds of tiles: accumulators written on either way cost copies
#pragma unroll
      for (int y = 0; y < 8; ++y) next_products(y, 0, 8);
    }
    TL_STAMP(5);
#ifdef ARMT_GEMM_TIMELINE
    if (tl_on && tid == 0) tl[6] = __builtin_amdgcn_s_memrealtime();
#endif
    if (SHORT) {
      if (next < 0) break;
      tile = next == ct.r ? ct : tile_from(next);
    } else {
      if (ct.r < 0) break;
      tile = ct;                                               // (at its third k-tile)
    }
    behind_epilogue = 1;
  }
  mf_wait_vmcnt<0>();                                          // the copies behind the last k-tile write LDS of this workgroup
}

template <int EPI, bool TAIL, int HB>
__global__ __launch_bounds__(256) void gemm_tile256_kernel(const GemmGroup* __restrict__ table, int first, GemmShape s, TileWalk w) {
  tile256<EPI, TAIL, HB, false>(table, first, s, w);
}
// TAIL 2
template <int EPI, int HB>
__global__ __launch_bounds__(256) void gemm_tile272_kernel(const GemmGroup* __restrict__ table, int first, GemmShape s, TileWalk w) {
  tile256<EPI, 2, HB, false>(table, first, s, w);
}
template <int EPI, int TAIL>
__global__ __launch_bounds__(256) void gemm_short256_kernel(const GemmGroup* __restrict__ table, int first, GemmShape s, TileWalk w) {
  tile256<EPI, TAIL, 0, true>(table, first, s, w);
}

}  // namespace armt
