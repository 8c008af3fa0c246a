// Register-window x pass of the row-lane refocus (the first of its two sums,
//     T(plane, y_b, y, x_r) = sum over x_b of  wx0 * view(y, xc) + wx1 * view(y, xc + 1),
// see kernels_refocus_rows.hip for the decomposition and the fold).
//
// What bounds it: two multiply-adds per (plane, x_r, view row, x_b) on the
// vector ALUs (no packed FP32): 7 ms at Da 256 x 256, Db 128 x 128 and 128
// planes if nothing else were issued and every row and column were needed (of
// which the skipped ones leave 6.0).
// The LDS-tap form (k_ref_rows) reads 16 bytes per lane, pair and view from
// LDS instead; there the LDS sets the pace.
//
// Here a wave keeps the view's window in registers.  Lanes are view rows (two
// per lane), so a pair's column cell is the same for every lane and a tap is
// a register whose number is uniform: the VGPR index mode (s_set_gpr_idx_*)
// adds the cell's column to the number of the window's first register.  The
// weights come from one lane of each row of 16 by DPP: a DPP multiply-add in
// index mode issues as fast as a plain one (measured: 256 of them 1193 clocks
// against 1173, two waves per SIMD).  So a pair costs four multiply-adds and
// one scalar instruction, and no LDS read.  Weights as scalar operands were
// slower: streamed through the scalar cache they arrive at one 64-byte line
// in about 38 clocks per CU.  The cells do come that way: a scalar register
// holds two, as M0 takes them, so that a pair's index is one scalar move.
//
// LDS only hands the window over: a work-group (four waves, 256 (plane,
// column) pairs, 128 view rows) copies the union of its waves' windows there
// directly from memory, each wave reads its own columns once per view, and
// from then on that LDS space is free for a later view, whose copy flies
// during the multiply-adds.
//
// Split: 64 pairs x 2 rows of sums, 40 columns x 2 rows of window, the weights
// and about 30 others fit the 256 registers of two waves per SIMD, and two
// work-groups' 80 KB of LDS a CU, so that one's hand-over overlaps the other's
// multiply-adds.  View rows are taken in units of 64 from the first row that
// the planes sample (planes with |alpha| < 1 sample only part of a view), and
// 16-pair chunks whose samples all fall outside the view are skipped.
//
// Measured, x pass and whole refocus: Da 256 x 256, Db 128 x 128, 128 planes
// 18.8 -> 11.1 ms and 20.1 -> 12.4 ms; Da 128 x 128, Db 64 x 64, 32 planes 0.465 ->
// 0.24 ms and 0.470 -> 0.28 ms; results bit-identical to k_ref_rows.  What is left
// (large size, by the counters): the vector ALUs are busy 57% of the time, 95% of
// that with multiply-adds (6.0 ms); 0.59 scalar and 0.12 other instructions go
// with each multiply-add, two waves per SIMD overlap them only in part, and the
// waves wait for memory or a barrier in a quarter of their cycles.  No LDS bank
// conflicts; Gamma is fetched 15 times (65 GB), T written once.  Raising the
// priority of waves that multiply (the other wave of the SIMD fills their gaps)
// gave 2%, whole-line copies of 32 columns nothing, and reading the next window
// under the multiply-adds, into the half of the registers that a narrow one
// leaves, nothing.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.h"
#include "refocus_common.h"

namespace cpi {

namespace {

constexpr int kWinWaveWords = 176;   // table words per wave and view
static_assert(kWinWaveWords * 4 <= 12 * kWinPairs, "plan_refocus reserves 12 bytes per pair");
constexpr int kWinTabBytes = kWinWaves * 512;   // of which the weights are staged in LDS
constexpr int kWinMaxGroups = 64;    // plane groups per chunk (256 planes in groups of 4 or more)

// Column cells of every pair of work-group (group gq, tile t) against
// lens-plane column x_b.  Wave w of the work-group owns NP planes x XC
// columns (64 pairs, wave (w / CG, w % CG) of the PG x CG arrangement).  Its
// table:
//   words 0 .. 63 and 64 .. 127: weights w0 and w1, pair 16 k + i at word
//     4 i + k (lane i of every row of 16 lanes reads the pairs it broadcasts);
//   words 128 .. 159: 16 bits per pair, what the VGPR index mode takes from M0:
//     its cell's column in the wave's window, and the bit that puts the index on
//     the second operand;
//   words 160 .. 164: where the wave's first four 4-column chunks start in the
//     staged window (window_pack_chunks; to be exchanged (xor) with the lane's offset);
//     its number of chunks and, from bit 8, one bit per 16 pairs with a nonzero
//     weight; the work-group's first staged column (a multiple of 4) and number
//     of 16-column blocks staged;
//   words 165 and 166: the last two of view x_b + ahead (no blocks if there is
//     none).
// Pairs past the planes or columns, or whose taps fall outside the view, have
// zero weights.  One block per (gq, t, x_b).
template <int NP, int XC, int PG>
__global__ __launch_bounds__(256) void k_window_xtab(GeomI g, const int32_t* __restrict__ itab,
                                                     const float* __restrict__ ftab,
                                                     int64_t stride, int first, int count,
                                                     int tiles, int max_blocks, int ahead,
                                                     int32_t* __restrict__ xe) {
  constexpr int CG = kWinWaves / PG;
  const int64_t idx = blockIdx.x;
  const int xb = int(idx % g.wb);
  const int t = int((idx / g.wb) % tiles);
  const int gq = int(idx / (int64_t(g.wb) * tiles));
  const int wv = threadIdx.x >> 6, k = threadIdx.x & 63;
  const int pl = (gq * PG + wv / CG) * NP + k / XC;
  const int xr = (t * CG + wv % CG) * XC + k % XC;
  int c = 0;
  float w0 = 0.0f, w1 = 0.0f;
  if (pl < count && xr < g.out_w) {
    const int32_t* it = itab + int64_t(first + pl) * stride;
    const float* ft = ftab + int64_t(first + pl) * stride;
    const int e_bx = g.out_w + g.out_h;
    int x0 = it[xr] + it[e_bx + xb];
    float fx = ft[xr] + ft[e_bx + xb];
    if (fx >= 1.0f) {
      x0 += 1;
      fx -= 1.0f;
    }
    clamp_cell(x0, fx, g.wa, c, w0, w1);
  }
  const bool live = w0 != 0.0f || w1 != 0.0f;
  const uint64_t lives = __ballot(live);
  int lo = live ? c : 1 << 30, hi = live ? c : -1;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lo = min(lo, __shfl_xor(lo, o, 64));
    hi = max(hi, __shfl_xor(hi, o, 64));
  }
  __shared__ int slo[kWinWaves], shi[kWinWaves];
  if (k == 0) {
    slo[wv] = lo;
    shi[wv] = hi;
  }
  __syncthreads();
  int glo = slo[0], ghi = shi[0];
#pragma unroll
  for (int i = 1; i < kWinWaves; ++i) {
    glo = min(glo, slo[i]);
    ghi = max(ghi, shi[i]);
  }
  const int wx0 = ghi < 0 ? 0 : glo & ~3;
  // columns wx0 .. ghi + 1 are staged, in blocks of 16; the host's bounds keep
  // them and every wave's chunks within the LDS and the registers, the
  // clamps keep every access there regardless
  const int blocks = ghi < 0 ? 0 : min((ghi + 1 - wx0) / 16 + 1, max_blocks);
  const int q0 = lives ? min((lo - wx0) >> 2, 4 * blocks - 1) : 0;
  const int nq =
      lives ? min(min(((hi + 1 - wx0) >> 2) - q0 + 1, kWinCols / 4), 4 * blocks - q0) : 0;
  const int rel = live ? min(c - wx0 - 4 * q0, kWinCols - 2) : 0;
  constexpr int kStep = kWinWaves * kWinWaveWords;   // words per view
  int32_t* e = xe + (idx * kWinWaves + wv) * kWinWaveWords;
  const int slot = 4 * (k % 16) + k / 16;
  e[slot] = __builtin_bit_cast(int32_t, w0);
  e[64 + slot] = __builtin_bit_cast(int32_t, w1);
  reinterpret_cast<uint16_t*>(e + 128)[k] = uint16_t(0x2000 | rel);
  if (k == 0) {
    int bits = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) bits |= ((lives >> (16 * j)) & 0xffffu) ? 1 << j : 0;
    const int xa = int(window_pack_chunks(q0)), xc = int(window_pack_chunks(q0 + 2));
    const int nl = nq | bits << 8;
    e[160] = xa;
    e[161] = xc;
    e[162] = nl;
    e[163] = wx0;
    e[164] = blocks;
    if (xb >= ahead) {
      int32_t* b = e - ahead * kStep;
      b[165] = wx0;
      b[166] = blocks;
    }
    if (xb + ahead >= g.wb) e[165] = e[166] = 0;
  }
}

// ---- one view of a wave, as one block of assembly --------------------------
// The window lives in registers that only this block touches (40 for each of
// the lane's two rows, from v168 and v208), and so do the weights (v248 .. v251
// and v252 .. v255): the block has to hold all of a view's work.  That is the
// barrier after which the view's copies are in LDS and every wave has read the
// view before it, the wave's reads of its window and weights, the copies of a
// later view into the LDS space of the one before (a second barrier before
// them where there is only one space), and the multiply-adds.  The cells come
// through the scalar cache meanwhile, the next view's last words during the
// multiply-adds.

// waits until at most n copies of this wave are in flight: ever fewer, until
// n allows as many
#define CPI_WIN_WAIT(k)            \
  "s_waitcnt vmcnt(" #k ")\n"      \
  "s_cmp_ge_u32 %[fly], " #k "\n"  \
  "s_cbranch_scc1 Lwait%=\n"
#define CPI_WIN_WAITS                                                                     \
  CPI_WIN_WAIT(9) CPI_WIN_WAIT(7) CPI_WIN_WAIT(5) CPI_WIN_WAIT(3) CPI_WIN_WAIT(1)         \
  "s_waitcnt vmcnt(0)\n"                                                                  \
  "Lwait%=:\n"

// chunk i of the window (4 columns) for both rows, skipped past the wave's
// chunks
#define CPI_WIN_READ(i, a, v0, o0, v1, o1)             \
  "s_cmp_le_u32 %[nq], " #i "\n"                       \
  "s_cbranch_scc1 Lread%=\n"                           \
  "ds_read_b128 " v0 ", %[a" #a "] offset:" #o0 "\n"   \
  "ds_read_b128 " v1 ", %[a" #a "] offset:" #o1 "\n"
#define CPI_WIN_READS \
  CPI_WIN_READ(0, 0, "v[168:171]", 0, "v[208:211]", 4096) \
  CPI_WIN_READ(1, 1, "v[172:175]", 0, "v[212:215]", 4096) \
  CPI_WIN_READ(2, 2, "v[176:179]", 0, "v[216:219]", 4096) \
  CPI_WIN_READ(3, 3, "v[180:183]", 0, "v[220:223]", 4096) \
  CPI_WIN_READ(4, 0, "v[184:187]", 8192, "v[224:227]", 12288) \
  CPI_WIN_READ(5, 1, "v[188:191]", 8192, "v[228:231]", 12288) \
  CPI_WIN_READ(6, 2, "v[192:195]", 8192, "v[232:235]", 12288) \
  CPI_WIN_READ(7, 3, "v[196:199]", 8192, "v[236:239]", 12288) \
  CPI_WIN_READ(8, 0, "v[200:203]", 16384, "v[240:243]", 20480) \
  CPI_WIN_READ(9, 1, "v[204:207]", 16384, "v[244:247]", 20480)

// copies of 16-column block i of the wave's 32 rows, skipped past the staged
// blocks.  The LDS address is M0 plus the instruction's offset (64 i), so M0
// holds 8192 i less that.
#define CPI_WIN_COPY(i, o)                                              \
  "s_cmp_le_u32 %[nb], " #i "\n"                                        \
  "s_cbranch_scc1 Lcopy%=\n"                                            \
  "s_add_u32 m0, %[dst], 8128*" #i "\n"                                 \
  "s_nop 0\n"                                                           \
  "buffer_load_dwordx4 %[from], %[rs], 0 offen offset:" #o " lds\n"     \
  "s_add_u32 m0, %[dst], 8128*" #i "+1024\n"                            \
  "s_nop 0\n"                                                           \
  "buffer_load_dwordx4 %[from1], %[rs], 0 offen offset:" #o " lds\n"
#define CPI_WIN_COPIES \
  CPI_WIN_COPY(0, 0) \
  CPI_WIN_COPY(1, 64) \
  CPI_WIN_COPY(2, 128) \
  CPI_WIN_COPY(3, 192) \
  CPI_WIN_COPY(4, 256) \
  CPI_WIN_COPY(5, 320) \
  CPI_WIN_COPY(6, 384) \
  CPI_WIN_COPY(7, 448) \
  CPI_WIN_COPY(8, 512)

// the wave's weights of the same view: 512 bytes, by 32 lanes
#define CPI_WIN_TABLE                        \
  "s_mov_b32 m0, %[td]\n"                    \
  "s_mov_b32 exec_hi, 0\n"                   \
  "s_nop 0\n"                                \
  "global_load_lds_dwordx4 %[tl], %[tp]\n"   \
  "s_mov_b32 exec_hi, -1\n"

// one pair: the sums of its two rows; lane i of every row of 16 lanes hands
// its weights to the row (DPP), which costs a multiply-add nothing.
#define CPI_WIN_DPP(a, w, v, i) \
  "v_fmac_f32_dpp %" #a ", " #w ", " #v " row_newbcast:" #i " row_mask:0xf bank_mask:0xf\n"
#define CPI_WIN_PAIR(x, y, a, b, i)                              \
  CPI_WIN_DPP(a, x, v168, i)   CPI_WIN_DPP(b, x, v208, i)        \
  CPI_WIN_DPP(a, y, v169, i) CPI_WIN_DPP(b, y, v209, i)
// two pairs whose cells are the 16-bit halves of register c
#define CPI_WIN_TWO(c, x, y, a0, b0, i0, a1, b1, i1)                  \
  "s_mov_b32 m0, " #c "\n" CPI_WIN_PAIR(x, y, a0, b0, i0)             \
  "s_lshr_b32 m0, " #c ", 16\n" CPI_WIN_PAIR(x, y, a1, b1, i1)
#define CPI_WIN_CHUNK0 \
  CPI_WIN_TWO(s36, v248, v252, 0, 64, 0, 1, 65, 1) \
  CPI_WIN_TWO(s37, v248, v252, 2, 66, 2, 3, 67, 3) \
  CPI_WIN_TWO(s38, v248, v252, 4, 68, 4, 5, 69, 5) \
  CPI_WIN_TWO(s39, v248, v252, 6, 70, 6, 7, 71, 7) \
  CPI_WIN_TWO(s40, v248, v252, 8, 72, 8, 9, 73, 9) \
  CPI_WIN_TWO(s41, v248, v252, 10, 74, 10, 11, 75, 11) \
  CPI_WIN_TWO(s42, v248, v252, 12, 76, 12, 13, 77, 13) \
  CPI_WIN_TWO(s43, v248, v252, 14, 78, 14, 15, 79, 15)
#define CPI_WIN_CHUNK1 \
  CPI_WIN_TWO(s44, v249, v253, 16, 80, 0, 17, 81, 1) \
  CPI_WIN_TWO(s45, v249, v253, 18, 82, 2, 19, 83, 3) \
  CPI_WIN_TWO(s46, v249, v253, 20, 84, 4, 21, 85, 5) \
  CPI_WIN_TWO(s47, v249, v253, 22, 86, 6, 23, 87, 7) \
  CPI_WIN_TWO(s48, v249, v253, 24, 88, 8, 25, 89, 9) \
  CPI_WIN_TWO(s49, v249, v253, 26, 90, 10, 27, 91, 11) \
  CPI_WIN_TWO(s50, v249, v253, 28, 92, 12, 29, 93, 13) \
  CPI_WIN_TWO(s51, v249, v253, 30, 94, 14, 31, 95, 15)
#define CPI_WIN_CHUNK2 \
  CPI_WIN_TWO(s52, v250, v254, 32, 96, 0, 33, 97, 1) \
  CPI_WIN_TWO(s53, v250, v254, 34, 98, 2, 35, 99, 3) \
  CPI_WIN_TWO(s54, v250, v254, 36, 100, 4, 37, 101, 5) \
  CPI_WIN_TWO(s55, v250, v254, 38, 102, 6, 39, 103, 7) \
  CPI_WIN_TWO(s56, v250, v254, 40, 104, 8, 41, 105, 9) \
  CPI_WIN_TWO(s57, v250, v254, 42, 106, 10, 43, 107, 11) \
  CPI_WIN_TWO(s58, v250, v254, 44, 108, 12, 45, 109, 13) \
  CPI_WIN_TWO(s59, v250, v254, 46, 110, 14, 47, 111, 15)
#define CPI_WIN_CHUNK3 \
  CPI_WIN_TWO(s60, v251, v255, 48, 112, 0, 49, 113, 1) \
  CPI_WIN_TWO(s61, v251, v255, 50, 114, 2, 51, 115, 3) \
  CPI_WIN_TWO(s62, v251, v255, 52, 116, 4, 53, 117, 5) \
  CPI_WIN_TWO(s63, v251, v255, 54, 118, 6, 55, 119, 7) \
  CPI_WIN_TWO(s64, v251, v255, 56, 120, 8, 57, 121, 9) \
  CPI_WIN_TWO(s65, v251, v255, 58, 122, 10, 59, 123, 11) \
  CPI_WIN_TWO(s66, v251, v255, 60, 124, 12, 61, 125, 13) \
  CPI_WIN_TWO(s67, v251, v255, 62, 126, 14, 63, 127, 15)
#define CPI_WIN_SUM(c, CH)                    \
  "s_bitcmp1_b32 %[live], " #c "\n"           \
  "s_cbranch_scc0 Lskip" #c "%=\n" CH         \
  "Lskip" #c "%=:\n"

#define CPI_WIN_VIEW                                     \
  "s_load_dwordx16 s[36:51], %[th], 512\n"               \
  "s_load_dwordx16 s[52:67], %[th], 576\n"               \
  CPI_WIN_WAITS                                          \
  "s_barrier\n"                                          \
  "ds_read_b128 v[248:251], %[tw]\n"                     \
  "ds_read_b128 v[252:255], %[tw] offset:256\n"          \
  CPI_WIN_READS                                          \
  "Lread%=:\n"                                           \
  "s_cmp_eq_u32 %[spaces], 1\n"                            \
  "s_cbranch_scc0 Ltwo%=\n"                              \
  "s_waitcnt lgkmcnt(0)\n"                               \
  "s_barrier\n"                                          \
  "Ltwo%=:\n"                                            \
  CPI_WIN_COPIES                                         \
  "Lcopy%=:\n"                                           \
  CPI_WIN_TABLE                                          \
  "s_waitcnt lgkmcnt(0)\n"                               \
  "s_load_dwordx8 s[68:75], %[tn], 640\n"                \
  "s_setprio 2\n"                                        \
  "s_set_gpr_idx_on s36, 2\n"                            \
  CPI_WIN_SUM(0, CPI_WIN_CHUNK0)                         \
  CPI_WIN_SUM(1, CPI_WIN_CHUNK1)                         \
  CPI_WIN_SUM(2, CPI_WIN_CHUNK2)                         \
  CPI_WIN_SUM(3, CPI_WIN_CHUNK3)                         \
  "s_set_gpr_idx_off\n"                                  \
  "s_setprio 0\n"                                  \
  "s_waitcnt lgkmcnt(0)\n"

#define CPI_WIN_ACC \
  "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]), "+v"(acc[4]), "+v"(acc[5]), \
      "+v"(acc[6]), "+v"(acc[7]), "+v"(acc[8]), "+v"(acc[9]), "+v"(acc[10]), "+v"(acc[11]), \
      "+v"(acc[12]), "+v"(acc[13]), "+v"(acc[14]), "+v"(acc[15]), "+v"(acc[16]), \
      "+v"(acc[17]), "+v"(acc[18]), "+v"(acc[19]), "+v"(acc[20]), "+v"(acc[21]), \
      "+v"(acc[22]), "+v"(acc[23]), "+v"(acc[24]), "+v"(acc[25]), "+v"(acc[26]), \
      "+v"(acc[27]), "+v"(acc[28]), "+v"(acc[29]), "+v"(acc[30]), "+v"(acc[31]), \
      "+v"(acc[32]), "+v"(acc[33]), "+v"(acc[34]), "+v"(acc[35]), "+v"(acc[36]), \
      "+v"(acc[37]), "+v"(acc[38]), "+v"(acc[39]), "+v"(acc[40]), "+v"(acc[41]), \
      "+v"(acc[42]), "+v"(acc[43]), "+v"(acc[44]), "+v"(acc[45]), "+v"(acc[46]), \
      "+v"(acc[47]), "+v"(acc[48]), "+v"(acc[49]), "+v"(acc[50]), "+v"(acc[51]), \
      "+v"(acc[52]), "+v"(acc[53]), "+v"(acc[54]), "+v"(acc[55]), "+v"(acc[56]), \
      "+v"(acc[57]), "+v"(acc[58]), "+v"(acc[59]), "+v"(acc[60]), "+v"(acc[61]), \
      "+v"(acc[62]), "+v"(acc[63]), "+v"(acc[64]), "+v"(acc[65]), "+v"(acc[66]), \
      "+v"(acc[67]), "+v"(acc[68]), "+v"(acc[69]), "+v"(acc[70]), "+v"(acc[71]), \
      "+v"(acc[72]), "+v"(acc[73]), "+v"(acc[74]), "+v"(acc[75]), "+v"(acc[76]), \
      "+v"(acc[77]), "+v"(acc[78]), "+v"(acc[79]), "+v"(acc[80]), "+v"(acc[81]), \
      "+v"(acc[82]), "+v"(acc[83]), "+v"(acc[84]), "+v"(acc[85]), "+v"(acc[86]), \
      "+v"(acc[87]), "+v"(acc[88]), "+v"(acc[89]), "+v"(acc[90]), "+v"(acc[91]), \
      "+v"(acc[92]), "+v"(acc[93]), "+v"(acc[94]), "+v"(acc[95]), "+v"(acc[96]), \
      "+v"(acc[97]), "+v"(acc[98]), "+v"(acc[99]), "+v"(acc[100]), "+v"(acc[101]), \
      "+v"(acc[102]), "+v"(acc[103]), "+v"(acc[104]), "+v"(acc[105]), "+v"(acc[106]), \
      "+v"(acc[107]), "+v"(acc[108]), "+v"(acc[109]), "+v"(acc[110]), "+v"(acc[111]), \
      "+v"(acc[112]), "+v"(acc[113]), "+v"(acc[114]), "+v"(acc[115]), "+v"(acc[116]), \
      "+v"(acc[117]), "+v"(acc[118]), "+v"(acc[119]), "+v"(acc[120]), "+v"(acc[121]), \
      "+v"(acc[122]), "+v"(acc[123]), "+v"(acc[124]), "+v"(acc[125]), "+v"(acc[126]), \
      "+v"(acc[127])
#define CPI_WIN_CLOBBERS \
  "s36", "s37", "s38", "s39", "s40", "s41", "s42", "s43", "s44", "s45", "s46", "s47", "s48", \
      "s49", "s50", "s51", "s52", "s53", "s54", "s55", "s56", "s57", "s58", "s59", "s60", \
      "s61", "s62", "s63", "s64", "s65", "s66", "s67", "v168", "v169", "v170", "v171", \
      "v172", "v173", "v174", "v175", "v176", "v177", "v178", "v179", "v180", "v181", "v182", \
      "v183", "v184", "v185", "v186", "v187", "v188", "v189", "v190", "v191", "v192", "v193", \
      "v194", "v195", "v196", "v197", "v198", "v199", "v200", "v201", "v202", "v203", "v204", \
      "v205", "v206", "v207", "v208", "v209", "v210", "v211", "v212", "v213", "v214", "v215", \
      "v216", "v217", "v218", "v219", "v220", "v221", "v222", "v223", "v224", "v225", "v226", \
      "v227", "v228", "v229", "v230", "v231", "v232", "v233", "v234", "v235", "v236", "v237", \
      "v238", "v239", "v240", "v241", "v242", "v243", "v244", "v245", "v246", "v247", "v248", \
      "v249", "v250", "v251", "v252", "v253", "v254", "v255", "m0", "scc", "memory"

typedef int i4v __attribute__((ext_vector_type(4)));
typedef int i8v __attribute__((ext_vector_type(8)));

// (read through the scalar cache: the kernel does not write the tables)
typedef const __attribute__((address_space(4))) int32_t* TabPtr;

struct WindowUnits {
  uint8_t n[kWinMaxGroups];   // 64-row units per lens-plane row, by plane group
};

// Plane group gq has n[gq] units of 64 view rows for each lens-plane row (rows
// from the first one its planes sample at that y_b), in order, and a
// work-group takes two consecutive units.  Work-group (gq, t, p, j) belongs to the p-th
// lens-plane row, where its first unit lies, so that work-groups of different
// groups that run together read the same views.  False: no such work-group.
__device__ __forceinline__ bool window_first_unit(int n, int p, int j, int* u) {
  *u = kWinSlots * ((p * n + kWinSlots - 1) / kWinSlots + j);
  return *u < (p + 1) * n;
}

template <int NP, int XC, int PG>
__global__ __launch_bounds__(64 * kWinWaves, 2) void k_ref_window(
    const float* __restrict__ gamma, GeomI g, const int32_t* __restrict__ xe,
    const int2* __restrict__ yr, WindowUnits units, int groups, int tiles, int per_yb, int count,
    int stages, int stage_bytes, float* __restrict__ tout, int wout_pad) {
  constexpr int CG = kWinWaves / PG, PW = kWinPairs;
  static_assert(NP * XC == PW && XC % 4 == 0, "64 pairs per wave");
  __shared__ __attribute__((aligned(1024))) uint8_t ring[kWinLds + kWinMaxStages * kWinTabBytes];
  // All work-groups of one lens-plane row on one XCD (work-groups go to the
  // XCDs in turn), plane groups fastest, then column tiles: the work-groups
  // resident on an XCD at one time read the same rows of each view.
  const int xcd = blockIdx.x & 7;
  int rest = blockIdx.x >> 3;
  const int gq = rest % groups;
  rest /= groups;
  const int t = rest % tiles;
  rest /= tiles;
  const int j = rest % per_yb;
  const int p = rest / per_yb;
  const int yb0 = xcd * g.hb / 8, yb1 = (xcd + 1) * g.hb / 8;
  const int n = units.n[gq];
  int u0;
  if (yb0 + p >= yb1 || !window_first_unit(n, p, j, &u0)) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int2* yrg = yr + int64_t(gq) * g.hb;
  // unit u: its y_b (at or past yb1 if there is none), first row and the last
  // row of its y_b; false if it has no row
  auto unit = [&](int u, int* yb, int* row, int* last) {
    *yb = yb0 + u / n;
    if (*yb >= yb1) return false;
    const int2 r = yrg[*yb];
    *row = r.x + 64 * (u % n);
    *last = r.y;
    return *row <= r.y;
  };

  float acc[kWinSlots * PW];
#pragma unroll
  for (int i = 0; i < kWinSlots * PW; ++i) acc[i] = 0.0f;
  {
    // this wave copies 32 rows of unit u0 + wave / 2.  1 KB per instruction,
    // 16 rows x 16 columns; lane l writes slot l of the block, which holds row
    // l / 4 and columns 4 c .. 4 c + 3 with c = (l % 4) ^ ((l / 16) % 4), so
    // that 16 lanes reading one chunk of 16 rows cover all banks once.  Rows
    // past the view read as zero.  Block (16-column block cb, 16-row block rb)
    // is at 8192 cb + 1024 rb.
    int yb = 0, row = 0, row_last = 0;
    const bool mine = unit(u0 + wave / 2, &yb, &row, &row_last);
    const int pa = g.wa * g.ha;
    const float* view = gamma + (mine ? int64_t(yb) * g.wb * pa : 0);
    const uint32_t from = window_lane_offset(row, wave, lane, 0, g.wa);
    const uint32_t from1 = window_lane_offset(row, wave, lane, 1, g.wa);
    const uint32_t base = uint32_t(reinterpret_cast<uintptr_t>(ring));
    const uint32_t rd = uint32_t(64 * (lane & 15) + 1024 * (lane >> 4) + 16 * ((lane >> 2) & 3));
    const uint32_t tl = uint32_t(16 * (lane & 31));
    const uint32_t tab0 = base + uint32_t(kWinLds + wave * 512);
    constexpr int kStep = kWinWaves * kWinWaveWords;
    const int32_t* tp = xe + (int64_t(gq * tiles + t) * g.wb * kWinWaves + wave) * kWinWaveWords;
    TabPtr th = (TabPtr)tp;
    const int last = g.wb - 1;
    // descriptor of a view's columns from wx0
    auto desc = [&](int wx0) {
      const uint64_t a = reinterpret_cast<uint64_t>(view + wx0);
      return i4v{int(uint32_t(a)), int(uint32_t(a >> 32) & 0xffffu), (pa - wx0) * 4, 0x00020000};
    };
    // the copies of the first `ahead` views
    const int ahead = stages == 1 ? 1 : stages - 1;
    int f1 = 0;   // copies started last
    for (int k = 0; k < ahead; ++k) {
      const int kk = k < last ? k : last;
      const i4v rs = desc(th[kk * kStep + 163]);
      const int nb = mine && k <= last ? th[kk * kStep + 164] : 0;
      // (s_nop: a descriptor register may just have been written by a vector
      // instruction)
      asm volatile("s_nop 4\n" CPI_WIN_COPIES "Lcopy%=:\n" CPI_WIN_TABLE
                   :
                   : [nb] "s"(nb), [dst] "s"(base + uint32_t(k * stage_bytes + 2048 * wave)),
                     [rs] "s"(rs), [from] "v"(from), [from1] "v"(from1),
                     [td] "s"(tab0 + uint32_t(k * kWinTabBytes)), [tl] "v"(tl),
                     [tp] "s"(tp + kk * kStep)
                   : "m0", "scc", "memory");
      f1 = 2 * nb + 1;
      if (k < last) view += pa;
    }
    i8v head;
#pragma unroll
    for (int k = 0; k < 8; ++k) head[k] = th[160 + k];
    tp += int64_t(ahead <= last ? ahead : last) * kStep;
    int stage = 0, to = ahead % stages;   // of this view, and of the copies it starts
#pragma unroll 1
    for (int v = 0; v <= last; ++v) {
      TabPtr tn = v < last ? th + kStep : th;
      const int fly = ahead > 1 ? f1 : 0;
      const i4v rs = desc(head[5]);
      const int nb = mine ? head[6] : 0;
      const int xa = head[0], xc = head[1];
      const int nq = head[2] & 0xff, live = head[2] >> 8;
      const uint32_t sb = base + uint32_t(stage * stage_bytes);
      const uint32_t a0 = (rd ^ window_unpack_chunk(uint32_t(xa), 0)) + sb;
      const uint32_t a1 = (rd ^ window_unpack_chunk(uint32_t(xa), 1)) + sb;
      const uint32_t a2 = (rd ^ window_unpack_chunk(uint32_t(xc), 0)) + sb;
      const uint32_t a3 = (rd ^ window_unpack_chunk(uint32_t(xc), 1)) + sb;
      const uint32_t tw = tab0 + uint32_t(stage * kWinTabBytes) + uint32_t(16 * (lane & 15));
      i8v next;
      asm volatile(CPI_WIN_VIEW
                   : CPI_WIN_ACC, [next] "=&{s[68:75]}"(next)
                   : [fly] "s"(fly), [nq] "s"(nq), [nb] "s"(nb), [spaces] "s"(stages),
                     [dst] "s"(base + uint32_t(to * stage_bytes + 2048 * wave)), [rs] "s"(rs),
                     [live] "s"(live), [a0] "v"(a0), [a1] "v"(a1), [a2] "v"(a2), [a3] "v"(a3),
                     [from] "v"(from), [from1] "v"(from1),
                     [td] "s"(tab0 + uint32_t(to * kWinTabBytes)), [tl] "v"(tl), [tp] "s"(tp),
                     [th] "s"(th), [tn] "s"(tn), [tw] "v"(tw)
                   : CPI_WIN_CLOBBERS);
      head = next;
      th = tn;
      f1 = 2 * nb + 1;
      stage = stage + 1 == stages ? 0 : stage + 1;
      to = to + 1 == stages ? 0 : to + 1;
      if (v + ahead < last) {
        view += pa;
        tp += kStep;
      }
    }
    // (the last table copies are still in flight)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }

  const int64_t plane_stride = int64_t(g.hb) * g.ha * wout_pad;
  const int pl0 = (gq * PG + wave / CG) * NP;
  float* tw = tout + pl0 * plane_stride + (t * CG + wave % CG) * XC;
#pragma unroll
  for (int k = 0; k < kWinSlots; ++k) {
    int yb = 0, row = 0, row_last = -1;
    const bool live = unit(u0 + k, &yb, &row, &row_last);
    if (yb >= yb1) continue;
    float* d = tw + int64_t(yb) * g.ha * wout_pad;
    if (live && row + lane <= row_last) {
#pragma unroll
      for (int i = 0; i < PW; i += 4) {
        const float* s = acc + k * PW + i;
        if (pl0 + i / XC < count)
          *reinterpret_cast<float4*>(d + (i / XC) * plane_stride + int64_t(row + lane) * wout_pad +
                                     i % XC) = make_float4(s[0], s[1], s[2], s[3]);
      }
    }
    // The fold also reads, with zero weights, the rows next to the sampled
    // ones and the two at either end of the view: zeros, by the first unit of
    // each y_b, where no sum is written.
    if ((u0 + k) % n == 0 && lane < 6) {
      const int lo = yrg[yb].x, hi = yrg[yb].y;
      const int r = lane < 2 ? lane : lane < 4 ? g.ha - lane + 1 : lane == 4 ? lo - 1 : hi + 1;
      if (r >= 0 && r < g.ha && (r < lo || r > hi)) {
#pragma unroll
        for (int i = 0; i < PW; i += 4)
          if (pl0 + i / XC < count)
            *reinterpret_cast<float4*>(d + (i / XC) * plane_stride + int64_t(r) * wout_pad +
                                       i % XC) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      }
    }
  }
}

#undef CPI_WIN_TABLE
#undef CPI_WIN_DPP
#undef CPI_WIN_SUM
#undef CPI_WIN_CHUNK2
#undef CPI_WIN_CHUNK3
#undef CPI_WIN_WAIT
#undef CPI_WIN_WAITS
#undef CPI_WIN_READ
#undef CPI_WIN_READS
#undef CPI_WIN_COPY
#undef CPI_WIN_COPIES
#undef CPI_WIN_PAIR
#undef CPI_WIN_TWO
#undef CPI_WIN_CHUNK0
#undef CPI_WIN_CHUNK1
#undef CPI_WIN_VIEW
#undef CPI_WIN_ACC
#undef CPI_WIN_CLOBBERS

template <int NP, int XC, int PG>
hipError_t launch_window(const float* gamma, const RefGeom& g, const double* alphas,
                         const int32_t* itab, const float* ftab, int64_t stride, int first,
                         int count, int blocks, int32_t* xe, const int2* yr, float* t,
                         int wout_pad, hipStream_t s) {
  constexpr int NA = NP * PG, XR = XC * (kWinWaves / PG);
  const GeomI gi{g.wa, g.ha, g.wb, g.hb, g.out_w, g.out_h};
  const int tiles = (gi.out_w + XR - 1) / XR;
  const int groups = (count + NA - 1) / NA;
  const int64_t nx = int64_t(groups) * tiles * gi.wb;
  if (nx > 0x7fffffff || groups > kWinMaxGroups) return hipErrorInvalidValue;
  WindowUnits units = {};
  int per_yb = 1;   // work-groups of a lens-plane row at most
  for (int q = 0; q < groups; ++q) {
    const int rows = window_rows(g, alphas, first + q * NA, first + std::min((q + 1) * NA, count));
    if ((rows + 63) / 64 > 255) return hipErrorInvalidValue;
    units.n[q] = uint8_t(std::max(1, (rows + 63) / 64));
    per_yb = std::max(per_yb, (units.n[q] + kWinSlots - 1) / kWinSlots);
  }
  const int64_t nwg = int64_t(8) * ((gi.hb + 7) / 8) * per_yb * tiles * groups;
  const int stages = std::min(kWinMaxStages, kWinBlocks / blocks);
  if (nwg > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_window_xtab<NP, XC, PG>), dim3(unsigned(nx)), dim3(256), 0, s, gi, itab,
                     ftab, stride, first, count, tiles, blocks, stages == 1 ? 1 : stages - 1, xe);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_ref_window<NP, XC, PG>), dim3(unsigned(nwg)), dim3(64 * kWinWaves), 0, s,
                     gamma, gi, xe, yr, units, groups, tiles, per_yb, count, stages,
                     blocks * kWinBlockBytes, t, wout_pad);
  return hipGetLastError();
}

}  // namespace

hipError_t window_xpass(const float* gamma, const RefGeom& g, const double* alphas,
                        const WindowSplit& w, const int32_t* itab, const float* ftab,
                        int64_t stride, int first, int count, int32_t* xe, const int2* yr,
                        float* t, int wout_pad, hipStream_t s) {
#define CPI_WIN_CASE(NP_, XC_, PG_)                                                              \
  if (w.np == NP_ && w.xc == XC_ && w.pg == PG_)                                                 \
    return launch_window<NP_, XC_, PG_>(gamma, g, alphas, itab, ftab, stride, first, count,    \
                                        w.blocks, xe, yr, t, wout_pad, s);
  CPI_WIN_CASE(8, 8, 2)
  CPI_WIN_CASE(4, 16, 2)
  CPI_WIN_CASE(4, 16, 1)
#undef CPI_WIN_CASE
  return hipErrorInvalidValue;
}

}  // namespace cpi
