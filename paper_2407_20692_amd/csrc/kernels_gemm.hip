// Sum of products S_ab = A^T B on matrix cores (int8 or FP4 operands),
// followed by the exact combination of Eq. (1):
//     numer = N * S_ab - S_a * S_b        (int64)
//     gamma = fl64(fl64(numer) / fl64(N * N))
//     gamma_f32 = fl32(gamma)
//
// Operands are pixel-major rows (frames contiguous) built by the ingest
// kernels.  M = detector-B pixels (views), N = detector-A pixels, so the
// matrix-core output rows are views and its columns run along detector-A
// pixels, which is the view-major storage of Gamma.
//
// Each 64-byte segment of a row holds 512 frames as bits or 64 frames as
// bytes.  Lane l of a wave reads 16 bytes of row (16*f + l%16) at byte
// 16*(l/16) of the segment.  For byte rows those 16 bytes are the lane's
// 16 K values of one MFMA (k_gemm_bytes).  For bit rows they are four 32-bit words; word w
// shifted right by s and masked with 0x01010101 gives four bytes holding the
// frames 8*b + s of that word (b = 0..3), so shifts 4h..4h+3 make one 16-byte
// MFMA operand and every word feeds two MFMAs.  Both operands use the same
// lane/byte -> frame assignment, so every product pairs A and B of the same
// frame, whatever order the hardware sums the K index in.
//
// Bit rows can instead feed the FP4 matrix-core op
// (v_mfma_f32_16x16x128_f8f6f4 with E2M1 operands, no block scales).  Word w
// of a lane supplies the lane's 32 K values of one such op: nibble k of
// dword d holds frame 4k + d of the word.  A single set bit is an exact
// E2M1 value (bit 0: 0.5, bit 1: 1, bit 2: 2), so a dword can often be cut
// out of the word with one AND: the N operand takes dwords 0, 1, 2 as
// w & 0x1..., w & 0x2..., w & 0x4... (values 0.5, 1, 2), and the M rows are
// stored with bits 0 and 2 of every 4-bit group exchanged, so the same ANDs
// give it values 2, 1, 0.5 for the same frames.  Frame 4k + 3 sits on the
// sign bit and is shifted to bit 1 (value 1) on both sides.  Every product
// of two set bits is then exactly 1, the FP32 accumulator holds integers
// exactly up to 2^24, and the sums equal the int8 ones bit for bit as long
// as one launch covers at most 2^24 frames.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdlib>
#include <cstring>
#include <type_traits>

#include "kernels.h"

namespace cpi {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

// Scale operands 0 select the unscaled form of the op (plain products),
// which issues faster than the block-scaled one.
constexpr int kNoScale = 0;
constexpr int kFmtE2M1 = 4;

// The four E2M1 dwords (32 K values) of bit word x of an N row (plain
// layout: frames 4k + 0, 1, 2 at values 0.5, 1, 2; frame 4k + 3 at 1) ...
__device__ __forceinline__ v8i fp4_operand_n(uint32_t x) {
  return v8i{int(x & 0x11111111u), int(x & 0x22222222u), int(x & 0x44444444u),
             int((x >> 2) & 0x22222222u), 0, 0, 0, 0};
}
// ... and of an M row stored with bits 0 and 2 of each group exchanged
// (frames 4k + 0, 1, 2 at values 2, 1, 0.5; frame 4k + 3 at 1).
__device__ __forceinline__ v8i fp4_operand_m(uint32_t x) {
  return v8i{int(x & 0x44444444u), int(x & 0x22222222u), int(x & 0x11111111u),
             int((x >> 2) & 0x22222222u), 0, 0, 0, 0};
}

// Work-group b executes on XCD b % 8.  Give each XCD a contiguous range of
// output tiles so that tiles sharing operand rows share that XCD's L2.
__device__ __forceinline__ int xcd_remap(int b, int nwg) {
  const int per = nwg >> 3, rem = nwg & 7;
  const int x = b & 7, i = b >> 3;
  return (x < rem ? x * (per + 1) : rem * (per + 1) + (x - rem) * per) + i;
}

// Tile of work-group b: XCD-contiguous ranges, walked in groups of 8 tile
// rows, so that the work-groups resident on one XCD at a time cover about
// 8 x 8 tiles and re-use each other's operand rows in its L2.
__device__ __forceinline__ void tile_of(int b, int nwg, int tiles_m, int* tm, int* tn) {
  constexpr int kGroup = 8;
  const int id = xcd_remap(b, nwg);
  const int tiles_n = nwg / tiles_m;
  const int per_group = kGroup * tiles_n;
  const int grp = id / per_group;
  const int m0 = grp * kGroup;
  const int gm = (tiles_m - m0) < kGroup ? (tiles_m - m0) : kGroup;
  const int in = id - grp * per_group;
  *tm = m0 + in % gm;
  *tn = in / gm;
}

// Epilogue fields, copied out of the kernel argument block into registers.
struct Epi {
  int mode, layout;
  int64_t pa, pb, n, kchunk;
  const int64_t* sum_a;
  const int64_t* sum_b;
  const int64_t* csum_a;
  const int64_t* csum_b;
  double* gamma;
  float* gamma_f32;
  int64_t* numer;
  int64_t* acc64;
  int32_t* acc32;
};

// a / nn rounded once (IEEE), with y the rounded reciprocal of nn: two Newton
// steps from a * y by fused multiply-adds.  The first gives a quotient within
// one unit in the last place, the second rounds it correctly (Markstein's
// theorem; it excludes nn with a mantissa of all ones, which no square has).
// Values stay far from overflow and underflow: |a| is 0 or in [1, 2^63], nn
// in [1, 2^53).  Five instructions instead of the fourteen of a division.
__device__ __forceinline__ double quotient(double a, double nn, double y) {
  double q = a * y;
  q = __builtin_fma(__builtin_fma(-nn, q, a), y, q);
  return __builtin_fma(__builtin_fma(-nn, q, a), y, q);
}

// Output stores: past the caches (written once, not read back here) where a
// wave's stores cover whole lines, else through them, so that the lines two
// stores share are put together there.
template <typename T>
__device__ __forceinline__ void store_out(T v, T* p, bool past) {
  if (past)
    __builtin_nontemporal_store(v, p);
  else
    *p = v;
}

// The sum of a row or column of outputs: S and, in EPI_STREAM64, the chunk's.
struct SideSum {
  int64_t s, c;
};
template <int MODE>
__device__ __forceinline__ SideSum side_sum(const int64_t* sum, const int64_t* csum, int64_t i) {
  SideSum v{0, 0};
  if constexpr (MODE != EPI_STORE64 && MODE != EPI_ADD64) v.s = sum[i];
  if constexpr (MODE == EPI_STREAM64) v.c = csum[i];
  return v;
}
template <int MODE, bool VM>
__device__ __forceinline__ void store_result(const Epi& g, double y, bool past, int64_t q,
                                             int64_t p, int64_t s, int64_t o, SideSum a,
                                             SideSum b) {
  // s: sum of products in the operand domain; o: operand offset (0 or 128)
  const int64_t idx_vm = q * g.pa + p;
  const int64_t n = g.n;
  switch (MODE) {
    case EPI_STORE64:
      g.acc64[idx_vm] = s;
      return;
    case EPI_ADD64:
      g.acc64[idx_vm] += s;
      return;
    case EPI_FINAL_ACC64:
      s += g.acc64[idx_vm];
      break;
    case EPI_STREAM32: {
      const int32_t t = g.acc32[idx_vm] + int32_t(s);
      g.acc32[idx_vm] = t;
      s = t;
      o = 0;
      break;
    }
    case EPI_STREAM64: {
      // back to raw values: sum (a-o)(b-o) = S_ab - o S_a - o S_b + k o^2
      const int64_t raw = s + o * (a.c + b.c) - g.kchunk * o * o;
      const int64_t t = g.acc64[idx_vm] + raw;
      g.acc64[idx_vm] = t;
      s = t;
      o = 0;
      break;
    }
    default:
      break;
  }
  const int64_t sa = a.s - o * n;
  const int64_t sb = b.s - o * n;
  const int64_t numer = n * s - sa * sb;
  const double gam = quotient(double(numer), double(n) * double(n), y);
  const int64_t idx = VM ? idx_vm : p * g.pb + q;
  if (g.gamma) store_out(gam, g.gamma + idx, past);
  if (g.gamma_f32) store_out(float(gam), g.gamma_f32 + idx, past);
  if (g.numer) store_out(numer, g.numer + idx, past);
}

// Four consecutive detector-A pixels p..p+3 of view q in view-major order, all
// inside the detector and 16-byte aligned; s[] in the operand domain, o its
// offset.
template <int MODE>
__device__ __forceinline__ void store_quad(const Epi& g, double y, int64_t q, int64_t p,
                                           const int32_t (&s)[4], int64_t o) {
  const int64_t idx_vm = q * g.pa + p;
  int64_t t[4];
  if constexpr (MODE == EPI_STREAM32) {
    int4 a = *reinterpret_cast<const int4*>(g.acc32 + idx_vm);
    a.x += s[0];
    a.y += s[1];
    a.z += s[2];
    a.w += s[3];
    *reinterpret_cast<int4*>(g.acc32 + idx_vm) = a;
    t[0] = a.x;
    t[1] = a.y;
    t[2] = a.z;
    t[3] = a.w;
  } else if constexpr (MODE == EPI_STREAM64) {
    longlong2 a0 = *reinterpret_cast<const longlong2*>(g.acc64 + idx_vm);
    longlong2 a1 = *reinterpret_cast<const longlong2*>(g.acc64 + idx_vm + 2);
    // back to raw values: sum (a-o)(b-o) = S_ab - o S_a - o S_b + k o^2
    int64_t r[4] = {s[0], s[1], s[2], s[3]};
    if (o)
#pragma unroll
      for (int k = 0; k < 4; ++k)
        r[k] += o * (g.csum_a[p + k] + g.csum_b[q]) - g.kchunk * o * o;
    o = 0;
    a0.x += r[0];
    a0.y += r[1];
    a1.x += r[2];
    a1.y += r[3];
    *reinterpret_cast<longlong2*>(g.acc64 + idx_vm) = a0;
    *reinterpret_cast<longlong2*>(g.acc64 + idx_vm + 2) = a1;
    t[0] = a0.x;
    t[1] = a0.y;
    t[2] = a1.x;
    t[3] = a1.y;
  } else {
    static_assert(MODE == EPI_FINAL, "quad epilogue modes");
#pragma unroll
    for (int k = 0; k < 4; ++k) t[k] = s[k];
  }
  const int64_t on = o * g.n;
  const int64_t sb = g.sum_b[q] - on;
  const longlong2 sa01 = *reinterpret_cast<const longlong2*>(g.sum_a + p);
  const longlong2 sa23 = *reinterpret_cast<const longlong2*>(g.sum_a + p + 2);
  const int64_t sa[4] = {sa01.x - on, sa01.y - on, sa23.x - on, sa23.y - on};
  const double nn = double(g.n) * double(g.n);
  int64_t num[4];
  double gam[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    // (bits, and bytes in one pass of at most 131008 frames: n, S_a, S_b and
    // an int32 state all fit 32 bits)
    if constexpr (MODE == EPI_STREAM64)
      num[k] = g.n * t[k] - sa[k] * sb;
    else
      num[k] = int64_t(int32_t(g.n)) * int32_t(t[k]) - int64_t(int32_t(sa[k])) * int32_t(sb);
    gam[k] = quotient(double(num[k]), nn, y);
  }
  // The outputs are written once and not read back here: non-temporal
  // stores stream them past the caches, which keep the operand rows (at
  // 65536 x 65536 pairs this cut the contraction from 18.4 to 12.0 ms).
  typedef double d2v __attribute__((ext_vector_type(2)));
  typedef float f4v __attribute__((ext_vector_type(4)));
  typedef int64_t l2v __attribute__((ext_vector_type(2)));
  if (g.gamma) {
    __builtin_nontemporal_store(d2v{gam[0], gam[1]}, reinterpret_cast<d2v*>(g.gamma + idx_vm));
    __builtin_nontemporal_store(d2v{gam[2], gam[3]}, reinterpret_cast<d2v*>(g.gamma + idx_vm + 2));
  }
  if (g.gamma_f32)
    __builtin_nontemporal_store(f4v{float(gam[0]), float(gam[1]), float(gam[2]), float(gam[3])},
                                reinterpret_cast<f4v*>(g.gamma_f32 + idx_vm));
  if (g.numer) {
    __builtin_nontemporal_store(l2v{num[0], num[1]}, reinterpret_cast<l2v*>(g.numer + idx_vm));
    __builtin_nontemporal_store(l2v{num[2], num[3]}, reinterpret_cast<l2v*>(g.numer + idx_vm + 2));
  }
}

// Row pitch of a tile of sums staged in LDS: for quads (16-byte reads, rows 4
// banks apart) or, where the lanes of a wave read down a column, odd.
__device__ __forceinline__ int tile_pitch(const Epi& g, int cols) {
  return g.layout == CPI_GAMMA_VIEW_MAJOR ? cols + 4 : cols + 1;
}

// ROWS x COLS sums (views q0 .., detector-A pixels p0 ..), less `pad`, from LDS to the
// outputs, by a work-group of T threads.  Consecutive lanes take consecutive
// output elements: along the pixels in view-major order, four at a time where
// they are aligned, along the views in pixel-major order.  (Four elements of
// one view per lane, stored one by one, wrote 7575 x 1353 pixel-major
// numerators from 12345 frames in 265 us; this takes 82 us.)  Elements stored one
// by one take the sums of their row and column from LDS behind the tile, where
// stage_sums put them before the barrier that the tile is read behind: read from
// memory for each element, they made a small call wait 32 times (Da 644, Db 32
// pixels, 199 packed frames, pixel-major: 33.3 -> 28.7 us), and kept for several
// elements at a time in registers, they cost the bit kernels their third wave.
template <bool QUADS>
__device__ __forceinline__ bool in_quads(const Epi& g) {
  return QUADS && g.layout == CPI_GAMMA_VIEW_MAJOR && (g.pa & 3) == 0;
}
constexpr int sums_bytes(int rows, int cols) { return (rows + cols) * int(sizeof(SideSum)); }
template <int MODE, bool QUADS, int ROWS, int COLS>
__device__ __forceinline__ void stage_sums(const Epi& g, SideSum* sums, int64_t q0, int64_t p0) {
  if (in_quads<QUADS>(g)) return;
  for (int t = threadIdx.x; t < COLS + ROWS; t += blockDim.x) {
    SideSum v{0, 0};
    if (t < COLS) {
      if (p0 + t < g.pa) v = side_sum<MODE>(g.sum_a, g.csum_a, p0 + t);
    } else if (q0 + t - COLS < g.pb) {
      v = side_sum<MODE>(g.sum_b, g.csum_b, q0 + t - COLS);
    }
    sums[t] = v;   // columns, then rows
  }
}
template <int MODE, bool QUADS, int ROWS, int COLS, int T>
__device__ __forceinline__ void store_tile(const Epi& g, const int32_t* tile,
                                           const SideSum* sums, int pitch, int64_t q0,
                                           int64_t p0, int64_t o, int32_t pad) {
  static_assert(T % (COLS / 4) == 0 && COLS % 4 == 0, "tile shape");
  const int t = threadIdx.x;
  const double y = 1.0 / (double(g.n) * double(g.n));
  const bool vm = g.layout == CPI_GAMMA_VIEW_MAJOR;
  if constexpr (QUADS) {
    if (in_quads<QUADS>(g)) {
      const int cq = 4 * (t % (COLS / 4));
      const int64_t p = p0 + cq;
      if (p >= g.pa) return;
#pragma unroll 1
      for (int row = t / (COLS / 4); row < ROWS && q0 + row < g.pb; row += T / (COLS / 4)) {
        const int4 v = *reinterpret_cast<const int4*>(tile + row * pitch + cq);
        const int32_t s[4] = {v.x - pad, v.y - pad, v.z - pad, v.w - pad};
        store_quad<MODE>(g, y, q0 + row, p, s, o);
      }
      return;
    }
  }
  // Element by element: a thread keeps its column (view-major) or row; past the
  // caches where the 64 elements of 4 bytes that a wave stores at a time are whole
  // 128-byte lines.
  static_assert(T % COLS == 0 && T % ROWS == 0, "tile shape");
  const int32_t rows = int32_t(g.pb - q0 < ROWS ? g.pb - q0 : ROWS);
  const int32_t cols = int32_t(g.pa - p0 < COLS ? g.pa - p0 : COLS);
  auto run = [&](auto view_major, int fixed, int fixed_n, int first, int step, int n) {
    constexpr bool VM = decltype(view_major)::value;
    if (fixed >= fixed_n) return;
    const bool past = ((VM ? g.pa : g.pb) & 31) == 0;
    const SideSum own = sums[VM ? fixed : COLS + fixed];
    // (two elements with their states would cost the bit kernels their third wave)
    constexpr int kUnroll = MODE == EPI_STREAM32 || MODE == EPI_STREAM64 ? 1 : 2;
#pragma unroll kUnroll
    for (int k = first; k < n; k += step) {
      const int row = VM ? k : fixed, col = VM ? fixed : k;
      const SideSum other = sums[VM ? COLS + k : k];
      store_result<MODE, VM>(g, y, past, q0 + row, p0 + col, tile[row * pitch + col] - pad, o,
                             VM ? own : other, VM ? other : own);
    }
  };
  if (vm)
    run(std::true_type{}, t % COLS, cols, t / COLS, T / COLS, rows);
  else
    run(std::false_type{}, t % ROWS, rows, t / ROWS, T / ROWS, cols);
}

// Register-fed contraction of bit rows (for comparison: CPI_GEMM_FEED=regs).
template <int FM, int FN, int MODE, bool F4>
__global__ __launch_bounds__(256) void k_gemm(GemmArgs g) {
  if (g.cond) {
    const uint32_t mx = g.stats[0];
    if ((g.cond == 1) != (mx <= 1u)) return;
  }
  constexpr int WM = 16 * FM, WN = 16 * FN;
  const int tiles_m = int(g.m_pad / (2 * WM));
  int tm, tn;
  tile_of(blockIdx.x, gridDim.x, tiles_m, &tm, &tn);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = lane & 15, kg = lane >> 4;
  const int64_t m0 = int64_t(tm) * (2 * WM) + (wave & 1) * WM;
  const int64_t n0 = int64_t(tn) * (2 * WN) + (wave >> 1) * WN;
  const uint8_t* pm = g.opm + (m0 + r) * g.row_bytes + g.k_byte_off + kg * 16;
  const uint8_t* pn = g.opn + (n0 + r) * g.row_bytes + g.k_byte_off + kg * 16;
  const int64_t fstride = 16 * g.row_bytes;

  using Acc = std::conditional_t<F4, v4f, v4i>;
  Acc acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = Acc{0, 0, 0, 0};

  v4i am[FM], bn[FN];
#pragma unroll
  for (int i = 0; i < FM; ++i) am[i] = *reinterpret_cast<const v4i*>(pm + i * fstride);
#pragma unroll
  for (int j = 0; j < FN; ++j) bn[j] = *reinterpret_cast<const v4i*>(pn + j * fstride);

  for (int64_t kb = 0; kb < g.kblocks; ++kb) {
    // next block's operands, loaded while this block is multiplied
    const int64_t nx = (kb + 1 < g.kblocks ? kb + 1 : kb) * 64;
    v4i am2[FM], bn2[FN];
#pragma unroll
    for (int i = 0; i < FM; ++i) am2[i] = *reinterpret_cast<const v4i*>(pm + i * fstride + nx);
#pragma unroll
    for (int j = 0; j < FN; ++j) bn2[j] = *reinterpret_cast<const v4i*>(pn + j * fstride + nx);

    if constexpr (F4) {
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        v8i ea[FM], eb[FN];
#pragma unroll
        for (int i = 0; i < FM; ++i) ea[i] = fp4_operand_m(uint32_t(am[i][w]));
#pragma unroll
        for (int j = 0; j < FN; ++j) eb[j] = fp4_operand_n(uint32_t(bn[j][w]));
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                ea[i], eb[j], acc[i][j], kFmtE2M1, kFmtE2M1, 0, kNoScale, 0, kNoScale);
      }
    } else {
      const int mask = 0x01010101;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          v4i ea[FM], eb[FN];
#pragma unroll
          for (int i = 0; i < FM; ++i) {
            const uint32_t x = uint32_t(am[i][w]);
            ea[i] = v4i{int((x >> (4 * h + 0)) & mask), int((x >> (4 * h + 1)) & mask),
                        int((x >> (4 * h + 2)) & mask), int((x >> (4 * h + 3)) & mask)};
          }
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            const uint32_t x = uint32_t(bn[j][w]);
            eb[j] = v4i{int((x >> (4 * h + 0)) & mask), int((x >> (4 * h + 1)) & mask),
                        int((x >> (4 * h + 2)) & mask), int((x >> (4 * h + 3)) & mask)};
          }
#pragma unroll
          for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ea[i], eb[j], acc[i][j], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) am[i] = am2[i];
#pragma unroll
    for (int j = 0; j < FN; ++j) bn[j] = bn2[j];
  }

  const Epi e{g.mode,   g.layout, g.pa,        g.pb,    g.n,     g.kchunk, g.sum_a, g.sum_b,
              g.csum_a, g.csum_b, g.gamma,     g.gamma_f32, g.numer, g.acc64,  g.acc32};
  const double y = 1.0 / (double(g.n) * double(g.n));
  // Output element (row 4*kg + t, column r) of each 16 x 16 tile.
#pragma clang loop unroll(full)
  for (int i = 0; i < FM; ++i)
#pragma clang loop unroll(full)
    for (int j = 0; j < FN; ++j)
#pragma clang loop unroll(full)
      for (int t = 0; t < 4; ++t) {
        const int64_t q = m0 + 16 * i + 4 * kg + t;
        const int64_t p = n0 + 16 * j + r;
        if (q >= e.pb || p >= e.pa) continue;
        const SideSum a = side_sum<MODE>(e.sum_a, e.csum_a, p);
        const SideSum b = side_sum<MODE>(e.sum_b, e.csum_b, q);
        if (e.layout == CPI_GAMMA_VIEW_MAJOR)
          store_result<MODE, true>(e, y, true, q, p, int64_t(acc[i][j][t]), 0, a, b);
        else
          store_result<MODE, false>(e, y, true, q, p, int64_t(acc[i][j][t]), 0, a, b);
      }
}

// ---- Bit-row contraction fed through an LDS pipeline ----------------------
// FP4 (k_gemm_f4lds) or int8 (k_gemm_i8lds) matrix-core ops on bit rows, with
// the expansions of the register-fed kernel above.
// A work-group computes a 128 x 128 tile (2 x 2 waves of 64 x 64).  Each
// 512-frame block needs 256 operand rows x 64 bytes = 16 KB, which direct
// global->LDS copies (no registers) bring into one of S stages, S - 1 blocks
// ahead of the block being multiplied; one barrier per block.  Each row
// segment is fetched once per work-group.
//
// Stage layout: 16 groups of 16 rows (groups 0-7: M rows, 8-15: N rows),
// 1 KB each, one copy instruction per group.  Chunk c (16 bytes) of row r of
// a group sits at slot 4r + (c ^ lds_swizzle(r)).
//
// LDS reads are issued by inline asm: the compiler would otherwise wait for
// every outstanding global->LDS copy before each LDS read, serializing the
// pipeline.  Ordering is explicit instead: each wave waits for its own copies
// of the block (vmcnt), then a barrier makes every wave's copies visible and
// guarantees that the stage about to be refilled has been read by all waves.
typedef __attribute__((address_space(3))) void* lds_ptr_t;

// A 16-byte LDS read serves 16 lanes at a time: lanes 0-3, 12-15 and 20-27
// together, and 4-11, 16-19 and 28-31 (likewise in the upper half).  A
// fragment's lane 16 kg + r reads chunk kg of row r, so a group holds rows 0-3
// and 12-15 of one chunk and rows 4-11 of the next, or the reverse: with this
// exchange of the chunks of rows 4q .. 4q + 3 (0, 2, 3, 1 for q = 0 .. 3) either
// covers all banks once.  (With q itself every read took 12 clocks instead of
// 8: 1.2e8 conflict cycles per 1.4 ms byte contraction.)
__device__ __forceinline__ int lds_swizzle(int r) { return (0x78 >> (2 * (r >> 2))) & 3; }

// Eight 16-byte LDS reads and the wait for them, as one unit.
__device__ __forceinline__ void lds_read8(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3,
                                          uint32_t a4, uint32_t a5, uint32_t a6, uint32_t a7,
                                          v4i (&x)[4], v4i (&y)[4]) {
  asm volatile(
      "ds_read_b128 %0, %8\n"
      "ds_read_b128 %1, %9\n"
      "ds_read_b128 %2, %10\n"
      "ds_read_b128 %3, %11\n"
      "ds_read_b128 %4, %12\n"
      "ds_read_b128 %5, %13\n"
      "ds_read_b128 %6, %14\n"
      "ds_read_b128 %7, %15\n"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(y[0]), "=&v"(y[1]),
        "=&v"(y[2]), "=&v"(y[3])
      : "v"(a0), "v"(a1), "v"(a2), "v"(a3), "v"(a4), "v"(a5), "v"(a6), "v"(a7));
}

template <int S>
__device__ __forceinline__ void wait_copies() {
  // s_waitcnt vmcnt(4 * (S - 2)), expcnt and lgkmcnt left open
  static_assert(S >= 2 && 4 * (S - 2) < 16, "stage count");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (4 * (S - 2)));
}

// __launch_bounds__(256, 2) makes the compiler fit the kernel in about 168
// registers (no spills), so that three work-groups share a CU (the LDS limit):
// measured 12% faster than its unconstrained allocation (240 registers, two
// work-groups) on Da 128 x 128, Db 64 x 64, 20000 frames.
constexpr int kLdsStage = 16384;   // bytes per stage

template <int MODE, int S, bool I8>
__device__ __forceinline__ void gemm_lds(const GemmArgs& g, uint8_t* stage) {
  if (g.cond) {
    const uint32_t mx = g.stats[0];
    if ((g.cond == 1) != (mx <= 1u)) return;
  }
  constexpr int kStage = kLdsStage;
  const int tiles_m = int(g.m_pad / 128);
  int tm, tn;
  tile_of(blockIdx.x, gridDim.x, tiles_m, &tm, &tn);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int64_t mb = int64_t(tm) * 128, nb = int64_t(tn) * 128;

  // copy side: waves 0-1 copy the 128 M rows, waves 2-3 the 128 N rows, 64
  // rows (4 groups) each; lane -> (row, chunk) within a group
  const int cr = lane >> 2;
  const int cc = (lane & 3) ^ lds_swizzle(cr);
  const uint8_t* wbase = wave < 2 ? g.opm + (mb + 64 * wave) * g.row_bytes
                                  : g.opn + (nb + 64 * (wave - 2)) * g.row_bytes;
  // wave-uniform base + 32-bit lane offset (scalar-base addressing)
  const uint8_t* ubase = wbase + g.k_byte_off;
  const uint32_t loff = uint32_t(cr * g.row_bytes + 16 * cc);
  const int64_t gstride = 16 * g.row_bytes;
  const uint32_t lds0 = uint32_t(reinterpret_cast<uintptr_t>(stage));
  auto copy_block = [&](int64_t kb, int st) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      __builtin_amdgcn_global_load_lds(ubase + (q * gstride + kb * 64) + loff,
                                       (lds_ptr_t)(stage + st * kStage + (wave * 4 + q) * 1024),
                                       16, 0, 0);
  };

  // read side
  const int wm = wave & 1, wn = wave >> 1;
  const int r = lane & 15, kg = lane >> 4;
  const uint32_t roff = uint32_t(r * 64 + 16 * (kg ^ lds_swizzle(r)));

  using Acc = std::conditional_t<I8, v4i, v4f>;
  Acc acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = Acc{0, 0, 0, 0};

  const int64_t last = g.kblocks - 1;
#pragma unroll
  for (int p = 0; p < S - 1; ++p) copy_block(p < last ? p : last, p);

  int st = 0;
  for (int64_t kb = 0; kb < g.kblocks; ++kb) {
    wait_copies<S>();
    __builtin_amdgcn_s_barrier();
    {
      const int64_t nxt = kb + S - 1;
      const int ns = st == 0 ? S - 1 : st - 1;   // (kb + S - 1) % S
      copy_block(nxt < last ? nxt : last, ns);
    }
    const uint32_t base = lds0 + uint32_t(st * kStage) + roff;
    const uint32_t ba = base + wm * 4096, bb = base + 8192 + wn * 4096;
    v4i am[4], bn[4];
    lds_read8(ba, ba + 1024, ba + 2048, ba + 3072, bb, bb + 1024, bb + 2048, bb + 3072, am, bn);
    if constexpr (I8) {
      const int mask = 0x01010101;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          v4i ea[4], eb[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const uint32_t x = uint32_t(am[i][w]);
            ea[i] = v4i{int((x >> (4 * h + 0)) & mask), int((x >> (4 * h + 1)) & mask),
                        int((x >> (4 * h + 2)) & mask), int((x >> (4 * h + 3)) & mask)};
          }
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const uint32_t x = uint32_t(bn[j][w]);
            eb[j] = v4i{int((x >> (4 * h + 0)) & mask), int((x >> (4 * h + 1)) & mask),
                        int((x >> (4 * h + 2)) & mask), int((x >> (4 * h + 3)) & mask)};
          }
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ea[i], eb[j], acc[i][j], 0, 0, 0);
        }
      }
    } else {
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        v8i ea[4], eb[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) ea[i] = fp4_operand_m(uint32_t(am[i][w]));
#pragma unroll
        for (int j = 0; j < 4; ++j) eb[j] = fp4_operand_n(uint32_t(bn[j][w]));
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                ea[i], eb[j], acc[i][j], kFmtE2M1, kFmtE2M1, 0, kNoScale, 0, kNoScale);
      }
    }
    st = st == S - 1 ? 0 : st + 1;
  }
  // the last copies (clamped repeats of the final block) are still in flight;
  // every wave must also be done with the stages before they are reused
  __builtin_amdgcn_s_waitcnt(0x0F70);
  __syncthreads();

  // Epilogue through LDS, one half of the tile (64 rows) at a time: the two
  // waves owning those rows store their sums (exact integers) into a padded
  // row-major tile, which the whole work-group then writes out.
  static_assert(64 * 132 * 4 + sums_bytes(64, 128) <= S * kStage, "epilogue tile fits the stages");
  int32_t* tile = reinterpret_cast<int32_t*>(stage);
  SideSum* sums = reinterpret_cast<SideSum*>(stage + 64 * 132 * 4);
  const Epi e{g.mode,   g.layout, g.pa,        g.pb,    g.n,     g.kchunk, g.sum_a, g.sum_b,
              g.csum_a, g.csum_b, g.gamma,     g.gamma_f32, g.numer, g.acc64,  g.acc32};
  const int pitch = tile_pitch(e, 128);
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    if (wm == h) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int u = 0; u < 4; ++u)
            tile[(16 * i + 4 * kg + u) * pitch + wn * 64 + 16 * j + r] = int32_t(acc[i][j][u]);
    }
    stage_sums<MODE, true, 64, 128>(e, sums, mb + 64 * h, nb);
    __syncthreads();
    store_tile<MODE, true, 64, 128, 256>(e, tile, sums, pitch, mb + 64 * h, nb, 0, 0);
    __syncthreads();
  }
}

template <int MODE, int S>
__global__ __launch_bounds__(256, 2) void k_gemm_f4lds(GemmArgs g) {
  __shared__ __attribute__((aligned(16))) uint8_t stage[S * kLdsStage];
  gemm_lds<MODE, S, false>(g, stage);
}

template <int MODE, int S>
__global__ __launch_bounds__(256, 2) void k_gemm_i8lds(GemmArgs g) {
  __shared__ __attribute__((aligned(16))) uint8_t stage[S * kLdsStage];
  gemm_lds<MODE, S, true>(g, stage);
}

// ---- Byte-row contraction --------------------------------------------------
// int8 matrix-core ops on byte rows.  A K step covers only 64 frames of a
// 64-byte row segment (a bit row's covers 512), so operand bytes per
// multiply-add are eight times those of the bit kernel and the tile has to be
// larger: 256 x 256 per work-group (8 waves of 128 x 64, two per SIMD) moves
// 32 KB into LDS per 1024 matrix-core clocks of a CU, half of what its L1
// delivers; a 128 x 128 tile would need all of it.  Small problems, whose
// 256 x 256 tiles would leave most CUs idle, take 64 x 64 tiles (4 waves of
// 32 x 32).  Stages, copies, swizzle and waits are those of the bit kernel.
// Values above 127 (stats[1]) are offset by -128 in registers: the sign bit of
// every byte is flipped.  The zero bytes of pad frames then count 128 * 128
// each, which the epilogue subtracts.
// Measured (Da 128 x 128, Db 64 x 64, 20000 frames): 1.24 ms, 2.2 POP/s; the
// register-fed form with its element-wise epilogue took 3.66 ms.

// The 16-byte LDS reads of a K step's fragments (2048 bytes apart in the large
// tile's stages, 1024 in the small one's) and the wait for them, as one unit.
__device__ __forceinline__ void lds_read_frags(uint32_t a, uint32_t b, v4i (&x)[8], v4i (&y)[4]) {
  asm volatile(
      "ds_read_b128 %0, %12\n"
      "ds_read_b128 %8, %13\n"
      "ds_read_b128 %9, %13 offset:2048\n"
      "ds_read_b128 %10, %13 offset:4096\n"
      "ds_read_b128 %11, %13 offset:6144\n"
      "ds_read_b128 %1, %12 offset:2048\n"
      "ds_read_b128 %2, %12 offset:4096\n"
      "ds_read_b128 %3, %12 offset:6144\n"
      "ds_read_b128 %4, %12 offset:8192\n"
      "ds_read_b128 %5, %12 offset:10240\n"
      "ds_read_b128 %6, %12 offset:12288\n"
      "ds_read_b128 %7, %12 offset:14336\n"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(x[4]), "=&v"(x[5]),
        "=&v"(x[6]), "=&v"(x[7]), "=&v"(y[0]), "=&v"(y[1]), "=&v"(y[2]), "=&v"(y[3])
      : "v"(a), "v"(b));
}
__device__ __forceinline__ void lds_read_frags(uint32_t a, uint32_t b, v4i (&x)[2], v4i (&y)[2]) {
  asm volatile(
      "ds_read_b128 %0, %4\n"
      "ds_read_b128 %2, %5\n"
      "ds_read_b128 %1, %4 offset:1024\n"
      "ds_read_b128 %3, %5 offset:1024\n"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(x[0]), "=&v"(x[1]), "=&v"(y[0]), "=&v"(y[1])
      : "v"(a), "v"(b));
}

// One K step of the 256 x 256 tile as one block: the reads of the next step's
// fragments (xn, yn) from LDS are issued ahead of this step's matrix ops on
// (x, y) and waited for behind them.  All waves of a work-group run in step, so
// a read that is waited for before its own matrix ops leaves the matrix cores
// idle meanwhile.  The last sums are still being written when the block ends:
// between two blocks nothing but matrix ops may touch them, which the compiler
// does not know and test_host_mfma_wait checks in its output.  (Waiting inside the
// block, 11 states, took a call on 20000 frames of counts, Da 128 x 128, Db
// 64 x 64, from 1539 to 1563 us.)
__device__ __forceinline__ void bytes_step(uint32_t a, uint32_t b, const v4i (&x)[8],
                                           const v4i (&y)[4], v4i (&xn)[8], v4i (&yn)[4],
                                           v4i (&acc)[8][4]) {
  asm volatile(
      "ds_read_b128 %[x0], %[pa]\n"
      "ds_read_b128 %[y0], %[pb]\n"
      "ds_read_b128 %[y1], %[pb] offset:2048\n"
      "ds_read_b128 %[y2], %[pb] offset:4096\n"
      "ds_read_b128 %[y3], %[pb] offset:6144\n"
      "ds_read_b128 %[x1], %[pa] offset:2048\n"
      "ds_read_b128 %[x2], %[pa] offset:4096\n"
      "ds_read_b128 %[x3], %[pa] offset:6144\n"
      "ds_read_b128 %[x4], %[pa] offset:8192\n"
      "ds_read_b128 %[x5], %[pa] offset:10240\n"
      "ds_read_b128 %[x6], %[pa] offset:12288\n"
      "ds_read_b128 %[x7], %[pa] offset:14336\n"
      "v_mfma_i32_16x16x64_i8 %0, %[a0], %[b0], %0\n"
      "v_mfma_i32_16x16x64_i8 %1, %[a0], %[b1], %1\n"
      "v_mfma_i32_16x16x64_i8 %2, %[a0], %[b2], %2\n"
      "v_mfma_i32_16x16x64_i8 %3, %[a0], %[b3], %3\n"
      "v_mfma_i32_16x16x64_i8 %4, %[a1], %[b0], %4\n"
      "v_mfma_i32_16x16x64_i8 %5, %[a1], %[b1], %5\n"
      "v_mfma_i32_16x16x64_i8 %6, %[a1], %[b2], %6\n"
      "v_mfma_i32_16x16x64_i8 %7, %[a1], %[b3], %7\n"
      "v_mfma_i32_16x16x64_i8 %8, %[a2], %[b0], %8\n"
      "v_mfma_i32_16x16x64_i8 %9, %[a2], %[b1], %9\n"
      "v_mfma_i32_16x16x64_i8 %10, %[a2], %[b2], %10\n"
      "v_mfma_i32_16x16x64_i8 %11, %[a2], %[b3], %11\n"
      "v_mfma_i32_16x16x64_i8 %12, %[a3], %[b0], %12\n"
      "v_mfma_i32_16x16x64_i8 %13, %[a3], %[b1], %13\n"
      "v_mfma_i32_16x16x64_i8 %14, %[a3], %[b2], %14\n"
      "v_mfma_i32_16x16x64_i8 %15, %[a3], %[b3], %15\n"
      "v_mfma_i32_16x16x64_i8 %16, %[a4], %[b0], %16\n"
      "v_mfma_i32_16x16x64_i8 %17, %[a4], %[b1], %17\n"
      "v_mfma_i32_16x16x64_i8 %18, %[a4], %[b2], %18\n"
      "v_mfma_i32_16x16x64_i8 %19, %[a4], %[b3], %19\n"
      "v_mfma_i32_16x16x64_i8 %20, %[a5], %[b0], %20\n"
      "v_mfma_i32_16x16x64_i8 %21, %[a5], %[b1], %21\n"
      "v_mfma_i32_16x16x64_i8 %22, %[a5], %[b2], %22\n"
      "v_mfma_i32_16x16x64_i8 %23, %[a5], %[b3], %23\n"
      "v_mfma_i32_16x16x64_i8 %24, %[a6], %[b0], %24\n"
      "v_mfma_i32_16x16x64_i8 %25, %[a6], %[b1], %25\n"
      "v_mfma_i32_16x16x64_i8 %26, %[a6], %[b2], %26\n"
      "v_mfma_i32_16x16x64_i8 %27, %[a6], %[b3], %27\n"
      "v_mfma_i32_16x16x64_i8 %28, %[a7], %[b0], %28\n"
      "v_mfma_i32_16x16x64_i8 %29, %[a7], %[b1], %29\n"
      "v_mfma_i32_16x16x64_i8 %30, %[a7], %[b2], %30\n"
      "v_mfma_i32_16x16x64_i8 %31, %[a7], %[b3], %31\n"
      "s_waitcnt lgkmcnt(0)"
      : "+v"(acc[0][0]), "+v"(acc[0][1]), "+v"(acc[0][2]), "+v"(acc[0][3]), "+v"(acc[1][0]),
        "+v"(acc[1][1]), "+v"(acc[1][2]), "+v"(acc[1][3]), "+v"(acc[2][0]), "+v"(acc[2][1]),
        "+v"(acc[2][2]), "+v"(acc[2][3]), "+v"(acc[3][0]), "+v"(acc[3][1]), "+v"(acc[3][2]),
        "+v"(acc[3][3]), "+v"(acc[4][0]), "+v"(acc[4][1]), "+v"(acc[4][2]), "+v"(acc[4][3]),
        "+v"(acc[5][0]), "+v"(acc[5][1]), "+v"(acc[5][2]), "+v"(acc[5][3]), "+v"(acc[6][0]),
        "+v"(acc[6][1]), "+v"(acc[6][2]), "+v"(acc[6][3]), "+v"(acc[7][0]), "+v"(acc[7][1]),
        "+v"(acc[7][2]), "+v"(acc[7][3]),
        [x0] "=&v"(xn[0]), [x1] "=&v"(xn[1]), [x2] "=&v"(xn[2]), [x3] "=&v"(xn[3]),
        [x4] "=&v"(xn[4]), [x5] "=&v"(xn[5]), [x6] "=&v"(xn[6]), [x7] "=&v"(xn[7]),
        [y0] "=&v"(yn[0]), [y1] "=&v"(yn[1]), [y2] "=&v"(yn[2]), [y3] "=&v"(yn[3])
      : [pa] "v"(a), [pb] "v"(b), [a0] "v"(x[0]), [a1] "v"(x[1]), [a2] "v"(x[2]), [a3] "v"(x[3]),
        [a4] "v"(x[4]), [a5] "v"(x[5]), [a6] "v"(x[6]), [a7] "v"(x[7]), [b0] "v"(y[0]),
        [b1] "v"(y[1]), [b2] "v"(y[2]), [b3] "v"(y[3]));
}

// Epilogue of a byte tile through LDS (BYTES of it), 16 FM' rows of every wave
// row at a time (FM' = 4 or FM): 64 rows or the whole tile.
template <int MODE, int FM, int FN, int WM, int WN, int BYTES>
__device__ __forceinline__ void bytes_epilogue(const GemmArgs& g, uint8_t* stage,
                                               const v4i (&acc)[FM][FN], int64_t mb, int64_t nb,
                                               bool offset) {
  constexpr int TM = 16 * FM * WM, TN = 16 * FN * WN, T = 64 * WM * WN;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int wm = wave % WM, wn = wave / WM;
  const int r = lane & 15, kg = lane >> 4;
  constexpr int FP = FM < 4 ? FM : 4;            // fragment rows per pass
  constexpr int ROWS = FM < 4 ? TM : 16 * FP;    // rows staged per pass
  constexpr int PASSES = TM / ROWS;
  static_assert(ROWS * (TN + 4) * 4 + sums_bytes(ROWS, TN) <= BYTES,
                "epilogue tile fits the stages");
  constexpr bool quads = MODE == EPI_FINAL || MODE == EPI_STREAM64;
  static_assert(PASSES == 1 || PASSES == WM * FM / FP, "epilogue passes");
  int32_t* tile = reinterpret_cast<int32_t*>(stage);
  SideSum* sums = reinterpret_cast<SideSum*>(stage + ROWS * (TN + 4) * 4);
  const Epi e{g.mode,   g.layout, g.pa,        g.pb,    g.n,     g.kchunk, g.sum_a, g.sum_b,
              g.csum_a, g.csum_b, g.gamma,     g.gamma_f32, g.numer, g.acc64,  g.acc32};
  const int64_t o = offset ? 128 : 0;
  const int32_t pad = offset ? int32_t(g.pad_frames) << 14 : 0;
  const int pitch = tile_pitch(e, TN);
#pragma unroll
  for (int h = 0; h < PASSES; ++h) {
    if (PASSES == 1 || wm == h / (FM / FP)) {
#pragma unroll
      for (int i = 0; i < FP; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
          for (int u = 0; u < 4; ++u)
            tile[((PASSES == 1 ? wm * 16 * FM : 0) + 16 * i + 4 * kg + u) * pitch +
                 wn * 16 * FN + 16 * j + r] = acc[h % (FM / FP) * FP + i][j][u];
    }
    stage_sums<MODE, quads, ROWS, TN>(e, sums, mb + ROWS * h, nb);
    __syncthreads();
    store_tile<MODE, quads, ROWS, TN, T>(e, tile, sums, pitch, mb + ROWS * h, nb, o, pad);
    __syncthreads();
  }
}

template <int N>
__device__ __forceinline__ void flip_signs(v4i (&x)[N]) {
  const int m = int(0x80808080u);
#pragma unroll
  for (int i = 0; i < N; ++i) x[i] ^= v4i{m, m, m, m};
}

template <int MODE, int FM, int FN, int WM, int WN, int S>
__device__ __forceinline__ void gemm_bytes(const GemmArgs& g, uint8_t* stage) {
  constexpr int NW = WM * WN, T = 64 * NW;
  constexpr int TM = 16 * FM * WM, TN = 16 * FN * WN;
  constexpr int kStage = (TM + TN) * 64;            // bytes per stage
  constexpr int CPW = (TM + TN) / 16 / NW;          // copies (16 rows, 1 KB) per wave
  static_assert(CPW * NW * 16 == TM + TN && CPW * (S - 2) < 16, "copies per wave");
  if (g.cond) {
    const uint32_t mx = g.stats[0];
    if ((g.cond == 1) != (mx <= 1u)) return;
  }
  int tm, tn;
  tile_of(blockIdx.x, gridDim.x, int(g.m_pad / TM), &tm, &tn);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int64_t mb = int64_t(tm) * TM, nb = int64_t(tn) * TN;

  // copy side: wave w copies row groups w CPW .. (groups of 16 rows, M rows
  // first); lane -> (row, chunk) within a group
  const int cr = lane >> 2;
  const int cc = (lane & 3) ^ lds_swizzle(cr);
  const uint32_t loff = uint32_t(cr * g.row_bytes + 16 * cc);
  const uint32_t lds0 = uint32_t(reinterpret_cast<uintptr_t>(stage));
  const uint8_t* src[CPW];
#pragma unroll
  for (int q = 0; q < CPW; ++q) {
    const int r = 16 * (wave * CPW + q);
    src[q] = (r < TM ? g.opm + (mb + r) * g.row_bytes : g.opn + (nb + r - TM) * g.row_bytes) +
             g.k_byte_off;
  }
  auto copy_block = [&](int64_t kb, int st) {
#pragma unroll
    for (int q = 0; q < CPW; ++q)
      __builtin_amdgcn_global_load_lds(src[q] + kb * 64 + loff,
                                       (lds_ptr_t)(stage + st * kStage + (wave * CPW + q) * 1024),
                                       16, 0, 0);
  };

  // read side
  const int wm = wave % WM, wn = wave / WM;
  const int r = lane & 15, kg = lane >> 4;
  const uint32_t roff = uint32_t(r * 64 + 16 * (kg ^ lds_swizzle(r)));
  const uint32_t ra = lds0 + roff + uint32_t(wm * FM * 1024);
  const uint32_t rb = lds0 + roff + uint32_t(TM * 64 + wn * FN * 1024);

  v4i acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = v4i{0, 0, 0, 0};

  const bool offset = g.offset_from_stats && g.stats[1] > 127u;
  const int64_t last = g.kblocks - 1;
#pragma unroll
  for (int p = 0; p < S - 1; ++p) copy_block(p < last ? p : last, p);

  int st = 0;
  for (int64_t kb = 0; kb < g.kblocks; ++kb) {
    // this wave's copies of block kb have landed; then everyone's have, and
    // the stage to be refilled has been read by all
    __builtin_amdgcn_s_waitcnt(0x0F70 | (CPW * (S - 2)));
    __builtin_amdgcn_s_barrier();
    const int64_t nxt = kb + S - 1;
    copy_block(nxt < last ? nxt : last, st == 0 ? S - 1 : st - 1);
    v4i am[FM], bn[FN];
    lds_read_frags(ra + uint32_t(st * kStage), rb + uint32_t(st * kStage), am, bn);
    if (offset) {
      flip_signs(am);
      flip_signs(bn);
    }
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(am[i], bn[j], acc[i][j], 0, 0, 0);
    st = st == S - 1 ? 0 : st + 1;
  }
  // the last copies (clamped repeats of the final block) are still in flight;
  // every wave must also be done with the stages before they are reused
  __builtin_amdgcn_s_waitcnt(0x0F70);
  __syncthreads();

  bytes_epilogue<MODE, FM, FN, WM, WN, S * kStage>(g, stage, acc, mb, nb, offset);
}

template <int MODE, int FM, int FN, int WM, int WN, int S>
__global__ __launch_bounds__(64 * WM * WN, 2) void k_gemm_bytes(GemmArgs g) {
  __shared__ __attribute__((aligned(16))) uint8_t stage[S * 16 * (FM * WM + FN * WN) * 64];
  gemm_bytes<MODE, FM, FN, WM, WN, S>(g, stage);
}

// The 256 x 256 tile.  Copies take 128 bytes (two K steps) of a row at a time, whole
// lines, which L2 serves faster than 64-byte pieces (times below).
// Rows of a workspace of the reported size start at multiples of 128 bytes.
// Stage: 8 rows x 128 bytes per copy instruction, chunk c (16 bytes) of row r
// at slot 8 (r % 8) + (c ^ swz(r)), swz chosen as lds_swizzle is, for 128-byte
// rows.  Two stages of 64 KB; a stage is refilled as soon as the fragments of
// its second half are in registers, half a stage's work before the other stage
// runs out.  An odd last K step is read as the second half of the row's last
// 128 bytes.
// Measured (Da 128 x 128, Db 64 x 64, 20000 frames): 1.24 ms; with 64-byte copies
// 1.39 ms (four or five stages alike), with 128-byte copies of rows that start
// at odd multiples of 64 bytes 1.33 ms.  The matrix ops take 0.60 ms of it at the
// rate of a register-only loop of them (4.46 POP/s).
constexpr int kBigStage = 65536;

template <int MODE>
__device__ __forceinline__ void gemm_bytes_big(const GemmArgs& g, uint8_t* stage) {
  constexpr int FM = 8, FN = 4, WM = 2, WN = 4, CPW = 8;
  if (g.cond) {
    const uint32_t mx = g.stats[0];
    if ((g.cond == 1) != (mx <= 1u)) return;
  }
  int tm, tn;
  tile_of(blockIdx.x, gridDim.x, int(g.m_pad / 256), &tm, &tn);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int64_t mb = int64_t(tm) * 256, nb = int64_t(tn) * 256;

  // copy side: waves 0-3 copy the 256 M rows, 4-7 the N rows, 64 rows each;
  // lane: row lane / 8 of the instruction's 8, 16 bytes of it
  auto swz = [](int r) { return ((r >> 1) & 1) << 1 | ((r >> 3) & 1) << 2; };
  const uint8_t* src = (wave < 4 ? g.opm + (mb + 64 * wave) * g.row_bytes
                                 : g.opn + (nb + 64 * (wave - 4)) * g.row_bytes) +
                       g.k_byte_off;
  const int cr = lane >> 3;
  const uint32_t l0 = uint32_t(cr * g.row_bytes) + uint32_t(16 * ((lane & 7) ^ swz(cr)));
  const uint32_t l1 = uint32_t(cr * g.row_bytes) + uint32_t(16 * ((lane & 7) ^ swz(8 + cr)));
  const uint32_t lds0 = uint32_t(reinterpret_cast<uintptr_t>(stage));
  const int64_t lastoff = 64 * g.kblocks - 128;
  auto copy = [&](int64_t d) {   // 128 bytes of every row, double step d
    const int64_t off = 128 * d < lastoff ? 128 * d : lastoff;
    uint8_t* dst = stage + (d & 1) * kBigStage + wave * (CPW * 1024);
#pragma unroll
    for (int q = 0; q < CPW; ++q)
      __builtin_amdgcn_global_load_lds(src + (8 * q * g.row_bytes + off) + ((q & 1) ? l1 : l0),
                                       (lds_ptr_t)(dst + q * 1024), 16, 0, 0);
  };

  // read side: fragment i of 16 rows at 2048 i; K half h at address ^ 64 h
  const int wm = wave % WM, wn = wave / WM;
  const int r = lane & 15, kg = lane >> 4;
  const uint32_t roff = uint32_t((r >> 3) * 1024 + (r & 7) * 128 + 16 * (kg ^ swz(r)));
  const uint32_t ra = lds0 + uint32_t(wm * FM * 2048) + roff;
  const uint32_t rb = lds0 + uint32_t(32768 + wn * FN * 2048) + roff;

  v4i acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = v4i{0, 0, 0, 0};
  const bool offset = g.offset_from_stats && g.stats[1] > 127u;
  const int64_t full = g.kblocks / 2;             // whole double steps
  const int64_t last = (g.kblocks + 1) / 2 - 1;   // last double step
  v4i x0[FM], y0[FN], x1[FM], y1[FN];
  copy(0);
  __builtin_amdgcn_s_waitcnt(0x0F70);
  __builtin_amdgcn_s_barrier();
  if (last > 0) copy(1);
  lds_read_frags(ra, rb, x0, y0);
  if (offset) {
    flip_signs(x0);
    flip_signs(y0);
  }
  for (int64_t d = 0; d < full; ++d) {
    const uint32_t s0 = uint32_t((d & 1) * kBigStage), s1 = kBigStage - s0;
    // first half (in x0, y0) while the second is read
    bytes_step((ra + s0) ^ 64u, (rb + s0) ^ 64u, x0, y0, x1, y1, acc);
    if (offset) {
      flip_signs(x1);
      flip_signs(y1);
    }
    // the next double step has landed for this wave, then for all; and all
    // have read this one's stage, which the one after next refills
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __builtin_amdgcn_s_barrier();
    if (d + 2 <= last) copy(d + 2);
    const uint32_t h = d + 1 < full ? 0u : 64u;   // (an odd last step is a second half)
    bytes_step((ra + s1) ^ h, (rb + s1) ^ h, x1, y1, x0, y0, acc);
    if (offset) {
      flip_signs(x0);
      flip_signs(y0);
    }
  }
  if (g.kblocks & 1)   // (reads x1, y1 once more, not used)
    bytes_step(ra, rb, x0, y0, x1, y1, acc);
  // (the sums are read by ordinary instructions from here on, no earlier)
  asm volatile("s_nop 15\ns_nop 15" ::: "memory");
  __syncthreads();
  bytes_epilogue<MODE, FM, FN, WM, WN, 2 * kBigStage>(g, stage, acc, mb, nb, offset);
}

template <int MODE>
__global__ __launch_bounds__(512, 2) void k_gemm_bytes_big(GemmArgs g) {
  __shared__ __attribute__((aligned(1024))) uint8_t stage[2 * kBigStage];
  gemm_bytes_big<MODE>(g, stage);
}

// One thread per Gamma element of a streaming state.
__global__ __launch_bounds__(256) void k_state_gamma(const void* __restrict__ sab, int sab64,
                                                     const int64_t* __restrict__ sum_a,
                                                     const int64_t* __restrict__ sum_b, int64_t n,
                                                     int64_t pa, int64_t pb, int layout,
                                                     double* __restrict__ gamma,
                                                     float* __restrict__ gamma_f32,
                                                     int64_t* __restrict__ numer) {
  const int64_t count = pa * pb;
  const double nn = double(n) * double(n);
  for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < count;
       i += int64_t(gridDim.x) * 256) {
    const int64_t q = i / pa, p = i - q * pa;   // view-major element (q, p)
    const int64_t s = sab64 ? reinterpret_cast<const int64_t*>(sab)[i]
                            : int64_t(reinterpret_cast<const int32_t*>(sab)[i]);
    const int64_t num = n * s - sum_a[p] * sum_b[q];
    const double gam = double(num) / nn;
    const int64_t idx = (layout == CPI_GAMMA_VIEW_MAJOR) ? i : p * pb + q;
    if (gamma) __builtin_nontemporal_store(gam, gamma + idx);
    if (gamma_f32) __builtin_nontemporal_store(float(gam), gamma_f32 + idx);
    if (numer) __builtin_nontemporal_store(num, numer + idx);
  }
}

// CPI_GEMM_FEED=regs selects the register-fed kernels for bit rows
// (measurement runs); the default feeds the matrix cores through the LDS
// pipeline.
bool fp4_from_registers() {
  static const bool on = [] {
    const char* v = std::getenv("CPI_GEMM_FEED");
    return v && std::strcmp(v, "regs") == 0;
  }();
  return on;
}

template <int FM, int FN, int MODE, bool F4>
hipError_t launch_gemm(const GemmArgs& a, hipStream_t s) {
  const int64_t tiles_m = a.m_pad / (32 * FM);
  const int64_t tiles_n = a.n_pad / (32 * FN);
  if (tiles_m * (32 * FM) != a.m_pad || tiles_n * (32 * FN) != a.n_pad) return hipErrorInvalidValue;
  const int64_t nwg = tiles_m * tiles_n;
  if (nwg <= 0 || nwg > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_gemm<FM, FN, MODE, F4>), dim3(unsigned(nwg)), dim3(256), 0, s, a);
  return hipGetLastError();
}

// Matrix-core encoding of bit rows (CPI_MMA_AUTO or CPI_MMA_INT8), process-wide.
std::atomic<int> g_mma_encoding{[] {
  const char* v = std::getenv("CPI_GEMM_ENC");
  return (v && std::strcmp(v, "int8") == 0) ? int(CPI_MMA_INT8) : int(CPI_MMA_AUTO);
}()};

bool fp4_enabled() { return g_mma_encoding.load(std::memory_order_relaxed) == CPI_MMA_AUTO; }

constexpr int64_t kFp4MaxFrames = int64_t(1) << 24;

template <int MODE, int S, bool I8>
hipError_t launch_lds(const GemmArgs& a, hipStream_t s) {
  const int64_t tiles_m = a.m_pad / 128, tiles_n = a.n_pad / 128;
  if (tiles_m * 128 != a.m_pad || tiles_n * 128 != a.n_pad || a.kblocks < 1)
    return hipErrorInvalidValue;
  const int64_t nwg = tiles_m * tiles_n;
  if (nwg > 0x7fffffff) return hipErrorInvalidValue;
  if constexpr (I8)
    hipLaunchKernelGGL((k_gemm_i8lds<MODE, S>), dim3(unsigned(nwg)), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL((k_gemm_f4lds<MODE, S>), dim3(unsigned(nwg)), dim3(256), 0, s, a);
  return hipGetLastError();
}

template <int MODE>
hipError_t launch_bits(const GemmArgs& a, hipStream_t s) {
  if (a.fp4) {
    if (a.kblocks * 512 > kFp4MaxFrames) return hipErrorInvalidValue;
    if (fp4_from_registers()) return launch_gemm<4, 4, MODE, true>(a, s);
    return launch_lds<MODE, 3, false>(a, s);
  }
  if (fp4_from_registers()) return launch_gemm<4, 4, MODE, false>(a, s);
  return launch_lds<MODE, 3, true>(a, s);
}

// 256 x 256 tiles when they occupy at least half of the CUs (three quarters
// where K is short and filling the chip counts for more than operand traffic),
// else 64 x 64 tiles.  Whole calls with Da of 4096 pixels, small / large, us:
//   8000 frames, 64 tiles: 140 / 170, 96: 183 / 183, 128: 215 / 185, 192: 279 / 184
//   1000 frames, 128 tiles: 57 / 63, 192: 68 / 68, 256: 79 / 71
template <int MODE>
hipError_t launch_bytes(const GemmArgs& a, hipStream_t s) {
  if (a.m_pad % 256 != 0 || a.n_pad % 256 != 0 || a.kblocks < 1) return hipErrorInvalidValue;
  const int64_t big = (a.m_pad / 256) * (a.n_pad / 256);
  if (big * 16 > 0x7fffffff) return hipErrorInvalidValue;
  if (a.kblocks >= 2 && big >= (a.kblocks < 64 ? 192 : 128))
    hipLaunchKernelGGL((k_gemm_bytes_big<MODE>), dim3(unsigned(big)), dim3(512), 0, s, a);
  else
    hipLaunchKernelGGL((k_gemm_bytes<MODE, 2, 2, 2, 2, 4>), dim3(unsigned(16 * big)), dim3(256), 0,
                       s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t gemm_correlate(const GemmArgs& a, bool bits, hipStream_t s) {
  switch (a.mode) {
    case EPI_FINAL:
      return bits ? launch_bits<EPI_FINAL>(a, s) : launch_bytes<EPI_FINAL>(a, s);
    case EPI_STREAM64:
      return bits ? launch_bits<EPI_STREAM64>(a, s) : launch_bytes<EPI_STREAM64>(a, s);
    case EPI_STREAM32:
      return bits ? launch_bits<EPI_STREAM32>(a, s) : hipErrorInvalidValue;
    case EPI_FINAL_ACC64:
      return bits ? hipErrorInvalidValue : launch_bytes<EPI_FINAL_ACC64>(a, s);
    case EPI_STORE64:
      return bits ? hipErrorInvalidValue : launch_bytes<EPI_STORE64>(a, s);
    case EPI_ADD64:
      return bits ? hipErrorInvalidValue : launch_bytes<EPI_ADD64>(a, s);
    default:
      return hipErrorInvalidValue;
  }
}

bool bits_use_fp4(int64_t kblocks) { return fp4_enabled() && kblocks * 512 <= kFp4MaxFrames; }

void set_mma_encoding(int enc) { g_mma_encoding.store(enc, std::memory_order_relaxed); }
int get_mma_encoding() { return g_mma_encoding.load(std::memory_order_relaxed); }

hipError_t state_gamma(const void* sab, bool sab64, const int64_t* sum_a, const int64_t* sum_b,
                       int64_t n, int64_t pa, int64_t pb, int layout, double* gamma,
                       float* gamma_f32, int64_t* numer, hipStream_t s) {
  int64_t gr = (pa * pb + 255) / 256;
  if (gr > 65536) gr = 65536;
  hipLaunchKernelGGL(k_state_gamma, dim3(unsigned(gr)), dim3(256), 0, s, sab, sab64 ? 1 : 0, sum_a,
                     sum_b, n, pa, pb, layout, gamma, gamma_f32, numer);
  return hipGetLastError();
}

}  // namespace cpi
