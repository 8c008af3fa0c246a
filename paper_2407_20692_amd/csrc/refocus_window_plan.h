// Host-side plan of the register-window x pass of the refocus (no HIP
// dependencies, so that it can be built and tested with a plain host
// compiler), and the offsets that its kernels share.
#pragma once

#include <cstdint>

namespace cpi {

struct RefGeom {
  int wa, ha, wb, hb, out_w, out_h;
  double mag_x, mag_y, ca_x, ca_y, cb_x, cb_y;
};

constexpr int kWinSlots = 2;         // 64-row units per work-group, one row of each per lane
constexpr int kWinWaves = 4;         // waves per work-group
constexpr int kWinPairs = 64;        // (plane, column) pairs per wave
constexpr int kWinCols = 40;         // window columns a wave keeps in registers
constexpr int kWinBlocks = 9;        // 16-column blocks (8 KB each) that the LDS holds
constexpr int kWinBlockBytes = kWinSlots * 64 * 16 * 4;
constexpr int kWinLds = kWinBlocks * kWinBlockBytes;
constexpr int kWinMaxStages = 3;     // views staged at a time at most

// A staged window is a run of 4-column chunks, four to a 16-column block.
// Byte offset of chunk q from the window's start in LDS.
constexpr uint32_t window_chunk_at(int q) {
  return (uint32_t(q >> 2) * uint32_t(kWinBlockBytes)) | (uint32_t(q & 3) << 4);
}

// Where chunks q and q + 1 are, in one table word: in units of 16 bytes, 16
// bits each (nine blocks need 17 bits in bytes).
constexpr uint32_t window_pack_chunks(int q) {
  return (window_chunk_at(q) >> 4) | (window_chunk_at(q + 1) >> 4) << 16;
}
constexpr uint32_t window_unpack_chunk(uint32_t word, int k) {
  return (k ? word >> 16 : word & 0xffffu) << 4;
}
// (a wave's first chunk is one of the 4 kWinBlocks staged; its first four are packed)
static_assert((window_chunk_at(4 * kWinBlocks + 2) >> 4) <= 0xffffu,
              "chunk offsets fit their field");

// Byte offset, from a view's first staged column, of what lane `lane` of wave
// `wave` copies of each block's half `half`: four columns of one view row, of 16
// rows per half and two halves per wave, the unit's first row being `row`.  The
// whole row goes into this lane offset, so that rows past the view lie past the
// view's buffer descriptor, which then delivers zeros.  (A scalar offset for the
// second half would not be sure to count in that check, nor could it be taken
// off the descriptor's size where views have fewer than 16 rows.)
constexpr uint32_t window_lane_offset(int row, int wave, int lane, int half, int wa) {
  return uint32_t((row + 32 * (wave & 1) + 16 * half + (lane >> 2)) * wa +
                  4 * ((lane & 3) ^ ((lane >> 4) & 3))) *
         4u;
}

// Work split of the pass for a geometry and plane set, planes in chunks of
// `chunk`; false if it does not take them.
struct WindowSplit {
  int np = 0, xc = 0, pg = 0;   // planes x columns per wave, plane groups per work-group
  int na = 0, xr = 0;           // planes x columns per work-group
  int blocks = 0;               // 16-column blocks its windows take
};
bool window_split(const RefGeom& g, const double* alphas, int n_alpha, int64_t chunk,
                  WindowSplit* out);

// View rows that the samples of planes [p0, p1) span at most at any
// lens-plane row.
int window_rows(const RefGeom& g, const double* alphas, int p0, int p1);

}  // namespace cpi
