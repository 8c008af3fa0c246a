// Host-only checks of the register-window x pass's plan (no HIP): for evenly
// spaced, clustered, unordered and drawn plane lists, the windows of every
// work-group and wave at every view, as the column table forms them, lie in
// what the plan stages, and the chunk offsets read back from the table are
// those of the chunks; and copies of rows past a view are out of its bounds.  Built with the sanitizers.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "refocus_window_plan.h"

static int failures = 0;
#define CHECK(c)                                                        \
  do {                                                                  \
    if (!(c)) {                                                         \
      if (failures < 20) std::fprintf(stderr, "FAIL %s:%d: %s\n", __FILE__, __LINE__, #c); \
      ++failures;                                                       \
    }                                                                   \
  } while (0)

using namespace cpi;

static RefGeom geom(int wa, int ha, int wb, int hb, int out_w, int out_h) {
  return RefGeom{wa, ha, wb, hb, out_w, out_h, double(wa) / wb, double(ha) / hb, (wa - 1) / 2.0,
                 (ha - 1) / 2.0, (wb - 1) / 2.0, (hb - 1) / 2.0};
}

// the cell of pair (plane, column) at a view: first sample and whether it has one
static bool cell(const RefGeom& g, double al, int xr, int xb, int* c) {
  const double u = al * (xr - g.ca_x) + g.ca_x + (1.0 - al) * g.mag_x * (xb - g.cb_x);
  const double i = std::floor(u);
  if (i < -1 || i > g.wa - 1 || (i == -1 && u == i)) return false;
  *c = std::min(std::max(int(i), 0), g.wa - 2);
  return true;
}

static int far_waves = 0;   // waves whose first four chunks lie past the eighth block

static bool walk(const RefGeom& g, const std::vector<double>& al, WindowSplit* used = nullptr) {
  WindowSplit w;
  const int n = int(al.size());
  if (!window_split(g, al.data(), n, (n + 15) / 16 * 16, &w)) return false;
  if (used) *used = w;
  const int cg = kWinWaves / w.pg;
  const int tiles = (g.out_w + w.xr - 1) / w.xr, groups = (n + w.na - 1) / w.na;
  for (int gq = 0; gq < groups; ++gq)
    for (int t = 0; t < tiles; ++t)
      for (int xb = 0; xb < g.wb; ++xb) {
        int lo[kWinWaves], hi[kWinWaves];
        for (int wv = 0; wv < kWinWaves; ++wv) {
          lo[wv] = 1 << 30;
          hi[wv] = -1;
          for (int k = 0; k < kWinPairs; ++k) {
            const int pl = (gq * w.pg + wv / cg) * w.np + k / w.xc;
            const int xr = (t * cg + wv % cg) * w.xc + k % w.xc;
            int c = 0;
            if (pl >= n || xr >= g.out_w || !cell(g, al[size_t(pl)], xr, xb, &c)) continue;
            lo[wv] = std::min(lo[wv], c);
            hi[wv] = std::max(hi[wv], c);
          }
        }
        const int glo = *std::min_element(lo, lo + kWinWaves);
        const int ghi = *std::max_element(hi, hi + kWinWaves);
        if (ghi < 0) continue;
        const int wx0 = glo & ~3, blocks = (ghi + 1 - wx0) / 16 + 1;
        CHECK(blocks <= w.blocks && w.blocks <= kWinBlocks);
        for (int wv = 0; wv < kWinWaves; ++wv) {
          if (hi[wv] < 0) continue;
          const int q0 = (lo[wv] - wx0) >> 2, nq = ((hi[wv] + 1 - wx0) >> 2) - q0 + 1;
          CHECK(nq <= kWinCols / 4 && q0 + nq <= 4 * blocks);
          CHECK(hi[wv] - wx0 - 4 * q0 <= kWinCols - 2);
          const uint32_t word[2] = {window_pack_chunks(q0), window_pack_chunks(q0 + 2)};
          for (int i = 0; i < nq; ++i) {
            // chunk i is read 8 KB further on than chunk i - 4
            const uint32_t at = window_unpack_chunk(word[i >> 1 & 1], i & 1) +
                                uint32_t(i >> 2) * uint32_t(kWinBlockBytes);
            CHECK(at == window_chunk_at(q0 + i));
            CHECK(at < uint32_t(kWinLds));
          }
          if (q0 + std::min(nq, 4) > 32) ++far_waves;
        }
      }
  return true;
}

// Copies of views of every height around a wave's rows: what the buffer
// descriptor checks (the lane offset and the instruction's) is at or past the
// view's records exactly where the row is past the view.
static void copies(int wa, int ha) {
  for (int wx0 = 0; wx0 < wa - 1; wx0 += 4 * (1 + wa / 9)) {
    const uint32_t records = uint32_t(wa * ha - wx0) * 4;
    for (int row = 0; row < ha; row += 1 + ha / 7)
      for (int wave = 0; wave < kWinWaves; ++wave)
        for (int lane = 0; lane < 64; ++lane)
          for (int half = 0; half < 2; ++half) {
            const int r = row + 32 * (wave & 1) + 16 * half + (lane >> 2);
            const uint32_t at = window_lane_offset(row, wave, lane, half, wa);
            if (r >= ha) CHECK(at >= records);
            // (columns past the row's end are the next row's)
            if (r < ha - 1 && wx0 + 16 * kWinBlocks <= wa)
              CHECK(at + 64 * (kWinBlocks - 1) + 16 <= records);
          }
  }
}

static std::vector<double> clusters(double a, double b, double step, int each) {
  std::vector<double> v;
  for (double c : {a, b})
    for (int i = 0; i < each; ++i) v.push_back(c + i * step);
  return v;
}

// The split of one geometry and plane list: wa ha wb hb out_w out_h mag_x mag_y
// ca_x ca_y cb_x cb_y alpha ..
static int print_split(int argc, char** argv) {
  std::vector<double> v;
  for (int i = 1; i < argc; ++i) v.push_back(std::atof(argv[i]));
  const RefGeom g{int(v[0]), int(v[1]), int(v[2]), int(v[3]), int(v[4]), int(v[5]),
                  v[6],      v[7],      v[8],      v[9],      v[10],     v[11]};
  const std::vector<double> al(v.begin() + 12, v.end());
  WindowSplit w;
  if (window_split(g, al.data(), int(al.size()), (int64_t(al.size()) + 15) / 16 * 16, &w))
    std::printf("%d %d %d %d\n", w.np, w.xc, w.pg, w.blocks);
  else
    std::printf("none\n");
  return 0;
}

int main(int argc, char** argv) {
  if (argc > 13) return print_split(argc, argv);
  for (int ha : {2, 3, 8, 15, 16, 17, 31, 33, 47, 63, 64, 65, 100, 128, 200})
    for (int wa : {64, 65, 150, 256}) copies(wa, ha);
  // evenly spaced planes
  for (int n : {1, 5, 16, 33, 128}) {
    std::vector<double> al;
    for (int i = 0; i < n; ++i) al.push_back(n > 1 ? 0.5 + double(i) / (n - 1) : 1.0);
    walk(geom(128, 96, 64, 48, 128, 96), al);
    walk(geom(255, 130, 7, 2, 300, 140), al);
  }
  // two clusters of planes and unordered ones: nine blocks, waves at the far end
  WindowSplit w;
  CHECK(walk(geom(160, 120, 48, 36, 160, 120), clusters(0.3, 1.4, 0.004, 4), &w));
  CHECK(w.blocks == kWinBlocks && far_waves > 0);
  int before = far_waves;
  CHECK(walk(geom(160, 120, 48, 36, 160, 120),
             {0.300, 0.304, 0.308, 0.312, 1.412, 1.400, 1.408, 1.404}, &w));
  CHECK(far_waves > before);
  // drawn: views of up to 256 columns, crops, clusters (of as many planes as
  // half a plane group of either size) at most of the distances that fit
  uint32_t x = 1;
  auto rnd = [&](double a, double b) {
    x = x * 1664525u + 1013904223u;
    return a + (b - a) * (x >> 8) / double(1 << 24);
  };
  int taken = 0, shapes[3] = {0, 0, 0};
  before = far_waves;
  for (int k = 0; k < 3000; ++k) {
    const int wa = int(rnd(140, 257)), wb = int(rnd(1, 24));
    const int ow = rnd(0, 1) < 0.2 ? wa : int(rnd(8, 33));
    const double a = rnd(0.2, 1.0), b = rnd(1.0, 1.8);
    const int each = rnd(0, 1) < 0.5 ? 4 : 8;
    RefGeom g = geom(wa, 32, wb, 4, ow, 32);
    g.ca_x = rnd(0, 1) < 0.5 ? g.ca_x : rnd(0, wa - 1);
    g.mag_x *= rnd(0.3, 1);
    const int far0 = far_waves;
    if (!walk(g, clusters(a, b, rnd(0.0002, 0.004), each), &w)) continue;
    ++taken;
    if (far_waves > far0) ++shapes[w.np == 8 ? 0 : w.pg == 2 ? 1 : 2];
  }
  CHECK(taken > 500 && shapes[0] > 0 && shapes[1] > 0);
  if (failures) {
    std::fprintf(stderr, "%d failures\n", failures);
    return 1;
  }
  std::printf("window tests passed: %d drawn cases, %d waves past the eighth block (%d %d %d)\n",
              taken, far_waves, shapes[0], shapes[1], shapes[2]);
  return 0;
}
