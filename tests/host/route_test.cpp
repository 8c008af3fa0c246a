// Host-only checks of the rule that takes stacks by direct gathers (no HIP): the
// forms it must refuse, sizes measured faster by the gathers and sizes measured
// slower.  Built with the sanitizers.  With arguments, the rule's answer for one
// stack: wa ha wb hb out_w out_h n lo hi row_lane.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "refocus_route.h"

static int failures = 0;
#define CHECK(c)                                                        \
  do {                                                                  \
    if (!(c)) {                                                         \
      std::fprintf(stderr, "FAIL %s:%d: %s\n", __FILE__, __LINE__, #c); \
      ++failures;                                                       \
    }                                                                   \
  } while (0)

using namespace cpi;

static RefGeom geom(int wa, int ha, int wb, int hb, int out_w, int out_h) {
  return RefGeom{wa, ha, wb, hb, out_w, out_h, double(wa) / wb, double(ha) / hb, (wa - 1) / 2.0,
                 (ha - 1) / 2.0, (wb - 1) / 2.0, (hb - 1) / 2.0};
}

static bool gathers(const RefGeom& g, int n, double lo, double hi, bool row_lane = false) {
  std::vector<double> al;
  for (int i = 0; i < n; ++i) al.push_back(n > 1 ? lo + (hi - lo) * i / (n - 1) : lo);
  RefocusOther o;
  o.row_lane = row_lane;
  o.rows = g.out_h >= 16 ? 16 : 8;
  const long tiles = long((g.out_w + 63) / 64) * ((g.out_h + o.rows - 1) / o.rows) * ((n + 3) / 4);
  while (o.splits * 2 <= (g.hb < 16 ? g.hb : 16) && tiles * o.splits < 8192) o.splits *= 2;
  return refocus_gather_surely(g, n) || refocus_gather_wins(g, al.data(), n, o);
}

static bool square(int wa, int ha, int wb, int hb, int n, double lo, double hi,
                   bool row_lane = false) {
  return gathers(geom(wa, ha, wb, hb, wa, ha), n, lo, hi, row_lane);
}

int main(int argc, char** argv) {
  if (argc == 11) {
    std::vector<double> v;
    for (int i = 1; i < argc; ++i) v.push_back(std::atof(argv[i]));
    std::printf("%d\n", gathers(geom(int(v[0]), int(v[1]), int(v[2]), int(v[3]), int(v[4]), int(v[5])),
                                int(v[6]), v[7], v[8], v[9] != 0));
    return 0;
  }
  // what the kernel does not take
  CHECK(!square(1, 8, 2, 2, 1, 1, 1) && !square(8, 1, 2, 2, 1, 1, 1));
  CHECK(!square(4, 4, 1023, 2, 3, 0.7, 1.3) && square(4, 4, 1023, 1, 3, 0.7, 1.3));
  // measured faster: small stacks, and few planes whose windows are too wide
  CHECK(square(32, 32, 16, 16, 5, 0.5, 1.5) && square(32, 32, 16, 16, 32, 0.5, 1.5));
  CHECK(square(64, 64, 16, 16, 16, 0.5, 1.5, true));
  CHECK(square(48, 48, 48, 48, 8, 0.5, 1.5));
  CHECK(square(128, 128, 64, 64, 2, 0.5, 1.5) && square(128, 128, 64, 64, 8, 0.5, 1.5));
  CHECK(square(150, 233, 100, 128, 6, 0.5, 1.5));
  CHECK(square(63, 146, 134, 56, 4, 0.7, 1.3) && square(158, 277, 160, 6, 5, 0.5, 1.5));
  // measured slower: few views per pixel, full tiles whose windows fit, tiles
  // enough for every compute unit, few pixels of many views beside a row-lane pass
  CHECK(!square(1000, 1000, 2, 2, 4, 0.6, 1.4) && !square(224, 154, 1, 3, 80, 0.53, 1.53, true));
  CHECK(!square(44, 167, 24, 46, 8, 0.96, 1.0) && !square(288, 64, 12, 274, 8, 0.7, 1.3));
  CHECK(!square(37, 186, 14, 300, 8, 0.98, 1.02) && !square(60, 106, 8, 247, 6, 0.98, 1.02));
  CHECK(!square(60, 60, 200, 200, 8, 0.6, 1.4) && !square(63, 500, 60, 60, 8, 0.6, 1.4));
  CHECK(!square(49, 119, 40, 58, 8, 0.83, 0.87) && !square(62, 226, 8, 91, 8, 1.05, 1.09));
  CHECK(!square(68, 5, 73, 109, 2, 0.98, 1.02, true));
  // not candidates
  CHECK(!square(48, 48, 48, 48, 16, 0.5, 1.5) && !square(256, 256, 64, 64, 4, 0.5, 1.5));
  CHECK(!square(128, 128, 64, 64, 8, 0.5, 1.5, true));
  // crops, one pixel, one view
  CHECK(gathers(geom(200, 200, 32, 32, 1, 1), 4, 0.5, 1.5));
  CHECK(square(2, 2, 1, 1, 1, 1, 1));
  if (failures) return 1;
  std::printf("route tests passed\n");
  return 0;
}
