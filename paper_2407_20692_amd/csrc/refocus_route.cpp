// Which untuned stacks are refocused by direct gathers.
#include "refocus_route.h"

#include <algorithm>
#include <cmath>

namespace cpi {

namespace {

// Stacks of up to so many (plane, output pixel, view) triples are candidates ..
constexpr double kSmallWork = double(1 << 24);
// .. and, where no row-lane pass applies, those of so few planes and output
// pixels in all: the column-sum kernel, of four planes per work-group, hardly
// gains from fewer, and they do not fill its work-groups.
constexpr int kFewPlanes = 8;
constexpr double kFewPixels = double(1 << 18);

// The estimates' constants are fits to whole calls of 770 stacks (views of 2 to 400
// rows and columns, 1 to 400 lens-plane rows and columns, 1 to 80 planes spread
// by 0.04 to 1), each timed with the gathers, without them, and with the library
// of before them.  Of the 538 candidates among them, taking all made 15 over 10%
// slower than before (Da 62 x 226, Db 8 x 91, 8 planes 103 -> 250 us; Da 44 x 167, Db
// 24 x 46, 8 planes 94 -> 180; and beside them Da 1000 x 1000, Db 2 x 2, 4 planes
// 59 -> 204; Da 288 x 64, Db 12 x 274, 8 planes 305 -> 1285); taking the 516 that the
// estimates favour makes one 10% slower (71 -> 80) and the candidates 3.38 times as
// fast as before on average (all: 3.35; always the faster way: 3.39).

double triples(const RefGeom& g, int n_alpha) {
  return double(g.out_w) * g.out_h * n_alpha * g.wb * g.hb;
}

}  // namespace

bool refocus_gather_takes(const RefGeom& g, int n_alpha) {
  return g.wa >= 2 && g.ha >= 2 && int64_t(g.wb) + g.hb <= kGatherViews && n_alpha <= 65535 &&
         int64_t(g.wa) * g.ha < (int64_t(1) << 31) &&
         int64_t(g.out_w) * g.out_h < (int64_t(1) << 31);
}

// Launches; then the serial loop over a thread's views, or loads (16 pixels and 16
// views at a time, padded to that) and a work-group's start and sum.
double refocus_gather_us(const RefGeom& g, int n_alpha) {
  const double groups = std::ceil(double(g.out_w) * g.out_h / 16) * n_alpha;
  const double steps = std::ceil(double(g.wb) * g.hb / 16);
  return 10 + std::max(0.35 * steps, groups * (steps * 256 * 48 / kSmallWork + 0.0006));
}

double refocus_other_us(const RefGeom& g, const double* alphas, int n_alpha,
                        const RefocusOther& other) {
  // row-lane: launches, and the serial loop over lens-plane columns
  if (other.row_lane) return 45 + 1.1 * g.wb + 2.2 * triples(g, n_alpha) / kSmallWork;
  // column sums: the serial loop over a split's views, 1.2 us each, and 6 to 8 if
  // some group's window (four planes; 128 columns, twice the tile's rows) exceeds
  // the LDS, so that views are read directly, at some lens-plane row: the largest
  // share of those rows is sampled over groups and tiles
  const int groups = (n_alpha + 3) / 4;
  const int tx = (g.out_w + 63) / 64, ty = (g.out_h + other.rows - 1) / other.rows;
  auto span = [&](double mag, double ca, double cb, int size, int o0, int o1, double b, double a0,
                  double a1) {
    double lo = 1e300, hi = -1e300;
    for (double a : {a0, a1})
      for (int o : {o0, o1}) {
        const double u = a * (o - ca) + ca + (1.0 - a) * mag * (b - cb);
        lo = std::min(lo, u);
        hi = std::max(hi, u);
      }
    lo = std::min(std::max(std::floor(lo), 0.0), size - 2.0);
    hi = std::min(std::max(std::floor(hi) + 1, 0.0), size - 2.0) + 1;
    return hi - lo + 1;
  };
  const int gstep = std::max(1, groups / 4), xstep = std::max(1, tx / 4);
  const int ystep = std::max(1, ty / 16);
  int most = 0;   // of eight sampled lens-plane rows
  for (int q = 0; q < groups && most < 8; q += gstep) {
    double a0 = alphas[4 * q], a1 = a0;
    for (int k = 4 * q; k < std::min(4 * q + 4, n_alpha); ++k) {
      a0 = std::min(a0, alphas[k]);
      a1 = std::max(a1, alphas[k]);
    }
    for (int t = 0; t < tx; t += xstep)
      for (int b : {0, g.wb - 1})
        if (span(g.mag_x, g.ca_x, g.cb_x, g.wa, 64 * t, std::min(64 * t + 63, g.out_w - 1), b, a0,
                 a1) > 128)
          most = 8;
    for (int t = 0; t < ty; t = t + ystep < ty || t == ty - 1 ? t + ystep : ty - 1) {
      int wide = 0;
      for (int i = 0; i < 8; ++i)
        wide += span(g.mag_y, g.ca_y, g.cb_y, g.ha, other.rows * t,
                     std::min(other.rows * (t + 1), g.out_h) - 1, (i + 0.5) / 8 * g.hb - 0.5, a0,
                     a1) > 2 * other.rows;
      most = std::max(most, wide);
    }
  }
  const double view = most == 0 ? 1.2 : 6 + 0.25 * most;
  const int splits = std::max(1, std::min(other.splits, g.hb));
  const double views = double((g.hb + splits - 1) / splits) * g.wb;
  const double rounds = std::max(1.0, double(tx) * ty * groups * splits / 1024);
  return 30 + views * view * rounds;
}

// (the fastest of the 770 took 27.7 us without gathers)
bool refocus_gather_surely(const RefGeom& g, int n_alpha) {
  return refocus_gather_takes(g, n_alpha) && triples(g, n_alpha) <= kSmallWork &&
         refocus_gather_us(g, n_alpha) < 27;
}

bool refocus_gather_wins(const RefGeom& g, const double* alphas, int n_alpha,
                         const RefocusOther& other) {
  if (!refocus_gather_takes(g, n_alpha)) return false;
  const bool few = !other.row_lane && n_alpha <= kFewPlanes &&
                   double(g.out_w) * g.out_h * n_alpha < kFewPixels;
  if (!few && triples(g, n_alpha) > kSmallWork) return false;
  return refocus_gather_us(g, n_alpha) < refocus_other_us(g, alphas, n_alpha, other);
}

}  // namespace cpi
