// Host-side plan of the register-window x pass of the refocus.
#include "refocus_window_plan.h"

#include <algorithm>
#include <cmath>

namespace cpi {

namespace {

// One axis of the geometry.
struct Axis {
  double mag, ca, cb;
  int na, nb, out;   // detector-A, detector-B and output sizes
};

// Most samples that the cells of planes [p0, p1) and output pixels [x0, x1]
// span on an axis at any lens-plane position, from the first cell's to the
// last cell's second sample.  u = alpha (x_r - ca) + ca + (1 - alpha) mag (x_b - cb)
// is bilinear in (alpha, x_r), so the samples lie between its values at the
// four corners (alpha_min or alpha_max, first or last pixel).  Along x_b the
// corners are straight lines: where the view's edges do not cut them their
// largest distance is a convex function, and where one edge does, it still
// is, so it is largest at an end of the x_b range or where a corner crosses
// an edge.
int axis_span(const Axis& g, const double* alphas, int p0, int p1, int x0, int x1) {
  const double s0 = g.mag * (0 - g.cb), s1 = g.mag * (g.nb - 1 - g.cb);
  const double smin = std::fmin(s0, s1), smax = std::fmax(s0, s1);
  double al[2] = {alphas[p0], alphas[p0]};
  for (int k = p0; k < p1; ++k) {
    al[0] = std::fmin(al[0], alphas[k]);
    al[1] = std::fmax(al[1], alphas[k]);
  }
  double c0[4], c1[4];   // corner i: u = c0 + c1 s
  for (int i = 0; i < 4; ++i) {
    c0[i] = al[i >> 1] * ((i & 1 ? x1 : x0) - g.ca) + g.ca;
    c1[i] = 1.0 - al[i >> 1];
  }
  int need = 0;
  for (int k = 0; k < 10; ++k) {
    double s = k == 8 ? smin : smax;
    if (k < 8) {
      const int i = k >> 1;
      if (c1[i] == 0.0) continue;
      s = ((k & 1 ? double(g.na) : -1.0) - c0[i]) / c1[i];
      if (!(s > smin && s < smax)) continue;
    }
    double lo = 1e300, hi = -1e300;
    for (int i = 0; i < 4; ++i) {
      const double u = c0[i] + c1[i] * s;
      lo = std::fmin(lo, u);
      hi = std::fmax(hi, u);
    }
    lo = std::fmax(lo, -1.0);
    hi = std::fmin(hi, double(g.na));
    // (the device's coordinates are within 2^-22 of these)
    if (hi >= lo) need = std::max(need, int(hi - lo + 1e-5) + 3);
  }
  return need;
}

// the most over all groups of na planes and tiles of xr output columns
int window_span(const RefGeom& g, const double* alphas, int n_alpha, int na, int xr) {
  const Axis x{g.mag_x, g.ca_x, g.cb_x, g.wa, g.wb, g.out_w};
  int need = 0;
  for (int p = 0; p < n_alpha; p += na)
    for (int c = 0; c < g.out_w; c += xr)
      need = std::max(need, axis_span(x, alphas, p, std::min(p + na, n_alpha), c,
                                      std::min(c + xr, g.out_w) - 1));
  return need;
}

// 16-column blocks that windows of `cols` columns take, starting at a
// multiple of 4 columns
int staged_blocks(int cols) { return (cols + 3 + 15) / 16; }

}  // namespace

int window_rows(const RefGeom& g, const double* alphas, int p0, int p1) {
  const Axis y{g.mag_y, g.ca_y, g.cb_y, g.ha, g.hb, g.out_h};
  return std::min(g.ha, axis_span(y, alphas, p0, p1, 0, g.out_h - 1));
}

bool window_split(const RefGeom& g, const double* alphas, int n_alpha, int64_t chunk,
                  WindowSplit* out) {
  // byte offsets within a view stay below 2^31, units per y_b below 256
  if (chunk < 16 || chunk % 16 != 0 || g.wa < 2 || g.ha < 2 || g.ha > 255 * 64 ||
      int64_t(g.wa) * g.ha >= (int64_t(1) << 29))
    return false;
  // Of the shapes of a wave (planes x columns) and arrangements of the four
  // waves, the one that moves the fewest window columns per pair: those
  // staged once per work-group, and those each wave then reads (3 columns
  // more: windows start at multiples of 4).
  struct Shape {
    int np, xc, pg;
  };
  double best = -1.0;
  for (const Shape& c : {Shape{8, 8, 2}, Shape{4, 16, 2}, Shape{4, 16, 1}}) {
    const int na = c.np * c.pg, xr = c.xc * (kWinWaves / c.pg);
    const int mine = window_span(g, alphas, n_alpha, c.np, c.xc) + 3;
    if (mine > kWinCols) continue;
    const int span = window_span(g, alphas, n_alpha, na, xr);
    if (staged_blocks(span) > kWinBlocks) continue;
    const double cost = (double(span + 3) / (4 * kWinPairs) + double(mine) / kWinPairs) *
                        ((n_alpha + na - 1) / na * na) * ((g.out_w + xr - 1) / xr * xr);
    if (best < 0 || cost < best) {
      best = cost;
      out->np = c.np;
      out->xc = c.xc;
      out->pg = c.pg;
      out->na = na;
      out->xr = xr;
      out->blocks = staged_blocks(span);
    }
  }
  return best >= 0;
}

}  // namespace cpi
