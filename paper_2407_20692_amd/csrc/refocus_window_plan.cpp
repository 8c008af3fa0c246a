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

// The largest and smallest of a group of planes' alpha, and what follows from
// them for an axis.
struct Group {
  double al[2], slope[2], inv[2];   // alpha, 1 - alpha, 1 / (1 - alpha)
  double smin, smax;                // mag (x_b - cb) at the lens-plane ends
};
Group group_of(const Axis& g, const double* alphas, int p0, int p1) {
  Group r;
  const double s0 = g.mag * (0 - g.cb), s1 = g.mag * (g.nb - 1 - g.cb);
  r.smin = std::fmin(s0, s1);
  r.smax = std::fmax(s0, s1);
  r.al[0] = r.al[1] = alphas[p0];
  for (int k = p0; k < p1; ++k) {
    r.al[0] = std::fmin(r.al[0], alphas[k]);
    r.al[1] = std::fmax(r.al[1], alphas[k]);
  }
  for (int i = 0; i < 2; ++i) {
    r.slope[i] = 1.0 - r.al[i];
    r.inv[i] = 1.0 / r.slope[i];
  }
  return r;
}

// Most samples that the cells of a group of planes and output pixels [x0, x1]
// span on an axis at any lens-plane position, from the first cell's to the last
// cell's second sample.  u = alpha (x_r - ca) + ca + (1 - alpha) mag (x_b - cb) is
// bilinear in (alpha, x_r), so the samples lie between its values at the four
// corners (alpha_min or alpha_max, first or last pixel).  Along s = mag (x_b - cb)
// the largest corner is the larger of two straight lines (one per alpha, of its
// larger intercept), the smallest the smaller of two.  Cut at the view's edges
// their distance is convex between the points where one of the first two lines
// crosses the far edge or one of the others the near one, so it is largest at
// such a point or at an end of the range.
int axis_span(const Axis& g, const Group& r, int x0, int x1) {
  const double near = -1.0, far = double(g.na);
  double top[2], bot[2], at[6];
  for (int i = 0; i < 2; ++i) {
    const double a = r.al[i] * (x0 - g.ca) + g.ca, b = r.al[i] * (x1 - g.ca) + g.ca;
    top[i] = std::max(a, b);
    bot[i] = std::min(a, b);
    // (an alpha of 1 gives no crossing: infinite or no number)
    at[i] = (far - top[i]) * r.inv[i];
    at[2 + i] = (near - bot[i]) * r.inv[i];
  }
  at[4] = r.smin;
  at[5] = r.smax;
  double most = -1.0;
  for (const double s : at) {
    if (!(s >= r.smin && s <= r.smax)) continue;
    const double hi = std::max(top[0] + r.slope[0] * s, top[1] + r.slope[1] * s);
    const double lo = std::min(bot[0] + r.slope[0] * s, bot[1] + r.slope[1] * s);
    most = std::max(most, std::min(hi, far) - std::max(lo, near));
  }
  // (the device's coordinates are within 2^-22 of these)
  return most >= 0 ? int(most + 1e-5) + 3 : 0;
}

// the most over all groups of na planes and tiles of xr output columns; looked for
// up to the first above `limit`
int window_span(const RefGeom& g, const double* alphas, int n_alpha, int na, int xr, int limit) {
  const Axis x{g.mag_x, g.ca_x, g.cb_x, g.wa, g.wb, g.out_w};
  int need = 0;
  for (int p = 0; p < n_alpha; p += na) {
    const Group r = group_of(x, alphas, p, std::min(p + na, n_alpha));
    for (int c = 0; c < g.out_w; c += xr) {
      need = std::max(need, axis_span(x, r, c, std::min(c + xr, g.out_w) - 1));
      if (need > limit) return need;
    }
  }
  return need;
}

// 16-column blocks that windows of `cols` columns take, starting at a
// multiple of 4 columns
int staged_blocks(int cols) { return (cols + 3 + 15) / 16; }

}  // namespace

int window_rows(const RefGeom& g, const double* alphas, int p0, int p1) {
  const Axis y{g.mag_y, g.ca_y, g.cb_y, g.ha, g.hb, g.out_h};
  return std::min(g.ha, axis_span(y, group_of(y, alphas, p0, p1), 0, g.out_h - 1));
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
  int mine = 0;
  for (const Shape& c : {Shape{8, 8, 2}, Shape{4, 16, 2}, Shape{4, 16, 1}}) {
    const int na = c.np * c.pg, xr = c.xc * (kWinWaves / c.pg);
    if (c.pg == 2)   // (the last two shapes have the same waves)
      mine = window_span(g, alphas, n_alpha, c.np, c.xc, kWinCols - 3) + 3;
    if (mine > kWinCols) continue;
    const int span = window_span(g, alphas, n_alpha, na, xr, 16 * kWinBlocks - 3);
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
