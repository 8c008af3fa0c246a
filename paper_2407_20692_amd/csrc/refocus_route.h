// Which untuned stacks are refocused by direct gathers (host; no HIP
// dependencies, so that it can be built and tested with a plain host compiler).
#pragma once

#include "refocus_window_plan.h"

namespace cpi {

constexpr int kGatherViews = 1024;   // lens-plane columns and rows that the gathers hold in LDS

// What the gathers can take at all.
bool refocus_gather_takes(const RefGeom& g, int n_alpha);

// What would be taken otherwise: a row-lane x pass and fold, or the column-sum
// kernel in tiles of `rows` output rows with `splits` view-row splits.
struct RefocusOther {
  bool row_lane = false;
  int rows = 16, splits = 1;
};

// Estimated microseconds of a whole call.
double refocus_gather_us(const RefGeom& g, int n_alpha);
double refocus_other_us(const RefGeom& g, const double* alphas, int n_alpha,
                        const RefocusOther& other);

// Whether a stack is a candidate (small, or of few planes) and, with `other`,
// whether the gathers are estimated to be faster.  Stacks whose gathers take less
// than any of the others' launches need no `other` (refocus_gather_surely).
bool refocus_gather_surely(const RefGeom& g, int n_alpha);
bool refocus_gather_wins(const RefGeom& g, const double* alphas, int n_alpha,
                         const RefocusOther& other);

}  // namespace cpi
