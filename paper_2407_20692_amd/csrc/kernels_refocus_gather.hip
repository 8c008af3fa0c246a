// Refocus by direct gathers, for small stacks and for those of a few planes.
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "refocus_common.h"
#include "refocus_route.h"

namespace cpi {

namespace {

// Small stacks: direct gathers, the views of a pixel split over 16 threads.
// Such a call is bound by launches and latency: of the batched kernel's five
// launches this takes two, no window is staged, and a thread's loads over its
// views are independent.  A work-group takes 16 consecutive output pixels of a
// plane; thread (slice, pixel) sums the views slice, slice + 16, ..., and the
// slices are added in order, in double (in float the sums, longer than the
// batched kernels', had up to twice their error).  Cells outside a view contribute nothing.
// (refocus_route.cpp says which stacks are taken and what they cost.)
__global__ __launch_bounds__(256) void k_ref_gather(const float* __restrict__ gamma, GeomI g,
                                                    const int32_t* __restrict__ itab,
                                                    const float* __restrict__ ftab,
                                                    int64_t stride, float* __restrict__ out) {
  __shared__ int bi[kGatherViews];
  __shared__ float bf[kGatherViews];
  __shared__ double red[16][17];
  const int t = threadIdx.x, slice = t >> 4, plane = blockIdx.y;
  const int64_t opix = int64_t(g.out_w) * g.out_h;
  const int64_t pix = int64_t(blockIdx.x) * 16 + (t & 15);
  const int32_t* it = itab + int64_t(plane) * stride;
  const float* ft = ftab + int64_t(plane) * stride;
  const int out_n = g.out_w + g.out_h;
  for (int i = t; i < g.wb + g.hb; i += 256) {   // columns, then rows
    bi[i] = it[out_n + i];
    bf[i] = ft[out_n + i];
  }
  __syncthreads();
  double acc = 0.0;
  if (pix < opix) {
    const int xr = int(pix % g.out_w), yr = int(pix / g.out_w);
    const int iax = it[xr], iay = it[g.out_w + yr];
    const float fax = ft[xr], fay = ft[g.out_w + yr];
    const int64_t pa = int64_t(g.wa) * g.ha;
    const int nv = g.wb * g.hb;
    int yb = slice / g.wb, xb = slice % g.wb;
    const int dy = 16 / g.wb, dx = 16 % g.wb;
#pragma unroll 4
    for (int v = slice; v < nv; v += 16) {
      int x0 = iax + bi[xb], y0 = iay + bi[g.wb + yb];
      float fx = fax + bf[xb], fy = fay + bf[g.wb + yb];
      if (fx >= 1.0f) {
        x0 += 1;
        fx -= 1.0f;
      }
      if (fy >= 1.0f) {
        y0 += 1;
        fy -= 1.0f;
      }
      int cx, cy;
      float wx0, wx1, wy0, wy1;
      clamp_cell(x0, fx, g.wa, cx, wx0, wx1);
      clamp_cell(y0, fy, g.ha, cy, wy0, wy1);
      const float* p = gamma + int64_t(v) * pa + (cy * g.wa + cx);
      const float top = wx0 * p[0] + wx1 * p[1];
      const float bot = wx0 * p[g.wa] + wx1 * p[g.wa + 1];
      const bool in = (wx0 != 0.0f || wx1 != 0.0f) && (wy0 != 0.0f || wy1 != 0.0f);
      acc += double(in ? wy0 * top + wy1 * bot : 0.0f);
      xb += dx;
      yb += dy;
      if (xb >= g.wb) {
        xb -= g.wb;
        ++yb;
      }
    }
  }
  red[slice][t & 15] = acc;
  __syncthreads();
  if (t < 16 && pix < opix) {
    double sum = 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) sum += red[k][t];
    out[int64_t(plane) * opix + pix] = float(sum);
  }
}

}  // namespace

hipError_t refocus_gather(const float* gamma, const RefGeom& g, const int32_t* itab,
                          const float* ftab, int64_t stride, int n_alpha, float* out,
                          hipStream_t s) {
  if (!refocus_gather_takes(g, n_alpha)) return hipErrorInvalidValue;
  const GeomI gi{g.wa, g.ha, g.wb, g.hb, g.out_w, g.out_h};
  const int64_t opix = int64_t(g.out_w) * g.out_h;
  hipLaunchKernelGGL(k_ref_gather, dim3(unsigned((opix + 15) / 16), unsigned(n_alpha)), dim3(256),
                     0, s, gamma, gi, itab, ftab, stride, out);
  return hipGetLastError();
}

}  // namespace cpi
