// Device helpers shared by the mesh-derived kernels (shallow-ice guess, column features).
#pragma once

#include <hip/hip_runtime.h>

#include "fo_internal.h"

namespace fo {

// Gradient of the interpolated surface on base cell t, and its area (triangles: P1 gradient;
// quads: bilinear gradient at the centre).
__device__ __forceinline__ void cell_surface_gradient(const MeshView &m, int t, double &gx, double &gy,
                                                      double &area) {
  const int nv = m.nv;
  double px[4], py[4], ps[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const int w = m.cells[int64_t(t) * nv + (a < nv ? a : 0)];
    const double4 g = m.geo[w];
    px[a] = g.x; py[a] = g.y; ps[a] = m.sb[w].x;
  }
  if (nv == 3) {
    const double area2 = (px[1] - px[0]) * (py[2] - py[0]) - (px[2] - px[0]) * (py[1] - py[0]);
    gx = ((ps[1] - ps[0]) * (py[2] - py[0]) - (ps[2] - ps[0]) * (py[1] - py[0])) / area2;
    gy = ((ps[2] - ps[0]) * (px[1] - px[0]) - (ps[1] - ps[0]) * (px[2] - px[0])) / area2;
    area = 0.5 * area2;
  } else {
    const double dxi[4] = {-0.5, 0.5, 0.5, -0.5}, deta[4] = {-0.5, -0.5, 0.5, 0.5};
    double j00 = 0, j01 = 0, j10 = 0, j11 = 0, d0 = 0, d1 = 0;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      j00 += px[a] * dxi[a]; j01 += px[a] * deta[a];
      j10 += py[a] * dxi[a]; j11 += py[a] * deta[a];
      d0 += ps[a] * dxi[a];  d1 += ps[a] * deta[a];
    }
    const double det = j00 * j11 - j01 * j10;
    gx = (j11 * d0 - j10 * d1) / det;
    gy = (-j01 * d0 + j00 * d1) / det;
    double sh = 0.0;
#pragma unroll
    for (int a = 0; a < 4; ++a) sh += px[a] * py[(a + 1) & 3] - px[(a + 1) & 3] * py[a];
    area = 0.5 * fabs(sh);
  }
}

// Lanes that share a base vertex in the kernels over vertices: a cell, a neighbour or a level each.
// One thread per vertex walked these one after the other, each a chain of loads.
constexpr int VERT_LANES = 8;

// Area-weighted mean over the base cells around vertex v of the cells' surface gradients, in every one
// of the vertex's lanes (sub: this lane's number).  The sums run in the order of the cells.
__device__ __forceinline__ void vertex_surface_gradient(const MeshView &m, const int32_t *__restrict__ vc_ptr,
                                                        const int32_t *__restrict__ vc_idx, int v, int sub,
                                                        double &gx_out, double &gy_out) {
  double wsum = 0.0, gxs = 0.0, gys = 0.0;
  const int p0 = vc_ptr[v], p1 = vc_ptr[v + 1];
  for (int p = p0; p < p1; p += VERT_LANES) {
    double gx = 0.0, gy = 0.0, area = 0.0;
    if (p + sub < p1) cell_surface_gradient(m, vc_idx[p + sub], gx, gy, area);
    for (int i = 0; i < VERT_LANES && p + i < p1; ++i) {
      const double a = __shfl(area, i, VERT_LANES);
      wsum += a;
      gxs += a * __shfl(gx, i, VERT_LANES);
      gys += a * __shfl(gy, i, VERT_LANES);
    }
  }
  gx_out = gxs / wsum;
  gy_out = gys / wsum;
}

}  // namespace fo
