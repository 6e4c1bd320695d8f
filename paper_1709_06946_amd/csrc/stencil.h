// The Gaussian stencils, shared by the list builders (lists.hip) and the grid
// kernels (grid.hip).
#pragma once

#include <cmath>

#include "pse_internal.h"

namespace pse {

__device__ __forceinline__ int wrapi(int i, int n) {
  i %= n;
  return i < 0 ? i + n : i;
}

// First stencil index and the grid offset of a particle coordinate.
__device__ __forceinline__ int stencil_start(double xc, double h, int P) {
  const double f = xc / h;
  return (P & 1) ? (int)floor(f + 0.5) - (P - 1) / 2 : (int)floor(f) - P / 2 + 1;
}

inline GridGeom geom(const Handle &h) {
  GridGeom g;
  g.ng = h.d.grid;
  g.P = h.d.support;
  g.L = h.p.box;
  g.h = h.d.h;
  const double xi2 = h.d.xi * h.d.xi;
  g.kcoef = 2.0 * xi2 / h.d.eta_s;
  g.knorm = sqrt(2.0 * xi2 / (M_PI * h.d.eta_s));
  g.def = h.def.on;
  for (int i = 0; i < 6; ++i) g.G[i] = h.def.G[i];
  return g;
}

// The particles' weight rows that spreading onto grids of T reads.
template <typename T> inline const T *weights(const Handle &h) {
  if constexpr (sizeof(T) == 8) return h.wt64;
  else return h.wt32;
}

}  // namespace pse
