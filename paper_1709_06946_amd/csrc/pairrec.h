// The pair list's records and the pair geometry shared by the list builders
// (lists.hip) and the pair sums (real.hip).
#pragma once

#include "pse_internal.h"

namespace pse {

// Records lie in blocks of REC_BLOCK entries, field by field within a block: a
// lane reaches every field of its entry from one address, and the six fields
// of the stresslet-strain sum are one contiguous run of a block (2*10^5
// spheres, 111 neighbours each, FP32: 349 -> 305 us for the whole sum, 213 ->
// 190 for that block, against one array per field; FP64 at 2*10^4: 26 -> 24).
constexpr int PAIR_REC = 10;
constexpr int REC_BLOCK = 16;
// fields: d2 d3 d4, the unit vector, a b, c1 c2 (see the list of radial
// coefficients above)
enum { F_D2 = 0, F_D3, F_D4, F_E, F_A = F_E + 3, F_B, F_C1, F_C2 };

// Entry s of the records: field f at [f].
template <typename R> struct Entry {
  R *p;
  __device__ __forceinline__ Entry(R *rec, uint32_t s)
      : p(rec + (size_t)(s / REC_BLOCK) * (PAIR_REC * REC_BLOCK) + s % REC_BLOCK) {}
  __device__ __forceinline__ R &operator[](int f) const { return p[f * REC_BLOCK]; }
};

// Separation x_i - x_j of wrapped positions: nearest image, and on a
// deformed lattice mapped from lattice offsets to Cartesian ones (the cutoff
// is at most a third of the cell's thinnest width, so the image is the
// nearest one).
__device__ __forceinline__ void separation(const double *__restrict__ xw, double xi0, double xi1,
                                           double xi2, int j, double L, int def, const double *A,
                                           double *d) {
  d[0] = xi0 - xw[3 * j];
  d[1] = xi1 - xw[3 * j + 1];
  d[2] = xi2 - xw[3 * j + 2];
  // positions are wrapped into [0, L): one image shift per axis suffices
  const double hL = 0.5 * L;
#pragma unroll
  for (int k = 0; k < 3; ++k) d[k] += d[k] > hL ? -L : (d[k] < -hL ? L : 0.0);
  if (def) {
    const double e[3] = {d[0], d[1], d[2]};
#pragma unroll
    for (int r = 0; r < 3; ++r) d[r] = A[3 * r] * e[0] + A[3 * r + 1] * e[1] + A[3 * r + 2] * e[2];
  }
}

// The seven radial coefficients at distance r from the table.
template <typename T>
__device__ __forceinline__ void lookup(const T *__restrict__ tab, T r, T inv_dr,
                                       int n2a, int ntab, T *co) {
  const T f = r * inv_dr;
  int i0 = (int)f;
  int base;
  if (i0 < n2a) {
    base = i0 - 1;
    if (base < 0) base = 0;
    if (base > n2a - 3) base = n2a - 3;
  } else {
    base = i0 - 1;
    if (base < n2a) base = n2a;
    if (base > ntab - 4) base = ntab - 4;
  }
  const T t = f - (T)base;
  const T w0 = -(t - 1) * (t - 2) * (t - 3) / (T)6;
  const T w1 = t * (t - 2) * (t - 3) / (T)2;
  const T w2 = -t * (t - 1) * (t - 3) / (T)2;
  const T w3 = t * (t - 1) * (t - 2) / (T)6;
  const T *p = tab + (size_t)base * NCOEF;
#pragma unroll
  for (int j = 0; j < NCOEF; ++j)
    co[j] = w0 * p[j] + w1 * p[NCOEF + j] + w2 * p[2 * NCOEF + j] + w3 * p[3 * NCOEF + j];
}

}  // namespace pse
