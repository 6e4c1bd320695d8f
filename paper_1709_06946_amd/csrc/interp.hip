// Interpolation from the grids to the particles (handles with spreading tiles):
// the values of the velocity grids, and with derivative gridding the gradients
// of v = 3 f1(ka) u^'s grids, weighted with the particles' weight rows.
//
// One wavefront per particle, particles in cell order, each XCD taking a
// contiguous range of them so that neighbouring stencils share its L2.  Lane l
// owns the x-y columns l, l + 64, ... of the P^2; the Gaussian factorises, so
// a column's z sum needs one product per point with a weight that is the same
// for every lane (a scalar register), the planes' addresses are scalar too,
// and the x and y weights come in once per column.  A point costs one load and
// one or two multiply-adds; with weights and offsets formed per point the
// arithmetic was as long as the loads (633 vector instructions per particle at
// support 8, 2400 at support 10; now 240 and 390 with three and five components
// from FP32 grids).  Weights, products and sums are FP64 on FP32 grids too:
// rounded one-dimensional weights share their errors over whole rows and planes
// of the stencil (5.5e-8 of the value, rms, against 3.4e-8 with each point's
// weight rounded once).  FP64 takes 1 to 6 % of these kernels' time.  Against
// weights formed per point, gradient interpolation at 512^3, N = 10^6: 1.89 ->
// 1.47 ms, at 192^3, N = 2*10^5: 345 -> 221 us; five components at 384^3, N =
// 2*10^5, support 10: 1.17 -> 1.03 ms; six grids at 512^3 in one launch 2.92 ->
// 3.02 ms.  What bounds it now is the L1's misses: of 295 accesses a particle at
// 512^3 216 go on to the L2, and the L1 stalls on them for 70 % of the kernel's
// cycles (at 192^3 175 of 310 and 56 %).
#include <type_traits>

#include "fftreg.h"
#include "stencil.h"

namespace pse {

// Value of the same lane of the row rotated by R.
template <int R> __device__ __forceinline__ double rotated(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x120 + R, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x120 + R, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// a's upper and b's lower halves exchanged (rows of 16: a's odd with b's even
// rows), then added: lane sums of a and b side by side in one register.
__device__ __forceinline__ double fold32(double a, double b) {
  const auto l = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a),
                                                  (unsigned)__double2loint(b), false, false);
  const auto h = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a),
                                                  (unsigned)__double2hiint(b), false, false);
  return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
}
__device__ __forceinline__ double fold16(double a, double b) {
  const auto l = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(a),
                                                  (unsigned)__double2loint(b), false, false);
  const auto h = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(a),
                                                  (unsigned)__double2hiint(b), false, false);
  return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
}

// Wavefront sums of four values: the sum of value SUM_OF[r] in every lane of
// row r.
__device__ __forceinline__ double wave_sum4(double a, double b, double c, double d) {
  double v = fold16(fold32(a, b), fold32(c, d));
  v += rotated<8>(v);
  v += rotated<4>(v);
  v += rotated<2>(v);
  v += rotated<1>(v);
  return v;
}
// rows hold a, c, b, d
__device__ __forceinline__ int sum_of(int row) { return row == 1 ? 2 : (row == 2 ? 1 : row); }

// Wavefront sums of r[0..M), value k handed to store(k, sum) in one lane.
template <int M, typename Store>
__device__ __forceinline__ void wave_sums(int lane, const double (&r)[M], Store store) {
#pragma unroll
  for (int k = 0; k < M; k += 4) {
    const double v = wave_sum4(r[k], k + 1 < M ? r[k + 1] : 0.0, k + 2 < M ? r[k + 2] : 0.0,
                               k + 3 < M ? r[k + 3] : 0.0);
    const int j = k + sum_of(lane / 16);
    if (lane % 16 == 0 && j < M) store(j, v);
  }
}

struct InterpArgs {
  const int *order;     // traversal of the particles
  int64_t n;
  int ng, P, rw, pad;   // grid, support, entries and zeros of a weight row
  double h;             // grid spacing
  size_t ngrid;
  Layout lo;
  int accumulate;
  double scale;
};

// Supports whose planes an instance unrolls exactly (see with_planes).
constexpr bool exact_planes(int PZ) { return PZ >= 5; }

// What the lanes of a particle's wavefront share and own: its particle, the
// columns' places in a plane and weights (zero beyond P^2), its planes and
// their weights (beyond P: the last plane with weight zero).
template <typename T, typename W, int PZ> struct Columns {
  static constexpr int NJ = (PZ * PZ + 63) / 64;
  int p;
  uint32_t at[NJ];      // bytes within a plane
  size_t plane[PZ];     // bytes within a grid
  W X[NJ], Y[NJ], Z[PZ];

  __device__ __forceinline__ Columns(const InterpArgs &ia, const double *__restrict__ x,
                                     const W *__restrict__ wt, int64_t t, int lane) {
    p = __builtin_amdgcn_readfirstlane(ia.order ? ia.order[t] : (int)t);
    const int P = exact_planes(PZ) ? PZ : ia.P, ng = ia.ng;
    const int ix0 = stencil_start(x[3 * (size_t)p], ia.h, P);
    const int iy0 = stencil_start(x[3 * (size_t)p + 1], ia.h, P);
    int iz = __builtin_amdgcn_readfirstlane(stencil_start(x[3 * (size_t)p + 2], ia.h, P));
    const W *w = wt + (size_t)p * (3 * ia.rw) + ia.pad;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int s = lane + 64 * j, b = s / P, a = s - b * P;
      const bool in = b < P;
      // (stencils of wrapped positions start above -ng and end below 2 ng)
      int ix = ix0 + a, iy = iy0 + (in ? b : P - 1);
      ix += ix < 0 ? ng : (ix >= ng ? -ng : 0);
      iy += iy < 0 ? ng : (iy >= ng ? -ng : 0);
      at[j] = (uint32_t)(iy * ng + ix) * (uint32_t)sizeof(T);
      X[j] = w[a];
      Y[j] = w[ia.rw + (in ? b : P - 1)];
      if (!in) X[j] = W{};
    }
    iz += iz < 0 ? ng : (iz >= ng ? -ng : 0);
    const size_t step = (size_t)ng * ng * sizeof(T);
    size_t off = (size_t)iz * step;
#pragma unroll
    for (int c = 0; c < PZ; ++c) {
      plane[c] = off;
      Z[c] = w[2 * ia.rw + (c < P ? c : P - 1)];
      if (c >= P) Z[c] = W{};
      if (c + 1 < P) {
        ++iz;
        off = iz == ng ? 0 : off + step;
        if (iz == ng) iz = 0;
      }
    }
  }
  // Column j's point in plane c of a grid.  The plane's address stays in
  // scalar registers (the compiler would add it to each lane's), so that a
  // load takes no vector instruction of its own.
  __device__ __forceinline__ T load(const T *__restrict__ g, int j, int c) const {
    using Global = const __attribute__((address_space(1))) char;
    Global *q = (Global *)g + plane[c];
    asm("" : "+s"(q));
    return *(const __attribute__((address_space(1))) T *)(q + at[j]);
  }
};

// the weight of a row's entry
__device__ __forceinline__ double plain(double w) { return w; }
__device__ __forceinline__ double plain(const double2 &w) { return w.x; }

// Components cs of the particles' vectors from one grid each (M of them;
// those beyond cs.n read the last grid again and are dropped).
template <typename T, typename W, int PZ, int M>
__global__ void __launch_bounds__(256)
interp_kernel(const double *__restrict__ x, const T *__restrict__ grids,
              const W *__restrict__ wt, InterpArgs ia, CompSet cs, double *__restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)xcd_block(blockIdx.x, gridDim.x) * 4 +
                    __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (t >= ia.n) return;
  const Columns<T, W, PZ> C(ia, x, wt, t, lane);
  constexpr int NJ = Columns<T, W, PZ>::NJ;
  double acc[M];
#pragma unroll
  for (int k = 0; k < M; ++k) {
    const T *g = grids + (size_t)min(k, cs.n - 1) * ia.ngrid;
    T v[NJ][PZ];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int c = 0; c < PZ; ++c) v[j][c] = C.load(g, j, c);
    double a = 0.0;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      double s = 0.0;
#pragma unroll
      for (int c = 0; c < PZ; ++c) s += (double)v[j][c] * plain(C.Z[c]);
      a += s * (plain(C.X[j]) * plain(C.Y[j]));
    }
    acc[k] = a;
  }
  wave_sums<M>(lane, acc, [&](int k, double v) {
    if (k >= cs.n) return;
    double *o = out + (size_t)C.p * ia.lo.stride + cs.idx[k] - ia.lo.off;
    const double r = ia.scale * v;
    *o = ia.accumulate ? *o + r : r;
  });
}

// Rotation and strain from derivative gridding: with v = the three velocity
// grids of the k-space factor 3 f1(ka) u^, and the sums
// G_ij = sum_n v_i(x_n) dK/dx_j (x_n - x_p) = -(d v_i / d x_j)(x_p) (the
// interpolation of grad v with the gradient moved onto the Gaussian), the
// strain is e_q = Y_q : grad v and the rotation curl v / 2 (the adjoints of
// the stresslet and torque columns).  With HU the three grids of j0(ka) u^
// come first and give the velocity by plain interpolation; ROT: the rotation
// too.  mask: bit c for each output component c (velocity 0-2, rotation 3-5,
// strain 6-10).
template <typename T, int PZ, bool HU, bool ROT>
__global__ void __launch_bounds__(256)
interp_deriv_kernel(const double *__restrict__ x, const T *__restrict__ grids,
                    const double2 *__restrict__ wt, InterpArgs ia, int mask,
                    double *__restrict__ out) {
  using W = double2;   // (weight, gradient weight)
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)xcd_block(blockIdx.x, gridDim.x) * 4 +
                    __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (t >= ia.n) return;
  const Columns<T, W, PZ> C(ia, x, wt, t, lane);
  constexpr int NJ = Columns<T, W, PZ>::NJ, NU = HU ? 3 : 0, NR = ROT ? 3 : 0;
  double G[3][3], U[3];
#pragma unroll
  for (int k = 0; k < 3 + NU; ++k) {
    const T *g = grids + (size_t)k * ia.ngrid;
    T v[NJ][PZ];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int c = 0; c < PZ; ++c) v[j][c] = C.load(g, j, c);
    double a[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      // the column's sums with the weight and the gradient weight along z
      double s = 0.0, z = 0.0;
#pragma unroll
      for (int c = 0; c < PZ; ++c) {
        s += (double)v[j][c] * C.Z[c].x;
        if (k >= NU) z += (double)v[j][c] * C.Z[c].y;
      }
      const W X = C.X[j], Y = C.Y[j];
      if (k < NU) {
        a[0] += (X.x * Y.x) * s;
      } else {
        a[0] += (X.y * Y.x) * s;
        a[1] += (X.x * Y.y) * s;
        a[2] += (X.x * Y.x) * z;
      }
    }
    if (k < NU) {
      U[k] = a[0];
    } else {
#pragma unroll
      for (int i = 0; i < 3; ++i) G[k - NU][i] = a[i];
    }
  }
  double r[5 + NR + NU];
  r[0] = G[0][1] + G[1][0];
  r[1] = G[0][2] + G[2][0];
  r[2] = G[1][2] + G[2][1];
  r[3] = G[0][0] - G[1][1];
  r[4] = G[0][0] + G[1][1] - 2.0 * G[2][2];
  if constexpr (ROT) {
    r[5] = G[2][1] - G[1][2];
    r[6] = G[0][2] - G[2][0];
    r[7] = G[1][0] - G[0][1];
  }
  if constexpr (HU)
#pragma unroll
    for (int k = 0; k < 3; ++k) r[5 + NR + k] = U[k];
  wave_sums<5 + NR + NU>(lane, r, [&](int k, double v) {
    const int c = k < 5 ? 6 + k : (k < 5 + NR ? k - 2 : k - 5 - NR);
    if (!((mask >> c) & 1)) return;
    const double f = c < 3 ? 1.0
                           : (c < 6 ? -0.5 : (c < 10 ? -0.70710678118654752440
                                                     : -0.40824829046386301637));
    double *o = out + (size_t)C.p * ia.lo.stride + c - ia.lo.off;
    const double s = ia.scale * f * v;
    *o = ia.accumulate ? *o + s : s;
  });
}

template <typename T>
static InterpArgs interp_args(const Handle &h, Layout lo, bool accumulate, double scale) {
  const GridGeom g = geom(h);
  InterpArgs ia;
  ia.order = h.cells.trav;
  ia.n = h.n;
  ia.ng = g.ng;
  ia.P = g.P;
  ia.rw = weight_row(g.P, h.stile);
  ia.pad = h.stile - 1;
  ia.h = g.h;
  ia.ngrid = h.ngrid;
  ia.lo = lo;
  ia.accumulate = accumulate ? 1 : 0;
  ia.scale = scale;
  return ia;
}

// Instances by support: a wavefront's unrolled planes.  From 5 on each support
// has its own; below, four planes, those beyond P reading the last one once more
// (stencils so small are bound by their launch).  Padded to the next instance
// support 11 took 1315 against 904 us and 13 2006 against 1409 (N = 10^5, eleven
// components at 128^3 in FP32).
template <typename F> static void with_planes(int P, F f) {
  if (P <= 4) f(std::integral_constant<int, 4>());
  else if (P == 5) f(std::integral_constant<int, 5>());
  else if (P == 6) f(std::integral_constant<int, 6>());
  else if (P == 7) f(std::integral_constant<int, 7>());
  else if (P == 8) f(std::integral_constant<int, 8>());
  else if (P == 9) f(std::integral_constant<int, 9>());
  else if (P == 10) f(std::integral_constant<int, 10>());
  else if (P == 11) f(std::integral_constant<int, 11>());
  else if (P == 12) f(std::integral_constant<int, 12>());
  else if (P == 13) f(std::integral_constant<int, 13>());
  else if (P == 14) f(std::integral_constant<int, 14>());
  else if (P == 15) f(std::integral_constant<int, 15>());
  else throw Error{PSE_ERR_INVALID, "interpolation: support beyond 15"};
}

template <typename F> static void with_count(int n, F f) {
  if (n <= 3) f(std::integral_constant<int, 3>());
  else if (n <= 5) f(std::integral_constant<int, 5>());
  else if (n <= 8) f(std::integral_constant<int, 8>());
  else f(std::integral_constant<int, NC>());
}

template <typename T>
void interpolate(Handle &h, const double *x, const T *grids, const CompSet &cs, double *out,
                 Layout lo, bool accumulate, double scale) {
  if (!h.stile) {
    interp_generic<T>(h, x, grids, cs, out, lo, accumulate, scale);
    return;
  }
  if (cs.n < 1) return;
  ProfScope ps(h, PK_INTERP, (double)cs.n * h.ngrid * sizeof(T) + (double)h.n * (3 + cs.n) * 8);
  const InterpArgs ia = interp_args<T>(h, lo, accumulate, scale);
  with_planes(ia.P, [&](auto planes) {
    with_count(cs.n, [&](auto count) {
      constexpr int PZ = decltype(planes)::value, M = decltype(count)::value;
      if constexpr (PZ <= 10)   // derivative gridding's supports
        if (h.deriv) {
          hipLaunchKernelGGL((interp_kernel<T, double2, PZ, M>), dim3(nblocks(h.n, 4)), dim3(256),
                             0, h.stream, x, grids, reinterpret_cast<const double2 *>(h.wt64), ia,
                             cs, out);
          return;
        }
      hipLaunchKernelGGL((interp_kernel<T, double, PZ, M>), dim3(nblocks(h.n, 4)), dim3(256), 0,
                         h.stream, x, grids, (const double *)h.wt64, ia, cs, out);
    });
  });
  PSE_LAUNCH_CHECK();
}

// Velocity (with hu), rotation and strain components cs of out in layout lo
// from the grids of derivative gridding.
template <typename T>
void interp_deriv(Handle &h, const double *x, const T *grids, bool hu, const CompSet &cs,
                  double *out, Layout lo, bool accumulate, double scale) {
  const double2 *wt = reinterpret_cast<const double2 *>(h.wt64);
  ProfScope ps(h, PK_INTERP, (hu ? 6.0 : 3.0) * h.ngrid * sizeof(T) + (double)h.n * (3 + cs.n) * 8);
  const InterpArgs ia = interp_args<T>(h, lo, accumulate, scale);
  int mask = 0;
  for (int k = 0; k < cs.n; ++k) mask |= 1 << cs.idx[k];
  const bool rot = mask & (7 << 3);
  with_planes(ia.P, [&](auto planes) {
    constexpr int PZ = decltype(planes)::value;
    const auto launch = [&](auto u, auto r) {
      if constexpr (PZ <= 10)
        hipLaunchKernelGGL((interp_deriv_kernel<T, PZ, decltype(u)::value, decltype(r)::value>),
                           dim3(nblocks(h.n, 4)), dim3(256), 0, h.stream, x, grids, wt, ia, mask,
                           out);
      else throw Error{PSE_ERR_INVALID, "derivative gridding supports P <= 10"};
    };
    const std::true_type yes;
    const std::false_type no;
    if (hu && rot) launch(yes, yes);
    else if (hu) launch(yes, no);
    else if (rot) launch(no, yes);
    else launch(no, no);
  });
  PSE_LAUNCH_CHECK();
}

#define INST(T)                                                                             \
  template void interpolate<T>(Handle &, const double *, const T *, const CompSet &,        \
                               double *, Layout, bool, double);                             \
  template void interp_deriv<T>(Handle &, const double *, const T *, bool, const CompSet &, \
                                double *, Layout, bool, double);
INST(double)
INST(float)
#undef INST

}  // namespace pse
