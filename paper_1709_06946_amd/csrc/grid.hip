// Wave-space stages of the NUFFT mobility (Sec. II.C, Eq. WSops2) and of the
// wave-space square root (Sec. III.C, Eq. FFTsqrt).
//
// Grids: each of the G real components of one operator application has its
// own real grid [c][z][y][x]; the real FFT turns it in place into a half
// spectrum [c][kz][ky][kx < n/2] (fft.hip), so the k-space kernels act on one
// wave vector at a time and the other half follows by Hermitian symmetry.
//
// Gaussian kernel (Sec. II.C): K(r) = (2 xi^2/(pi eta_s))^(3/2)
// exp(-2 xi^2 r^2 / eta_s), truncated to the P^3 nearest grid points, whose
// Fourier transform is exp(-eta_s k^2 / 8 xi^2).  Spreading and
// interpolation each contribute that factor once; the k-space scaling
// divides both out again.
#include <algorithm>
#include <type_traits>

#include "fftreg.h"
#include "stencil.h"

namespace pse {

// ------------------------------------------------------------- spreading --

// Grids without spreading tiles: one wavefront per particle, its lanes covering
// the P^3 stencil, added to cleared grids.
template <typename T>
__global__ void __launch_bounds__(256)
spread_kernel(const double *__restrict__ x, const double *__restrict__ q,
              Layout lq, CompSet cs, GridGeom g, const int *__restrict__ order,
              int64_t n, T *__restrict__ grids, size_t ngrid) {
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= n) return;
  const int64_t p = order ? order[t] : t;
  const double px = x[3 * p], py = x[3 * p + 1], pz = x[3 * p + 2];
  const int P = g.P, P3 = P * P * P;
  const int ix0 = stencil_start(px, g.h, P);
  const int iy0 = stencil_start(py, g.h, P);
  const int iz0 = stencil_start(pz, g.h, P);
  T qv[NC];
#pragma unroll
  for (int k = 0; k < NC; ++k)
    qv[k] = k < cs.n ? (T)q[p * lq.stride + cs.idx[k] - lq.off] : (T)0;
  const double kn3 = g.knorm * g.knorm * g.knorm;
  for (int s = lane; s < P3; s += 64) {
    const int a = s % P, b = (s / P) % P, c = s / (P * P);
    const double dx = (ix0 + a) * g.h - px;
    const double dy = (iy0 + b) * g.h - py;
    const double dz = (iz0 + c) * g.h - pz;
    const double r2 = g.def ? qform(g.G, dx, dy, dz) : dx * dx + dy * dy + dz * dz;
    const T w = (T)(kn3 * exp(-g.kcoef * r2));
    const size_t gi = ((size_t)wrapi(iz0 + c, g.ng) * g.ng + wrapi(iy0 + b, g.ng)) * g.ng
                      + wrapi(ix0 + a, g.ng);
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      if (k < cs.n) atomicAdd(grids + (size_t)k * ngrid + gi, w * qv[k]);
    }
  }
}

// Gather form of the spreading sum: one wavefront per tile of S^3 grid points
// goes through the tile's candidates (TileRec: a particle and where the tile's
// window lies in its weight rows).  The Gaussian factorises over the axes, and
// a lane owns one z-column of an 8^3 tile (ZPT of its points; on grids below
// 24, tiles of 4^3 points, one point).  TCH candidates at a time are staged in
// the wavefront's own part of LDS -- their windows by half a wavefront each,
// their moments by one lane each -- with all loads in flight together, so a
// tile pays the memory's latency once per chunk, and no barrier.  (Loads by
// scalar instructions one candidate ahead were bound by that latency: 1.45
// against 1.01 ms per gradient spreading at 512^3, N = 10^6, and 1.33 for
// records of weights written per tile and candidate.)  z planes that the
// stencil does not reach are skipped, four of eight on average at support 8.
// Every grid point is written exactly once: no atomics and no zeroing pass.
// Neighbouring tiles, in blocks of 4^3, run on one XCD, whose L2 they share
// their particles' rows and complete their cache lines in.
constexpr int TCH = 16;

template <int S, int ZPT> struct TileLane {
  int tile, tc[3], lx, ly, z0;    // z0: first z point; S = 4: the lane's own
  __device__ __forceinline__ TileLane(int nb) {
    constexpr int PARTS = S == 8 ? 8 / ZPT : 1;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int unit = (int)xcd_block(blockIdx.x, gridDim.x) * 4 + wave;
    const int lane = threadIdx.x & 63, u = unit / PARTS;
    if (nb % 4 == 0) {
      const int b = u / 64, i = u % 64, n4 = nb / 4;
      tc[0] = (b % n4) * 4 + i % 4;
      tc[1] = (b / n4) % n4 * 4 + i / 4 % 4;
      tc[2] = b / (n4 * n4) * 4 + i / 16;
    } else {
      tc[0] = u % nb;
      tc[1] = u / nb % nb;
      tc[2] = u / (nb * nb);
    }
    tile = (tc[2] * nb + tc[1]) * nb + tc[0];
    lx = lane % S;
    ly = (lane / S) % S;
    z0 = S == 8 ? (unit % PARTS) * ZPT : lane / (S * S);
  }
  __device__ __forceinline__ size_t point(int ng, int z) const {
    return ((size_t)(tc[2] * S + z0 + z) * ng + tc[1] * S + ly) * ng + tc[0] * S + lx;
  }
};

// Stages up to TCH candidates rec[0..cnt): item i of candidate c's windows
// (axis i / S, position i % S) at items[c * 3 S + i], W = entry(row index).
// Two candidates per step, half a wavefront each.
template <typename W, int S, typename Entry>
__device__ __forceinline__ void stage_windows(const TileRec &r, int cnt, int rw, W *items,
                                              Entry entry) {
  constexpr int NI = 3 * S;
  const int lane = threadIdx.x & 63, i = lane & 31, axis = min(i / S, 2);
  const bool upper = lane >= 32;
  W v[TCH / 2];
#pragma unroll
  for (int k = 0; k < TCH / 2; ++k) {
    if (2 * k >= cnt) break;
    const int c1 = min(2 * k + 1, cnt - 1);
    const int p0 = __builtin_amdgcn_readlane(r.p, 2 * k), p1 = __builtin_amdgcn_readlane(r.p, c1);
    const int w0 = __builtin_amdgcn_readlane(r.win, 2 * k),
              w1 = __builtin_amdgcn_readlane(r.win, c1);
    const int p = upper ? p1 : p0, win = upper ? w1 : w0;
    // (lanes past the items read a window's entry too and drop it)
    v[k] = entry((size_t)p * (3 * rw) + axis * rw + ((win >> (8 * axis)) & 255) + i % S);
  }
  if (i >= NI) return;
#pragma unroll
  for (int k = 0; k < TCH / 2; ++k) {
    if (2 * k >= cnt) break;
    items[(2 * k + (lane >> 5)) * NI + i] = v[k];
  }
}

// Moments: component k of grid k is sum_b q_bk K(x_n - x_b).
template <typename T, int E, int S, int NCM, int ZPT>
__global__ void __launch_bounds__(256)
spread_tile_kernel(const double *__restrict__ q, Layout lq, CompSet cs, int ng, int P, int nb,
                   const int *__restrict__ tstart, const TileRec *__restrict__ rec,
                   const T *__restrict__ wt, int rw, T *__restrict__ grids, size_t ngrid) {
  constexpr int NI = 3 * S, NQ = (NCM + 3) / 4 * 4;
  __shared__ __align__(16) T lds_w[4][TCH * NI], lds_q[4][TCH * NQ];
  const TileLane<S, ZPT> L(nb);
  if (L.tile >= nb * nb * nb) return;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  T *items = lds_w[wave], *mom = lds_q[wave];
  const int lo = tstart[L.tile], hi = tstart[L.tile + 1];
  T acc[ZPT][NCM];
#pragma unroll
  for (int z = 0; z < ZPT; ++z)
#pragma unroll
    for (int k = 0; k < NCM; ++k) acc[z][k] = (T)0;
  for (int base = lo; base < hi; base += TCH) {
    const int cnt = min(TCH, hi - base);
    const TileRec r = rec[base + min(lane, cnt - 1)];
    double qv[NCM];
    if (lane < cnt) {
      const double *qp = q + (size_t)r.p * lq.stride - lq.off;
#pragma unroll
      for (int k = 0; k < NCM; ++k) qv[k] = k < cs.n ? qp[cs.idx[k]] : 0.0;
    }
    stage_windows<T, S>(r, cnt, rw, items, [&](size_t e) { return wt[e * E]; });
    if (lane < cnt)
#pragma unroll
      for (int k = 0; k < NCM; ++k) mom[lane * NQ + k] = (T)qv[k];
    wave_lds_sync();
    for (int c = 0; c < cnt; ++c) {
      const int wz = __builtin_amdgcn_readlane(r.win, c) >> 16;
      const T *w = items + c * NI;
      const T wxy = w[L.lx] * w[S + L.ly];
      T f[NCM];
#pragma unroll
      for (int k = 0; k < NCM; ++k) f[k] = mom[c * NQ + k] * wxy;
      T zw[ZPT];
#pragma unroll
      for (int z = 0; z < ZPT; ++z) zw[z] = w[2 * S + L.z0 + z];
#pragma unroll
      for (int z = 0; z < ZPT; ++z) {
        if (S == 8 && (unsigned)(wz + L.z0 + z - (S - 1)) >= (unsigned)P) continue;
#pragma unroll
        for (int k = 0; k < NCM; ++k) acc[z][k] += zw[z] * f[k];
      }
    }
    wave_lds_sync();
  }
#pragma unroll
  for (int z = 0; z < ZPT; ++z) {
    const size_t gi = L.point(ng, z);
#pragma unroll
    for (int k = 0; k < NCM; ++k)
      if (k < cs.n) grids[(size_t)k * ngrid + gi] = acc[z][k];
  }
}

// Deformed lattices: the Gaussian takes an exponential per point.  A wavefront
// per tile and z part as above, but without lists or weight rows: the lanes
// test the particles of the 27 bins around the tile, 64 at a time, and stage
// those whose stencils meet it.  Bound by the exponentials.  (5003 spheres, 11
// components at 96^3 in FP64, support 9: 51 us; one wavefront per particle
// adding to the grid with atomics took 402 and a pass to clear the grids.)
template <typename T, int NCM, int ZPT>
__global__ void __launch_bounds__(256)
spread_deformed_kernel(const double *__restrict__ x, const double *__restrict__ q, Layout lq,
                       CompSet cs, GridGeom g, int nb, const int *__restrict__ bstart,
                       const int *__restrict__ bperm, T *__restrict__ grids, size_t ngrid) {
  constexpr int S = 8;
  __shared__ double lds_x[4][64][3];
  __shared__ int lds_o[4][64][6];   // tile's first point and its place in the stencil
  __shared__ T lds_q[4][64][NCM];
  const TileLane<S, ZPT> L(nb);
  if (L.tile >= nb * nb * nb) return;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int P = g.P, ng = g.ng;
  int first, pre, total;
  nbr27_setup(lane, L.tc[0], L.tc[1], L.tc[2], nb, bstart, first, pre, total);
  T acc[ZPT][NCM];
#pragma unroll
  for (int z = 0; z < ZPT; ++z)
#pragma unroll
    for (int k = 0; k < NCM; ++k) acc[z][k] = (T)0;
  const double kn3 = g.knorm * g.knorm * g.knorm;
  for (int base = 0; base < total; base += 64) {
    const int idx = base + lane;
    const int s = nbr27_slot(idx, first, pre);
    bool ok = idx < total;
    int p = 0, at[3] = {}, off[3] = {};
    double xp[3] = {};
    if (ok) {
      p = bperm[s];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        xp[d] = x[3 * (size_t)p + d];
        const int st = stencil_start(xp[d], g.h, P);
        int o = (st - L.tc[d] * S) % ng;
        o += o < 0 ? ng : 0;
        o -= o >= S ? ng : 0;
        off[d] = o;
        at[d] = st - o;   // the tile's first point, next to the particle
        ok = ok && o > -P;
      }
      ok = ok && off[2] < L.z0 + ZPT && off[2] + P > L.z0;
    }
    const unsigned long long m = __ballot(ok);
    const int cnt = __popcll(m);
    if (ok) {
      const int c = __popcll(m & ((1ull << lane) - 1ull));
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        lds_x[wave][c][d] = xp[d];
        lds_o[wave][c][d] = at[d];
        lds_o[wave][c][3 + d] = off[d];
      }
      const double *qp = q + (size_t)p * lq.stride - lq.off;
#pragma unroll
      for (int k = 0; k < NCM; ++k) lds_q[wave][c][k] = k < cs.n ? (T)qp[cs.idx[k]] : (T)0;
    }
    wave_lds_sync();
    for (int c = 0; c < cnt; ++c) {
      const double *xc = lds_x[wave][c];
      const int *o = lds_o[wave][c];
      const bool in = (unsigned)(L.lx - o[3]) < (unsigned)P && (unsigned)(L.ly - o[4]) < (unsigned)P;
      const double dx = (o[0] + L.lx) * g.h - xc[0], dy = (o[1] + L.ly) * g.h - xc[1];
      const double exy = g.G[0] * dx * dx + g.G[1] * dy * dy + 2.0 * g.G[3] * dx * dy;
      const double lin = 2.0 * (g.G[4] * dx + g.G[5] * dy);
      const int oz = __builtin_amdgcn_readfirstlane(o[5]);
      T mom[NCM];
#pragma unroll
      for (int k = 0; k < NCM; ++k) mom[k] = lds_q[wave][c][k];
#pragma unroll
      for (int z = 0; z < ZPT; ++z) {
        if ((unsigned)(L.z0 + z - oz) >= (unsigned)P) continue;
        const double dz = (o[2] + L.z0 + z) * g.h - xc[2];
        const double e = exp(-g.kcoef * (exy + (lin + g.G[2] * dz) * dz));
        const T w = in ? (T)(kn3 * e) : (T)0;
#pragma unroll
        for (int k = 0; k < NCM; ++k) acc[z][k] += w * mom[k];
      }
    }
    wave_lds_sync();
  }
#pragma unroll
  for (int z = 0; z < ZPT; ++z) {
    const size_t gi = L.point(ng, z);
#pragma unroll
    for (int k = 0; k < NCM; ++k)
      if (k < cs.n) grids[(size_t)k * ngrid + gi] = acc[z][k];
  }
}

// Derivative gridding of the couplets: three grids
// D_i(x_n) = sum_b sum_j C_b,ij dK/dx_j (x_n - x_b), with C_b = S_b + A_b the
// particle's couplet, S_b the symmetric traceless stresslet of its five
// components in the Y_q basis and A_b x = (1/2) L_b x x its torque.  Their
// transform is i C^ k K^, so the k-space factors of the stresslet column,
// -3 i f1(ka) Y_q k, and of the torque column, (3/2) i f1(ka) k x e_c,
// become one factor -3 f1(ka) on D^ (Eq. WSops with the gradient moved onto
// the Gaussian).  Torques (HL) and stresslets (HS), either or both, start at
// components iL and iS of the vector.  Per point
//   D_i = (C_ix g_x w_y + C_iy w_x g_y) w_z + C_iz w_x w_y g_z,
// the two brackets constant along the lane's z-column.
template <typename T, int S, int ZPT, bool HL, bool HS>
__global__ void __launch_bounds__(256)
spread_deriv_kernel(const double *__restrict__ q, Layout lq, int iL, int iS, int ng, int P, int nb,
                    const int *__restrict__ tstart, const TileRec *__restrict__ rec,
                    const cplx<T> *__restrict__ wt, int rw, T *__restrict__ grids, size_t ngrid) {
  using W = cplx<T>;   // (weight, gradient weight)
  constexpr int NI = 3 * S, NQ = 12;
  __shared__ __align__(16) W lds_w[4][TCH * NI];
  __shared__ __align__(16) T lds_c[4][TCH * NQ];
  const TileLane<S, ZPT> L(nb);
  if (L.tile >= nb * nb * nb) return;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  W *items = lds_w[wave];
  T *cpl = lds_c[wave];
  const int lo = tstart[L.tile], hi = tstart[L.tile + 1];
  T acc[ZPT][3];
#pragma unroll
  for (int z = 0; z < ZPT; ++z)
#pragma unroll
    for (int k = 0; k < 3; ++k) acc[z][k] = (T)0;
  for (int base = lo; base < hi; base += TCH) {
    const int cnt = min(TCH, hi - base);
    const TileRec r = rec[base + min(lane, cnt - 1)];
    double sv[5] = {}, lv[3] = {};
    if (lane < cnt) {
      const double *qp = q + (size_t)r.p * lq.stride - lq.off;
      if constexpr (HS)
#pragma unroll
        for (int k = 0; k < 5; ++k) sv[k] = qp[iS + k];
      if constexpr (HL)
#pragma unroll
        for (int k = 0; k < 3; ++k) lv[k] = qp[iL + k];
    }
    stage_windows<W, S>(r, cnt, rw, items, [&](size_t e) { return wt[e]; });
    if (lane < cnt) {
      const T r2 = (T)0.70710678118654752440, r6 = (T)0.40824829046386301637;
      const T xy = r2 * (T)sv[0], xz = r2 * (T)sv[1], yz = r2 * (T)sv[2], a = r2 * (T)sv[3],
              b = r6 * (T)sv[4];
      const T lx = (T)0.5 * (T)lv[0], ly = (T)0.5 * (T)lv[1], lz = (T)0.5 * (T)lv[2];
      T *o = cpl + lane * NQ;   // rows of C, four apart
      o[0] = b + a;      o[1] = xy - lz;  o[2] = xz + ly;
      o[4] = xy + lz;    o[5] = b - a;    o[6] = yz - lx;
      o[8] = xz - ly;    o[9] = yz + lx;  o[10] = (T)-2 * b;
    }
    wave_lds_sync();
    for (int c = 0; c < cnt; ++c) {
      const int wz = __builtin_amdgcn_readlane(r.win, c) >> 16;
      const W *w = items + c * NI;
      const T *C = cpl + c * NQ;
      const W X = w[L.lx], Y = w[S + L.ly];
      const T gxwy = X.y * Y.x, wxgy = X.x * Y.y, wxwy = X.x * Y.x;
      T a[3], b[3];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        a[i] = C[4 * i] * gxwy + C[4 * i + 1] * wxgy;
        b[i] = C[4 * i + 2] * wxwy;
      }
      W zw[ZPT];
#pragma unroll
      for (int z = 0; z < ZPT; ++z) zw[z] = w[2 * S + L.z0 + z];
#pragma unroll
      for (int z = 0; z < ZPT; ++z) {
        if (S == 8 && (unsigned)(wz + L.z0 + z - (S - 1)) >= (unsigned)P) continue;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          acc[z][i] += a[i] * zw[z].x;
          acc[z][i] += b[i] * zw[z].y;
        }
      }
    }
    wave_lds_sync();
  }
#pragma unroll
  for (int z = 0; z < ZPT; ++z) {
    const size_t gi = L.point(ng, z);
#pragma unroll
    for (int k = 0; k < 3; ++k) grids[(size_t)k * ngrid + gi] = acc[z][k];
  }
}

// --------------------------------------------------------- interpolation --

// Deformed lattices, where the Gaussian does not factorise over the lattice
// axes, and grids without spreading tiles, whose handles keep no weight rows:
// one wavefront per particle, lane s covering stencil points s, s + 64, ...
// (interp.hip has the others' kernels).
template <typename T>
__global__ void __launch_bounds__(256)
interp_generic_kernel(const double *__restrict__ x, const T *__restrict__ grids,
                       size_t ngrid, CompSet cs, GridGeom g, const int *__restrict__ order,
                       int64_t n, double *__restrict__ out, Layout lo, int accumulate,
                       double scale) {
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)xcd_block(blockIdx.x, gridDim.x) * 4 + (threadIdx.x >> 6);
  if (t >= n) return;
  const int64_t p = order ? order[t] : t;
  const double px = x[3 * p], py = x[3 * p + 1], pz = x[3 * p + 2];
  const int P = g.P, P3 = P * P * P;
  const int ix0 = stencil_start(px, g.h, P);
  const int iy0 = stencil_start(py, g.h, P);
  const int iz0 = stencil_start(pz, g.h, P);
  T acc[NC];
#pragma unroll
  for (int k = 0; k < NC; ++k) acc[k] = (T)0;
  const double kn3 = g.knorm * g.knorm * g.knorm;
  // U points at a time, their loads in flight together (points beyond the
  // stencil: weight zero at its first point)
  constexpr int U = 4;
  for (int s0 = lane; s0 < P3; s0 += 64 * U) {
    T w[U];
    uint32_t gi[U];   // offsets within one grid: below 2^31
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int s = s0 + 64 * u < P3 ? s0 + 64 * u : 0;
      const int a = s % P, b = (s / P) % P, c = s / (P * P);
      const double dx = (ix0 + a) * g.h - px;
      const double dy = (iy0 + b) * g.h - py;
      const double dz = (iz0 + c) * g.h - pz;
      const double r2 = g.def ? qform(g.G, dx, dy, dz) : dx * dx + dy * dy + dz * dz;
      w[u] = s0 + 64 * u < P3 ? (T)(kn3 * exp(-g.kcoef * r2)) : (T)0;
      gi[u] = ((uint32_t)wrapi(iz0 + c, g.ng) * g.ng + wrapi(iy0 + b, g.ng)) * g.ng
              + wrapi(ix0 + a, g.ng);
    }
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      if (k >= cs.n) break;
      T v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = grids[(size_t)k * ngrid + gi[u]];
#pragma unroll
      for (int u = 0; u < U; ++u) acc[k] += w[u] * v[u];
    }
  }
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    if (k < cs.n) {
      T v = acc[k];
      for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
      acc[k] = v;
    }
  }
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      if (k < cs.n) {
        double *o = out + p * lo.stride + cs.idx[k] - lo.off;
        const double v = scale * (double)acc[k];
        *o = accumulate ? *o + v : v;
      }
    }
  }
}

// ------------------------------------------------------ k-space kernels --

// Wave vector of grid index i (FFT order).
__device__ __forceinline__ int kidx(int i, int n) { return i < n / 2 ? i : i - n; }

// Shape factors j0(x) = sin x / x and f1(x) = (sin x - x cos x)/x^3
// (Eq. WSops); series below x = 0.1 where the closed form cancels.
__device__ __forceinline__ void shape_factors(double x, double &j0, double &f1) {
  if (x < 0.1) {
    const double x2 = x * x;
    j0 = 1.0 - x2 / 6.0 * (1.0 - x2 / 20.0 * (1.0 - x2 / 42.0));
    f1 = 1.0 / 3.0 - x2 / 30.0 * (1.0 - x2 / 28.0 * (1.0 - x2 / 54.0));
  } else {
    double s, c;
    sincos(x, &s, &c);
    j0 = s / x;
    f1 = (s - x * c) / (x * x * x);
  }
}

// k-table entry type per precision: double4 for the FP64 kernels, float4
// (the same values rounded) for the FP32 ones.
template <typename T> struct TabT;
template <> struct TabT<double> { using type = double4; };
template <> struct TabT<float> { using type = float4; };

struct KGeom {
  int ng;
  double twopi_L;     // 2 pi / L
  double a;
  double inv4xi2;     // 1 / (4 xi^2)
  double one_m_etas;  // 1 - eta_s
  double pref_m;      // mobility: h^6 / (V eta)
  double pref_n;      // noise: h^3 / sqrt(V eta)
  int def;            // deformed lattice: k = (2 pi / L) A^-T n
  double Ai[9];       // A^-1 (row-major)
};

// Wave vector of the integer index (i, j, l): (2 pi / L) A^-T (i, j, l).
__device__ __forceinline__ void deformed_k(const KGeom &kg, int i, int j, int l, double *kv) {
#pragma unroll
  for (int r = 0; r < 3; ++r)
    kv[r] = kg.twopi_L * (kg.Ai[r] * i + kg.Ai[3 + r] * j + kg.Ai[6 + r] * l);
}

// Radial factors of a wave number with square k2:
//   x = j0(ka), y = f1(ka), z = h^6/(V eta) (1 + u) e^{-(1 - eta_s) u} / k^2,
//   w = h^3/sqrt(V eta) sqrt(1 + u) e^{-(1 - eta_s) u / 2} / k,  u = k^2 / 4 xi^2
// (the mobility scaling of Eq. WSops2 with both Gaussian factors divided out,
// and the amplitude of Eq. FFTsqrt).
__device__ __forceinline__ double4 radial_factors(const KGeom &kg, double k2) {
  const double k = sqrt(k2);
  double j0, f1;
  shape_factors(k * kg.a, j0, f1);
  const double u = k2 * kg.inv4xi2;
  const double mob = kg.pref_m * (1.0 + u) * exp(-kg.one_m_etas * u) / k2;
  const double amp = kg.pref_n * sqrt(1.0 + u) * exp(-0.5 * kg.one_m_etas * u) / k;
  return double4{j0, f1, mob, amp};
}

// Every stored wave vector of the cube is k = (2 pi / L) (i, j, l) with
// integers, so its radial factors depend on the integer n2 = i^2 + j^2 + l^2 <=
// 3 (N/2)^2 only: a table of them, entry 0 (k = 0) zero.
__global__ void __launch_bounds__(256)
ktable_kernel(KGeom kg, int len, double4 *__restrict__ tab) {
  const int n2 = blockIdx.x * blockDim.x + threadIdx.x;
  if (n2 >= len) return;
  tab[n2] = n2 == 0 ? double4{0, 0, 0, 0}
                    : radial_factors(kg, kg.twopi_L * kg.twopi_L * (double)n2);
}

// Column of P(k) for moment component c (0..10), as (coef, col): the
// contribution to rho is coef * col * g with coef real for F (j0) and
// imaginary for L and s:
//   F_c:  j0 e_c;   L_l: (3i/2) f1 (k x e_l);   s_q: -3i f1 Y_q k.
// R is the arithmetic type (double, or float in the FP32 kernels).
template <typename R>
__device__ __forceinline__ void p_column(int c, R kx, R ky, R kz, R j0, R f1, bool &imag,
                                         R &cx, R &cy, R &cz) {
  const R r2 = (R)0.70710678118654752440, r6 = (R)0.40824829046386301637;
  imag = c >= 3;
  const R a = (R)1.5 * f1, b = (R)-3.0 * f1;
  switch (c) {
    case 0: cx = j0;  cy = 0;   cz = 0;   break;
    case 1: cx = 0;   cy = j0;  cz = 0;   break;
    case 2: cx = 0;   cy = 0;   cz = j0;  break;
    case 3: cx = 0;   cy = a * kz;  cz = -a * ky; break;       // k x e_x
    case 4: cx = -a * kz; cy = 0;   cz = a * kx;  break;       // k x e_y
    case 5: cx = a * ky;  cy = -a * kx; cz = 0;   break;       // k x e_z
    case 6: cx = b * r2 * ky; cy = b * r2 * kx; cz = 0; break;
    case 7: cx = b * r2 * kz; cy = 0; cz = b * r2 * kx; break;
    case 8: cx = 0; cy = b * r2 * kz; cz = b * r2 * ky; break;
    case 9: cx = b * r2 * kx; cy = -b * r2 * ky; cz = 0; break;
    default: cx = b * r6 * kx; cy = b * r6 * ky; cz = (R)-2.0 * b * r6 * kz; break;
  }
}

// P_c as a linear form in the integer wave vector n, P_c(k) = B + (2 pi / L) CK
// A n without its radial factor: B = e_c for forces (real), A for couplets
// (times i; the column of p_column with f1 = 1).  With CK and 2 pi / L apart, n
// and nearly all of A are exact in FP32 too; the constants join the radial
// factors in FP64 before those are rounded (rounded into the columns they shift
// every mode alike: -3 / sqrt 2 alone the stresslet-strain block by 9e-8).
constexpr double CK = -3.0 * 0.70710678118654752440;
template <typename R> struct ColumnForm {
  R A[3][3], B[3];
  __device__ __forceinline__ explicit ColumnForm(int c) {
    const R r2 = (R)1, r6 = (R)0.57735026918962576451;   // 1 / sqrt 3
    const R a = (R)-0.70710678118654752440;              // 1.5 / CK
#pragma unroll
    for (int m = 0; m < 3; ++m) B[m] = c == m ? (R)1 : (R)0;
    A[0][0] = c == 9 ? r2 : (c == 10 ? r6 : (R)0);
    A[1][1] = c == 9 ? -r2 : (c == 10 ? r6 : (R)0);
    A[2][2] = c == 10 ? (R)-2 * r6 : (R)0;
    A[0][1] = c == 6 ? r2 : (c == 5 ? a : (R)0);
    A[1][0] = c == 6 ? r2 : (c == 5 ? -a : (R)0);
    A[0][2] = c == 7 ? r2 : (c == 4 ? -a : (R)0);
    A[2][0] = c == 7 ? r2 : (c == 4 ? a : (R)0);
    A[1][2] = c == 8 ? r2 : (c == 3 ? a : (R)0);
    A[2][1] = c == 8 ? r2 : (c == 3 ? -a : (R)0);
  }
  // the part of a column that n_x and n_y give
  __device__ __forceinline__ void fixed(R kx, R ky, R *o) const {
#pragma unroll
    for (int m = 0; m < 3; ++m) o[m] = B[m] + A[m][0] * kx + A[m][1] * ky;
  }
};

// rho += P_c(k) g
template <typename C, typename R>
__device__ __forceinline__ void add_P(int c, C gv, const R *kv, R j0, R f1, C *rho) {
  bool imag;
  R cx, cy, cz;
  p_column<R>(c, kv[0], kv[1], kv[2], j0, f1, imag, cx, cy, cz);
  const R gx = (R)gv.x, gy = (R)gv.y;
  if (!imag) {
    rho[0].x += cx * gx; rho[0].y += cx * gy;
    rho[1].x += cy * gx; rho[1].y += cy * gy;
    rho[2].x += cz * gx; rho[2].y += cz * gy;
  } else {
    // i col g = col (-g.y, g.x)
    rho[0].x -= cx * gy; rho[0].y += cx * gx;
    rho[1].x -= cy * gy; rho[1].y += cy * gx;
    rho[2].x -= cz * gy; rho[2].y += cz * gx;
  }
}

// W_c = P_c^+ u = conj(coef) col . u
template <typename C, typename R>
__device__ __forceinline__ C apply_Pdag(int c, const C *u, const R *kv, R j0, R f1) {
  bool imag;
  R cx, cy, cz;
  p_column<R>(c, kv[0], kv[1], kv[2], j0, f1, imag, cx, cy, cz);
  const R re = cx * (R)u[0].x + cy * (R)u[1].x + cz * (R)u[2].x;
  const R im = cx * (R)u[0].y + cy * (R)u[1].y + cz * (R)u[2].y;
  C w;
  if (!imag) {
    w.x = re;
    w.y = im;
  } else {
    // conj(i) = -i: -i (re + i im) = im - i re
    w.x = im;
    w.y = -re;
  }
  return w;
}

// Stored half-spectrum mode (ix < n/2, iy, iz) that is zeroed: a Nyquist
// index in y or z, or k = 0 (the x Nyquist column is not stored).
__device__ __forceinline__ bool zero_mode(int ix, int iy, int iz, int n) {
  const int h = n / 2;
  return iy == h || iz == h || (ix == 0 && iy == 0 && iz == 0);
}

// Fused z transform + k-space kernel + inverse z transform (Eq. WSops2 from
// the half spectra after the x and y transforms back to them).  A workgroup
// owns TL neighbouring kx columns at one ky, i.e. TL z-lines, each
// transformed by TPL threads that hold E modes in registers.  For every input
// component the z transform runs in registers and the mode is folded at
// once into rho(k) = sum_c P_c(k) G_c(k) (three complex numbers per mode,
// kept in registers), so the inputs stream through one at a time.  Then
// u = scale (I - k^k^) rho, and for every output component P_q^+ u is formed
// in the same registers -- the inverse transform runs the passes in reverse
// order, so its input layout is the forward output layout -- transformed back
// along z and stored.  One read of the inputs and one write of the outputs.
// DG (derivative gridding): the components are grid codes, 0-2 the force
// grids F^ (factor j0(ka)) and 3-5 the couplet grids D^ spread with the
// Gaussian's gradient (factor -3 f1(ka)) on input, so rho = j0 F^ - 3 f1 D^;
// on output 0-2 the velocity grids j0(ka) u^ and 3-5 the grids
// v^ = 3 f1(ka) u^ whose gradient the interpolation takes.
// The radial factors j0 and f1 come out of the sums over components of one
// kind (forces, couplets): with one kind on a side its factor is applied with
// the projection's scale, once per mode; with both, the inputs' couplets come
// first, the accumulator takes f1, and the forces follow with j0 each, and the
// outputs' forces come first (KOrder).  With the factors out of the inner
// loops and the columns as linear forms an FP32 thread has registers for
// twice the modes, and a line takes half the exchanges.  Bound by the memory
// and the exchanges' barriers: five components each way at 384^3 in FP32 1.31
// -> 0.82 ms (1.8 -> 2.8 TB/s), six in and five out 1.52 -> 1.3 ms; at 128^3
// in FP64, six in and three out, 44 -> 35 us.  At 512^3 in FP32, six in and
// three out, it is 3 % slower (2.09 -> 2.15 ms).
struct KOrder {
  int n, both;             // both kinds present
  int kind;                // else the kind: 0 forces, 1 couplets
  int slot[NC], comp[NC];  // grid slots and their components
};

template <typename T, int N, bool DG>
__global__ void __launch_bounds__(512)
kspace_fused_kernel(const cplx<T> *__restrict__ in, KOrder cin, cplx<T> *__restrict__ out,
                    KOrder cout, KGeom kg, const typename TabT<T>::type *__restrict__ ktab,
                    const cplx<T> *__restrict__ tw, int TL) {
  using C = cplx<T>;
  constexpr int E = fused_e<T>(N), M = N / 2;
  using S = Shape<N, E>;
  constexpr int R0 = S::first(false), RL = S::last(false);
  extern __shared__ unsigned char smem_raw[];
  C *lds = reinterpret_cast<C *>(smem_raw);
  const int tiles = M / TL;
  // neighbouring x tiles share the cache lines of their row segments (TL
  // complex numbers, 32 or 64 bytes at long lines): they run on one XCD, so
  // its L2 fetches each line once (at 512^3 in FP32 the HBM reads were five
  // times the data with tiles spread over the XCDs)
  const int lb = (int)xcd_block(blockIdx.x, gridDim.x);
  const int xt = lb % tiles, iy = lb / tiles;
  const int line = threadIdx.x % TL, t = threadIdx.x / TL;
  const int ix = xt * TL + line;
  const int ky = kidx(iy, N);
  const size_t hsz = (size_t)M * N * N, plane = (size_t)N * M;
  const size_t base = (size_t)iy * M + ix;
  // the couplets' constant (ColumnForm), and with that of the sides whose
  // factor joins the projection's scale
  const double ck = kg.twopi_L * CK;
  const double cks = (!cin.both && cin.kind ? ck : 1.0) * (!cout.both && cout.kind ? ck : 1.0);
  C rho[E][3];
#pragma unroll
  for (int e = 0; e < E; ++e)
#pragma unroll
    for (int m = 0; m < 3; ++m) rho[e][m] = C{(T)0, (T)0};
  // table entry of the thread's mode e
  const auto entry = [&](int e) {
    const int kz = kidx(reg_pos<N, E, RL>(t, e / RL, e % RL), N);
    return ktab[ix * ix + ky * ky + kz * kz];
  };
  // factors of both kinds: where registers allow, read once and kept; else j0
  // is read for a side's forces and f1 on the spot
  constexpr bool KEEP = N % 3 != 0;
  const bool both = cin.both || cout.both;
  T j0[E], f1[KEEP ? E : 1];
  const auto read_j0 = [&] {
#pragma unroll
    for (int e = 0; e < E; ++e) j0[e] = (T)entry(e).x;
  };
  if constexpr (KEEP)
    if (both)
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const auto tb = entry(e);
        j0[e] = (T)tb.x;
        f1[e] = (T)tb.y;
      }
  const auto times_f1 = [&] {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      T f;
      if constexpr (KEEP) f = f1[e];
      else f = (T)entry(e).y;
      if constexpr (!DG) f = (T)(ck * (double)f);
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        rho[e][m].x *= f;
        rho[e][m].y *= f;
      }
    }
  };
  // where registers allow, the next component's z-line is loaded while the
  // current one is transformed (the barriers of the exchanges wait on LDS
  // traffic only)
  constexpr bool AHEAD = E <= 8;
  const C tw0 = tw_fetch<C, N>(tw);
  C v[E], vn[AHEAD ? E : 1];
  const auto load = [&](C *dst, int p) {
    const C *src = in + (size_t)cin.slot[p] * hsz + base;
#pragma unroll
    for (int b = 0; b < E / R0; ++b)
#pragma unroll
      for (int r = 0; r < R0; ++r) dst[b * R0 + r] = src[reg_pos<N, E, R0>(t, b, r) * plane];
  };
  if constexpr (AHEAD) load(vn, 0);
  C *twl = lds + (size_t)TL * N;
  tw_store<C, N>(twl, tw0, tw);
  for (int p = 0; p < cin.n; ++p) {
    if constexpr (AHEAD) {
#pragma unroll
      for (int e = 0; e < E; ++e) v[e] = vn[e];
      if (p + 1 < cin.n) load(vn, p + 1);
    } else {
      load(v, p);
    }
    reg_fft_forward<T, N, E>(v, t, lds, TL, line, twl);
    const int c = cin.comp[p];
    if (cin.both && c < 3) {
      if (cin.comp[p - 1] >= 3) {
        times_f1();
        if constexpr (!KEEP) read_j0();
      }
#pragma unroll
      for (int e = 0; e < E; ++e) {
        v[e].x *= j0[e];
        v[e].y *= j0[e];
      }
    }
    // (zeroed modes are zeroed at the fold)
    if constexpr (DG) {
      const T f = c < 3 ? (T)1 : (T)-3;
#pragma unroll
      for (int m = 0; m < 3; ++m)
        if (m == c % 3)
#pragma unroll
          for (int e = 0; e < E; ++e) {
            rho[e][m].x += f * v[e].x;
            rho[e][m].y += f * v[e].y;
          }
    } else {
      const ColumnForm<T> F(c);
      T col0[3];
      F.fixed((T)ix, (T)ky, col0);
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const T kz = (T)kidx(reg_pos<N, E, RL>(t, e / RL, e % RL), N);
        const T gx = c < 3 ? v[e].x : -v[e].y, gy = c < 3 ? v[e].y : v[e].x;
#pragma unroll
        for (int m = 0; m < 3; ++m) {
          const T col = col0[m] + F.A[m][2] * kz;
          rho[e][m].x += col * gx;
          rho[e][m].y += col * gy;
        }
      }
    }
  }
  // u = scale (I - k^k^) rho
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int iz = reg_pos<N, E, RL>(t, e / RL, e % RL);
    const int kz = kidx(iz, N);
    const int n2 = ix * ix + ky * ky + kz * kz;
    const auto tb = ktab[n2];
    if (zero_mode(ix, iy, iz, N)) {
#pragma unroll
      for (int m = 0; m < 3; ++m) rho[e][m] = C{(T)0, (T)0};
      continue;
    }
    T scale = (T)tb.z;
    if (!cin.both) scale *= cin.kind ? (T)tb.y : (T)tb.x;
    if (!cout.both) scale *= cout.kind ? (T)tb.y : (T)tb.x;
    if constexpr (!DG) scale = (T)(cks * (double)scale);
    const T kv[3] = {(T)ix, (T)ky, (T)kz};
    const T inv = (T)1 / (T)n2;
    T krx = 0, kry = 0;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      krx += kv[m] * rho[e][m].x;
      kry += kv[m] * rho[e][m].y;
    }
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      rho[e][m].x = scale * (rho[e][m].x - kv[m] * krx * inv);
      rho[e][m].y = scale * (rho[e][m].y - kv[m] * kry * inv);
    }
  }
  if constexpr (!KEEP)
    if (cout.both) read_j0();
  for (int q = 0; q < cout.n; ++q) {
    const int c = cout.comp[q];
    if (cout.both && c >= 3 && cout.comp[q - 1] < 3) times_f1();
    if constexpr (DG) {
      const T f = c < 3 ? (T)1 : (T)3;
#pragma unroll
      for (int m = 0; m < 3; ++m)
        if (m == c % 3)
#pragma unroll
          for (int e = 0; e < E; ++e) v[e] = C{f * rho[e][m].x, f * rho[e][m].y};
    } else {
      const ColumnForm<T> F(c);
      T col0[3];
      F.fixed((T)ix, (T)ky, col0);
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const T kz = (T)kidx(reg_pos<N, E, RL>(t, e / RL, e % RL), N);
        T re = (T)0, im = (T)0;
#pragma unroll
        for (int m = 0; m < 3; ++m) {
          const T col = col0[m] + F.A[m][2] * kz;
          re += col * rho[e][m].x;
          im += col * rho[e][m].y;
        }
        // conj(i) = -i on couplets
        v[e] = c < 3 ? C{re, im} : C{im, -re};
      }
    }
    if (cout.both && c < 3)
#pragma unroll
      for (int e = 0; e < E; ++e) {
        v[e].x *= j0[e];
        v[e].y *= j0[e];
      }
    reg_fft_inverse<T, N, E>(v, t, lds, TL, line, twl);
    C *dst = out + (size_t)cout.slot[q] * hsz + base;
#pragma unroll
    for (int b = 0; b < E / R0; ++b)
#pragma unroll
      for (int r = 0; r < R0; ++r) dst[reg_pos<N, E, R0>(t, b, r) * plane] = v[b * R0 + r];
  }
}

// Derivative gridding on long lines with all three grids in registers: a
// workgroup owns TL neighbouring kx columns at one ky (row segments of up to
// 128 bytes), and the TPL threads of a line hold E modes of each of the
// three couplet grids D^.  Every load is issued before the first transform; the
// three forward z transforms run one after the other through one LDS area;
// each mode is then folded with its three components at hand,
// out = -9 f1^2 scale (I - k^k^) D^; and the three inverse transforms
// follow.  No accumulator and no prefetch copy: 3 E complex numbers per
// thread, so E can be as large as the line passes' (fewer exchanges).
template <typename T, int N, int E>
__global__ void __launch_bounds__(512)
kspace_dg3_kernel(const cplx<T> *__restrict__ in, cplx<T> *__restrict__ out, KGeom kg,
                  const T *__restrict__ kdg, const cplx<T> *__restrict__ tw, int TL) {
  using C = cplx<T>;
  constexpr int M = N / 2;
  using S = Shape<N, E>;
  constexpr int R0 = S::first(false), RL = S::last(false);
  extern __shared__ unsigned char smem_raw[];
  C *lds = reinterpret_cast<C *>(smem_raw);
  const int tiles = M / TL;
  const int lb = (int)xcd_block(blockIdx.x, gridDim.x);
  const int xt = lb % tiles, iy = lb / tiles;
  const int line = threadIdx.x % TL, t = threadIdx.x / TL;
  const int ix = xt * TL + line;
  const int ky = kidx(iy, N);
  const size_t hsz = (size_t)M * N * N, plane = (size_t)N * M;
  const size_t base = (size_t)iy * M + ix;
  const C tw0 = tw_fetch<C, N>(tw);
  C v[3][E];
#pragma unroll
  for (int m = 0; m < 3; ++m)
#pragma unroll
    for (int b = 0; b < E / R0; ++b)
#pragma unroll
      for (int r = 0; r < R0; ++r)
        v[m][b * R0 + r] = in[m * hsz + base + reg_pos<N, E, R0>(t, b, r) * plane];
  C *twl = lds + (size_t)TL * N;
  tw_store<C, N>(twl, tw0, tw);
#pragma unroll
  for (int m = 0; m < 3; ++m) reg_fft_forward<T, N, E>(v[m], t, lds, TL, line, twl);
  // the factors of the thread's modes are loaded in groups of KG before
  // their first use (every mode's |k|^2 is inside the table, the zeroed
  // modes' included) instead of one round trip per mode
  constexpr int KG = sizeof(T) == 8 ? 2 : (E % 8 == 0 ? 8 : 6);
  static_assert(E % KG == 0, "whole groups");
#pragma unroll
  for (int g0 = 0; g0 < E; g0 += KG) {
    T sk[KG];
#pragma unroll
    for (int i = 0; i < KG; ++i) {
      const int e = g0 + i;
      const int kz = kidx(reg_pos<N, E, RL>(t, e / RL, e % RL), N);
      sk[i] = kdg[ix * ix + ky * ky + kz * kz];
    }
#pragma unroll
    for (int i = 0; i < KG; ++i) {
      const int e = g0 + i;
      const int iz = reg_pos<N, E, RL>(t, e / RL, e % RL);
      if (zero_mode(ix, iy, iz, N)) {
#pragma unroll
        for (int m = 0; m < 3; ++m) v[m][e] = C{(T)0, (T)0};
        continue;
      }
      const int kz = kidx(iz, N);
      const int n2 = ix * ix + ky * ky + kz * kz;
      const T s = sk[i];
      const T kv[3] = {(T)ix, (T)ky, (T)kz};
      const T inv = (T)1 / (T)n2;
      T krx = 0, kry = 0;
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        krx += kv[m] * v[m][e].x;
        kry += kv[m] * v[m][e].y;
      }
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        v[m][e].x = s * (v[m][e].x - kv[m] * krx * inv);
        v[m][e].y = s * (v[m][e].y - kv[m] * kry * inv);
      }
    }
  }
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    reg_fft_inverse<T, N, E>(v[m], t, lds, TL, line, twl);
#pragma unroll
    for (int b = 0; b < E / R0; ++b)
#pragma unroll
      for (int r = 0; r < R0; ++r)
        out[m * hsz + base + reg_pos<N, E, R0>(t, b, r) * plane] = v[m][b * R0 + r];
  }
}

// ----------------------------------------------------- Philox4x32-10 RNG --
// Counter-based generator of Salmon, Moraes, Dror & Shaw (SC'11), written
// from its published definition.

struct u4 { uint32_t x, y, z, w; };

__device__ __forceinline__ u4 philox4x32_10(u4 c, uint32_t k0, uint32_t k1) {
  const uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;
  const uint32_t W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)M0 * c.x, p1 = (uint64_t)M1 * c.z;
    const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
    const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
    c = u4{hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0};
    k0 += W0;
    k1 += W1;
  }
  return c;
}

// Four standard normals from one Philox block (Box-Muller).
__device__ __forceinline__ void normals4(u4 r, double *z) {
  const double s = 2.3283064365386963e-10;  // 2^-32
  const double u1 = ((double)r.x + 0.5) * s, u2 = ((double)r.y + 0.5) * s;
  const double u3 = ((double)r.z + 0.5) * s, u4v = ((double)r.w + 0.5) * s;
  const double ra = sqrt(-2.0 * log(u1)), rb = sqrt(-2.0 * log(u3));
  double sa, ca, sb, cb;
  sincospi(2.0 * u2, &sa, &ca);
  sincospi(2.0 * u4v, &sb, &cb);
  z[0] = ra * ca; z[1] = ra * sa; z[2] = rb * cb; z[3] = rb * sb;
}

// The same in FP32 (the wave noise of mixed-precision handles, whose grids
// are FP32): u in (0, 1] from the same 32-bit words.
__device__ __forceinline__ void normals4f(u4 r, double *z) {
  const float s = 2.3283064365386963e-10f;  // 2^-32
  const float u1 = ((float)r.x + 0.5f) * s, u2 = ((float)r.y + 0.5f) * s;
  const float u3 = ((float)r.z + 0.5f) * s, u4v = ((float)r.w + 0.5f) * s;
  const float ra = sqrtf(-2.0f * logf(u1)), rb = sqrtf(-2.0f * logf(u3));
  float sa, ca, sb, cb;
  sincospif(2.0f * u2, &sa, &ca);
  sincospif(2.0f * u4v, &sb, &cb);
  z[0] = ra * ca; z[1] = ra * sa; z[2] = rb * cb; z[3] = rb * sb;
}

template <bool F32 = false>
__device__ __forceinline__ void philox_normals(uint64_t seed, uint64_t counter,
                                               uint32_t stream, uint32_t index,
                                               int nblk, double *z) {
  for (int b = 0; b < nblk; ++b) {
    u4 c{index, stream * 16u + (uint32_t)b, (uint32_t)counter, (uint32_t)(counter >> 32)};
    const u4 r = philox4x32_10(c, (uint32_t)seed, (uint32_t)(seed >> 32));
    if constexpr (F32) normals4f(r, z + 4 * b);
    else normals4(r, z + 4 * b);
  }
}

enum : uint32_t { STREAM_REAL = 1, STREAM_WAVE = 2 };

// u(k) of the wave noise at stored mode (ix, iy, iz) (not a zeroed mode) and
// its radial factors tb and wave vector kv (see kspace_noise_kernel).
template <bool F32>
__device__ __forceinline__ void noise_mode(const double2 *__restrict__ psi, uint64_t seed,
                                           uint64_t counter, const KGeom &kg,
                                           const double4 *__restrict__ ktab, int ix, int iy,
                                           int iz, double2 uu[3], double4 &tb, double kv[3]) {
  const int n = kg.ng, hx = n / 2, hp = n / 2 + 1;
  // canonical member: kx > 0; or kx = 0 and ky in (0, n/2); or kx = ky = 0, kz in (0, n/2)
  const bool canon = ix > 0 || (iy > 0 && iy < hx) || (iy == 0 && iz < hx);
  const int cy = canon ? iy : (n - iy) % n, cz = canon ? iz : (n - iz) % n;
  const size_t cidx = ((size_t)cz * n + cy) * hp + ix;   // index in the noise layout
  double2 ps[3];
  if (psi) {
    const size_t psz = (size_t)n * n * hp;
    for (int m = 0; m < 3; ++m) ps[m] = psi[m * psz + cidx];
  } else {
    double z[8];
    philox_normals<F32>(seed, counter, STREAM_WAVE, (uint32_t)cidx, 2, z);
    const double s = 0.70710678118654752440;
    for (int m = 0; m < 3; ++m) ps[m] = double2{s * z[2 * m], s * z[2 * m + 1]};
  }
  if (!canon)
    for (int m = 0; m < 3; ++m) ps[m].y = -ps[m].y;
  const int ky = kidx(iy, n), kz = kidx(iz, n);
  double iv[3], inv;
  if (kg.def) {
    // deformed lattice: the projection and the radial factors of the true k
    deformed_k(kg, ix, ky, kz, kv);
    const double k2 = kv[0] * kv[0] + kv[1] * kv[1] + kv[2] * kv[2];
    tb = radial_factors(kg, k2);
    for (int m = 0; m < 3; ++m) iv[m] = kv[m];
    inv = 1.0 / k2;
  } else {
    const int n2 = ix * ix + ky * ky + kz * kz;
    tb = ktab[n2];
    kv[0] = kg.twopi_L * ix;
    kv[1] = kg.twopi_L * ky;
    kv[2] = kg.twopi_L * kz;
    iv[0] = (double)ix;
    iv[1] = (double)ky;
    iv[2] = (double)kz;
    inv = 1.0 / (double)n2;
  }
  double2 kr{0, 0};
  for (int m = 0; m < 3; ++m) {
    kr.x += iv[m] * ps[m].x;
    kr.y += iv[m] * ps[m].y;
  }
  for (int m = 0; m < 3; ++m) {
    uu[m].x = tb.w * (ps[m].x - iv[m] * kr.x * inv);
    uu[m].y = tb.w * (ps[m].y - iv[m] * kr.y * inv);
  }
}

// Wave-space square root (Eq. FFTsqrt): for each stored mode k,
//   u(k) = h^3 / sqrt(V eta) sqrt(1 + k^2/4xi^2) exp(-(1 - eta_s) k^2/8xi^2) / k
//          (I - kk) psi(k),   W_c(k) = P_c^+(k) u(k),
// with psi read (or drawn) at the canonical member of {k, -k}; the stored
// modes with kx = 0 outside the canonical half take conj psi(-k), so that the
// spectrum is Hermitian.
template <typename T>
__global__ void __launch_bounds__(256)
kspace_noise_kernel(const double2 *__restrict__ psi, uint64_t seed, uint64_t counter,
                    cplx<T> *__restrict__ out, CompSet cout, int dg, KGeom kg,
                    const double4 *__restrict__ ktab, const uint64_t *counter_dev) {
  using C = cplx<T>;
  const int n = kg.ng, hx = n / 2;
  const size_t hsz = (size_t)hx * n * n;
  const size_t tid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (tid >= hsz) return;
  if (counter_dev) counter = *counter_dev;
  const int ix = (int)(tid % hx);
  const int iy = (int)((tid / hx) % n);
  const int iz = (int)(tid / ((size_t)hx * n));
  if (zero_mode(ix, iy, iz, n)) {
    for (int q = 0; q < cout.n; ++q) out[q * hsz + tid] = C{(T)0, (T)0};
    return;
  }
  double2 uu[3];
  double4 tb;
  double kv[3];
  noise_mode<sizeof(T) == 4>(psi, seed, counter, kg, ktab, ix, iy, iz, uu, tb, kv);
  for (int q = 0; q < cout.n; ++q) {
    const int c = cout.idx[q];
    double2 w;
    if (dg) {
      // grid codes of derivative gridding: j0(ka) u^ (0-2), 3 f1(ka) u^ (3-5)
      const double f = c < 3 ? tb.x : 3.0 * tb.y;
      w = double2{f * uu[c % 3].x, f * uu[c % 3].y};
    } else {
      w = apply_Pdag<double2, double>(c, uu, kv, tb.x, tb.y);
    }
    out[q * hsz + tid] = C{(T)w.x, (T)w.y};
  }
}


// The wave noise of derivative gridding with the inverse z transform fused
// (cubic lattice, long lines): a workgroup owns TL neighbouring kx columns
// at one ky as the k-space kernels do; each thread forms u(k) of its E modes
// (noise_mode), keeps them with the factors j0(ka) and 3 f1(ka), and for
// every output grid code (0-2: j0 u^, 3-5: 3 f1 u^) transforms the line back
// along z and stores it -- the grids the y and x passes take next, without
// the round trip through HBM of a separate noise kernel and z pass.
template <typename T, int N, int E>
__global__ void __launch_bounds__(512)
kspace_noise_z_kernel(const double2 *__restrict__ psi, uint64_t seed, uint64_t counter,
                      cplx<T> *__restrict__ out, CompSet cout, KGeom kg,
                      const double4 *__restrict__ ktab, const cplx<T> *__restrict__ tw, int TL,
                      const uint64_t *counter_dev) {
  using C = cplx<T>;
  constexpr int M = N / 2;
  using S = Shape<N, E>;
  constexpr int R0 = S::first(false), RL = S::last(false);
  extern __shared__ unsigned char smem_raw[];
  C *lds = reinterpret_cast<C *>(smem_raw);
  if (counter_dev) counter = *counter_dev;
  const int tiles = M / TL;
  const int lb = (int)xcd_block(blockIdx.x, gridDim.x);
  const int xt = lb % tiles, iy = lb / tiles;
  const int line = threadIdx.x % TL, t = threadIdx.x / TL;
  const int ix = xt * TL + line;
  const size_t hsz = (size_t)M * N * N, plane = (size_t)N * M;
  const size_t base = (size_t)iy * M + ix;
  C *twl = lds + (size_t)TL * N;
  tw_store<C, N>(twl, tw_fetch<C, N>(tw), tw);
  C u[3][E];
  T fj[E], ff[E];
#pragma unroll
  for (int b = 0; b < E / RL; ++b)
#pragma unroll
    for (int r = 0; r < RL; ++r) {
      const int e = b * RL + r;
      const int iz = reg_pos<N, E, RL>(t, b, r);
      if (zero_mode(ix, iy, iz, N)) {
#pragma unroll
        for (int m = 0; m < 3; ++m) u[m][e] = C{(T)0, (T)0};
        fj[e] = ff[e] = (T)0;
        continue;
      }
      double2 uu[3];
      double4 tb;
      double kv[3];
      noise_mode<sizeof(T) == 4>(psi, seed, counter, kg, ktab, ix, iy, iz, uu, tb, kv);
#pragma unroll
      for (int m = 0; m < 3; ++m) u[m][e] = C{(T)uu[m].x, (T)uu[m].y};
      fj[e] = (T)tb.x;
      ff[e] = (T)(3.0 * tb.y);
    }
  for (int q = 0; q < cout.n; ++q) {
    const int c = cout.idx[q];
    C v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const T f = c < 3 ? fj[e] : ff[e];
#pragma unroll
      for (int m = 0; m < 3; ++m)
        if (m == c % 3) v[e] = C{f * u[m][e].x, f * u[m][e].y};
    }
    reg_fft_inverse<T, N, E>(v, t, lds, TL, line, twl);
    C *dst = out + (size_t)q * hsz + base;
#pragma unroll
    for (int b = 0; b < E / R0; ++b)
#pragma unroll
      for (int r = 0; r < R0; ++r) dst[reg_pos<N, E, R0>(t, b, r) * plane] = v[b * R0 + r];
  }
}

// k-space kernel of a deformed lattice on full 3D half spectra (x, y and z
// transformed): per stored mode, rho = sum_c P_c(k) G_c, u = scale
// (I - k^k^) rho, W_q = P_q^+ u, with k = (2 pi / L) A^-T n and the radial
// factors of that k (no |k|^2 table: k^2 is no longer an integer multiple
// of (2 pi / L)^2).  One thread per mode; in and out may be the same.
template <typename T>
__global__ void __launch_bounds__(256)
kspace_deformed_kernel(const cplx<T> *__restrict__ in, CompSet cin, cplx<T> *__restrict__ out,
                       CompSet cout, KGeom kg) {
  using C = cplx<T>;
  const int n = kg.ng, hx = n / 2;
  const size_t hsz = (size_t)hx * n * n;
  const size_t tid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (tid >= hsz) return;
  const int ix = (int)(tid % hx);
  const int iy = (int)((tid / hx) % n);
  const int iz = (int)(tid / ((size_t)hx * n));
  if (zero_mode(ix, iy, iz, n)) {
    for (int q = 0; q < cout.n; ++q) out[q * hsz + tid] = C{(T)0, (T)0};
    return;
  }
  double kv[3];
  deformed_k(kg, ix, kidx(iy, n), kidx(iz, n), kv);
  const double k2 = kv[0] * kv[0] + kv[1] * kv[1] + kv[2] * kv[2];
  const double4 tb = radial_factors(kg, k2);
  double2 rho[3] = {{0, 0}, {0, 0}, {0, 0}};
  for (int p = 0; p < cin.n; ++p) {
    const C g = in[p * hsz + tid];
    add_P<double2, double>(cin.idx[p], double2{(double)g.x, (double)g.y}, kv, tb.x, tb.y, rho);
  }
  double2 kr{0, 0};
  for (int m = 0; m < 3; ++m) {
    kr.x += kv[m] * rho[m].x;
    kr.y += kv[m] * rho[m].y;
  }
  for (int m = 0; m < 3; ++m) {
    rho[m].x = tb.z * (rho[m].x - kv[m] * kr.x / k2);
    rho[m].y = tb.z * (rho[m].y - kv[m] * kr.y / k2);
  }
  for (int q = 0; q < cout.n; ++q) {
    const double2 w = apply_Pdag<double2, double>(cout.idx[q], rho, kv, tb.x, tb.y);
    out[q * hsz + tid] = C{(T)w.x, (T)w.y};
  }
}

// Real-space noise psi1 ~ N(0, I), 11 per particle, from Philox.
__global__ void real_noise_kernel(uint64_t seed, uint64_t counter, int64_t n, int ncomp,
                                  const int *__restrict__ order, double *__restrict__ out,
                                  const uint64_t *counter_dev) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  if (counter_dev) counter = *counter_dev;
  double z[12];
  philox_normals(seed, counter, STREAM_REAL, (uint32_t)order[i], 3, z);
  for (int c = 0; c < ncomp; ++c) out[i * ncomp + c] = z[c];
}

// --------------------------------------------------------- small kernels --

template <typename T>
__global__ void __launch_bounds__(256) zero_kernel(T *g, size_t n) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256)
    g[i] = (T)0;
}

template <typename T>
__global__ void from_double_kernel(const double *src, size_t n, T *dst) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = (T)src[i];
}

template <typename T>
__global__ void to_double_kernel(const T *src, size_t n, double *dst, const int *stopped,
                                 int call) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n && !(stopped && *stopped == call)) dst[i] = (double)src[i];
}

// ----------------------------------------------------------- host side --

static KGeom kgeom(const Handle &h) {
  KGeom k;
  k.ng = h.d.grid;
  k.twopi_L = 2.0 * M_PI / h.p.box;
  k.a = h.p.radius;
  k.inv4xi2 = 1.0 / (4.0 * h.d.xi * h.d.xi);
  k.one_m_etas = 1.0 - h.d.eta_s;
  const double V = h.p.box * h.p.box * h.p.box;
  const double h3 = h.d.h * h.d.h * h.d.h;
  k.pref_n = h3 / sqrt(V * h.p.viscosity);
  k.pref_m = h3 * h3 / (V * h.p.viscosity);
  k.def = h.def.on;
  for (int i = 0; i < 9; ++i) k.Ai[i] = h.def.Ai[i];
  return k;
}

int ktable_len(int grid) { return 3 * (grid / 2) * (grid / 2) + 1; }

__global__ void __launch_bounds__(256)
ktable_to_float_kernel(const double4 *__restrict__ src, int len, float4 *__restrict__ dst) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < len) dst[i] = float4{(float)src[i].x, (float)src[i].y, (float)src[i].z, (float)src[i].w};
}

// The constraint operator's k-space factor of derivative gridding,
// -9 f1(ka)^2 times the mobility factor, one number per |k|^2 (the fold of
// kspace_dg3_kernel reads only this; a quarter of the four-factor entry).
__global__ void __launch_bounds__(256)
kdg_table_kernel(const double4 *__restrict__ tab, int len, double *__restrict__ d,
                 float *__restrict__ f) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= len) return;
  const double4 t = tab[i];
  const double v = -9.0 * t.y * t.y * t.z;
  d[i] = v;
  if (f) f[i] = (float)v;
}

void build_ktable(Handle &h) {
  const int len = ktable_len(h.d.grid);
  hipLaunchKernelGGL(ktable_kernel, dim3(nblocks(len, 256)), dim3(256), 0, h.stream, kgeom(h),
                     len, (double4 *)h.ktab);
  PSE_LAUNCH_CHECK();
  if (h.ktab32) {
    hipLaunchKernelGGL(ktable_to_float_kernel, dim3(nblocks(len, 256)), dim3(256), 0, h.stream,
                       (const double4 *)h.ktab, len, (float4 *)h.ktab32);
    PSE_LAUNCH_CHECK();
  }
  if (h.kdg) {
    hipLaunchKernelGGL(kdg_table_kernel, dim3(nblocks(len, 256)), dim3(256), 0, h.stream,
                       (const double4 *)h.ktab, len, h.kdg, h.kdg32);
    PSE_LAUNCH_CHECK();
  }
}

namespace {

// Component-count buckets: kernels keep NCM accumulators per point.
template <typename F> void with_ncm(int n, F f) {
  if (n <= 3) f(std::integral_constant<int, 3>());
  else if (n <= 5) f(std::integral_constant<int, 5>());
  else if (n <= 6) f(std::integral_constant<int, 6>());
  else f(std::integral_constant<int, NC>());
}

}  // namespace

// Workgroups of the tile kernels: four wavefronts each, `parts` per tile.
static dim3 tile_blocks(const Handle &h, int parts) {
  const size_t nb = (size_t)h.sbins.nc;
  return dim3(nblocks(nb * nb * nb * parts, 4));
}

static void check_tiles(const Handle &h) {
  if (!h.tiles_current)
    throw Error{PSE_ERR_INVALID, "spreading tile lists not built for these positions"};
}

template <typename T>
void spread(Handle &h, const double *x, const double *q, Layout lq, const CompSet &cs,
            T *grids) {
  const GridGeom g = geom(h);
  if (h.stile) {
    check_tiles(h);
    ProfScope ps(h, PK_SPREAD, (double)cs.n * h.ngrid * sizeof(T) + (double)h.n * (3 + cs.n) * 8);
    const int rw = weight_row(g.P, h.stile);
    const auto launch = [&](auto e, auto s, auto m, auto z) {
      constexpr int E = decltype(e)::value, S = decltype(s)::value, M = decltype(m)::value,
                    Z = decltype(z)::value;
      hipLaunchKernelGGL((spread_tile_kernel<T, E, S, M, Z>), tile_blocks(h, S == 8 ? 8 / Z : 1),
                         dim3(256), 0, h.stream, q, lq, cs, g.ng, g.P, h.sbins.nc,
                         (const int *)h.tl_start, (const TileRec *)h.tl_rec, weights<T>(h), rw,
                         grids, h.ngrid);
    };
    with_ncm(cs.n, [&](auto m) {
      // a lane's whole column while its accumulators leave room for several
      // wavefronts, half of it for the 11-component product
      using Z8 = std::integral_constant<int, decltype(m)::value <= 6 ? 8 : 4>;
      using I1 = std::integral_constant<int, 1>;
      using I2 = std::integral_constant<int, 2>;
      using I4 = std::integral_constant<int, 4>;
      using I8 = std::integral_constant<int, 8>;
      if (h.deriv) {
        if (h.stile == 8) launch(I2(), I8(), m, Z8());
        else launch(I2(), I4(), m, I1());
      } else {
        if (h.stile == 8) launch(I1(), I8(), m, Z8());
        else launch(I1(), I4(), m, I1());
      }
    });
    PSE_LAUNCH_CHECK();
    return;
  }
  if (h.sbins.nc) {   // deformed lattices (bin_tile)
    if (!h.tiles_current)
      throw Error{PSE_ERR_INVALID, "spreading tiles not built for these positions"};
    ProfScope ps(h, PK_SPREAD, (double)cs.n * h.ngrid * sizeof(T) + (double)h.n * (3 + cs.n) * 8);
    with_ncm(cs.n, [&](auto m) {
      constexpr int M = decltype(m)::value, Z = 4;
      hipLaunchKernelGGL((spread_deformed_kernel<T, M, Z>), tile_blocks(h, 8 / Z), dim3(256), 0,
                         h.stream, x, q, lq, cs, g, h.sbins.nc, (const int *)h.sbins.start,
                         (const int *)h.sbins.perm, grids, h.ngrid);
    });
    PSE_LAUNCH_CHECK();
    return;
  }
  zero_grids<T>(h, grids, cs.n);
  ProfScope ps(h, PK_SPREAD, (double)cs.n * h.ngrid * sizeof(T) + (double)h.n * (3 + cs.n) * 8);
  hipLaunchKernelGGL(spread_kernel<T>, dim3(nblocks(h.n, 4)), dim3(256), 0,
                     h.stream, x, q, lq, cs, g, (const int *)h.cells.perm, h.n,
                     grids, h.ngrid);
  PSE_LAUNCH_CHECK();
}

template <typename T>
void interp_generic(Handle &h, const double *x, const T *grids, const CompSet &cs, double *out,
                     Layout lo, bool accumulate, double scale) {
  ProfScope ps(h, PK_INTERP, (double)cs.n * h.ngrid * sizeof(T) + (double)h.n * (3 + cs.n) * 8);
  hipLaunchKernelGGL(interp_generic_kernel<T>, dim3(nblocks(h.n, 4)), dim3(256), 0, h.stream, x,
                     grids, h.ngrid, cs, geom(h), (const int *)h.cells.trav, h.n, out, lo,
                     accumulate ? 1 : 0, scale);
  PSE_LAUNCH_CHECK();
}

// Derivative gridding of couplets (tile lists required): the torques (hasL)
// and stresslets (hasS) of q in layout lq onto three grids with the Gaussian's
// gradient.
template <typename T>
void spread_deriv(Handle &h, const double *q, Layout lq, bool hasL, bool hasS, T *grids) {
  if (!h.stile) throw Error{PSE_ERR_INVALID, "derivative gridding unavailable"};
  check_tiles(h);
  const GridGeom g = geom(h);
  const int ncomp = (hasL ? 3 : 0) + (hasS ? 5 : 0);
  ProfScope ps(h, PK_SPREAD, 3.0 * h.ngrid * sizeof(T) + (double)h.n * (3 + ncomp) * 8);
  const int rw = weight_row(g.P, h.stile);
  const auto launch = [&](auto s, auto z, auto hl, auto hs) {
    constexpr int S = decltype(s)::value, Z = decltype(z)::value;
    hipLaunchKernelGGL((spread_deriv_kernel<T, S, Z, decltype(hl)::value, decltype(hs)::value>),
                       tile_blocks(h, 1), dim3(256), 0, h.stream, q, lq, 3, 6, g.ng, g.P,
                       h.sbins.nc, (const int *)h.tl_start, (const TileRec *)h.tl_rec,
                       reinterpret_cast<const cplx<T> *>(weights<T>(h)), rw, grids, h.ngrid);
  };
  const auto tile = [&](auto hl, auto hs) {
    if (h.stile == 8)
      launch(std::integral_constant<int, 8>(), std::integral_constant<int, 8>(), hl, hs);
    else launch(std::integral_constant<int, 4>(), std::integral_constant<int, 1>(), hl, hs);
  };
  if (hasL && hasS) tile(std::true_type(), std::true_type());
  else if (hasL) tile(std::true_type(), std::false_type());
  else tile(std::false_type(), std::true_type());
  PSE_LAUNCH_CHECK();
}

namespace {

template <typename T, int N>
void launch_fused(Handle &h, const cplx<T> *in, const CompSet &cin, cplx<T> *out,
                  const CompSet &cout, const cplx<T> *tw, bool dg) {
  using Tab = typename TabT<T>::type;
  const Tab *tab = sizeof(T) == 8 ? (const Tab *)h.ktab : (const Tab *)h.ktab32;
  // the constraint operator's derivative gridding (couplet grids each way):
  // all three grids in registers, row segments of up to 128 bytes (against
  // the accumulating form: 512^3 1.63 -> 1.14 ms in FP32 and 3.10 -> 2.32 in
  // FP64, 192^3 64 -> 46 us in FP32, 128^3 35 -> 22 us in FP64)
  const auto couplet3 = [](const CompSet &c) {
    return c.n == 3 && c.idx[0] == 3 && c.idx[1] == 4 && c.idx[2] == 5;
  };
  // exchange area of l lines and the twiddle table
  const auto lds_of = [](int l) { return (size_t)(l + 1) * N * sizeof(cplx<T>); };
  if constexpr (N >= 32) {
    if (dg && couplet3(cin) && couplet3(cout)) {
      constexpr int E = dg3_e<T>(N), TPL = N / E;
      int tl = (int)(128 / sizeof(cplx<T>));
      while (tl > 1 && (N / 2 % tl || tl * TPL > 512 || lds_of(tl) > (size_t)h.max_lds)) tl /= 2;
      const unsigned nb = (unsigned)(N * (N / 2 / tl));
      const T *kdg = sizeof(T) == 8 ? (const T *)h.kdg : (const T *)h.kdg32;
      if (!kdg) throw Error{PSE_ERR_INVALID, "k-space factor of derivative gridding missing"};
      hipLaunchKernelGGL((kspace_dg3_kernel<T, N, E>), dim3(nb), dim3(tl * TPL), lds_of(tl),
                         h.stream, in, out, kgeom(h), kdg, tw, tl);
      PSE_LAUNCH_CHECK();
      return;
    }
  }
  constexpr int TPL = N / fused_e<T>(N);
  // at least 64-byte row segments per workgroup on long lines (FP32 at 512^3,
  // six grids in and three out: 2.93 ms with 32 bytes, 2.13 with 64)
  const int tl = lines_per_block(N, TPL, N * sizeof(cplx<T>), (size_t)N / 2,
                                 TPL >= 64 ? 512 : 256);
  if (lds_of(tl) > (size_t)h.max_lds)
    throw Error{PSE_ERR_HIP, "k-space kernel: LDS beyond the device's per-workgroup limit"};
  // the slots with couplets first (inputs) or last (outputs)
  const auto order = [](const CompSet &c, bool couplets_first) {
    KOrder o{};
    for (int pass = 0; pass < 2; ++pass)
      for (int k = 0; k < c.n; ++k)
        if ((c.idx[k] >= 3) == (couplets_first == (pass == 0))) {
          o.slot[o.n] = k;
          o.comp[o.n++] = c.idx[k];
        }
    o.kind = o.n && o.comp[0] >= 3;
    o.both = o.n && (o.comp[0] >= 3) != (o.comp[o.n - 1] >= 3);
    return o;
  };
  const KOrder oin = order(cin, true), oout = order(cout, false);
  const unsigned nb = (unsigned)(N * (N / 2 / tl));
  if (dg)
    hipLaunchKernelGGL((kspace_fused_kernel<T, N, true>), dim3(nb), dim3(tl * TPL), lds_of(tl),
                       h.stream, in, oin, out, oout, kgeom(h), tab, tw, tl);
  else
    hipLaunchKernelGGL((kspace_fused_kernel<T, N, false>), dim3(nb), dim3(tl * TPL), lds_of(tl),
                       h.stream, in, oin, out, oout, kgeom(h), tab, tw, tl);
  PSE_LAUNCH_CHECK();
}

}  // namespace

#define PSE_CASE_F(NN) case NN: launch_fused<T, NN>(h, in, cin, out, cout, tw, dg); break;

template <typename T>
void kspace_fused(Handle &h, const cplx<T> *in, const CompSet &cin, cplx<T> *out,
                  const CompSet &cout, const cplx<T> *tw, bool dg) {
  const size_t hsz = h.ngrid / 2;
  ProfScope ps(h, PK_KSPACE, (double)(cin.n + cout.n) * hsz * sizeof(cplx<T>));
  switch (h.d.grid) {
    PSE_FOR_EACH_N(PSE_CASE_F)
    default: throw Error{PSE_ERR_INVALID, "unsupported FFT length"};
  }
}

template <typename T>
void kspace_deformed(Handle &h, const cplx<T> *in, const CompSet &cin, cplx<T> *out,
                     const CompSet &cout) {
  const size_t hsz = h.ngrid / 2;
  ProfScope ps(h, PK_KSPACE, (double)(cin.n + cout.n) * hsz * sizeof(cplx<T>));
  hipLaunchKernelGGL(kspace_deformed_kernel<T>, dim3(nblocks(hsz, 256)), dim3(256), 0,
                     h.stream, in, cin, out, cout, kgeom(h));
  PSE_LAUNCH_CHECK();
}

template <typename T>
bool kspace_noise_z(Handle &h, const double *psi, uint64_t seed, uint64_t counter,
                    cplx<T> *out, const CompSet &cout, const cplx<T> *tw) {
  // long power-of-two lines of a cubic lattice (measured at 512)
  if (h.def.on || h.d.grid != 512) return false;
  constexpr int N = 512, E = 8, TPL = N / E;
  const int tl = 512 / TPL;
  const size_t hsz = h.ngrid / 2;
  ProfScope ps(h, PK_NOISE, (double)cout.n * hsz * sizeof(cplx<T>) + (psi ? 3.0 * hsz * 16 : 0.0));
  // exchange area and the twiddle table
  const size_t lds = (size_t)(tl + 1) * N * sizeof(cplx<T>);
  if (lds > (size_t)h.max_lds) return false;
  const unsigned nb = (unsigned)(N * (N / 2 / tl));
  hipLaunchKernelGGL((kspace_noise_z_kernel<T, N, E>), dim3(nb), dim3(tl * TPL), lds,
                     h.stream, (const double2 *)psi, seed, counter, out, cout, kgeom(h),
                     (const double4 *)h.ktab, tw, tl, h.counter_dev);
  PSE_LAUNCH_CHECK();
  return true;
}

template <typename T>
void kspace_noise(Handle &h, const double *psi, uint64_t seed, uint64_t counter,
                  cplx<T> *out, const CompSet &cout, bool dg) {
  const size_t hsz = h.ngrid / 2;
  ProfScope ps(h, PK_NOISE, (double)cout.n * hsz * sizeof(cplx<T>) + (psi ? 3.0 * hsz * 16 : 0.0));
  hipLaunchKernelGGL(kspace_noise_kernel<T>, dim3(nblocks(hsz, 256)), dim3(256),
                     0, h.stream, (const double2 *)psi, seed, counter, out, cout, dg ? 1 : 0,
                     kgeom(h), (const double4 *)h.ktab, h.counter_dev);
  PSE_LAUNCH_CHECK();
}

void real_noise(Handle &h, uint64_t seed, uint64_t counter, double *out, int ncomp) {
  hipLaunchKernelGGL(real_noise_kernel, dim3(nblocks(h.n, 256)), dim3(256), 0,
                     h.stream, seed, counter, h.n, ncomp, (const int *)h.order, out, h.counter_dev);
  PSE_LAUNCH_CHECK();
}

template <typename T> void zero_grids(Handle &h, T *g, int ncomp) {
  const size_t n = (size_t)ncomp * h.ngrid;
  ProfScope ps(h, PK_ZERO, (double)n * sizeof(T));
  // (a launch has fewer than 2^32 threads; eleven grids of 768^3 points have more)
  const unsigned nb = (unsigned)std::min<size_t>((n + 255) / 256, size_t(1) << 23);
  hipLaunchKernelGGL(zero_kernel<T>, dim3(nb), dim3(256), 0, h.stream, g, n);
  PSE_LAUNCH_CHECK();
}

template <typename T> void from_double(Handle &h, const double *src, size_t n, T *dst) {
  hipLaunchKernelGGL(from_double_kernel<T>, dim3(nblocks(n, 256)), dim3(256), 0, h.stream,
                     src, n, dst);
  PSE_LAUNCH_CHECK();
}

template <typename T>
void to_double(Handle &h, const T *src, size_t n, double *dst, const int *stopped) {
  hipLaunchKernelGGL(to_double_kernel<T>, dim3(nblocks(n, 256)), dim3(256), 0, h.stream,
                     src, n, dst, stopped, h.call);
  PSE_LAUNCH_CHECK();
}

#define INST(T)                                                                 \
  template void spread<T>(Handle &, const double *, const double *, Layout,      \
                          const CompSet &, T *);                                 \
  template void interp_generic<T>(Handle &, const double *, const T *,           \
                                  const CompSet &, double *, Layout, bool, double); \
  template void kspace_deformed<T>(Handle &, const cplx<T> *, const CompSet &,   \
                                   cplx<T> *, const CompSet &);                  \
  template void kspace_noise<T>(Handle &, const double *, uint64_t, uint64_t,    \
                                cplx<T> *, const CompSet &, bool);               \
  template bool kspace_noise_z<T>(Handle &, const double *, uint64_t, uint64_t,  \
                                  cplx<T> *, const CompSet &, const cplx<T> *);  \
  template void kspace_fused<T>(Handle &, const cplx<T> *, const CompSet &,      \
                                cplx<T> *, const CompSet &, const cplx<T> *,     \
                                bool);                                           \
  template void spread_deriv<T>(Handle &, const double *, Layout, bool, bool, T *); \
  template void zero_grids<T>(Handle &, T *, int);                               \
  template void from_double<T>(Handle &, const double *, size_t, T *);           \
  template void to_double<T>(Handle &, const T *, size_t, double *, const int *);
INST(double)
INST(float)
#undef INST

}  // namespace pse
