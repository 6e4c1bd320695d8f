// Real-space part of the Ewald sum (Sec. II.C.1, Eqs. MUFr-MDCr, pairsums).
//
// Pair functions.  Writing T_pq for the inverse transform of
// f_p f_q (I - kk) / (eta k^2) (f_0 = j0(ka), f_1 = (sin ka - ka cos ka)/(ka)^3,
// the shape factors of Eqs. MUF-MDC), with k_n <-> -i d_n:
//   M_UF = T00,  M_UC_imn = -3 d_n T01_im,  M_DF_ijm = 3 d_j T01_im,
//   M_DC_ijmn = -9 d_j d_n T11_im,   T_pq = (grad grad - I lap) phi_pq,
// phi_pq the inverse transform of f_p f_q / (eta k^4).  With
// Phi_n = ((1/r) d/dr)^n phi every block follows from seven radial
// coefficients (the count of the paper's F1 F2 / G1 G2 / K1 K2 K3):
//   a = -(r^2 Phi2 + 2 Phi1), b = r^2 Phi2                 (pq = 00)
//   c1 = r^3 Phi3, c2 = r Phi2                             (pq = 01)
//   d2 = Phi2, d3 = r^2 Phi3, d4 = r^4 Phi4                (pq = 11)
// The real-space part (factor 1 - H) is "free space" minus "H part":
//  * free space: f_0 and f_1 transform to a shell density
//    delta(r - a)/(4 pi a^2) and a ball density 1/(4 pi a^3), and 1/k^4 to
//    -r/(8 pi), so phi_pq = -(1/8 pi eta) (shell/ball autocorrelation * r).
//    Carrying out the radial integrals gives, with A = -1/(8 pi eta),
//      phi00 = A (4a/3 + r^2/3a - r^3/24a^2),              r < 2a
//            = A (r + 2a^2/3r),                             r >= 2a
//      phi01 = A (2a/5 + r^2/9a - r^4/120a^3 + r^5/720a^4), r < 2a
//            = A (r/3 + 8a^2/45r),                          r >= 2a
//      phi11 = A (4a/35 + 2r^2/45a - r^4/180a^3 + r^5/720a^4
//                 - r^7/40320a^6),                          r < 2a
//            = A (r/9 + 2a^2/45r),                          r >= 2a
//    whose Phi_n are written out in free_coefficients();
//  * H part: Phi_n^H(r) = 1/(2 pi^2 eta) int_0^inf H(k) f_p f_q (-1)^n
//    k^(2n-2) j_n(kr)/(kr)^n dk, by the trapezoidal rule, which converges
//    geometrically for this even, Gaussian-damped integrand.
// Both are tabulated once per handle on the GPU (FP64) on a uniform r grid
// with a node at r = 2a, and interpolated with 4-point Lagrange stencils that
// never straddle r = 2a.
#include "listsum.h"
#include "pairrec.h"

namespace pse {

// ------------------------------------------------------------- tables --

// j_n(x)/x^n, n = 0..4 (out[n]): power series below x = 4, upward recurrence
// above.  The series' ratios are compile-time constants (a division per term
// was most of the table kernel's arithmetic); 20 terms leave less than 1e-19
// of the first at x = 4.
constexpr int JN_TERMS = 20;

template <int NMAX>
__device__ __forceinline__ void jn_over_xn(double x, double *out) {
  if (x < 4.0) {
    const double t = -0.5 * x * x;
    double df = 1.0;
#pragma unroll
    for (int n = 0; n <= NMAX; ++n) {
      df *= 2 * n + 1;
      // Horner form of sum_k t^k / prod_{i<=k} i (2 n + 2 i + 1)
      double acc = 1.0;
#pragma unroll
      for (int k = JN_TERMS; k >= 1; --k) acc = 1.0 + acc * (t * (1.0 / (k * (2 * n + 2 * k + 1))));
      out[n] = acc / df;
    }
    return;
  }
  double s, c;
  sincos(x, &s, &c);
  const double ix = 1.0 / x;
  double jm = s * ix;                       // j0
  double j = (s * ix - c) * ix;             // j1
  double p = ix;                            // 1 / x^n
  out[0] = jm;
#pragma unroll
  for (int n = 1; n <= NMAX; ++n) {
    out[n] = j * p;
    const double jp = (2 * n + 1) * ix * j - jm;
    jm = j;
    j = jp;
    p *= ix;
  }
}

__device__ void free_coefficients(double r, double a, double eta, double *co) {
  const double A = -1.0 / (8.0 * M_PI * eta);
  double v[NCOEF];
  if (r < 2.0 * a) {
    const double a2 = a * a, a3 = a2 * a, a4 = a3 * a, a6 = a3 * a3;
    const double r2 = r * r, r3 = r2 * r;
    // phi00: Phi1 = 2/3a - r/8a^2, Phi2 = -1/(8 a^2 r)
    v[0] = -4.0 / (3.0 * a) + 3.0 * r / (8.0 * a2);
    v[1] = -r / (8.0 * a2);
    // phi01: Phi2 = -1/15a^3 + r/48a^4, Phi3 = 1/(48 a^4 r)
    v[2] = r2 / (48.0 * a4);
    v[3] = -r / (15.0 * a3) + r2 / (48.0 * a4);
    // phi11: Phi2 = -2/45a^3 + r/48a^4 - r^3/1152a^6,
    //        Phi3 = 1/(48 a^4 r) - r/384a^6, Phi4 = -1/(48 a^4 r^3) - 1/(384 a^6 r)
    v[4] = -2.0 / (45.0 * a3) + r / (48.0 * a4) - r3 / (1152.0 * a6);
    v[5] = r / (48.0 * a4) - r3 / (384.0 * a6);
    v[6] = -r / (48.0 * a4) - r3 / (384.0 * a6);
  } else {
    const double a2 = a * a, r2 = r * r, r3 = r2 * r, r4 = r2 * r2, r5 = r4 * r;
    // phi00: Phi1 = 1/r - 2a^2/3r^3, Phi2 = -1/r^3 + 2a^2/r^5
    v[0] = -(1.0 / r + 2.0 * a2 / (3.0 * r3));
    v[1] = -1.0 / r + 2.0 * a2 / r3;
    // phi01: Phi2 = -1/3r^3 + 8a^2/15r^5, Phi3 = 1/r^5 - 8a^2/3r^7
    v[2] = 1.0 / r2 - 8.0 * a2 / (3.0 * r4);
    v[3] = -1.0 / (3.0 * r2) + 8.0 * a2 / (15.0 * r4);
    // phi11: Phi2 = -1/9r^3 + 2a^2/15r^5, Phi3 = 1/3r^5 - 2a^2/3r^7,
    //        Phi4 = -5/3r^7 + 14a^2/3r^9
    v[4] = -1.0 / (9.0 * r3) + 2.0 * a2 / (15.0 * r5);
    v[5] = 1.0 / (3.0 * r3) - 2.0 * a2 / (3.0 * r5);
    v[6] = -5.0 / (3.0 * r3) + 14.0 * a2 / (3.0 * r5);
  }
  for (int i = 0; i < NCOEF; ++i) co[i] = A * v[i];
}

// One wavefront forms TAB_ROWS nodes: its lanes share the quadrature's wave
// numbers, so a node's sum of nk + 1 (50 to 120) terms runs in parallel and the
// factors of a wave number are formed once for the wavefront's nodes; the
// lanes' partial sums are added by shuffles.  (One thread per node left 97
// wavefronts on the chip for a table of 6200 nodes, bound by their serial
// chains: 483 us, now 20.)
constexpr int TAB_ROWS = 4;

__global__ void __launch_bounds__(256)
table_kernel(double *__restrict__ tab, float *__restrict__ tab32, int ntab, double dr, double a,
             double eta, double xi, double dk, int nk) {
  const int lane = threadIdx.x & 63;
  const int i0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * TAB_ROWS;
  if (i0 >= ntab) return;
  // H part: Phi1_00, Phi2_00, Phi2_01, Phi3_01, Phi2_11, Phi3_11, Phi4_11
  double S[TAB_ROWS][7];
#pragma unroll
  for (int r = 0; r < TAB_ROWS; ++r)
#pragma unroll
    for (int j = 0; j < 7; ++j) S[r][j] = 0.0;
  const double inv4xi2 = 1.0 / (4.0 * xi * xi);
  for (int m = lane; m <= nk; m += 64) {
    const double k = m * dk;
    const double w = (m == 0) ? 0.5 * dk : dk;
    const double u = k * k * inv4xi2;
    double f[2];
    jn_over_xn<1>(k * a, f);
    const double k2 = k * k, wh = w * (1.0 + u) * exp(-u);
    const double w00 = wh * f[0] * f[0], w01 = wh * f[0] * f[1] * k2, w11 = wh * f[1] * f[1] * k2;
#pragma unroll
    for (int r = 0; r < TAB_ROWS; ++r) {
      double J[5];
      jn_over_xn<4>(k * ((i0 + r) * dr), J);
      S[r][0] -= w00 * J[1];
      S[r][1] += w00 * k2 * J[2];
      S[r][2] += w01 * J[2];
      S[r][3] -= w01 * k2 * J[3];
      S[r][4] += w11 * J[2];
      S[r][5] -= w11 * k2 * J[3];
      S[r][6] += w11 * k2 * k2 * J[4];
    }
  }
  const double c = 1.0 / (2.0 * M_PI * M_PI * eta);
#pragma unroll
  for (int r = 0; r < TAB_ROWS; ++r)
#pragma unroll
    for (int j = 0; j < 7; ++j) {
      double v = S[r][j];
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
      S[r][j] = v * c;
    }
  // lane r finishes node r
#pragma unroll
  for (int r = 0; r < TAB_ROWS; ++r) {
    const int i = i0 + r;
    if (lane != r || i >= ntab) continue;
    const double x = i * dr, r2 = x * x;
    double fc[NCOEF];
    free_coefficients(x, a, eta, fc);
    const double hc[NCOEF] = {-(r2 * S[r][1] + 2.0 * S[r][0]), r2 * S[r][1], r2 * x * S[r][3],
                              x * S[r][2], S[r][4], r2 * S[r][5], r2 * r2 * S[r][6]};
    for (int j = 0; j < NCOEF; ++j) {
      const double v = fc[j] - hc[j];
      tab[(size_t)i * NCOEF + j] = v;
      tab32[(size_t)i * NCOEF + j] = (float)v;
    }
  }
}

void build_tables(Handle &h) {
  const double a = h.p.radius, xi = h.d.xi;
  h.n2a = 2048;
  h.dr = 2.0 * a / h.n2a;
  h.ntab = (int)std::ceil(h.d.rcut / h.dr) + 8;
  handle_alloc(h, (void **)&h.g64.table, (size_t)h.ntab * NCOEF * sizeof(double));
  handle_alloc(h, (void **)&h.g32.table, (size_t)h.ntab * NCOEF * sizeof(float));
  const double rmax = h.ntab * h.dr;
  const double dk = M_PI / (2.0 * a + rmax + 7.0 / xi);
  const double kmax = 2.0 * xi * std::sqrt(50.0);
  const int nk = (int)std::ceil(kmax / dk);
  hipLaunchKernelGGL(table_kernel, dim3(nblocks(h.ntab, 4 * TAB_ROWS)), dim3(256),
                     0, h.stream, h.g64.table, h.g32.table, h.ntab, h.dr, a,
                     h.p.viscosity, xi, dk, nk);
  PSE_LAUNCH_CHECK();
}

// ------------------------------------------------------------ pair sum --

// Acting with the pair block M(r) on (F, C) of the partner; adds to U and D.
// UF, UC: forces, couplets present; OU, OD: velocity, gradient wanted (the
// coefficients a, b serve F -> U; c1, c2 serve F -> D and C -> U; d2, d3, d4
// serve C -> D; only those of the selected couplings are read).
template <typename T, bool UF, bool UC, bool OU, bool OD>
__device__ __forceinline__ void pair_action(const T *co, const T *e, const T *F,
                                                const T (*C)[3], T *U, T (*D)[3]) {
  const T a = co[0], b = co[1], c1 = co[2], c2 = co[3];
  const T d2 = co[4], d3 = co[5], d4 = co[6];
  const T c14 = c1 + (T)4 * c2;
  if constexpr (UF) {
    const T eF = e[0] * F[0] + e[1] * F[1] + e[2] * F[2];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      if constexpr (OU) U[i] += a * F[i] + b * e[i] * eF;
      if constexpr (OD)
#pragma unroll
        for (int j = 0; j < 3; ++j)
          D[i][j] += (T)3 * (c1 * e[i] * e[j] * eF + c2 * ((i == j ? eF : (T)0) + F[j] * e[i])
                             - c14 * F[i] * e[j]);
    }
  }
  if constexpr (UC) {
    T Ce[3], CTe[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      Ce[i] = C[i][0] * e[0] + C[i][1] * e[1] + C[i][2] * e[2];
      CTe[i] = C[0][i] * e[0] + C[1][i] * e[1] + C[2][i] * e[2];
    }
    const T eCe = e[0] * Ce[0] + e[1] * Ce[1] + e[2] * Ce[2];
    const T k7 = (T)7 * d3 + d4, k5 = (T)5 * d2 + d3;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      if constexpr (OU) U[i] += (T)(-3) * (c1 * e[i] * eCe + c2 * CTe[i] - c14 * Ce[i]);
      if constexpr (OD)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          const T s = d4 * e[i] * e[j] * eCe
                      + d3 * ((i == j ? eCe : (T)0) + e[j] * Ce[i] + e[j] * CTe[i]
                              + e[i] * Ce[j] + e[i] * CTe[j])
                      + d2 * (C[i][j] + C[j][i]) - k7 * e[j] * Ce[i] - k5 * C[i][j];
          D[i][j] += (T)(-9) * s;
        }
    }
  }
}

// Where a pair sum reads the partners' moments: the vector's own rows (double,
// component c of particle j at v[j stride + c - off]), or (PACK) a packed copy
// in the sum's precision, 12 numbers a particle (F, L, s1..s5, 0) read as
// three 16-byte loads (FP32; FP64 six).  The copy costs a launch, which few
// particles (below PACK_MIN) do not repay (N = 2*10^4, FP64: 29 + 5 us with
// it, 24 without).  A copy by component instead, whose loads touch fewer cache
// lines, was slower (N = 10^6, FP32, 11 components: 536 against 409 us).
template <typename T> struct Moments {
  const double *v;
  Layout l;
  const T *packed;
};

template <typename T>
__global__ void __launch_bounds__(256)
pack_moments_kernel(const double *__restrict__ in, Layout lin, int mask, int64_t n,
                    T *__restrict__ out) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n * 12) return;
  const int64_t p = t / 12;
  const int c = (int)(t % 12);
  const int grp = c < 3 ? 1 : (c < 6 ? 2 : 4);
  out[t] = (c < NC && (mask & grp)) ? (T)in[p * lin.stride + c - lin.off] : (T)0;
}

// Force F and couplet C (force index first) of particle j; groups absent
// from the mask are zero and not read.
template <typename T, bool PACK>
__device__ __forceinline__ void load_moments(const Moments<T> &m, int j, int mask, T *F,
                                             T (*C)[3]) {
  T v[12];
  if constexpr (PACK) {
    const T *q = m.packed + (size_t)j * 12;
    if constexpr (sizeof(T) == 4) {
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const float4 a = reinterpret_cast<const float4 *>(q)[k];
        v[4 * k] = a.x; v[4 * k + 1] = a.y; v[4 * k + 2] = a.z; v[4 * k + 3] = a.w;
      }
    } else {
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        const double2 a = reinterpret_cast<const double2 *>(q)[k];
        v[2 * k] = a.x; v[2 * k + 1] = a.y;
      }
    }
  } else {
    const double *q = m.v + (size_t)j * m.l.stride - m.l.off;
#pragma unroll
    for (int k = 0; k < NC; ++k) v[k] = (T)0;
    if (mask == 7) {
#pragma unroll
      for (int k = 0; k < NC; ++k) v[k] = (T)q[k];
    } else {
      if (mask & 1)
#pragma unroll
        for (int k = 0; k < 3; ++k) v[k] = (T)q[k];
      if (mask & 2)
#pragma unroll
        for (int k = 3; k < 6; ++k) v[k] = (T)q[k];
      if (mask & 4)
#pragma unroll
        for (int k = 6; k < NC; ++k) v[k] = (T)q[k];
    }
  }
  const T r2 = (T)0.70710678118654752440, r6 = (T)0.40824829046386301637;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    F[i] = v[i];
#pragma unroll
    for (int k = 0; k < 3; ++k) C[i][k] = (T)0;
  }
  if (mask & 2) {
    // C^A_mn = -1/2 eps_mnk L_k
    const T Lx = v[3], Ly = v[4], Lz = v[5];
    C[0][1] -= (T)0.5 * Lz; C[1][0] += (T)0.5 * Lz;
    C[0][2] += (T)0.5 * Ly; C[2][0] -= (T)0.5 * Ly;
    C[1][2] -= (T)0.5 * Lx; C[2][1] += (T)0.5 * Lx;
  }
  if (mask & 4) {
    const T *q = v + 6;
    C[0][1] += r2 * q[0]; C[1][0] += r2 * q[0];
    C[0][2] += r2 * q[1]; C[2][0] += r2 * q[1];
    C[1][2] += r2 * q[2]; C[2][1] += r2 * q[2];
    C[0][0] += r2 * q[3] + r6 * q[4];
    C[1][1] += -r2 * q[3] + r6 * q[4];
    C[2][2] += (T)(-2) * r6 * q[4];
  }
}

// A group of GROUP lanes works on one particle.  One thread per particle
// would leave most of the chip idle for N ~ 1e4.
constexpr int GROUP = 16;

// A group is one row of the wavefront, summed by rotations within it (an
// add per step instead of a shuffle through LDS); every lane gets the sum.
static_assert(GROUP == 16, "rows of 16 lanes");
template <int R> __device__ __forceinline__ float row_rotate(float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + R, 0xf, 0xf, true));
}
template <int R> __device__ __forceinline__ double row_rotate(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x120 + R, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x120 + R, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

template <typename T>
__device__ __forceinline__ T group_sum(T v) {
  v += row_rotate<8>(v);
  v += row_rotate<4>(v);
  v += row_rotate<2>(v);
  v += row_rotate<1>(v);
  return v;
}

struct RealArgs {
  int64_t n;
  int in_mask;    // 1: F, 2: L, 4: S
  int out_mask;   // 1: U, 2: Omega, 4: E
  Layout lout;
  int limit;      // entries the pair list holds (none beyond was written)
  double L;       // box; deformed lattice: separations mapped by A
  int def;
  double A[9];
  double inv_dr;  // radial table: spacing, rows of the near part, rows
  int n2a, ntab;
};

// The data of one pair formed from the positions (lists without records in
// this precision).
template <typename T>
__device__ __forceinline__ void pair_data(const double *__restrict__ xw, double xi0, double xi1,
                                          double xi2, int j, const RealArgs &ra,
                                          const T *__restrict__ tab, T *co, T *e) {
  double d[3];
  separation(xw, xi0, xi1, xi2, j, ra.L, ra.def, ra.A, d);
  const double r = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
  const double inv = r > 0 ? 1.0 / r : 0.0;
  lookup<T>(tab, (T)r, (T)ra.inv_dr, ra.n2a, ra.ntab, co);
#pragma unroll
  for (int k = 0; k < 3; ++k) e[k] = (T)(d[k] * inv);
}

// M_r applied from the pair list: the self block (r = 0: only the isotropic
// coefficients, table row 0) plus one pair block per stored neighbour.
// UF, UC: forces / couplets among the inputs; OU, OD: velocity / gradient
// outputs (from ra's masks); a stored entry's fields are read only when one
// of the selected couplings uses them.  REC: the list holds records in this
// precision (else the pair data are formed from the positions).
template <typename T, bool REC, bool PACK, bool UF, bool UC, bool OU, bool OD>
__global__ void __launch_bounds__(256)
real_pair_kernel(const double *__restrict__ xw, Moments<T> in,
                 double *__restrict__ out, const int *__restrict__ perm,
                 const int *__restrict__ start, const int *__restrict__ nbr,
                 const T *__restrict__ rec, const T *__restrict__ tab, RealArgs ra) {
  const int64_t t =
      ((int64_t)xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x) / GROUP;
  const int lane = threadIdx.x % GROUP;
  if (t >= ra.n) return;
  const int i = perm[t];
  T U[3] = {0, 0, 0};
  T D[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
  T F[3], C[3][3];
  if (lane == 0) {
    T co[NCOEF];
    for (int j = 0; j < NCOEF; ++j) co[j] = tab[j];
    const T e0[3] = {0, 0, 0};
    load_moments<T, PACK>(in, i, ra.in_mask, F, C);
    pair_action<T, UF, UC, OU, OD>(co, e0, F, C, U, D);
  }
  constexpr bool NEED_AB = UF && OU, NEED_C12 = (UF && OD) || (UC && OU), NEED_D = UC && OD;
  const int s1 = list_row_end(start[t + 1], ra.limit);
  const auto record = [&](int s, T *co, T *e) {
    const Entry<const T> p(rec, (uint32_t)s);
    if constexpr (NEED_AB) {
      co[0] = p[F_A];
      co[1] = p[F_B];
    }
    if constexpr (NEED_C12) {
      co[2] = p[F_C1];
      co[3] = p[F_C2];
    }
    if constexpr (NEED_D) {
      co[4] = p[F_D2];
      co[5] = p[F_D3];
      co[6] = p[F_D4];
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) e[k] = p[F_E + k];
  };
  int s = start[t] + lane;
  if constexpr (REC) {
    // the next entry's index and record are in flight while the current
    // neighbour's moments arrive
    int jn = 0;
    T con[NCOEF] = {}, en[3] = {};
    if (s < s1) {
      jn = nbr[s];
      record(s, con, en);
    }
    for (; s < s1; s += GROUP) {
      const int j = jn;
      T co[NCOEF], e[3];
#pragma unroll
      for (int k = 0; k < NCOEF; ++k) co[k] = con[k];
#pragma unroll
      for (int k = 0; k < 3; ++k) e[k] = en[k];
      load_moments<T, PACK>(in, j, ra.in_mask, F, C);
      if (s + GROUP < s1) {
        jn = nbr[s + GROUP];
        record(s + GROUP, con, en);
      }
      pair_action<T, UF, UC, OU, OD>(co, e, F, C, U, D);
    }
  } else {
    const double xi0 = xw[3 * i], xi1 = xw[3 * i + 1], xi2 = xw[3 * i + 2];
    for (; s < s1; s += GROUP) {
      const int j = nbr[s];
      T co[NCOEF], e[3];
      pair_data<T>(xw, xi0, xi1, xi2, j, ra, tab, co, e);
      load_moments<T, PACK>(in, j, ra.in_mask, F, C);
      pair_action<T, UF, UC, OU, OD>(co, e, F, C, U, D);
    }
  }
  if constexpr (OU)
#pragma unroll
    for (int k = 0; k < 3; ++k) U[k] = group_sum(U[k]);
  if constexpr (OD)
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) D[a][b] = group_sum(D[a][b]);
  if (lane != 0) return;
  // component c of the output at out[row + c - off]
  const size_t row = (size_t)i * ra.lout.stride;
  auto O = [&](int c) -> double & { return out[row + c - ra.lout.off]; };
  const double r2 = 0.70710678118654752440, r6 = 0.40824829046386301637;
  if (ra.out_mask & 1) {
    for (int k = 0; k < 3; ++k) O(k) = (double)U[k];
  }
  if (ra.out_mask & 2) {
    // Omega = -1/2 eps : D
    const double om[3] = {-0.5 * ((double)D[1][2] - D[2][1]),
                          -0.5 * ((double)D[2][0] - D[0][2]),
                          -0.5 * ((double)D[0][1] - D[1][0])};
    for (int k = 0; k < 3; ++k) O(3 + k) = om[k];
  }
  if (ra.out_mask & 4) {
    const double e5[5] = {r2 * ((double)D[0][1] + D[1][0]), r2 * ((double)D[0][2] + D[2][0]),
                          r2 * ((double)D[1][2] + D[2][1]), r2 * ((double)D[0][0] - D[1][1]),
                          r6 * ((double)D[0][0] + D[1][1] - 2.0 * D[2][2])};
    for (int k = 0; k < 5; ++k) O(6 + k) = e5[k];
  }
}

// The stresslet-strain block of M_r alone (the constraint operator and its
// preconditioner): out = alpha in + beta M_r,ES in.  Stresslets and strains
// are symmetric and traceless, so with S the partner's stresslet, w = S e and
// x = e.w the pair action of pair_action<T, false, true, false, true>
// reduces, in the Y_q components, to
//   E_q = -9 [ f s_q + Y_q : (e m + m e) ],   m = (d4/2) x e + h w,
//   f = -3 d2 - d3,  h = -(3 d3 + d4) / 2:
// five numbers in and out instead of nine, read from the vectors' own rows.
// Bound by the records, 28 bytes a pair (FP32) read once, and the arithmetic
// per neighbour; the next entry's record is in flight while the current
// neighbour's stresslet arrives.  N = 10^6, 28 neighbours: 276 + 36 (a packed
// copy) -> 235 us; 2*10^5, 111 neighbours: 239 + 7 -> 190 us; 10^4 in FP64:
// 9.4 + 4.2 -> 6.4 us.
template <typename T>
__device__ __forceinline__ void es_action(T d2, T d3, T d4, const T *e, const T *s, T *acc) {
  const T r2 = (T)0.70710678118654752440, r6 = (T)0.40824829046386301637;
  const T xy = r2 * s[0], xz = r2 * s[1], yz = r2 * s[2], a = r2 * s[3], b = r6 * s[4];
  const T w[3] = {(b + a) * e[0] + xy * e[1] + xz * e[2], xy * e[0] + (b - a) * e[1] + yz * e[2],
                  xz * e[0] + yz * e[1] - (T)2 * b * e[2]};
  const T x = e[0] * w[0] + e[1] * w[1] + e[2] * w[2];
  const T f = (T)-3 * d2 - d3, h = (T)-1.5 * d3 - (T)0.5 * d4, g = (T)0.5 * d4 * x;
  T m[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) m[k] = g * e[k] + h * w[k];
  const T c2 = (T)2 * r2, c6 = (T)2 * r6;
  const T xx = e[0] * m[0], yy = e[1] * m[1], zz = e[2] * m[2];
  acc[0] += f * s[0] + c2 * (e[0] * m[1] + e[1] * m[0]);
  acc[1] += f * s[1] + c2 * (e[0] * m[2] + e[2] * m[0]);
  acc[2] += f * s[2] + c2 * (e[1] * m[2] + e[2] * m[1]);
  acc[3] += f * s[3] + c2 * (xx - yy);
  acc[4] += f * s[4] + c6 * (xx + yy - (T)2 * zz);
}

template <typename T, bool REC>
__global__ void __launch_bounds__(256)
es_pair_kernel(const double *__restrict__ xw, const double *__restrict__ in, Layout lin,
               double *__restrict__ out, const int *__restrict__ perm,
               const int *__restrict__ start, const int *__restrict__ nbr,
               const T *__restrict__ rec, const T *__restrict__ tab, RealArgs ra, double alpha,
               double beta) {
  const int64_t t =
      ((int64_t)xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x) / GROUP;
  const int lane = threadIdx.x % GROUP;
  if (t >= ra.n) return;
  const int i = perm[t];
  const int s1 = list_row_end(start[t + 1], ra.limit);
  T acc[5] = {}, m[5], e[3];
  const double *in6 = in + 6 - lin.off;
  const auto moments = [&](int j) {
    const double *q = in6 + (size_t)j * lin.stride;
#pragma unroll
    for (int k = 0; k < 5; ++k) m[k] = (T)q[k];
  };
  int s = start[t] + lane;
  if constexpr (REC) {
    int jn = 0;
    T rn[6] = {};
    const auto record = [&](int p) {
      const Entry<const T> q(rec, (uint32_t)p);
#pragma unroll
      for (int k = 0; k < 6; ++k) rn[k] = q[k];
    };
    if (s < s1) {
      jn = nbr[s];
      record(s);
    }
    for (; s < s1; s += GROUP) {
      moments(jn);
      const T d2 = rn[0], d3 = rn[1], d4 = rn[2];
      e[0] = rn[3];
      e[1] = rn[4];
      e[2] = rn[5];
      if (s + GROUP < s1) {
        jn = nbr[s + GROUP];
        record(s + GROUP);
      }
      es_action(d2, d3, d4, e, m, acc);
    }
  } else {
    const double xi0 = xw[3 * i], xi1 = xw[3 * i + 1], xi2 = xw[3 * i + 2];
    for (; s < s1; s += GROUP) {
      const int j = nbr[s];
      T co[NCOEF];
      pair_data<T>(xw, xi0, xi1, xi2, j, ra, tab, co, e);
      moments(j);
      es_action(co[4], co[5], co[6], e, m, acc);
    }
  }
#pragma unroll
  for (int k = 0; k < 5; ++k) acc[k] = group_sum(acc[k]);
  if (lane >= 5) return;
  // lane k finishes component k in FP64; the self block is f s at r = 0 and the
  // larger part of a dilute sum
  T a = acc[0];
#pragma unroll
  for (int k = 1; k < 5; ++k) a = lane == k ? acc[k] : a;
  const double v = in[(size_t)i * lin.stride + 6 - lin.off + lane];
  const double f = -3.0 * (double)tab[4] - (double)tab[5];
  out[(size_t)i * ra.lout.stride + 6 - ra.lout.off + lane] =
      alpha * v + beta * (-9.0 * ((double)a + f * v));
}

static int mask_of(const CompSet &cs) {
  int m = 0;
  for (int k = 0; k < cs.n; ++k) {
    const int c = cs.idx[k];
    m |= c < 3 ? 1 : (c < 6 ? 2 : 4);
  }
  return m;
}

static RealArgs real_args(const Handle &h, int in_mask, Layout lout, int out_mask) {
  RealArgs ra;
  ra.n = h.n;
  ra.lout = lout;
  ra.in_mask = in_mask;
  ra.out_mask = out_mask;
  ra.limit = list_limit((int64_t)h.pl_cap);
  ra.L = h.p.box;
  ra.def = h.def.on;
  for (int k = 0; k < 9; ++k) ra.A[k] = h.def.A[k];
  ra.inv_dr = 1.0 / h.dr;
  ra.n2a = h.n2a;
  ra.ntab = h.ntab;
  return ra;
}

template <typename T> static void real_data(const Handle &h, const T *&tab, const T *&rec) {
  if constexpr (sizeof(T) == 8) {
    tab = h.g64.table;
    rec = h.pl_rec64;
  } else {
    tab = h.g32.table;
    rec = h.pl_rec32;
  }
}

// f(true_type) where the list holds records of T; FP32 sums run on mixed
// handles only, whose records are FP32.
template <typename T, typename F> static void with_records(const T *rec, F f) {
  if constexpr (sizeof(T) == 8) {
    if (rec) f(std::true_type());
    else f(std::false_type());
  } else {
    if (!rec) throw Error{PSE_ERR_INVALID, "pair records missing"};
    f(std::true_type());
  }
}

// Pairs that the stage profiler counts a sum with: the last length the host
// learned, or the list's capacity while it has learned none (asynchronous
// calls never tell).
static double profiled_pairs(const Handle &h) {
  return (double)(h.pl_pairs ? h.pl_pairs : h.pl_cap);
}

template <typename T>
void real_es(Handle &h, const double *xw, const double *in, Layout lin, double *out, Layout lout,
             double alpha, double beta) {
  const T *tab, *rec;
  real_data<T>(h, tab, rec);
  ProfScope ps(h, PK_REAL, profiled_pairs(h) * (4.0 + (rec ? 6 * sizeof(T) : 0)) +
                               (double)h.n * (5 * 8 * 2 + 8));
  with_records<T>(rec, [&](auto R) {
    hipLaunchKernelGGL((es_pair_kernel<T, decltype(R)::value>),
                       dim3(nblocks((size_t)h.n * GROUP, 256)), dim3(256), 0, h.stream, xw, in,
                       lin, out, h.cells.perm, h.pl_start, h.pl_nbr, rec, tab,
                       real_args(h, 4, lout, 4), alpha, beta);
  });
  PSE_LAUNCH_CHECK();
}

template <typename T>
void real_apply(Handle &h, const double *xw, const double *in, Layout lin, const CompSet &cin,
                double *out, Layout lout, const CompSet &cout) {
  const RealArgs ra = real_args(h, mask_of(cin), lout, mask_of(cout));
  if (ra.in_mask == 4 && ra.out_mask == 4) {
    real_es<T>(h, xw, in, lin, out, lout, 0.0, 1.0);
    return;
  }
  const T *tab, *rec;
  real_data<T>(h, tab, rec);
  ProfScope ps(h, PK_REAL, profiled_pairs(h) * (4.0 + (rec ? PAIR_REC * sizeof(T) : 0)) +
                               (double)h.n * (NC * 8 * 2 + 8 + 24));
  const bool uf = ra.in_mask & 1, uc = (ra.in_mask & 6) != 0;
  const bool ou = ra.out_mask & 1, od = (ra.out_mask & 6) != 0;
  Moments<T> m{in, lin, nullptr};
  if (h.n >= PACK_MIN) {
    T *mp = reinterpret_cast<T *>(h.mpack);
    hipLaunchKernelGGL(pack_moments_kernel<T>, dim3(nblocks((size_t)h.n * 12, 256)), dim3(256),
                       0, h.stream, in, lin, ra.in_mask, h.n, mp);
    PSE_LAUNCH_CHECK();
    m.packed = mp;
  }
  const dim3 grid(nblocks((size_t)h.n * GROUP, 256)), block(256);
  const auto launch = [&](auto UF, auto UC, auto OU, auto OD) {
    with_records<T>(rec, [&](auto R) {
      const auto go = [&](auto P) {
        hipLaunchKernelGGL((real_pair_kernel<T, decltype(R)::value, decltype(P)::value,
                                             decltype(UF)::value, decltype(UC)::value,
                                             decltype(OU)::value, decltype(OD)::value>),
                           grid, block, 0, h.stream, xw, m, out, h.cells.perm, h.pl_start,
                           h.pl_nbr, rec, tab, ra);
      };
      if (m.packed) go(std::true_type());
      else go(std::false_type());
    });
  };
  using Y = std::true_type;
  using N = std::false_type;
  if (uf && uc) {
    if (ou && od) launch(Y(), Y(), Y(), Y());
    else if (ou) launch(Y(), Y(), Y(), N());
    else launch(Y(), Y(), N(), Y());
  } else if (uf) {
    if (ou && od) launch(Y(), N(), Y(), Y());
    else if (ou) launch(Y(), N(), Y(), N());
    else launch(Y(), N(), N(), Y());
  } else {
    if (ou && od) launch(N(), Y(), Y(), Y());
    else if (ou) launch(N(), Y(), Y(), N());
    else launch(N(), Y(), N(), Y());
  }
  PSE_LAUNCH_CHECK();
}

template void real_es<double>(Handle &, const double *, const double *, Layout, double *, Layout,
                              double, double);
template void real_es<float>(Handle &, const double *, const double *, Layout, double *, Layout,
                             double, double);
template void real_apply<double>(Handle &, const double *, const double *, Layout,
                                 const CompSet &, double *, Layout, const CompSet &);
template void real_apply<float>(Handle &, const double *, const double *, Layout,
                                const CompSet &, double *, Layout, const CompSet &);

}  // namespace pse
