// FP64 vector kernels and small dense solvers of the Krylov iterations:
// the Lanczos square root of M_r (Sec. III.B, Chow & Saad) and GMRES on the
// stresslet constraint M_ES S = b (Eq. rigidconstraint).  All scalars stay
// on the device; kernels also write the few numbers that decide when to stop
// to host memory, which the host reads after waiting for the stream.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "pse_internal.h"

namespace pse {

constexpr int RED_BLOCKS = 1024;   // partial-sum blocks of a reduction

__global__ void zero_kernel_d(double *v, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) v[i] = 0.0;
}

__global__ void fill_kernel_i(int *v, size_t n, int value) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) v[i] = value;
}

__global__ void axpby_kernel(double a, const double *x, double b, double *y, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = a * x[i] + b * y[i];
}

__device__ __forceinline__ double lane_d(double v, int l) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
  return __hiloint2double(hi, lo);
}

// Sum over a wavefront (every lane gets it; all lanes active): rotations
// within the rows of 16 lanes, then the four rows' sums (shuffles go through
// LDS, six of them one after the other).
template <int R> __device__ __forceinline__ double row_rotated(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x120 + R, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x120 + R, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_sum(double v) {
  v += row_rotated<8>(v);
  v += row_rotated<4>(v);
  v += row_rotated<2>(v);
  v += row_rotated<1>(v);
  return (lane_d(v, 0) + lane_d(v, 16)) + (lane_d(v, 32) + lane_d(v, 48));
}

// One Gram-Schmidt step of a Krylov method (two classical passes, CGS2) takes
// w = V_m against V_0..V_{m-1}:
//   h1_j = V_j . w;  w -= sum_j h1_j V_j;
//   h2_j = V_j . w (j < m), h2_m = w . w;
//   w = (w - sum_j h2_j V_j) / nn,  nn = sqrt(h2_m - |h2_0..m-1|^2)
// and gives the method its column (Column below).  Three kernels -- dots, sub
// and dots, finish -- whose sums go from one to the next as block partials.
// How a step is launched depends on the vectors' length n alone (plan_of):
//  * ONE: one workgroup does the whole step (krylov_one_kernel).  A launch
//    takes 5 to 7 us of the stream whatever it does, and vectors this short
//    are read in less (n = 1100: one launch of 7 us instead of six of 2 to 6;
//    at n = 7655 it takes 25 us against 14 for the three).
//  * FEW: the three kernels on at most 64 workgroups, so that each consumer
//    adds up the 64 partials of a sum itself, one per lane (n = 110000: 20 us
//    a step against 32 with the sums in launches of their own).
//  * MANY: up to 1024 workgroups for the bandwidth, the partials added up by
//    launches of their own (each consumer reading 1024 of them would cost
//    more than the launch).
struct Plan {
  enum Kind { ONE, FEW, MANY } kind;
  int nb;   // workgroups of a sum
};

constexpr size_t ONE_MAX = 2048;
constexpr size_t FEW_MAX = size_t(1) << 18;

static Plan plan_of(size_t n) {
  const int nb = std::max(1, (int)std::min<size_t>(RED_BLOCKS, (n + 255) / 256));
  if (n <= ONE_MAX) return {Plan::ONE, 1};
  if (n <= FEW_MAX) return {Plan::FEW, std::min(nb, 64)};
  return {Plan::MANY, nb};
}

// h[j] = the sum of the nb <= 64 partials of sum j < cnt, by the block's
// wavefronts.
__device__ __forceinline__ void sum_partials(const double *__restrict__ partial, int nb, int cnt,
                                             double *h) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int j = wv; j < cnt; j += nw) {
    const double v = wave_sum(lane < nb ? partial[(size_t)j * nb + lane] : 0.0);
    if (lane == 0) h[j] = v;
  }
}

// Sums of NW wavefronts' accumulators: acc[k] into out[k], k < cnt <= 8
// (s: NW x 8 doubles; all threads call it, with a barrier after).
template <int NW>
__device__ __forceinline__ void block_sums8(const double *acc, int cnt, double (*s)[8],
                                            double *out, int stride) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    if (k >= cnt) break;
    const double v = wave_sum(acc[k]);
    if (lane == 0) s[wv][k] = v;
  }
  __syncthreads();
  if ((int)threadIdx.x < cnt) {
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) v += s[w][threadIdx.x];
    out[(size_t)threadIdx.x * stride] = v;
  }
  __syncthreads();
}

// f(integral_constant<int, k>) for k = cnt in 1..8: loops over a fixed number
// of vectors, so that all loads of an element are issued together.
template <typename F> __device__ __forceinline__ void fixed_count(int cnt, F f) {
  switch (cnt) {
    case 1: f(std::integral_constant<int, 1>()); break;
    case 2: f(std::integral_constant<int, 2>()); break;
    case 3: f(std::integral_constant<int, 3>()); break;
    case 4: f(std::integral_constant<int, 4>()); break;
    case 5: f(std::integral_constant<int, 5>()); break;
    case 6: f(std::integral_constant<int, 6>()); break;
    case 7: f(std::integral_constant<int, 7>()); break;
    default: f(std::integral_constant<int, 8>()); break;
  }
}

// w = (w - sum_{j<m} coef_j V_j) f over this thread's elements.
__device__ __forceinline__ void sub_of(double *w, const double *V, size_t ldv, int m,
                                       const double *coef, double f, size_t n, size_t i0,
                                       size_t step) {
  for (int j0 = 0; j0 < m; j0 += 8) {
    const int cnt = min(8, m - j0);
    const double *v0 = V + (size_t)j0 * ldv;
    const double fk = j0 + 8 >= m ? f : 1.0;
    fixed_count(cnt, [&](auto c) {
      constexpr int K = decltype(c)::value;
      double cf[K];
#pragma unroll
      for (int k = 0; k < K; ++k) cf[k] = coef[j0 + k];
#pragma unroll 4
      for (size_t i = i0; i < n; i += step) {
        double v[K], a = w[i];
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = v0[(size_t)k * ldv + i];
#pragma unroll
        for (int k = 0; k < K; ++k) a -= cf[k] * v[k];
        w[i] = a * fk;
      }
    });
  }
}

// Dots of w with V_0..V_{m-1} over this thread's elements i0, i0 + step, ...:
// eight vectors at a time, so w is read once per eight.
template <int NW>
__device__ __forceinline__ void dots_of(const double *V, size_t ldv, int m, const double *w,
                                        size_t n, size_t i0, size_t step, double (*s)[8],
                                        double *out, int stride) {
  for (int j0 = 0; j0 < m; j0 += 8) {
    const int cnt = min(8, m - j0);
    double acc[8] = {};
    const double *v0 = V + (size_t)j0 * ldv;
    fixed_count(cnt, [&](auto c) {
      constexpr int K = decltype(c)::value;
#pragma unroll 4
      for (size_t i = i0; i < n; i += step) {
        const double wi = w[i];
#pragma unroll
        for (int k = 0; k < K; ++k) acc[k] += v0[(size_t)k * ldv + i] * wi;
      }
    });
    block_sums8<NW>(acc, cnt, s, out + (size_t)j0 * stride, stride);
  }
}

// w -= sum_{j<m} coef_j V_j (coef in LDS), then the dots of the new w with
// V_0..V_{m-1} and itself.  Up to seven vectors every element is visited
// once; more take a pass for the update and one per eight dots.
template <int NW>
__device__ __forceinline__ void sub_dots_of(double *w, const double *V, size_t ldv, int m,
                                            const double *coef, size_t n, size_t i0, size_t step,
                                            double (*s)[8], double *out, int stride) {
  if (m <= 7) {
    double acc[8] = {};
    fixed_count(m, [&](auto c) {
      constexpr int K = decltype(c)::value < 8 ? decltype(c)::value : 7;
      double cf[K];
#pragma unroll
      for (int k = 0; k < K; ++k) cf[k] = coef[k];
#pragma unroll 4
      for (size_t i = i0; i < n; i += step) {
        double v[K], wn = w[i];
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = V[(size_t)k * ldv + i];
#pragma unroll
        for (int k = 0; k < K; ++k) wn -= cf[k] * v[k];
        w[i] = wn;
#pragma unroll
        for (int k = 0; k < K; ++k) acc[k] += v[k] * wn;
        acc[K] += wn * wn;
      }
    });
    block_sums8<NW>(acc, m + 1, s, out, stride);
    return;
  }
  sub_of(w, V, ldv, m, coef, 1.0, n, i0, step);
  // V_m is w itself
  dots_of<NW>(V, ldv, m + 1, w, n, i0, step, s, out, stride);
}

// Where a Krylov column goes.  GMRES (H not NULL): H[i][j] = h1_i + h2_i, the
// previous Givens rotations and a new one, g updated, |g_{j+1}| the residual.
// Lanczos: alpha_j = h1_j + h2_j and beta_j = nn.  vn_hist and res_hist keep
// nn and the residual per column on the device; host (may be NULL) is memory
// the host reads after a synchronisation: nn at [1 + j], the residual at
// [1 + hcap + j].
// Device-checked GMRES (sel not NULL): sel[0] is set at the first column whose
// residual met tol |b| or whose new vector vanished (nn <= 1e-15 |b|), sel[1]
// = its column count k (0 for b = 0); at the last column (last != 0) without
// one, k = j + 1 and sel[2] = 1 (not converged).
struct Column {
  double *H;
  int ldh;
  double *cs, *sn, *g, *res_hist;
  double *alpha, *beta;
  double *vn_hist;
  double *host;
  int hcap;
  int *sel;
  const double *bn;
  double tol;
  int last;
};

// One wavefront forms column j from h1[0..j] and h2[0..j+1] (LDS) and nn; cl,
// cs_l, sn_l: LDS scratch of j + 1 doubles each.
__device__ __forceinline__ void finish_column(const Column &c, int j, const double *h1,
                                              const double *h2, double nn, double *cl,
                                              double *cs_l, double *sn_l) {
  const int lane = threadIdx.x & 63;
  if (!c.H) {
    if (lane != 0) return;
    c.alpha[j] = h1[j] + h2[j];
    c.beta[j] = nn;
    c.vn_hist[j] = nn;
    if (c.host) c.host[1 + j] = nn;
    return;
  }
  for (int i = lane; i <= j; i += 64) cl[i] = h1[i] + h2[i];
  for (int i = lane; i < j; i += 64) {
    cs_l[i] = c.cs[i];
    sn_l[i] = c.sn[i];
  }
  wave_lds_sync();
  if (lane != 0) return;
  double *col = c.H + (size_t)j * c.ldh;
  double a = cl[0];
  for (int i = 0; i < j; ++i) {   // (cl[j] is the column's last entry)
    const double b = cl[i + 1];
    col[i] = cs_l[i] * a + sn_l[i] * b;
    a = -sn_l[i] * a + cs_l[i] * b;
  }
  const double r = hypot(a, nn);
  const double cn = r > 0 ? a / r : 1.0, sj = r > 0 ? nn / r : 0.0;
  c.cs[j] = cn;
  c.sn[j] = sj;
  col[j] = r;
  col[j + 1] = 0.0;
  const double gj = c.g[j], gn = -sj * gj, res = fabs(gn);
  c.g[j + 1] = gn;
  c.g[j] = cn * gj;
  c.vn_hist[j] = nn;
  c.res_hist[j] = res;
  if (c.host) {
    c.host[1 + j] = nn;
    c.host[1 + c.hcap + j] = res;
  }
  if (!c.sel || c.sel[0]) return;
  const double bn = *c.bn;
  const bool done = res < c.tol * bn || nn <= 1e-15 * bn;
  if (done || c.last) {
    c.sel[0] = 1;
    c.sel[1] = bn > 0.0 ? j + 1 : 0;
    c.sel[2] = done ? 0 : 1;
  }
}

// nn of the twice-orthogonalised w from h2[0..m] (LDS), by every wavefront.
__device__ __forceinline__ double new_norm(const double *h2, int m) {
  double p2 = 0.0;
  for (int i = threadIdx.x & 63; i < m; i += 64) p2 += h2[i] * h2[i];
  return sqrt(fmax(h2[m] - wave_sum(p2), 0.0));
}

// FEW and MANY: the first pass's dots, partial[j nb + blk].
__global__ void __launch_bounds__(256)
dots_kernel(const double *V, size_t ldv, int m, const double *w, size_t n,
            double *__restrict__ partial) {
  __shared__ double s[4][8];
  dots_of<4>(V, ldv, m, w, n, (size_t)blockIdx.x * 256 + threadIdx.x, (size_t)gridDim.x * 256, s,
             partial + blockIdx.x, gridDim.x);
}

__global__ void __launch_bounds__(256)
reduce_partial(const double *__restrict__ partial, int nb, double *__restrict__ out) {
  __shared__ double s[4][8];
  double acc = 0.0;
  for (int b = threadIdx.x; b < nb; b += 256) acc += partial[(size_t)blockIdx.x * nb + b];
  block_sums8<4>(&acc, 1, s, out + blockIdx.x, 1);
}

// The first pass's subtraction and the second pass's dots; nb1 > 0: h1 from
// nb1 partials each (kept in h1 by the first workgroup), else h1 given.
__global__ void __launch_bounds__(256)
sub_dots_kernel(double *w, const double *V, size_t ldv, int m, size_t n,
                const double *__restrict__ partial1, int nb1, double *__restrict__ h1,
                double *__restrict__ partial2) {
  __shared__ double s[4][8];
  extern __shared__ double h[];   // m
  if (nb1 > 0) sum_partials(partial1, nb1, m, h);
  else
    for (int j = threadIdx.x; j < m; j += 256) h[j] = h1[j];
  __syncthreads();
  if (nb1 > 0 && blockIdx.x == 0)
    for (int j = threadIdx.x; j < m; j += 256) h1[j] = h[j];
  sub_dots_of<4>(w, V, ldv, m, h, n, (size_t)blockIdx.x * 256 + threadIdx.x,
                 (size_t)gridDim.x * 256, s, partial2 + blockIdx.x, gridDim.x);
}

// The second subtraction, the scaling and (first workgroup) the column;
// nb2 > 0: h2 from nb2 partials each, else h2 given.
__global__ void __launch_bounds__(256)
finish_kernel(double *w, const double *V, size_t ldv, int m, size_t n,
              const double *__restrict__ h1, const double *__restrict__ partial2, int nb2,
              const double *__restrict__ h2, Column c) {
  extern __shared__ double h[];   // m + 1, then four times m + 1
  double *h1l = h + m + 1, *cl = h1l + m + 1, *cs = cl + m + 1, *sn = cs + m + 1;
  if (nb2 > 0) sum_partials(partial2, nb2, m + 1, h);
  else
    for (int j = threadIdx.x; j <= m; j += 256) h[j] = h2[j];
  __syncthreads();
  const double nn = new_norm(h, m), f = nn > 0.0 ? 1.0 / nn : 0.0;
  sub_of(w, V, ldv, m, h, f, n, (size_t)blockIdx.x * 256 + threadIdx.x,
         (size_t)gridDim.x * 256);
  if (blockIdx.x != 0 || threadIdx.x >= 64) return;
  for (int j = threadIdx.x; j < m; j += 64) h1l[j] = h1[j];
  wave_lds_sync();
  finish_column(c, m - 1, h1l, h, nn, cl, cs, sn);
}

// ONE: the whole step by one workgroup, w and up to eight vectors in
// registers (a thread holds ONE_E elements of each), more vectors read in
// chunks of eight for each phase.  A launch is one short chain -- two rounds of
// sums between barriers -- so the sums go over few wavefronts and the code is
// small (a version with loops unrolled per vector count spent its time
// fetching instructions).
constexpr int ONE_T = 512, ONE_E = (int)(ONE_MAX / ONE_T);
static_assert(ONE_E * ONE_T == ONE_MAX, "elements per thread");

__global__ void __launch_bounds__(ONE_T)
krylov_one_kernel(double *w, const double *V, size_t ldv, int m, int n, Column c) {
  __shared__ double s[ONE_T / 64][9];
  extern __shared__ double h1[];   // five times m + 1
  double *h2 = h1 + m + 1, *cl = h2 + m + 1, *cs = cl + m + 1, *sn = cs + m + 1;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  double x[ONE_E], v[8][ONE_E];
  const auto load = [&](int j0) {
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
      for (int e = 0; e < ONE_E; ++e) {
        const int i = tid + e * ONE_T;
        v[k][e] = (j0 + k < m && i < n) ? V[(size_t)(j0 + k) * ldv + i] : 0.0;
      }
  };
  // sums of the chunk's dots (and x . x with the last chunk) into out[j0 ..]
  const auto sums = [&](int j0, double *out, bool norm) {
    double a[9];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      a[k] = 0.0;
#pragma unroll
      for (int e = 0; e < ONE_E; ++e) a[k] += v[k][e] * x[e];
      a[k] = wave_sum(a[k]);
    }
    a[8] = 0.0;
    if (norm) {
#pragma unroll
      for (int e = 0; e < ONE_E; ++e) a[8] += x[e] * x[e];
      a[8] = wave_sum(a[8]);
    }
    if (lane == 0)
#pragma unroll
      for (int k = 0; k < 9; ++k) s[wv][k] = a[k];
    __syncthreads();
    if (tid < 9) {
      double t = 0.0;
#pragma unroll
      for (int k = 0; k < ONE_T / 64; ++k) t += s[k][tid];
      if (tid < 8 && j0 + tid < m) out[j0 + tid] = t;
      if (tid == 8 && norm) out[m] = t;
    }
    __syncthreads();
  };
  const auto subtract = [&](int j0, const double *h) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const double hk = j0 + k < m ? h[j0 + k] : 0.0;
#pragma unroll
      for (int e = 0; e < ONE_E; ++e) x[e] -= hk * v[k][e];
    }
  };
#pragma unroll
  for (int e = 0; e < ONE_E; ++e) {
    const int i = tid + e * ONE_T;
    x[e] = i < n ? w[i] : 0.0;
  }
  const bool hold = m <= 8;
  if (hold) load(0);
  for (int j0 = 0; j0 < m; j0 += 8) {
    if (!hold) load(j0);
    sums(j0, h1, false);
  }
  for (int j0 = 0; j0 < m; j0 += 8) {
    if (!hold) load(j0);
    subtract(j0, h1);
  }
  for (int j0 = 0; j0 < m; j0 += 8) {
    if (!hold) load(j0);
    sums(j0, h2, j0 + 8 >= m);
  }
  for (int j0 = 0; j0 < m; j0 += 8) {
    if (!hold) load(j0);
    subtract(j0, h2);
  }
  const double nn = new_norm(h2, m), f = nn > 0.0 ? 1.0 / nn : 0.0;
#pragma unroll
  for (int e = 0; e < ONE_E; ++e) {
    const int i = tid + e * ONE_T;
    if (i < n) w[i] = x[e] * f;
  }
  if (tid < 64) finish_column(c, m - 1, h1, h2, nn, cl, cs, sn);
}

// The start of a solve: bn = |b|, v = b / bn (0 for b = 0; v may be b), g =
// (bn, 0, ...) and, when given, clear0 and clear1 (len numbers) and sel (3)
// cleared.  nb > 0: |b|^2 from nb <= 64 partials; 0: given in norm2; -1:
// formed here (one workgroup).
__global__ void __launch_bounds__(1024)
krylov_start_kernel(const double *b, double *v, size_t n,
                    const double *__restrict__ partial, int nb, const double *norm2,
                    double *__restrict__ bn_out, double *__restrict__ g, int glen,
                    double *__restrict__ clear0, double *__restrict__ clear1, int len,
                    int *__restrict__ sel, double *__restrict__ host) {
  __shared__ double s[16][8];
  __shared__ double b2;
  if (nb > 0) sum_partials(partial, nb, 1, &b2);
  else if (nb == 0) {
    if (threadIdx.x == 0) b2 = norm2[0];
  } else {
    double acc = 0.0;
    for (size_t i = threadIdx.x; i < n; i += blockDim.x) acc += b[i] * b[i];
    block_sums8<16>(&acc, 1, s, &b2, 1);
  }
  __syncthreads();
  const double bn = sqrt(fmax(b2, 0.0)), f = bn != 0.0 ? 1.0 / bn : 0.0;
  const size_t step = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step)
    v[i] = b[i] * f;
  if (blockIdx.x != 0) return;
  if (threadIdx.x == 0) {
    *bn_out = bn;
    if (host) host[0] = bn;
  }
  for (int i = threadIdx.x; i < glen; i += blockDim.x) g[i] = i == 0 ? bn : 0.0;
  for (int i = threadIdx.x; i < len; i += blockDim.x) clear0[i] = clear1[i] = 0.0;
  if (sel && threadIdx.x < 3) sel[threadIdx.x] = 0;
}

// y = (acc ? y : 0) + alpha sum_j coef_j V_j (m from m_dev when given)
__global__ void gemv_small_kernel(const double *__restrict__ V, size_t ldv, int m,
                                  const double *__restrict__ coef, double *__restrict__ y,
                                  size_t n, double alpha, int accumulate,
                                  const int *__restrict__ m_dev) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  if (m_dev) m = *m_dev;
  double acc = 0.0;
  for (int j = 0; j < m; ++j) acc += coef[j] * V[(size_t)j * ldv + i];
  y[i] = (accumulate ? y[i] : 0.0) + alpha * acc;
}

// y = (acc ? y : 0) + V c with R c = g, R the k x k upper triangle of the
// columns H (k from k_dev when given): every workgroup solves the triangle
// itself (one launch instead of two, and the columns wait in LDS instead of a
// chain of global loads: 4.6 to 17 us for the solve alone).
constexpr int TRI_MAX = 48;   // columns staged in LDS

__global__ void __launch_bounds__(256)
solve_gemv_kernel(const double *__restrict__ V, size_t ldv, int k, const double *__restrict__ H,
                  int ldh, const double *__restrict__ g, double *__restrict__ y, size_t n,
                  int accumulate, const int *__restrict__ k_dev) {
  __shared__ double R[TRI_MAX * (TRI_MAX + 1) / 2];
  extern __shared__ double c[];   // the largest k
  if (k_dev) k = *k_dev;
  const bool staged = k <= TRI_MAX;
  if (staged)
    for (int e = threadIdx.x; e < k * k; e += 256) {
      const int j = e / k, i = e % k;
      if (i <= j) R[j * (j + 1) / 2 + i] = H[(size_t)j * ldh + i];
    }
  for (int i = threadIdx.x; i < k; i += 256) c[i] = g[i];
  __syncthreads();
  if (threadIdx.x < 64) {
    // columns from the last: c_j = g_j / R_jj, then g_i -= R_ij c_j for i < j
    for (int j = k - 1; j >= 0; --j) {
      const double *col = staged ? R + j * (j + 1) / 2 : H + (size_t)j * ldh;
      const double cj = c[j] / col[j];
      wave_lds_sync();
      for (int i = threadIdx.x; i < j; i += 64) c[i] -= col[i] * cj;
      if (threadIdx.x == 0) c[j] = cj;
      wave_lds_sync();
    }
  }
  __syncthreads();
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  double acc = accumulate ? y[i] : 0.0;
  for (int j = 0; j < k; ++j) acc += c[j] * V[(size_t)j * ldv + i];
  y[i] = acc;
}

// ------------------------------------------------------------ host glue --

void vzero(Handle &h, double *v, size_t n) {
  hipLaunchKernelGGL(zero_kernel_d, dim3(nblocks(n, 256)), dim3(256), 0, h.stream, v, n);
  PSE_LAUNCH_CHECK();
}
void fill_int(Handle &h, int *v, size_t n, int value) {
  hipLaunchKernelGGL(fill_kernel_i, dim3(nblocks(n, 256)), dim3(256), 0, h.stream, v, n,
                     value);
  PSE_LAUNCH_CHECK();
}

void vaxpby(Handle &h, double a, const double *x, double b, double *y, size_t n) {
  hipLaunchKernelGGL(axpby_kernel, dim3(nblocks(n, 256)), dim3(256), 0, h.stream, a, x,
                     b, y, n);
  PSE_LAUNCH_CHECK();
}

void gemv_small(Handle &h, const double *V, size_t ldv, int m, const double *coef_dev,
                double *y, size_t n, double alpha, bool accumulate, const int *m_dev) {
  ProfScope ps(h, PK_KRYLOV, (double)(m + 1 + (accumulate ? 1 : 0)) * n * 8);
  hipLaunchKernelGGL(gemv_small_kernel, dim3(nblocks(n, 256)), dim3(256), 0, h.stream, V,
                     ldv, m, coef_dev, y, n, alpha, accumulate ? 1 : 0, m_dev);
  PSE_LAUNCH_CHECK();
}

// ----------------------------------------------------- small dense work --

// Eigen-decomposition of the symmetric tridiagonal matrix (diag d, off-diag
// e) by the implicit QL iteration with Wilkinson-type shifts; z accumulates
// the eigenvectors (column k belongs to eigenvalue d[k]).  m <= ldz.  Run by
// one wavefront: every lane computes the scalar recurrences alike (each lane
// reads back only its own writes of d and e, which are the same in all
// lanes), and each plane rotation is applied to the rows of z in parallel,
// row k by lane k mod 64 (a lane touches only its own rows).
__device__ void tridiag_ql(double *d, double *e, double *z, int m, int ldz) {
  const int lane = threadIdx.x, nt = blockDim.x;
  for (int i = lane; i < m; i += nt)
    for (int j = 0; j < m; ++j) z[i * ldz + j] = (i == j) ? 1.0 : 0.0;
  if (m == 1) return;
  e[m - 1] = 0.0;
  for (int l = 0; l < m; ++l) {
    for (int iter = 0; iter < 60; ++iter) {
      int mm = l;
      for (; mm < m - 1; ++mm) {
        const double dd = fabs(d[mm]) + fabs(d[mm + 1]);
        if (fabs(e[mm]) <= 1e-16 * dd) break;
      }
      if (mm == l) break;
      double g = (d[l + 1] - d[l]) / (2.0 * e[l]);
      double r = hypot(g, 1.0);
      g = d[mm] - d[l] + e[l] / (g + (g >= 0 ? r : -r));
      double s = 1.0, c = 1.0, p = 0.0;
      int i = mm - 1;
      for (; i >= l; --i) {
        double f = s * e[i], b = c * e[i];
        r = hypot(f, g);
        e[i + 1] = r;
        if (r == 0.0) {
          d[i + 1] -= p;
          e[mm] = 0.0;
          break;
        }
        s = f / r;
        c = g / r;
        g = d[i + 1] - p;
        r = (d[i] - g) * s + 2.0 * c * b;
        p = s * r;
        d[i + 1] = g + p;
        g = c * r - b;
        for (int k = lane; k < m; k += nt) {
          const double zf = z[k * ldz + i + 1];
          z[k * ldz + i + 1] = s * z[k * ldz + i] + c * zf;
          z[k * ldz + i] = c * z[k * ldz + i] - s * zf;
        }
      }
      if (r == 0.0 && i >= l) continue;
      d[l] -= p;
      e[l] = g;
      e[mm] = 0.0;
    }
  }
}

// The same for m <= 64 with d and e in registers, entry i in lane i, and a
// rotation from one reciprocal square root (d and e are scaled to at most
// one): the recurrences are one dependent chain, and memory, hypot and two
// divisions per rotation were most of its length (m = 6: 21 -> 8 us).  The
// column of z that a rotation leaves to the next stays in a register.  z[i][j]
// (LDS, rows of m): row i belongs to lane i.
__device__ void tridiag_ql_lanes(double &d, double &e, double *z, int m) {
  const int lane = threadIdx.x;
  double *zr = z + lane * m;
  if (lane < m)
    for (int j = 0; j < m; ++j) zr[j] = lane == j ? 1.0 : 0.0;
  for (int l = 0; l < m; ++l) {
    for (int iter = 0; iter < 60; ++iter) {
      const double dn = __shfl_down(d, 1, 64);
      const unsigned long long small =
          __ballot(lane >= m - 1 || fabs(e) <= 1e-16 * (fabs(d) + fabs(dn)));
      const int mm = l + __builtin_ctzll(small >> l);
      if (mm == l) break;
      const double el = lane_d(e, l), dl = lane_d(d, l);
      double g = (lane_d(d, l + 1) - dl) / (2.0 * el);
      double r = sqrt(g * g + 1.0);
      g = lane_d(d, mm) - dl + el / (g + (g >= 0 ? r : -r));
      double s = 1.0, c = 1.0, p = 0.0;
      double zf = lane < m ? zr[mm] : 0.0;   // column i + 1
      int i = mm - 1;
      for (; i >= l; --i) {
        const double ei = lane_d(e, i), di1 = lane_d(d, i + 1), di = lane_d(d, i);
        const double zi = lane < m ? zr[i] : 0.0;
        const double f = s * ei, b = c * ei, h2 = f * f + g * g;
        if (h2 == 0.0) {
          if (lane == i + 1) {
            e = 0.0;
            d -= p;
          }
          if (lane == mm) e = 0.0;
          if (lane < m) zr[i + 1] = zf;
          break;
        }
        const double ir = rsqrt(h2);
        s = f * ir;
        c = g * ir;
        g = di1 - p;
        r = (di - g) * s + 2.0 * c * b;
        p = s * r;
        if (lane == i + 1) {
          e = h2 * ir;
          d = g + p;
        }
        g = c * r - b;
        if (lane < m) zr[i + 1] = s * zi + c * zf;
        zf = c * zi - s * zf;
      }
      if (i >= l) continue;
      if (lane < m) zr[l] = zf;
      if (lane == l) {
        d -= p;
        e = g;
      }
      if (lane == mm) e = 0.0;
    }
  }
}

// coef = bnorm * f(T) e_1 with f = sqrt, T = tridiag(alpha, beta) of size m;
// also the relative change against the previous coefficient vector
// (zero-padded), kept in chg_hist[m-1] and, when given, host_change[m-1].  One
// wavefront (64 threads): inputs
// loaded in parallel, the eigenproblem by tridiag_ql, coefficient i by lane
// i mod 64, the change summed in index order by lane 0.
// Device-checked solves (sel != NULL): sel[0] is set once the first
// iteration that met the tolerance (or broke down: vn_hist[m-1] <= 1e-14 |b|)
// is found, sel[1] holds its size m and coef_sel its coefficients; at the
// last iteration (last != 0) without one, m is taken and sel[2] = 1 (not
// converged).
__global__ void __launch_bounds__(64)
lanczos_sqrt_kernel(const double *alpha, const double *beta, int m, const double *bnorm_dev,
                    double *work, int ldz, double *coef, double *coef_prev, double *chg_hist,
                    double *host_change, int *sel, double *coef_sel, const double *vn_hist,
                    double tol, int last) {
  // LDS: the new and previous coefficients (2m), then d, e and z when they
  // fit (ldz == m; the host sizes the dynamic shared memory), else those
  // live in the global work area
  extern __shared__ double lds_work[];
  if (blockIdx.x != 0) return;
  const int lane = threadIdx.x, nt = blockDim.x;
  const double bnorm = *bnorm_dev;
  double *cbuf = lds_work, *pbuf = lds_work + m;
  double *base = ldz == m ? lds_work + 2 * m : work;
  double *d = base, *e = base + ldz, *z = base + 2 * ldz;
  if (m <= 64) {
    double di = lane < m ? alpha[lane] : 0.0, ei = lane + 1 < m ? beta[lane] : 0.0;
    if (lane < m) pbuf[lane] = lane < m - 1 ? coef_prev[lane] : 0.0;
    double big = fmax(fabs(di), fabs(ei));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) big = fmax(big, __shfl_xor(big, off, 64));
    const double f = big > 0.0 ? 1.0 / big : 1.0;
    di *= f;
    ei *= f;
    tridiag_ql_lanes(di, ei, z, m);
    if (lane < m) d[lane] = big > 0.0 ? di * big : di;
  } else {
    for (int i = lane; i < m; i += nt) {
      d[i] = alpha[i];
      e[i] = i + 1 < m ? beta[i] : 0.0;
      pbuf[i] = i < m - 1 ? coef_prev[i] : 0.0;
    }
    __syncthreads();
    tridiag_ql(d, e, z, m, ldz);
  }
  __syncthreads();
  // w_k = sqrt(lambda_k) z_0k (over e, which is done with)
  double *w = e;
  for (int k = lane; k < m; k += nt) w[k] = (d[k] > 0.0 ? sqrt(d[k]) : 0.0) * z[k];
  __syncthreads();
  for (int i = lane; i < m; i += nt) {
    double acc = 0.0;
    for (int k = 0; k < m; ++k) acc += z[i * ldz + k] * w[k];
    cbuf[i] = bnorm * acc;
    coef[i] = cbuf[i];
  }
  __syncthreads();
  if (lane != 0) return;
  double num = 0.0, den = 0.0;
  for (int i = 0; i < m; ++i) {
    const double c = cbuf[i], prev = pbuf[i];
    num += (c - prev) * (c - prev);
    den += c * c;
    coef_prev[i] = c;
  }
  const double change = den > 0.0 ? sqrt(num / den) : 0.0;
  chg_hist[m - 1] = change;
  if (host_change) host_change[m - 1] = change;
  if (!sel || sel[0]) return;
  const bool brk = vn_hist[m - 1] <= 1e-14 * bnorm;
  const bool conv = m > 1 && change < tol;
  if (brk || conv || last) {
    sel[0] = 1;
    sel[1] = m;
    sel[2] = (brk || conv) ? 0 : 1;
    for (int i = 0; i < m; ++i) coef_sel[i] = cbuf[i];
  }
}

// ---------------------------------------------------- host algorithms --

// Krylov scalars that kernels write to host memory (h.kry: |b| first, then
// two histories of hcap numbers), read after a synchronisation.  Any
// non-finite one among the first n of each history is reported as an error (a
// non-finite input vector or operator result).
static void host_scalars(Handle &h, int hcap, int n) {
  PSE_HIP(hipStreamSynchronize(h.stream));
  verify_lists(h);
  const volatile double *k = h.kry;
  bool ok = std::isfinite(k[0]);
  for (int i = 0; i < n; ++i) ok = ok && std::isfinite(k[1 + i]) && std::isfinite(k[1 + hcap + i]);
  if (!ok) throw Error{PSE_ERR_NONFINITE, "non-finite Krylov scalar"};
}

// dev_norm2 = v . v
void norm2_dev(Handle &h, const double *v, size_t n, double *dev_norm2) {
  const Plan p = plan_of(n);
  ProfScope ps(h, PK_KRYLOV, (double)n * 8);
  hipLaunchKernelGGL(dots_kernel, dim3(p.nb), dim3(256), 0, h.stream, v, n, 1, v, n,
                     p.nb == 1 ? dev_norm2 : h.dots);
  PSE_LAUNCH_CHECK();
  if (p.nb == 1) return;
  hipLaunchKernelGGL(reduce_partial, dim3(1), dim3(256), 0, h.stream, (const double *)h.dots,
                     p.nb, dev_norm2);
  PSE_LAUNCH_CHECK();
}

// Scalars of a solve's start (see krylov_start_kernel).
struct Start {
  double *bn, *g;
  int glen;
  double *clear0, *clear1;
  int len;
  int *sel;
  double *host;
};

static void krylov_start(Handle &h, const double *b, double *v, size_t n, double *norm2,
                         const Start &st) {
  const Plan p = plan_of(n);
  ProfScope ps(h, PK_KRYLOV, (double)(p.kind == Plan::ONE ? 2 : 3) * n * 8);
  int nb = -1;
  unsigned grid = 1, block = 1024;
  if (p.kind != Plan::ONE) {
    hipLaunchKernelGGL(dots_kernel, dim3(p.nb), dim3(256), 0, h.stream, b, n, 1, b, n, h.dots);
    PSE_LAUNCH_CHECK();
    nb = p.nb;
    if (p.kind == Plan::MANY) {
      hipLaunchKernelGGL(reduce_partial, dim3(1), dim3(256), 0, h.stream, (const double *)h.dots,
                         p.nb, norm2);
      PSE_LAUNCH_CHECK();
      nb = 0;
    }
    block = 256;
    grid = std::min(nblocks(n, 256), 2048u);
  }
  hipLaunchKernelGGL(krylov_start_kernel, dim3(grid), dim3(block), 0, h.stream, b, v, n,
                     (const double *)h.dots, nb, (const double *)norm2, st.bn, st.g, st.glen,
                     st.clear0, st.clear1, st.len, st.sel, st.host);
  PSE_LAUNCH_CHECK();
}

// One Gram-Schmidt step of w = V_m (leading dimension n) and its column.
static void krylov_step(Handle &h, const double *V, size_t n, int m, double *w, double *h1,
                        double *h2, const Column &c) {
  const Plan p = plan_of(n);
  const size_t hl = (size_t)(m + 1) * sizeof(double);
  ProfScope ps(h, PK_KRYLOV, (double)(3 * m + 5) * n * 8);
  if (p.kind == Plan::ONE) {
    hipLaunchKernelGGL(krylov_one_kernel, dim3(1), dim3(ONE_T), 5 * hl, h.stream, w, V, n, m,
                       (int)n, c);
    PSE_LAUNCH_CHECK();
    return;
  }
  const bool few = p.kind == Plan::FEW;
  double *p1 = h.dots, *p2 = few ? h.dots + (size_t)p.nb * m : h.dots;
  if ((size_t)(p2 - h.dots) + (size_t)p.nb * (m + 1) > h.dots_len)
    throw Error{PSE_ERR_INVALID, "reduction scratch too small"};
  hipLaunchKernelGGL(dots_kernel, dim3(p.nb), dim3(256), 0, h.stream, V, n, m, (const double *)w,
                     n, p1);
  PSE_LAUNCH_CHECK();
  if (!few) {
    hipLaunchKernelGGL(reduce_partial, dim3(m), dim3(256), 0, h.stream, (const double *)p1, p.nb,
                       h1);
    PSE_LAUNCH_CHECK();
  }
  hipLaunchKernelGGL(sub_dots_kernel, dim3(p.nb), dim3(256), hl, h.stream, w, V, n, m, n,
                     (const double *)p1, few ? p.nb : 0, h1, p2);
  PSE_LAUNCH_CHECK();
  if (!few) {
    hipLaunchKernelGGL(reduce_partial, dim3(m + 1), dim3(256), 0, h.stream, (const double *)p2,
                       p.nb, h2);
    PSE_LAUNCH_CHECK();
  }
  hipLaunchKernelGGL(finish_kernel, dim3(std::min(nblocks(n, 256), few ? 256u : 8192u)), dim3(256),
                     5 * hl, h.stream, w, V, n, m, n, (const double *)h1, (const double *)p2,
                     few ? p.nb : 0, (const double *)h2, c);
  PSE_LAUNCH_CHECK();
}

// Lanczos scratch in h.small for at most M iterations.
struct LanczosScratch {
  double *alpha, *beta, *h1, *h2, *norm2, *bn, *coef, *coef_prev, *vn_hist, *chg_hist, *coef_sel,
      *work;
  LanczosScratch(Handle &h, int M) {
    double *s = h.small;
    const auto take = [&](size_t n) { double *p = s; s += n; return p; };
    alpha = take(M + 1);
    beta = take(M + 1);
    h1 = take(M + 1);
    h2 = take(M + 2);
    norm2 = take(1);
    bn = take(1);
    coef = take(M + 1);
    coef_prev = take(M + 1);
    vn_hist = take(M + 1);
    chg_hist = take(M + 1);
    coef_sel = take(M + 1);
    work = s;
    if ((size_t)(work - h.small) + (size_t)(3 + M) * (M + 1) + 8 > h.small_len)
      throw Error{PSE_ERR_INVALID, "Lanczos scratch too small"};
  }
};

static void lanczos_coef(Handle &h, const LanczosScratch &z, int M, int mm, double *host_change,
                         int *sel, double tol, bool last) {
  // LDS holds the two coefficient vectors, and d, e and the mm^2 eigenvectors
  // when they fit in 48 KiB
  const size_t coefs = (size_t)2 * mm * sizeof(double);
  const size_t lds = coefs + (size_t)(2 * mm + mm * mm) * sizeof(double);
  const bool fits = lds <= 49152;
  hipLaunchKernelGGL(lanczos_sqrt_kernel, dim3(1), dim3(64), fits ? lds : coefs, h.stream,
                     (const double *)z.alpha, (const double *)z.beta, mm, (const double *)z.bn,
                     z.work, fits ? mm : M + 1, z.coef, z.coef_prev, z.chg_hist, host_change, sel,
                     z.coef_sel, (const double *)z.vn_hist, tol, last ? 1 : 0);
  PSE_LAUNCH_CHECK();
}

// The first iteration whose scalars the host looks at: the iteration counts
// of successive solves on a handle barely change, and a look stalls the
// stream, so they start shortly before the previous solve's count (two
// iterations; one where an iteration is short against the stall), at every
// iteration on a first solve.
static int first_look(const int *prev, size_t n) {
  if (!prev || *prev <= 3) return 0;
  return *prev - (plan_of(n).kind == Plan::MANY ? 2 : 1);
}

// Lanczos approximation of y = A^(1/2) b (Chow & Saad): full
// reorthogonalization, stop when the relative change of the iterate falls
// below tol.  The iterate is y_m = |b| V_m f(T_m) e_1; with V_m orthonormal
// its change is the change of the small coefficient vector.  The result does
// not depend on when the host looks (first_look): later iterations than the one
// that met the rule are discarded, and when the first look finds it met, the
// changes of the iterations before are formed too (their scalars are kept) and
// the first that met it is taken.
KrylovResult lanczos_sqrt(Handle &h, const Op &A, const double *b, size_t n, double *y,
                          int maxit, double tol, int *prev_iters) {
  const int M = maxit, hcap = M + 1;
  const LanczosScratch z(h, M);
  double *V = h.lz_V;
  KrylovResult res{0, 0.0, false, 0.0};
  // changes before the first look stay unset: zero, so that they read finite
  // (the stream has finished the last solve that wrote them)
  for (int i = 0; i < 2 * hcap; ++i) h.kry[1 + i] = 0.0;
  double *host_change = h.kry + 1 + hcap;
  krylov_start(h, b, V, n, z.norm2,
               Start{z.bn, nullptr, 0, z.coef_prev, z.chg_hist, M + 1, nullptr, h.kry});
  const int check_from = first_look(prev_iters, n);
  const volatile double *vh = h.kry + 1, *ch = host_change;
  int m = 0;
  bool looked = false;
  for (int j = 0; j < M; ++j) {
    double *w = V + (size_t)(j + 1) * n;
    A(V + (size_t)j * n, w);
    Column c{};
    c.alpha = z.alpha;
    c.beta = z.beta;
    c.vn_hist = z.vn_hist;
    c.host = h.kry;
    c.hcap = hcap;
    krylov_step(h, V, n, j + 1, w, z.h1, z.h2, c);
    // f(T) e_1 is needed from one iteration before the first look on (the
    // change there is taken against it)
    if (j + 2 >= check_from || j + 1 >= M)
      lanczos_coef(h, z, M, j + 1, host_change, nullptr, 0.0, false);
    m = j + 1;
    res.iters = m;
    if (m < check_from && m < M) continue;
    host_scalars(h, hcap, j + 1);
    res.bnorm = h.kry[0];
    if (!(res.bnorm > 0)) {
      vzero(h, y, n);
      return KrylovResult{0, 0.0, true, 0.0};
    }
    // a breakdown: the Krylov space is exhausted after i + 1 vectors
    const auto broke = [&](int i) { return vh[i] <= 1e-14 * res.bnorm; };
    int stop = 0;
    while (stop <= j && !broke(stop)) ++stop;
    if (stop > j && j > 0 && ch[j] < tol) stop = j;
    if (stop <= j) {
      int formed = j;   // f(T) e_1's iteration
      if (!looked && j > 0) {
        for (formed = 0; formed < stop; ++formed)
          lanczos_coef(h, z, M, formed + 1, host_change, nullptr, 0.0, false);
        lanczos_coef(h, z, M, stop + 1, host_change, nullptr, 0.0, false);
        host_scalars(h, hcap, j + 1);
        for (int i = 1; i < stop; ++i)
          if (ch[i] < tol) stop = i;
      }
      if (formed != stop) lanczos_coef(h, z, M, stop + 1, nullptr, nullptr, 0.0, false);
      m = res.iters = stop + 1;
      res.resid = ch[stop];
      res.converged = true;
      break;
    }
    looked = true;
    res.resid = ch[j];
  }
  if (prev_iters) *prev_iters = res.iters;
  gemv_small(h, V, n, m, z.coef, y, n, 1.0, false, nullptr);
  return res;
}

// GMRES scratch in h.small for at most R columns.
struct GmresScratch {
  double *H, *cs, *sn, *g, *h1, *h2, *norm2, *beta, *bn, *vn_hist, *res_hist;
  GmresScratch(Handle &h, int R) {
    double *s = h.small;
    const auto take = [&](size_t n) { double *p = s; s += n; return p; };
    H = take((size_t)(R + 1) * R);
    cs = take(R + 1);
    sn = take(R + 1);
    g = take(R + 1);
    h1 = take(R + 1);
    h2 = take(R + 2);
    norm2 = take(1);
    beta = take(1);
    bn = take(1);
    vn_hist = take(R + 1);
    res_hist = take(R + 1);
    if ((size_t)(s - h.small) + 8 > h.small_len)
      throw Error{PSE_ERR_INVALID, "GMRES scratch too small"};
  }
  Column column(int R) const {
    Column c{};
    c.H = H;
    c.ldh = R + 1;
    c.cs = cs;
    c.sn = sn;
    c.g = g;
    c.vn_hist = vn_hist;
    c.res_hist = res_hist;
    c.bn = bn;
    return c;
  }
};

// x = (acc ? x : 0) + V y, R y = g over k columns (k_dev: at most k).
static void gmres_update(Handle &h, const GmresScratch &z, int ldh, const double *V, size_t n,
                         int k, double *x, bool acc, const int *k_dev) {
  ProfScope ps(h, PK_KRYLOV, (double)(k + 1 + (acc ? 1 : 0)) * n * 8);
  hipLaunchKernelGGL(solve_gemv_kernel, dim3(nblocks(n, 256)), dim3(256),
                     (size_t)(k + 1) * sizeof(double), h.stream, V, n, k, (const double *)z.H, ldh,
                     (const double *)z.g, x, n, acc ? 1 : 0, k_dev);
  PSE_LAUNCH_CHECK();
}

// Restarted GMRES(restart) for A x = b from x = 0, stopping at relative
// residual tol or after maxit iterations.  Modified to classical
// Gram-Schmidt with a second pass (CGS2) so that each Arnoldi step costs two
// fused reductions; Givens rotations on the device.  The host looks at the
// residuals as in lanczos_sqrt; restarted cycles every step.
KrylovResult gmres(Handle &h, const Op &A, const double *b, size_t n, double *x,
                   int restart, int maxit, double tol, int *prev_iters) {
  const int R = restart, hcap = R + 1;
  const GmresScratch z(h, R);
  double *V = h.gm_V;
  KrylovResult res{0, 0.0, false, 0.0};
  const volatile double *vh = h.kry + 1, *rh = h.kry + 1 + hcap;
  double rel = 1.0, bnorm = 0.0;
  int total = 0;
  bool first = true;
  int check_from = first_look(prev_iters, n);
  while (total < maxit) {
    // r = b - A x; on the first cycle x = 0, so r = b and beta = |b|
    double *r = V;
    if (first) {
      krylov_start(h, b, r, n, z.norm2,
                   Start{z.bn, z.g, R + 1, nullptr, nullptr, 0, nullptr, h.kry});
    } else {
      A(x, r);
      vaxpby(h, 1.0, b, -1.0, r, n);
      check_from = 0;
      krylov_start(h, r, r, n, z.norm2,
                   Start{z.beta, z.g, R + 1, nullptr, nullptr, 0, nullptr, h.kry});
      host_scalars(h, hcap, 0);
      rel = h.kry[0] / bnorm;
      if (rel < tol) {
        res.converged = true;
        break;
      }
    }
    int k = 0;
    for (int j = 0; j < R && total < maxit; ++j) {
      double *w = V + (size_t)(j + 1) * n;
      A(V + (size_t)j * n, w);
      Column c = z.column(R);
      c.host = h.kry;
      c.hcap = hcap;
      krylov_step(h, V, n, j + 1, w, z.h1, z.h2, c);
      ++total;
      k = j + 1;
      if (k < check_from && j + 1 < R && total < maxit) continue;
      host_scalars(h, hcap, j + 1);
      if (first) {
        bnorm = h.kry[0];
        if (!(bnorm > 0)) {
          vzero(h, x, n);
          if (prev_iters) *prev_iters = 0;
          return KrylovResult{0, 0.0, true, 0.0};
        }
      }
      // first column at which the residual met tol or the space was exhausted;
      // later columns (and Givens entries) are not used by the update
      int stop = -1;
      for (int i = 0; i <= j; ++i)
        if (rh[i] / bnorm < tol || vh[i] <= 1e-15 * bnorm) {
          stop = i;
          break;
        }
      if (stop >= 0) {
        k = stop + 1;
        rel = rh[stop] / bnorm;
        break;
      }
      rel = rh[j] / bnorm;
    }
    gmres_update(h, z, R + 1, V, n, k, x, !first, nullptr);
    first = false;
    if (rel < tol) {
      res.converged = true;
      break;
    }
  }
  res.iters = total;
  res.resid = rel;
  res.bnorm = bnorm;
  if (prev_iters) *prev_iters = total;
  return res;
}

// ------------------------------------------- device-checked solves --
//
// Used by asynchronous handles: no host reads.  A solve runs exactly K
// iterations; kernels record on the device the first iteration that met the
// tolerance (or exhausted the Krylov space), and the result is formed from
// that iteration's quantities, so that it equals the result of stopping
// there (the later iterations are computed and discarded).  With no such
// iteration within K, the K-th iterate is taken and the solve is reported
// as not converged.

// stats after a Lanczos solve: iterations, last change, convergence
__global__ void lanczos_stats_kernel(const int *sel, const double *chg_hist, pse_stats *st) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const int m = sel[1];
  st->lanczos_iters = m;
  st->lanczos_change = m > 0 ? chg_hist[m - 1] : 0.0;
  if (sel[2]) st->converged = 0;
}

// stats after a GMRES solve (accumulated over refinement passes)
__global__ void gmres_stats_kernel(const int *sel, const double *res_hist, const double *bn,
                                   pse_stats *st) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const int k = sel[1];
  st->gmres_iters += k;
  st->gmres_residual = (k > 0 && bn[0] > 0.0) ? res_hist[k - 1] / bn[0] : 0.0;
  if (sel[2]) st->converged = 0;
}

void lanczos_sqrt_dev(Handle &h, const Op &A, const double *b, size_t n, double *y, int K,
                      double tol) {
  const LanczosScratch z(h, K);
  int *sel = h.dctl + CTL_LZ;
  double *V = h.lz_V;
  krylov_start(h, b, V, n, z.norm2,
               Start{z.bn, nullptr, 0, z.coef_prev, z.chg_hist, K + 1, sel, nullptr});
  for (int j = 0; j < K; ++j) {
    double *w = V + (size_t)(j + 1) * n;
    A(V + (size_t)j * n, w);
    Column c{};
    c.alpha = z.alpha;
    c.beta = z.beta;
    c.vn_hist = z.vn_hist;
    krylov_step(h, V, n, j + 1, w, z.h1, z.h2, c);
    lanczos_coef(h, z, K, j + 1, nullptr, sel, tol, j + 1 == K);
  }
  gemv_small(h, V, n, K, z.coef_sel, y, n, 1.0, false, sel + 1);
  hipLaunchKernelGGL(lanczos_stats_kernel, dim3(1), dim3(1), 0, h.stream, (const int *)sel,
                     (const double *)z.chg_hist, h.dstats);
  PSE_LAUNCH_CHECK();
}

void gmres_dev(Handle &h, const Op &A, const double *b, size_t n, double *x, int K,
               double tol) {
  const int R = K;
  const GmresScratch z(h, R);
  if ((size_t)R > (size_t)h.d.gmres_restart)
    throw Error{PSE_ERR_INVALID, "GMRES basis smaller than its iteration count"};
  int *sel = h.dctl + CTL_GM;
  double *V = h.gm_V;
  krylov_start(h, b, V, n, z.norm2,
               Start{z.bn, z.g, R + 1, nullptr, nullptr, 0, sel, nullptr});
  for (int j = 0; j < R; ++j) {
    double *w = V + (size_t)(j + 1) * n;
    A(V + (size_t)j * n, w);
    Column c = z.column(R);
    c.sel = sel;
    c.tol = tol;
    c.last = j + 1 == R ? 1 : 0;
    krylov_step(h, V, n, j + 1, w, z.h1, z.h2, c);
  }
  gmres_update(h, z, R + 1, V, n, R, x, false, sel + 1);
  hipLaunchKernelGGL(gmres_stats_kernel, dim3(1), dim3(1), 0, h.stream, (const int *)sel,
                     (const double *)z.res_hist, (const double *)z.bn, h.dstats);
  PSE_LAUNCH_CHECK();
}

}  // namespace pse
