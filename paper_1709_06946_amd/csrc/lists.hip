// Positions, bins and lists of one call: the particles' order, the real-space
// cells and the pair list, the spreading tiles' candidate lists and the
// particles' Gaussian weights (Sec. II.C; the pair sums and grid kernels read
// them over all the operator applications at fixed positions).
//
// Everything here is short: at N = 100 to 10^4 each launch does a few
// microseconds of work and takes five to seven of the stream, so the number of
// launches is what counts.  Up to ONE_WG_N particles the wrapping, both
// binnings and the particles' order are one workgroup's work (bins_one_kernel),
// and the passes of the pair list and of the tile lists share their launches.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "listsum.h"
#include "pairrec.h"
#include "stencil.h"

namespace pse {

// ---------------------------------------------------------- positions --

// Position i wrapped into [0, L)^3 (a deformed lattice's in lattice
// coordinates A^-1 x first).  Non-finite coordinates are reported and replaced
// by 0, so that every later kernel stays in bounds until the host reports the
// error.
__device__ __forceinline__ void wrapped_position(const double *__restrict__ x, int64_t i, double L,
                                                 const Deform &df, const Reports &rp, double *y) {
  const double p[3] = {x[3 * i], x[3 * i + 1], x[3 * i + 2]};
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    double v = df.on ? df.Ai[3 * d] * p[0] + df.Ai[3 * d + 1] * p[1] + df.Ai[3 * d + 2] * p[2]
                     : p[d];
    if (!isfinite(v)) {
      *rp.bad = 1;
      *rp.stopped = rp.call;
      atomicOr(rp.status, (int)PSE_STATUS_NONFINITE_POS);
      v = 0.0;
    }
    v -= L * floor(v / L);
    if (v >= L) v -= L;
    if (v < 0) v = 0;
    y[d] = v;
  }
}

// --------------------------------------------------------------- bins --

__device__ __forceinline__ int bin_of(const double *__restrict__ xw, int64_t i, int nc,
                                      double inv_cs) {
  int c[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int v = (int)(xw[3 * i + d] * inv_cs);
    c[d] = v < 0 ? 0 : (v >= nc ? nc - 1 : v);
  }
  return (c[2] * nc + c[1]) * nc + c[0];
}

// Prefix sums saturate (list_add): exclusive ones are the neighbour's
// inclusive ones, never a difference.

// Exclusive scan in chunks of 1024 (256 threads x 4).
__global__ void scan_block_kernel(const int *__restrict__ in, int *__restrict__ out,
                                  int *__restrict__ block_sums, int n) {
  __shared__ int s[256];
  const int base = blockIdx.x * 1024 + threadIdx.x * 4;
  int v[4], sum = 0;
  for (int j = 0; j < 4; ++j) {
    v[j] = base + j < n ? in[base + j] : 0;
    sum = list_add(sum, v[j]);
  }
  s[threadIdx.x] = sum;
  __syncthreads();
  for (int off = 1; off < 256; off <<= 1) {
    const int t = threadIdx.x >= off ? s[threadIdx.x - off] : 0;
    __syncthreads();
    s[threadIdx.x] = list_add(s[threadIdx.x], t);
    __syncthreads();
  }
  int run = threadIdx.x > 0 ? s[threadIdx.x - 1] : 0;
  for (int j = 0; j < 4; ++j) {
    if (base + j < n) out[base + j] = run;
    run = list_add(run, v[j]);
  }
  if (threadIdx.x == 255) block_sums[blockIdx.x] = s[255];
}

__global__ void scan_sums_kernel(int *__restrict__ sums, int nb, int *__restrict__ total,
                                 int *__restrict__ info) {
  // single block: exclusive scan of nb block sums with a running carry
  __shared__ int s[256];
  __shared__ int carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int b0 = 0; b0 < nb; b0 += 256) {
    const int i = b0 + threadIdx.x;
    const int v = i < nb ? sums[i] : 0;
    s[threadIdx.x] = v;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
      const int t = threadIdx.x >= off ? s[threadIdx.x - off] : 0;
      __syncthreads();
      s[threadIdx.x] = list_add(s[threadIdx.x], t);
      __syncthreads();
    }
    if (i < nb) sums[i] = list_add(carry, threadIdx.x > 0 ? s[threadIdx.x - 1] : 0);
    __syncthreads();
    if (threadIdx.x == 255) carry = list_add(carry, s[255]);
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *total = carry;
    if (info) *info = carry;
  }
}

__global__ void scan_add_kernel(int *__restrict__ out, const int *__restrict__ sums, int n) {
  const int i = blockIdx.x * 1024 + threadIdx.x * 4;
  const int add = sums[blockIdx.x];
  for (int j = 0; j < 4; ++j)
    if (i + j < n) out[i + j] = list_add(out[i + j], add);
}

// Exclusive prefix sums of n ints by one workgroup of 1024: thread t takes a
// contiguous chunk, the chunk totals are scanned within each wave (shuffles)
// and across the 16 waves (LDS), and every thread then writes its chunk's
// prefixes.  in and out may be the same; *total (may be NULL) is their sum.
__device__ __forceinline__ void scan_one(const int *in, int *out, int n, int *wsum,
                                         int *total, int *total2) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int per = (n + 1023) / 1024;
  const int lo = min(t * per, n), hi = min(lo + per, n);
  int incl = 0;
  for (int i = lo; i < hi; ++i) incl = list_add(incl, in[i]);
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int u = __shfl_up(incl, off, 64);
    if (lane >= off) incl = list_add(incl, u);
  }
  const int below = __shfl_up(incl, 1, 64);
  if (lane == 63) wsum[wv] = incl;
  __syncthreads();
  if (wv == 0) {
    int wi = lane < 16 ? wsum[lane] : 0;
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) {
      const int u = __shfl_up(wi, off, 64);
      if (lane >= off) wi = list_add(wi, u);
    }
    const int before = __shfl_up(wi, 1, 64);
    if (lane < 16) wsum[lane] = lane > 0 ? before : 0;
  }
  __syncthreads();
  int run = list_add(wsum[wv], lane > 0 ? below : 0);
  for (int i = lo; i < hi; ++i) {
    const int x = in[i];
    out[i] = run;
    run = list_add(run, x);
  }
  if (t == 1023) {
    if (total) *total = run;
    if (total2) *total2 = run;
  }
  __syncthreads();
}

// One scan per workgroup (one launch for lists of at most 1024 x SCAN1_PER
// entries; longer ones take three launches): out[n] = total, also at *info.
constexpr int SCAN1_PER = 32;
constexpr int SCAN1_MAX = 1024 * SCAN1_PER;

struct ScanJob {
  const int *in;
  int *out;
  int n;
  int *info;
  int *blocked;   // with nc: scan in's bins in block order, by way of this copy
  int nc;
};

// Bin b of an nc^3 lattice (x fastest) at its position in block order:
// blocks of BIN_BLOCK^3 bins in lexicographic order, bins lexicographic
// within a block (partial blocks at the far faces).
__device__ __forceinline__ int block_order_pos(int b, int nc) {
  const int bx = b % nc, by = (b / nc) % nc, bz = b / (nc * nc);
  const int B = BIN_BLOCK, nb = (nc + B - 1) / B;
  const int Bx = bx / B, By = by / B, Bz = bz / B;
  // bins before this block: full slabs and rows of blocks, with the widths
  // of the partial blocks at the far faces
  const auto w = [&](int blk) { return blk + 1 < nb ? B : nc - B * (nb - 1); };
  const int wx = w(Bx), wy = w(By);
  const int before = Bz * B * nc * nc + By * B * nc * w(Bz) + Bx * B * wy * w(Bz);
  const int lx = bx - Bx * B, ly = by - By * B, lz = bz - Bz * B;
  return before + (lz * wy + ly) * wx + lx;
}

// counts permuted into block order
__global__ void block_count_kernel(const int *__restrict__ count, int nc,
                                   int *__restrict__ bcount) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nc * nc * nc) return;
  bcount[block_order_pos(b, nc)] = count[b];
}

__global__ void __launch_bounds__(1024) scan_single_kernel(ScanJob a, ScanJob b, ScanJob c) {
  __shared__ int wsum[16];
  const ScanJob j = blockIdx.x == 0 ? a : (blockIdx.x == 1 ? b : c);
  const int *in = j.in;
  if (j.blocked) {
    for (int i = threadIdx.x; i < j.n; i += 1024) j.blocked[block_order_pos(i, j.nc)] = j.in[i];
    in = j.blocked;
    __threadfence_block();
    __syncthreads();
  }
  scan_one(in, j.out, j.n, wsum, j.out + j.n, j.info);
}

// The two binnings of a position update (real-space cells and, nc > 0,
// spreading tiles) pass by pass, both in every launch.
struct BinSet {
  int nc;
  double inv_cs;
  int *count, *start, *of, *slot, *scat, *perm, *trav, *bcount, *bstart;
  __host__ __device__ int bins() const { return nc * nc * nc; }
};

// x (may be NULL) wrapped into xu; counts cleared.
__global__ void __launch_bounds__(256)
bins_begin_kernel(const double *__restrict__ x, double *__restrict__ xu, int64_t n, double L,
                  Deform df, Reports rp, BinSet a, BinSet b) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (x && i < n) {
    double y[3];
    wrapped_position(x, i, L, df, rp, y);
#pragma unroll
    for (int d = 0; d < 3; ++d) xu[3 * i + d] = y[d];
  }
  if (i < a.bins()) a.count[i] = 0;
  if (i < b.bins()) b.count[i] = 0;
}

// each particle's bin and arrival slot
__global__ void __launch_bounds__(256)
bins_count_kernel(const double *__restrict__ xw, int64_t n, BinSet a, BinSet b) {
  const BinSet &s = blockIdx.y ? b : a;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int bin = bin_of(xw, i, s.nc, s.inv_cs);
  s.of[i] = bin;
  s.slot[i] = atomicAdd(&s.count[bin], 1);
}

// members of each bin in arrival order
__global__ void __launch_bounds__(256) bins_scatter_kernel(int64_t n, BinSet a, BinSet b) {
  const BinSet &s = blockIdx.y ? b : a;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  s.scat[s.start[s.of[i]] + s.slot[i]] = (int)i;
}

// The arrival order within a bin (atomic slots) varies from run to run; every
// later sum runs in bin order, so each bin's members are put in increasing
// particle index: one wavefront per bin, member p going to the position of
// its rank among the bin's indices.  Results are then reproducible bit for
// bit.  slot[t] becomes the bin of position t, trav lists the members with
// the bins in block order.
// SORT: the particles themselves take this order (the library's own order of
// a call, see prepare_positions): order[t] is the caller's index of particle t,
// xs its position, inv[order[t]] = t, and perm the identity.  map (not NULL):
// the members are the caller's indices, map[v] particle v's own.
template <bool SORT>
__device__ __forceinline__ void order_bin(unsigned blk, const BinSet &s,
                                          const double *__restrict__ x, int *__restrict__ order,
                                          double *__restrict__ xs, int *__restrict__ inv,
                                          const int *__restrict__ map) {
  const int bin = (int)blk * 4 + threadIdx.x / 64, lane = threadIdx.x % 64;
  if (bin >= s.bins()) return;
  const int lo = s.start[bin], k = s.start[bin + 1] - lo;
  const int dst = s.trav ? s.bstart[block_order_pos(bin, s.nc)] : 0;
  for (int p0 = 0; p0 < k; p0 += 64) {
    const int p = p0 + lane;
    int v = p < k ? s.scat[lo + p] : 0;
    if (map && p < k) v = map[v];
    int rank = 0;
    for (int q0 = 0; q0 < k; q0 += 64) {
      // members q0.. of the bin, one per lane, handed around the wavefront
      int u = v;
      if (q0 != p0) {
        u = q0 + lane < k ? s.scat[lo + q0 + lane] : 0;
        if (map && q0 + lane < k) u = map[u];
      }
      const int m = min(64, k - q0);
      for (int q = 0; q < m; ++q) rank += __builtin_amdgcn_readlane(u, q) < v ? 1 : 0;
    }
    if (p >= k) continue;
    const int t = lo + rank;
    s.slot[t] = bin;
    s.perm[t] = SORT ? t : v;
    if (s.trav) s.trav[dst + rank] = SORT ? t : v;
    if constexpr (SORT) {
      order[t] = v;
      inv[v] = t;
#pragma unroll
      for (int d = 0; d < 3; ++d) xs[3 * (size_t)t + d] = x[3 * (size_t)v + d];
    }
  }
}

template <bool SORT>
__global__ void __launch_bounds__(256)
bins_order_kernel(BinSet a, unsigned na, BinSet b, const double *__restrict__ x,
                  int *__restrict__ order, double *__restrict__ xs, int *__restrict__ inv,
                  const int *__restrict__ map) {
  if (blockIdx.x < na) order_bin<SORT>(blockIdx.x, a, x, order, xs, inv, map);
  else order_bin<false>(blockIdx.x - na, b, x, nullptr, nullptr, nullptr, map);
}

// The bins of one lattice for the single-workgroup build.
struct BinJob {
  const double *x;
  int nc;
  double inv_cs;
  int *start, *perm, *at, *trav;   // (trav may be NULL; see Bins)
};

// All of a binning in LDS: counts, prefix sums, members in arrival order and
// their ranks (the same order as the launches below give).  lds: two ints per
// bin, two 16-bit numbers per particle.
template <bool SORT>
__device__ __forceinline__ void bins_one(const BinJob &job, int n, int *lds, int *wsum,
                                         int *__restrict__ order, double *__restrict__ xs) {
  const int nc = job.nc, nb = nc * nc * nc, tid = threadIdx.x;
  int *cur = lds, *bpos = lds + nb;
  uint16_t *scat = reinterpret_cast<uint16_t *>(lds + 2 * nb), *sbin = scat + n;
  for (int b = tid; b < nb; b += 1024) cur[b] = 0;
  __syncthreads();
  for (int i = tid; i < n; i += 1024) atomicAdd(&cur[bin_of(job.x, i, nc, job.inv_cs)], 1);
  __syncthreads();
  if (job.trav) {
    for (int b = tid; b < nb; b += 1024) bpos[block_order_pos(b, nc)] = cur[b];
    __syncthreads();
    scan_one(bpos, bpos, nb, wsum, nullptr, nullptr);
  }
  scan_one(cur, cur, nb, wsum, job.start + nb, nullptr);
  for (int b = tid; b < nb; b += 1024) job.start[b] = cur[b];
  __syncthreads();
  for (int i = tid; i < n; i += 1024) {
    const int b = bin_of(job.x, i, nc, job.inv_cs);
    const int p = atomicAdd(&cur[b], 1);
    scat[p] = (uint16_t)i;
    sbin[p] = (uint16_t)b;
  }
  __syncthreads();
  // cur[b] is now the end of bin b
  for (int q = tid; q < n; q += 1024) {
    const int v = scat[q], b = sbin[q];
    const int lo = b > 0 ? cur[b - 1] : 0, hi = cur[b];
    int rank = 0;
    for (int r = lo; r < hi; ++r) rank += scat[r] < v ? 1 : 0;
    const int t = lo + rank;
    job.at[t] = b;
    job.perm[t] = SORT ? t : v;
    if (job.trav) job.trav[bpos[block_order_pos(b, nc)] + rank] = SORT ? t : v;
    if constexpr (SORT) {
      order[t] = v;
#pragma unroll
      for (int d = 0; d < 3; ++d) xs[3 * t + d] = job.x[3 * v + d];
    }
  }
  __syncthreads();
}

// SORT: the caller's positions x are wrapped (into xu), binned into the cells
// and put in cell order (order, xs), then the tiles (if any: tiles.nc > 0) are
// binned in that order.  Else workgroup 0 bins the cells, 1 the tiles.
template <bool SORT>
__global__ void __launch_bounds__(1024)
bins_one_kernel(const double *__restrict__ x, double *xu, int n, double L, Deform df, Reports rp,
                BinJob cells, BinJob tiles, int *order, double *xs) {
  extern __shared__ int bin_lds[];
  __shared__ int wsum[16];
  if constexpr (SORT) {
    for (int i = threadIdx.x; i < n; i += 1024) {
      double y[3];
      wrapped_position(x, i, L, df, rp, y);
#pragma unroll
      for (int d = 0; d < 3; ++d) xu[3 * i + d] = y[d];
    }
    // a thread bins the particles that it wrapped; the ordered positions are
    // read by others only after the barriers
    __threadfence_block();
    __syncthreads();
    bins_one<true>(cells, n, bin_lds, wsum, order, xs);
    __threadfence_block();
    __syncthreads();
    if (tiles.nc > 0) bins_one<false>(tiles, n, bin_lds, wsum, nullptr, nullptr);
  } else {
    bins_one<false>(blockIdx.x == 0 ? cells : tiles, n, bin_lds, wsum, nullptr, nullptr);
  }
}

// Particles up to which one workgroup builds the bins: its passes over the
// particles cost 4 us per 1000, the launches they replace 30 us (N = 10^4: 36
// against 30 us, 2*10^4: 105 against 40; its LDS holds the particles as 16-bit
// numbers).
constexpr int ONE_WG_N = 4096;
constexpr size_t ONE_WG_LDS = 150 * 1024;

static size_t one_wg_lds(int nc, int64_t n) {
  return (size_t)nc * nc * nc * 2 * sizeof(int) + (size_t)n * 2 * sizeof(uint16_t);
}

static bool one_wg(const Handle &h, const Bins &b) {
  return b.nc == 0 || (h.n <= ONE_WG_N && b.nc <= 40 && one_wg_lds(b.nc, h.n) <= ONE_WG_LDS &&
                       one_wg_lds(b.nc, h.n) <= (size_t)h.max_lds);
}

static BinJob bin_job(const Handle &h, const Bins &b, const double *x) {
  return BinJob{x, b.nc, b.nc / h.p.box, b.start, b.perm, b.slot, b.trav};
}

// Prefix sums of a list too long for one workgroup.
static void scan_long(Handle &h, const int *in, int *out, int *tmp, int n, int *info) {
  const int sb = (n + 1023) / 1024;
  hipLaunchKernelGGL(scan_block_kernel, dim3(sb), dim3(256), 0, h.stream, in, out, tmp, n);
  PSE_LAUNCH_CHECK();
  hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(256), 0, h.stream, tmp, sb, out + n, info);
  PSE_LAUNCH_CHECK();
  hipLaunchKernelGGL(scan_add_kernel, dim3(sb), dim3(256), 0, h.stream, out, tmp, n);
  PSE_LAUNCH_CHECK();
}

// The jobs' prefix sums: one launch where all are short, else the long ones'
// own (tmp: scratch of n/1024 + 8 ints each).
static void scan_jobs(Handle &h, const ScanJob *jobs, int *const *tmp, int count) {
  ScanJob small[3] = {};
  int ns = 0;
  for (int k = 0; k < count; ++k) {
    const ScanJob &j = jobs[k];
    if (j.n <= SCAN1_MAX) {
      small[ns++] = j;
      continue;
    }
    const int *in = j.in;
    if (j.blocked) {
      hipLaunchKernelGGL(block_count_kernel, dim3(nblocks(j.n, 256)), dim3(256), 0, h.stream,
                         j.in, j.nc, j.blocked);
      PSE_LAUNCH_CHECK();
      in = j.blocked;
    }
    scan_long(h, in, j.out, tmp[k], j.n, j.info);
  }
  if (ns == 0) return;
  hipLaunchKernelGGL(scan_single_kernel, dim3(ns), dim3(1024), 0, h.stream, small[0], small[1],
                     small[2]);
  PSE_LAUNCH_CHECK();
}

static BinSet bin_set(const Handle &h, const Bins &b) {
  return BinSet{b.nc, b.nc / h.p.box, b.count, b.start, b.of, b.slot, b.scat,
                b.perm, b.trav, b.bcount, b.bstart};
}

// ------------------------------------------------------------ pair list --
// The positions stay fixed over all the operator applications of a Krylov
// solve, so the neighbours within rcut are found once per position update
// and stored as a CSR list in cell order: row t holds the neighbours of
// particle perm[t].  Rows are filled in a fixed order (cells, then
// candidates, ranked with a ballot inside the group).  Each entry holds the
// neighbour index and the pair's data -- the seven interpolated radial
// coefficients and the unit vector -- in the precision of the handle's own
// pair sums (FP64 handles: doubles; mixed handles: floats, read by their
// FP32 sums).  A sum in the other precision (the FP64 residual of a mixed
// handle, once per step) forms the data from the positions itself.

struct PairArgs {
  int64_t n;
  int nc;
  double L, rcut2;
  double inv_cs, cs2;   // cells per unit length, squared cell side
  double inv_dr;
  int n2a, ntab;
  int limit;       // entries the pair list holds: those at or beyond are not written
  Reports rp;
  int def;         // deformed lattice: positions are lattice coordinates and
  double A[9];     // separations are mapped back by A
  const int *perm, *cell_start, *cell_at;
  int *cnt, *start, *nbr;
  double *rec64;
  float *rec32;
};

__device__ __forceinline__ bool near_pair(const double *__restrict__ xw, double xi0, double xi1,
                                          double xi2, int j, const PairArgs &pa, double *d) {
  separation(xw, xi0, xi1, xi2, j, pa.L, pa.def, pa.A, d);
  return d[0] * d[0] + d[1] * d[1] + d[2] * d[2] < pa.rcut2;
}

// FILL = false: count the neighbours of each row into cnt[t]; FILL = true:
// write them from start[t] on.  One wavefront per row enumerates the
// candidates of the 27 cells around the particle 64 at a time.
template <bool FILL>
__device__ __forceinline__ void pair_rows(unsigned blk, const double *__restrict__ xw,
                                          const PairArgs &pa) {
  const int *__restrict__ perm = pa.perm, *__restrict__ cell_start = pa.cell_start;
  const int *__restrict__ cell_at = pa.cell_at, *__restrict__ start = pa.start;
  int *__restrict__ cnt = pa.cnt, *__restrict__ nbr = pa.nbr;
  double *__restrict__ rec64 = pa.rec64;
  float *__restrict__ rec32 = pa.rec32;
  const int64_t t = ((int64_t)blk * 256 + threadIdx.x) / 64;
  const int lane = threadIdx.x % 64;
  if (t >= pa.n) return;
  const int i = perm[t];
  const double xi0 = xw[3 * i], xi1 = xw[3 * i + 1], xi2 = xw[3 * i + 2];
  const int nc = pa.nc;
  const int ci = cell_at[t];
  const int cc[3] = {ci % nc, (ci / nc) % nc, ci / (nc * nc)};
  // a neighbouring cell whose gap to the particle exceeds the cutoff holds no
  // neighbour: it is skipped (the list is the same; on a deformed lattice,
  // where cell units are not lengths, every cell is searched)
  bool skip = false;
  if (!pa.def && lane < 27) {
    const int off[3] = {lane % 3 - 1, (lane / 3) % 3 - 1, lane / 9 - 1};
    const double xi[3] = {xi0, xi1, xi2};
    double g2 = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double u = xi[d] * pa.inv_cs - cc[d];   // position in the cell, cell units
      const double gap = off[d] > 0 ? 1.0 - u : (off[d] < 0 ? u : 0.0);
      if (gap > 0.0) g2 += gap * gap;
    }
    skip = g2 * pa.cs2 > pa.rcut2 * (1.0 + 1e-9);
  }
  int first, pre, total;
  nbr27_setup(lane, cc[0], cc[1], cc[2], nc, cell_start, first, pre, total, skip);
  const int row = FILL ? start[t] : 0;
  int count = 0;
  for (int base = 0; base < total; base += 64) {
    const int idx = base + lane;
    const int s = nbr27_slot(idx, first, pre);
    double d[3];
    int j = -1;
    bool ok = false;
    if (idx < total) {
      j = perm[s];
      ok = j != i && near_pair(xw, xi0, xi1, xi2, j, pa, d);
    }
    if (!FILL) {
      count += ok ? 1 : 0;
    } else {
      const unsigned long long m = __ballot(ok);
      const int slot =
          list_slot(row, count + __popcll(m & ((1ull << lane) - 1ull)), pa.limit);
      if (ok && slot >= 0) {
        nbr[slot] = j;
        if (rec64 || rec32) {
          // the unit vector now, the distance in field d2 for
          // pair_coefficients (the table interpolation runs there on every
          // lane, not on the few lanes of a candidate batch that found a
          // neighbour)
          const double r = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
          const double inv = r > 0 ? 1.0 / r : 0.0;
          if (rec64) {
            const Entry<double> p(rec64, slot);
            p[F_D2] = r;
#pragma unroll
            for (int k = 0; k < 3; ++k) p[F_E + k] = d[k] * inv;
          } else {
            const Entry<float> p(rec32, slot);
            p[F_D2] = (float)r;
#pragma unroll
            for (int k = 0; k < 3; ++k) p[F_E + k] = (float)(d[k] * inv);
          }
        }
      }
      count += __popcll(m);
      if (m && list_slot(row, count - 1, pa.limit) < 0) {
        // the list is full: nothing more of this row fits
        if (lane == 0) {
          *pa.rp.stopped = pa.rp.call;
          atomicOr(pa.rp.status, (int)PSE_STATUS_PAIR_OVERFLOW);
        }
        return;
      }
    }
  }
  if (!FILL) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) count += __shfl_xor(count, off, 64);
    if (lane == 0) cnt[t] = count;
  }
}

// The seven radial coefficients of every stored pair, interpolated from the
// table at the distance the fill left in field d2 (entries up to the list's
// length, read on the device, and its capacity), in the records' precision,
// from the table of that precision: workgroup blk of nblk.
template <typename R>
__device__ __forceinline__ void pair_coefficients(unsigned blk, unsigned nblk, R *__restrict__ rec,
                                                  const R *__restrict__ tab, const PairArgs &pa) {
  const int64_t len = list_row_end(pa.start[pa.n], pa.limit);
  constexpr int field[NCOEF] = {F_A, F_B, F_C1, F_C2, F_D2, F_D3, F_D4};
  for (int64_t s = (int64_t)blk * blockDim.x + threadIdx.x; s < len;
       s += (int64_t)nblk * blockDim.x) {
    R co[NCOEF];
    const Entry<R> p(rec, (uint32_t)s);
    lookup<R>(tab, p[F_D2], (R)pa.inv_dr, pa.n2a, pa.ntab, co);
#pragma unroll
    for (int k = 0; k < NCOEF; ++k) p[field[k]] = co[k];
  }
}

// --------------------------------------------------------- tile lists --

struct TileArgs {
  GridGeom g;
  int S, nb;                    // points and tiles per side
  const int *bstart, *bperm;    // the spreading bins
  int *cnt, *start;
  TileRec *rec;
};

// FILL = false: count each tile's candidates; true: write their records from
// start[tile] on, in bin order and ranked with a ballot.  One wavefront per
// tile enumerates the particles of the 27 bins around it 64 at a time (bins
// are tiles; a stencil reaches at most one tile beyond its particle's).
template <bool FILL>
__device__ __forceinline__ void tile_rows(unsigned blk, const double *__restrict__ x,
                                          const TileArgs &ta) {
  const int tile = (int)blk * 4 + threadIdx.x / 64;
  const int lane = threadIdx.x % 64, nb = ta.nb, S = ta.S;
  if (tile >= nb * nb * nb) return;
  const int tc[3] = {tile % nb, (tile / nb) % nb, tile / (nb * nb)};
  const int P = ta.g.P, ng = ta.g.ng;
  int first, pre, total;
  nbr27_setup(lane, tc[0], tc[1], tc[2], nb, ta.bstart, first, pre, total);
  int pos = FILL ? ta.start[tile] : 0;
  int count = 0;
  for (int base = 0; base < total; base += 64) {
    const int idx = base + lane;
    const int s = nbr27_slot(idx, first, pre);
    bool ok = false;
    int p = 0, win = 0;
    if (idx < total) {
      p = ta.bperm[s];
      ok = true;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        // off: the stencil's first point relative to the tile's, in
        // (-P, S) where the two meet
        const int st = stencil_start(x[3 * p + d], ta.g.h, P);
        int off = (st - tc[d] * S) % ng;
        off += off < 0 ? ng : 0;
        off -= off >= S ? ng : 0;
        ok = ok && off > -P;
        win |= ((S - 1 - off) & 255) << (8 * d);
      }
    }
    if (!FILL) {
      count += ok ? 1 : 0;
    } else {
      const unsigned long long m = __ballot(ok);
      if (ok) ta.rec[(int64_t)pos + __popcll(m & ((1ull << lane) - 1ull))] = TileRec{p, win};
      pos += __popcll(m);
    }
  }
  if (!FILL) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) count += __shfl_xor(count, off, 64);
    if (lane == 0) ta.cnt[tile] = count;
  }
}

// Moment correction of the gradient weights of derivative gridding.  On the
// grid the gradient of the truncated Gaussian does not have the moments of
// the continuous one: along axis d its one-dimensional weights
// g_i = dK1/dx (x_i - x) sum to mu_d times the Gaussian's, sum_i g_i =
// mu_d sum_i w_i, with mu_d a small number that depends on the particle's
// offset from the grid, and their first moment sum_i d_i g_i (d_i = x_i - x)
// differs from -sum_i w_i, its continuous value.  A spread couplet then
// leaves a spurious monopole in the smallest wave numbers, where the Stokes
// kernel amplifies it, and the interpolated gradient of a smooth field picks
// up the field itself.  Spreading and interpolation take instead
// lambda_d (g_i - mu_d w_i), still separable, whose discrete sum is zero and
// whose first moment is -sum_i w_i: the gradient of a constant field is
// zero and that of a linear field exact, relative to the Gaussian's own
// normalisation.
//
// The one-dimensional weights are kept per particle and axis, formed once per
// position update, for spreading and interpolation: rows of rw = P + 2 (S - 1)
// entries, the P weights with S - 1 zeros on either side, so that any tile
// that a stencil meets reads its S weights as one window of the row; an entry
// is the weight, or with derivative gridding the weight and the corrected
// gradient weight.
struct WeightArgs {
  GridGeom g;
  int64_t n;
  int pad, rw;        // S - 1 zeros; entries of a row
  double *w64;
  float *w32;         // or NULL
};

constexpr int W_THREADS = 192;

// A workgroup forms W_THREADS rows, one per thread, in LDS and writes them as
// one contiguous block.
template <bool DERIV>
__device__ __forceinline__ void weight_rows(unsigned blk, const double *__restrict__ x,
                                            const WeightArgs &wa, double *lds) {
  const int tid = threadIdx.x;
  const int64_t t0 = (int64_t)blk * W_THREADS, t = t0 + tid;
  const int nrow = (int)min((int64_t)W_THREADS, 3 * wa.n - t0);
  const GridGeom &g = wa.g;
  // per row: P weights, then the first stencil point's offset, mu and lambda,
  // each W_THREADS apart
  double *const rowd = lds + g.P * W_THREADS;
  if (tid < nrow) {
    const double xc = x[t];
    const int i0 = stencil_start(xc, g.h, g.P);
    double s0 = 0.0, s1 = 0.0, sd = 0.0, sd1 = 0.0;
    for (int i = 0; i < g.P; ++i) {
      const double d = (i0 + i) * g.h - xc;
      const double w = exp(-g.kcoef * d * d);
      const double gi = -2.0 * g.kcoef * d * w;
      lds[i * W_THREADS + tid] = w;
      s0 += w;
      s1 += gi;
      sd += d * w;
      sd1 += d * gi;
    }
    rowd[tid] = i0 * g.h - xc;
    if constexpr (DERIV) {
      // sum_i d_i (g_i - m w_i) = sd1 - m sd
      const double m = s1 / s0, lam = -s0 / (sd1 - m * sd);
      rowd[W_THREADS + tid] = m;
      rowd[2 * W_THREADS + tid] = lam;
    }
  }
  __syncthreads();
  const size_t o0 = (size_t)t0 * wa.rw;
  int row = tid / wa.rw, e = tid % wa.rw;
  const int drow = W_THREADS / wa.rw, de = W_THREADS % wa.rw;
  for (int k = tid; k < nrow * wa.rw; k += W_THREADS) {
    const int a = e - wa.pad;
    double w = 0.0, gw = 0.0;
    if (a >= 0 && a < g.P) {
      w = g.knorm * lds[a * W_THREADS + row];
      if constexpr (DERIV)
        gw = rowd[2 * W_THREADS + row] *
             (-2.0 * g.kcoef * (rowd[row] + a * g.h) - rowd[W_THREADS + row]) * w;
    }
    if constexpr (DERIV) {
      reinterpret_cast<double2 *>(wa.w64)[o0 + k] = double2{w, gw};
      if (wa.w32) reinterpret_cast<float2 *>(wa.w32)[o0 + k] = float2{(float)w, (float)gw};
    } else {
      wa.w64[o0 + k] = w;
      if (wa.w32) wa.w32[o0 + k] = (float)w;
    }
    row += drow;
    e += de;
    if (e >= wa.rw) {
      e -= wa.rw;
      ++row;
    }
  }
}

// ------------------------------------------------------------- passes --

// Counting pass (FILL = false) and filling pass of the pair list (workgroups
// [0, nbp)) and of the tile lists (the rest).
template <bool FILL>
__global__ void __launch_bounds__(256)
list_pass_kernel(const double *__restrict__ x, PairArgs pa, unsigned nbp, TileArgs ta) {
  if (blockIdx.x < nbp) pair_rows<FILL>(blockIdx.x, x, pa);
  else tile_rows<FILL>(blockIdx.x - nbp, x, ta);
}

// The pairs' coefficients (workgroups [0, nbc)) and the particles' weights
// (the rest).
template <typename R, bool DERIV>
__global__ void __launch_bounds__(W_THREADS)
list_data_kernel(const double *__restrict__ x, PairArgs pa, R *__restrict__ rec,
                 const R *__restrict__ tab, unsigned nbc, WeightArgs wa) {
  extern __shared__ double w_lds[];
  if (blockIdx.x < nbc) pair_coefficients<R>(blockIdx.x, nbc, rec, tab, pa);
  else weight_rows<DERIV>(blockIdx.x - nbc, x, wa, w_lds);
}

static Reports reports(const Handle &h) {
  return Reports{h.info + INFO_BAD, h.dctl + CTL_STATUS, h.dctl + CTL_STOPPED, h.call};
}

// The pair list for the current cells and, with tiles, the tile lists and the
// particles' weights.  No host read in between: the list keeps its capacity,
// pairs beyond it are not written (and flagged in the device status), and a
// synchronous handle looks at the length where it waits for the stream next
// (verify_lists), before any result that depends on it is handed over.
static void build_lists(Handle &h, const double *xw, bool spreading) {
  const bool tiles = h.stile && spreading;
  h.tiles_current = h.sbins.nc && spreading;
  PairArgs pa;
  pa.n = h.n;
  pa.nc = h.cells.nc;
  pa.L = h.p.box;
  pa.rcut2 = h.d.rcut * h.d.rcut;
  // the cell assignment's own scale (cell = floor(x nc / L))
  pa.inv_cs = pa.nc / h.p.box;
  pa.cs2 = (h.p.box / pa.nc) * (h.p.box / pa.nc);
  pa.inv_dr = 1.0 / h.dr;
  pa.n2a = h.n2a;
  pa.ntab = h.ntab;
  pa.limit = list_limit((int64_t)h.pl_cap);
  pa.rp = reports(h);
  pa.def = h.def.on;
  for (int i = 0; i < 9; ++i) pa.A[i] = h.def.A[i];
  pa.perm = h.cells.perm;
  pa.cell_start = h.cells.start;
  pa.cell_at = h.cells.slot;
  pa.cnt = h.pl_cnt;
  pa.start = h.pl_start;
  pa.nbr = h.pl_nbr;
  pa.rec64 = h.pl_rec64;
  pa.rec32 = h.pl_rec32;
  TileArgs ta{};
  ta.g = geom(h);
  ta.S = h.stile;
  ta.nb = h.sbins.nc;
  ta.bstart = h.sbins.start;
  ta.bperm = h.sbins.perm;
  ta.cnt = h.tl_cnt;
  ta.start = h.tl_start;
  ta.rec = h.tl_rec;
  const int n = (int)h.n, ntile = tiles ? ta.nb * ta.nb * ta.nb : 0;
  const unsigned nbp = nblocks((size_t)h.n * 64, 256), nbt = (unsigned)((ntile + 3) / 4);
  hipLaunchKernelGGL(list_pass_kernel<false>, dim3(nbp + nbt), dim3(256), 0, h.stream, xw, pa, nbp,
                     ta);
  PSE_LAUNCH_CHECK();
  int *info = nullptr;
  if (!h.async) {
    if (h.lists_open == INFO_LISTS) throw Error{PSE_ERR_INVALID, "too many lists unverified"};
    info = h.info + INFO_PAIRS + h.lists_open++;
  }
  const ScanJob jobs[2] = {{h.pl_cnt, h.pl_start, n, info, nullptr, 0},
                           {h.tl_cnt, h.tl_start, ntile, nullptr, nullptr, 0}};
  int *const tmp[2] = {h.pl_scan, h.tl_scan};
  scan_jobs(h, jobs, tmp, tiles ? 2 : 1);
  hipLaunchKernelGGL(list_pass_kernel<true>, dim3(nbp + nbt), dim3(256), 0, h.stream, xw, pa, nbp,
                     ta);
  PSE_LAUNCH_CHECK();
  WeightArgs wa{};
  wa.g = ta.g;
  wa.n = h.n;
  wa.pad = h.stile - 1;
  wa.rw = weight_row(h.d.support, h.stile);
  // interpolation reads the FP64 rows, FP32 spreading the FP32 ones
  wa.w64 = h.wt64;
  wa.w32 = spreading ? h.wt32 : nullptr;
  // the coefficients' workgroups walk the list (its length is on the device)
  const unsigned nbc = std::min(nblocks(h.pl_cap, W_THREADS), (unsigned)h.num_cu * 32u);
  const unsigned nbw = !h.stile ? 0 : nblocks(3 * (size_t)h.n, W_THREADS);
  const size_t lds = nbw ? (size_t)W_THREADS * (h.d.support + 3) * sizeof(double) : 0;
  const auto launch = [&](auto *rec, auto *tab, auto deriv) {
    using R = std::remove_reference_t<decltype(*rec)>;
    hipLaunchKernelGGL((list_data_kernel<R, decltype(deriv)::value>), dim3(nbc + nbw),
                       dim3(W_THREADS), lds, h.stream, xw, pa, rec, (const R *)tab, nbc, wa);
  };
  if (h.mixed) {
    if (h.deriv) launch(h.pl_rec32, h.g32.table, std::true_type());
    else launch(h.pl_rec32, h.g32.table, std::false_type());
  } else {
    if (h.deriv) launch(h.pl_rec64, h.g64.table, std::true_type());
    else launch(h.pl_rec64, h.g64.table, std::false_type());
  }
  PSE_LAUNCH_CHECK();
}

// What the kernels of a synchronous call reported in h.info, read once the
// stream is idle: non-finite positions are an error; a pair list longer than
// its capacity makes the call start over with a longer one (Regrow).
void verify_lists(Handle &h) {
  if (h.async || h.lists_open == 0) return;
  int w[INFO_WORDS];
  if (h.arena) {
    PSE_HIP(hipMemcpyAsync(w, h.info, sizeof(w), hipMemcpyDeviceToHost, h.stream));
    PSE_HIP(hipStreamSynchronize(h.stream));
  } else {
    for (int i = 0; i < INFO_WORDS; ++i) w[i] = ((const volatile int *)h.info)[i];
  }
  int total = 0;
  for (int k = 0; k < h.lists_open; ++k) total = std::max(total, w[INFO_PAIRS + k]);
  h.lists_open = 0;
  if (w[INFO_BAD]) throw Error{PSE_ERR_NONFINITE, "non-finite particle position"};
  if (total >= LIST_MAX)
    throw Error{PSE_ERR_NOMEM, "real-space pair list beyond " + std::to_string(LIST_MAX) +
                                   " pairs"};
  if ((size_t)total > h.pl_cap) {
    if (h.arena)
      throw Error{PSE_ERR_NOMEM, "real-space pair list beyond its capacity in the "
                                 "allocation-free product (" + std::to_string(total) +
                                 " pairs)"};
    throw Regrow{(size_t)total};
  }
  h.pl_pairs = (size_t)total;
}

void begin_lists(Handle &h) {
  h.lists_open = 0;
  h.call = h.call < INT32_MAX ? h.call + 1 : 1;
  if (h.async) return;
  if (h.arena) fill_int(h, h.info, INFO_WORDS, 0);
  else
    for (int i = 0; i < INFO_WORDS; ++i) ((volatile int *)h.info)[i] = 0;
}

void regrow_pairs(Handle &h, size_t total) {
  clear_graphs(h);   // captured real-space launches hold the old buffers
  pair_storage(h, total + total / 4 + 1024, false);
}

void pair_storage(Handle &h, size_t cap, bool at_create) {
  if (!at_create) {
    dev_free(h.pl_nbr);
    dev_free(h.pl_rec64);
    dev_free(h.pl_rec32);
    h.pl_nbr = nullptr;
    h.pl_rec64 = nullptr;
    h.pl_rec32 = nullptr;
    h.pl_cap = 0;
  }
  const auto alloc = [&](void **ptr, size_t bytes) {
    if (at_create) handle_alloc(h, ptr, bytes);
    else dev_alloc(ptr, bytes);
  };
  cap = (cap + REC_BLOCK - 1) / REC_BLOCK * REC_BLOCK;   // whole blocks
  alloc((void **)&h.pl_nbr, cap * sizeof(int));
  if (h.mixed) alloc((void **)&h.pl_rec32, cap * PAIR_REC * sizeof(float));
  else alloc((void **)&h.pl_rec64, cap * PAIR_REC * sizeof(double));
  h.pl_cap = cap;
}

static double cells_bytes(const Handle &h, bool spreading) {
  const bool tiles = h.sbins.nc && spreading;
  const double nc3 = (double)h.cells.nc * h.cells.nc * h.cells.nc
                     + (tiles ? (double)h.sbins.nc * h.sbins.nc * h.sbins.nc : 0.0);
  return (double)h.n * (24 + 16) * (tiles ? 2 : 1) + 12.0 * nc3;
}

// The library's own order of the particles for one call: the caller's
// positions x are wrapped, binned into the real-space cells and put in cell
// order, xw[t] = wrapped x[order[t]].  Every particle vector of the call is
// kept in this order (gather_rows on the way in, scatter_rows on the way
// out), so neighbours' data lie next to each other whatever the caller's
// order: the pair sums gather moments, the list builders positions and the
// grid kernels weights and moments from near addresses (a caller's random
// order made each gather a line of its own).  N = 10^6 in random order: the
// constraint operator's pair sum 349 -> 276 us, the full one 564 -> 468, the
// list's counting pass 846 -> 704, gradient interpolation 2.02 -> 1.89 ms.
//
// The cells (x given: of the caller's positions, which take their order, else
// of the wrapped positions xw) and, with tiles, the spreading bins.
static void build_all_bins(Handle &h, const double *x, const double *xw, bool tiles) {
  Bins none;
  const Bins &tb = tiles ? h.sbins : none;
  if (one_wg(h, h.cells) && one_wg(h, tb)) {
    const size_t lds = std::max(one_wg_lds(h.cells.nc, h.n), one_wg_lds(tb.nc, h.n));
    static std::once_flag once[2];
    hipError_t attr = hipSuccess;
    std::call_once(once[x ? 1 : 0], [&] {
      attr = hipFuncSetAttribute(x ? (const void *)bins_one_kernel<true>
                                   : (const void *)bins_one_kernel<false>,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)ONE_WG_LDS);
    });
    PSE_HIP(attr);
    if (x)
      hipLaunchKernelGGL(bins_one_kernel<true>, dim3(1), dim3(1024), lds, h.stream, x, h.xh,
                         (int)h.n, h.p.box, h.def, reports(h), bin_job(h, h.cells, h.xh),
                         bin_job(h, tb, h.xw), h.order, h.xw);
    else
      hipLaunchKernelGGL(bins_one_kernel<false>, dim3(tiles ? 2 : 1), dim3(1024), lds, h.stream,
                         nullptr, nullptr, (int)h.n, h.p.box, h.def, reports(h),
                         bin_job(h, h.cells, xw), bin_job(h, tb, xw), nullptr, nullptr);
    PSE_LAUNCH_CHECK();
    return;
  }
  const BinSet cs = bin_set(h, h.cells), ts = bin_set(h, tb);
  double *xu = h.xh;   // wrapped, in the caller's order: the mid-point's buffer
  const double *xb = x ? xu : xw;
  const size_t most = std::max((size_t)std::max(cs.bins(), ts.bins()), x ? (size_t)h.n : 0);
  const unsigned jobs = tiles ? 2 : 1, np = nblocks(h.n, 256);
  hipLaunchKernelGGL(bins_begin_kernel, dim3(nblocks(most, 256)), dim3(256), 0, h.stream, x, xu,
                     h.n, h.p.box, h.def, reports(h), cs, ts);
  PSE_LAUNCH_CHECK();
  hipLaunchKernelGGL(bins_count_kernel, dim3(np, jobs), dim3(256), 0, h.stream, xb, h.n, cs, ts);
  PSE_LAUNCH_CHECK();
  const ScanJob sj[3] = {{cs.count, cs.start, cs.bins(), nullptr, nullptr, 0},
                         {cs.count, cs.bstart, cs.bins(), nullptr, cs.bcount, cs.nc},
                         {ts.count, ts.start, ts.bins(), nullptr, nullptr, 0}};
  int *const tmp[3] = {h.cells.scan_tmp, h.cells.scan_tmp, h.sbins.scan_tmp};
  scan_jobs(h, sj, tmp, tiles ? 3 : 2);
  hipLaunchKernelGGL(bins_scatter_kernel, dim3(np, jobs), dim3(256), 0, h.stream, h.n, cs, ts);
  PSE_LAUNCH_CHECK();
  const unsigned na = (unsigned)((cs.bins() + 3) / 4), nt = (unsigned)((ts.bins() + 3) / 4);
  if (!x) {
    hipLaunchKernelGGL(bins_order_kernel<false>, dim3(na + nt), dim3(256), 0, h.stream, cs, na, ts,
                       xb, nullptr, nullptr, nullptr, nullptr);
    PSE_LAUNCH_CHECK();
    return;
  }
  // the tiles' members need the cells' order (its inverse takes the place of
  // the particles' cells, not read any more)
  int *inv = cs.of;
  hipLaunchKernelGGL(bins_order_kernel<true>, dim3(na), dim3(256), 0, h.stream, cs, na, ts, xb,
                     h.order, h.xw, inv, nullptr);
  PSE_LAUNCH_CHECK();
  if (!tiles) return;
  hipLaunchKernelGGL(bins_order_kernel<false>, dim3(nt), dim3(256), 0, h.stream, cs, 0u, ts, xb,
                     nullptr, nullptr, nullptr, (const int *)inv);
  PSE_LAUNCH_CHECK();
}

void prepare_positions(Handle &h, const double *x, bool spreading) {
  ProfScope ps(h, PK_CELLS, cells_bytes(h, spreading));
  begin_lists(h);
  build_all_bins(h, x, nullptr, h.sbins.nc && spreading);
  build_lists(h, h.xw, spreading);
}

void build_cells(Handle &h, const double *xw, bool spreading) {
  ProfScope ps(h, PK_CELLS, cells_bytes(h, spreading));
  build_all_bins(h, nullptr, xw, h.sbins.nc && spreading);
  build_lists(h, xw, spreading);
}

// Rows of w numbers between the caller's order and the library's.
__global__ void __launch_bounds__(256)
gather_rows_kernel(const double *__restrict__ src, const int *__restrict__ order, int w,
                   int64_t nw, double *__restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nw) return;
  const int64_t t = i / w;
  dst[i] = src[(int64_t)order[t] * w + (i - t * w)];
}

// The components [lo, hi) of the rows, unless the call has stopped
// (stopped_word); *bad is raised (bad not NULL) by a non-finite number in any
// component of the rows as they are left.
__global__ void __launch_bounds__(256)
scatter_rows_kernel(const double *__restrict__ src, const int *__restrict__ order, int w, int lo,
                    int hi, int64_t nw, double *__restrict__ dst, int *__restrict__ bad,
                    const int *__restrict__ stopped, int call) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nw || (stopped && *stopped == call)) return;
  const int64_t t = i / w;
  const int c = (int)(i - t * w);
  double *o = dst + (int64_t)order[t] * w + c;
  double v;
  if (c >= lo && c < hi) *o = v = src[i];
  else if (bad) v = *o;
  else return;
  if (bad && !isfinite(v)) *bad = 1;
}

void gather_rows(Handle &h, const double *src, int w, double *dst) {
  hipLaunchKernelGGL(gather_rows_kernel, dim3(nblocks((size_t)h.n * w, 256)), dim3(256), 0,
                     h.stream, src, (const int *)h.order, w, h.n * w, dst);
  PSE_LAUNCH_CHECK();
}

void scatter_rows(Handle &h, const double *src, int w, int lo, int hi, double *dst, int *bad) {
  hipLaunchKernelGGL(scatter_rows_kernel, dim3(nblocks((size_t)h.n * w, 256)), dim3(256), 0,
                     h.stream, src, (const int *)h.order, w, lo, hi, h.n * w, dst, bad,
                     stopped_word(h), h.call);
  PSE_LAUNCH_CHECK();
}

}  // namespace pse
