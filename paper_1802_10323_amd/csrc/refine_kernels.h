// refine_kernels.h - FP64 kernels around the FP32 solve for iterative
// refinement: seven-point residual (Eq. (poi), finite-volume rows on the
// non-uniform axis), solution update, width-weighted means, and the norms
// that decide when to stop.  All reductions are fixed-order (per-block
// partial sums, then one block adding the partials in index order), so a
// result does not depend on scheduling.
//
// Device status block (doubles):
//   [0] skip flag (1 once refinement has converged: later sweeps return)
//   [1] weighted mean of Phi after the last update that ran (singular plans)
//   [2] converged flag
//   [3] relative update of the previous sweep
//   [4 + 2s], [5 + 2s]: ||e_s||^2 and ||Phi_s||^2 of sweep s (-1 if not run)
//   [REFINE_PARTIALS ...]: per-block partial sums (3 per block: ||e||^2,
//   ||Phi||^2 and the weighted sum of f or Phi)
//
// Bound: HBM.  The sweeps move pairs of neighbouring x points (16-byte
// accesses; single points where nx is odd) with several pairs of a thread in
// flight, and no sweep reads a field only to sum it where another one holds
// it already: the gauge's mean of Phi comes from the last update.  Measured
// on the 512 x 256 x 192 channel (singular), before -> after: mean of f 56 -> 31
// us, copy and cast 94 -> 85, residual 154 -> 112, update 84 -> 76, gauge 114 ->
// 57, four launches fewer; the refined solve 992 -> 844 us.
#pragma once
#include <algorithm>
#include <type_traits>

#include "device_common.h"

namespace poisson_dev {

static constexpr int REFINE_MAX_SWEEPS = 64;
static constexpr int REFINE_BLOCKS = 1024;
static constexpr int REFINE_NT = 256;
static constexpr int REFINE_PARTIALS = 4 + 2 * REFINE_MAX_SWEEPS + 8;
static constexpr int REFINE_STAT_SLOTS = REFINE_PARTIALS + 2 * REFINE_BLOCKS;
// Blocks of the element-wise sweeps: two per CU (more would only lengthen the
// partial sums that every block of the next sweep adds up).
static constexpr int REFINE_EBLOCKS = 512;
static_assert(3 * REFINE_EBLOCKS <= 2 * REFINE_BLOCKS, "three partial sums per block");

struct OpAxis {            // one axis of the operator: rows a, b, c and widths h
  const double* a;
  const double* b;
  const double* c;
  const double* h;
  int n;
};

struct RefineGeom {
  OpAxis ax[3];            // x, y, z
  long long npts;
  double* stats;
  double weight;           // total of the weights: nx ny times the sum of the z widths
};

__device__ __forceinline__ bool refine_skip(const double* stats) { return stats[0] != 0.0; }

// Sums over the block (fixed order), on every thread.
template <int NT>
__device__ __forceinline__ double block_sum(double a, double* sh) {
  const int tid = threadIdx.x;
  __syncthreads();
  sh[tid] = a;
  __syncthreads();
  for (int s = NT / 2; s > 0; s >>= 1) {
    if (tid < s) sh[tid] += sh[tid + s];
    __syncthreads();
  }
  return sh[0];
}

// Sum of partial sum `slot` over the blocks of a sweep.
__device__ __forceinline__ double refine_partials(const double* stats, int slot, int nblocks,
                                                  double* sh) {
  double a = 0.0;
  for (int i = threadIdx.x; i < nblocks; i += REFINE_NT) a += stats[REFINE_PARTIALS + 3 * i + slot];
  return block_sum<REFINE_NT>(a, sh);
}

// The thread's runs of V points of a field, U runs in flight: body(q, count)
// handles the runs q, q + step, ... (count of them; run q starts at point V q).
template <int V, int U, typename F>
__device__ __forceinline__ void refine_runs(long long npts, int block, int nblocks, F&& body) {
  const long long n = npts / V, step = (long long)nblocks * REFINE_NT;
  long long q = block * (long long)REFINE_NT + threadIdx.x;
  for (; q + (U - 1) * step < n; q += U * step) body(q, step, std::integral_constant<int, U>{});
  for (; q < n; q += step) body(q, step, std::integral_constant<int, 1>{});
}

// Grid position (i, j, k) of point idx, advanced by a fixed step without
// 64-bit divisions in the loop (only the set-up divides).
struct GridWalk {
  int i, j, k, di, dj, dk, nx, ny;
  __device__ GridWalk(long long idx, long long step, int nx_, int ny_) : nx(nx_), ny(ny_) {
    const long long plane = (long long)nx * ny;
    k = (int)(idx / plane);
    const int r = (int)(idx - k * plane);
    j = r / nx;
    i = r - j * nx;
    dk = (int)(step / plane);
    const int rs = (int)(step - dk * plane);
    dj = rs / nx;
    di = rs - dj * nx;
  }
  __device__ void advance() {
    i += di;
    int cj = 0;
    if (i >= nx) { i -= nx; cj = 1; }
    j += dj + cj;
    int ck = 0;
    if (j >= ny) { j -= ny; ck = 1; }
    k += dk + ck;
  }
};

// z index of the thread's successive runs (refine_runs order)
struct PlaneWalk {
  int k;
  long long r, dr, plane;
  int dk;
  __device__ PlaneWalk(long long point, long long step, long long plane_) : plane(plane_) {
    k = (int)(point / plane);
    r = point - k * plane;
    dk = (int)(step / plane);
    dr = step - dk * plane;
  }
  __device__ void advance() {
    r += dr;
    const bool carry = r >= plane;
    r -= carry ? plane : 0;
    k += dk + (carry ? 1 : 0);
  }
};

// Each kernel below is a device body over a block range, called by a
// kernel for one plan (blockIdx / gridDim) and by a batched kernel that
// runs the same body for every instance of a batch, each on its own block
// range (same blocks, same reduction order: bitwise the same result).

// reset the status block (a fill kernel rather than a memset, so the
// sequence can be captured in a graph)
__device__ __forceinline__ void refine_init_body(double* stats) {
  for (int i = threadIdx.x; i < REFINE_PARTIALS; i += blockDim.x) stats[i] = i >= 4 ? -1.0 : 0.0;
}

// Run q of V points, with the nontemporal hint (NT) or without.  The
// single-plan kernels take the hint on fields of 512 MiB and more: on the
// 512^3 cube the refined solve went 4.51-4.52 -> 4.44-4.46 ms with it;
// the batched kernels (many small instances) keep plain accesses.
template <bool NT, typename T, int V>
__device__ __forceinline__ void refine_ld(const T* p, long long q, T (&x)[V]) {
  using W = T __attribute__((ext_vector_type(V)));
  const W* w = reinterpret_cast<const W*>(p) + q;
  W t;
  if constexpr (NT) t = __builtin_nontemporal_load(w);
  else t = *w;
#pragma unroll
  for (int i = 0; i < V; ++i) x[i] = t[i];
}
template <bool NT, typename T, int V>
__device__ __forceinline__ void refine_st(T* p, long long q, const T (&x)[V]) {
  using W = T __attribute__((ext_vector_type(V)));
  W* w = reinterpret_cast<W*>(p) + q;
  W t;
#pragma unroll
  for (int i = 0; i < V; ++i) t[i] = x[i];
  if constexpr (NT) __builtin_nontemporal_store(t, w);
  else *w = t;
}

// partial weighted sums (slot 2) of x; the weights are the z widths (x and y
// are uniform)
template <int V>
__device__ __forceinline__ void refine_wsum_body(const double* __restrict__ x, const RefineGeom& G,
                                                 int block, int nblocks, double* sh) {
  double sx = 0.0;
  PlaneWalk at((block * (long long)REFINE_NT + threadIdx.x) * V, (long long)nblocks * REFINE_NT * V,
               (long long)G.ax[0].n * G.ax[1].n);
  refine_runs<V, 4>(G.npts, block, nblocks, [&](long long q, long long step, auto U) {
    double v[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u) refine_ld<false>(x, q + u * step, v[u]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      double t = 0.0;
#pragma unroll
      for (int i = 0; i < V; ++i) t += v[u][i];
      sx += G.ax[2].h[at.k] * t;
      at.advance();
    }
  });
  sx = block_sum<REFINE_NT>(sx, sh);
  if (threadIdx.x == 0) G.stats[REFINE_PARTIALS + 3 * block + 2] = sx;
}

// f64 = rhs - mean (the weighted mean of the partial sums, if `project`), e32 =
// (float) f64
template <bool NT, int V>
__device__ __forceinline__ void refine_prep_body(const double* __restrict__ rhs,
                                                 double* __restrict__ f64, float* __restrict__ e32,
                                                 const RefineGeom& G, int project, int block,
                                                 int nblocks, double* sh) {
  const double mean = project ? refine_partials(G.stats, 2, nblocks, sh) / G.weight : 0.0;
  refine_runs<V, 2>(G.npts, block, nblocks, [&](long long q, long long step, auto U) {
    double f[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u) refine_ld<NT>(rhs, q + u * step, f[u]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float e[V];
#pragma unroll
      for (int i = 0; i < V; ++i) {
        f[u][i] -= mean;
        e[i] = (float)f[u][i];
      }
      refine_st<NT>(f64, q + u * step, f[u]);
      refine_st<NT>(e32, q + u * step, e);
    }
  });
}

// x -= its weighted mean: stats[1], or (`summed`) that of the partial sums
template <int V>
__device__ __forceinline__ void refine_shift_body(double* __restrict__ x, const RefineGeom& G,
                                                  int summed, int block, int nblocks, double* sh) {
  const double mean = summed ? refine_partials(G.stats, 2, nblocks, sh) / G.weight : G.stats[1];
  refine_runs<V, 2>(G.npts, block, nblocks, [&](long long q, long long step, auto U) {
    double f[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u) refine_ld<false>(x, q + u * step, f[u]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int i = 0; i < V; ++i) f[u][i] -= mean;
      refine_st<false>(x, q + u * step, f[u]);
    }
  });
}

// phi += e; per-block partial ||e||^2, ||phi||^2 and weighted sum of phi
template <bool NT, int V>
__device__ __forceinline__ void refine_update_body(double* __restrict__ phi,
                                                   const float* __restrict__ e32,
                                                   const RefineGeom& G, int block, int nblocks,
                                                   double* sh) {
  if (refine_skip(G.stats)) return;
  double se = 0.0, sp = 0.0, sx = 0.0;
  PlaneWalk at((block * (long long)REFINE_NT + threadIdx.x) * V, (long long)nblocks * REFINE_NT * V,
               (long long)G.ax[0].n * G.ax[1].n);
  refine_runs<V, 2>(G.npts, block, nblocks, [&](long long q, long long step, auto U) {
    float e[U][V];
    double x[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      refine_ld<NT>(e32, q + u * step, e[u]);
      refine_ld<NT>(phi, q + u * step, x[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      double t = 0.0;
#pragma unroll
      for (int i = 0; i < V; ++i) {
        const double d = (double)e[u][i];
        x[u][i] += d;
        se += d * d;
        sp += x[u][i] * x[u][i];
        t += x[u][i];
      }
      refine_st<NT>(phi, q + u * step, x[u]);
      sx += G.ax[2].h[at.k] * t;
      at.advance();
    }
  });
  se = block_sum<REFINE_NT>(se, sh);
  sp = block_sum<REFINE_NT>(sp, sh);
  sx = block_sum<REFINE_NT>(sx, sh);
  if (threadIdx.x == 0) {
    G.stats[REFINE_PARTIALS + 3 * block] = se;
    G.stats[REFINE_PARTIALS + 3 * block + 1] = sp;
    G.stats[REFINE_PARTIALS + 3 * block + 2] = sx;
  }
}

// Record sweep `sweep`: rel = ||e|| / ||phi||; the error left after the
// update is estimated from the contraction rho = rel / rel_prev as
// rel * rho / (1 - rho) (rel_prev = 1 at the first sweep, whose correction
// measures the first FP32 solve's error); once that is <= tol / 10 the
// remaining sweeps are skipped.  The margin covers a contraction that
// differs between sweeps: the residual's spectrum is not f's, so the FP32
// solve of a correction can be several times less accurate than the first.
__device__ __forceinline__ void refine_status_body(const RefineGeom& G, int nblocks, int sweep,
                                                   double tol, double* sh) {
  double* stats = G.stats;
  if (refine_skip(stats)) return;
  const double a = refine_partials(stats, 0, nblocks, sh);
  const double b = refine_partials(stats, 1, nblocks, sh);
  const double x = refine_partials(stats, 2, nblocks, sh);
  if (threadIdx.x == 0) {
    stats[1] = x / G.weight;
    stats[4 + 2 * sweep] = a;
    stats[5 + 2 * sweep] = b;
    const double rel = b > 0.0 ? sqrt(a / b) : 0.0;
    const double prev = stats[3] > 0.0 ? stats[3] : 1.0;
    const double rho = rel / prev;
    const double est = rho < 1.0 ? rel * rho / (1.0 - rho) : rel;
    stats[3] = rel;
    if (est <= 0.1 * tol) {
      stats[2] = 1.0;
      stats[0] = 1.0;
    }
  }
}

// Launch shape of refine_residual_kernel: blocks of REFINE_NT runs of v points,
// 2^logtx runs along x by REFINE_NT / 2^logtx rows, each marching through `kz`
// consecutive planes; `blocks` is the block count rounded up to a multiple of
// 8 (see refine_residual_kernel).
struct ResidualGrid {
  int logtx, tiles_x, plane_blocks, kz, z_chunks, blocks;
};

inline ResidualGrid residual_grid(int nx, int ny, int nz, int v) {
  ResidualGrid r;
  r.logtx = 0;
  while (r.logtx < 6 && (v << r.logtx) < nx) ++r.logtx;
  const int rows = REFINE_NT >> r.logtx;
  r.tiles_x = (nx / v + (1 << r.logtx) - 1) >> r.logtx;
  r.plane_blocks = r.tiles_x * ((ny + rows - 1) / rows);
  // about two blocks per CU in all, at least 4 planes each: with the next plane
  // read ahead, long marches gain more than more waves (channel 512 x 256 x
  // 192: 512 blocks 112 us, 1024 125 us)
  r.kz = (int)std::max<long long>(4, ((long long)nz * r.plane_blocks + 511) / 512);
  r.kz = std::min(r.kz, nz);
  r.z_chunks = (nz + r.kz - 1) / r.kz;
  r.blocks = (r.plane_blocks * r.z_chunks + 7) / 8 * 8;
  return r;
}

// e32 = (float)(f64 - A phi), FP64 arithmetic.  One thread per V neighbouring x
// points, marching through kz planes with phi of the planes below, at and
// above in registers (each phi value is read from HBM about once; its x and
// y neighbours come from the caches: six loads for two points, where single
// points take twelve), the next plane's values read while the current one is
// computed.  A block covers several rows, so that most rows are fetched into
// its CU once and not three times.  The 8 XCDs receive consecutive
// blocks round-robin: block b works on chunk (b mod 8) * (blocks / 8) +
// b / 8, so each XCD sweeps a contiguous run of rows, whose y neighbours its
// own L2 holds.
template <bool NT, int V>
__device__ __forceinline__ void refine_residual_body(const double* __restrict__ phi,
                                                     const double* __restrict__ f64,
                                                     float* __restrict__ e32, const RefineGeom& G,
                                                     const ResidualGrid& rg, int block) {
  if (refine_skip(G.stats)) return;
  const int chunk = (block % 8) * (rg.blocks / 8) + block / 8;
  if (chunk >= rg.plane_blocks * rg.z_chunks) return;
  const int nx = G.ax[0].n, ny = G.ax[1].n, nz = G.ax[2].n;
  const int zc = chunk / rg.plane_blocks, pb = chunk - zc * rg.plane_blocks;
  const int ty = pb / rg.tiles_x, tx = pb - ty * rg.tiles_x;
  const int i = ((tx << rg.logtx) + ((int)threadIdx.x & ((1 << rg.logtx) - 1))) * V;
  const int j = ty * (REFINE_NT >> rg.logtx) + ((int)threadIdx.x >> rg.logtx);
  if (i >= nx || j >= ny) return;
  const int p = j * nx + i;
  const int k0 = zc * rg.kz;
  const int k1 = min(k0 + rg.kz, nz);
  const OpAxis& X = G.ax[0];
  const OpAxis& Y = G.ax[1];
  const OpAxis& Z = G.ax[2];
  // a_q phi_{q-1} + b_q phi_q + c_q phi_{q+1} per axis; a_0 / c_{n-1} are
  // the periodic wrap couplings (zero at a wall, where the ghost rule is in b)
  double ax[V], bx[V], cx[V];
#pragma unroll
  for (int t = 0; t < V; ++t) {
    ax[t] = X.a[i + t];
    bx[t] = X.b[i + t];
    cx[t] = X.c[i + t];
  }
  const double ay = Y.a[j], by = Y.b[j], cy = Y.c[j];
  const int xl = (i > 0 ? i - 1 : nx - 1) - i, xh = (i + V < nx ? i + V : 0) - i;
  const int yl = ((j > 0 ? j - 1 : ny - 1) - j) * nx, yh = ((j < ny - 1 ? j + 1 : 0) - j) * nx;
  const long long plane = (long long)nx * ny;
  // run at point offset o (a multiple of V)
  auto run = [&](long long o, double (&v)[V]) { refine_ld<false>(phi + o, 0, v); };
  double below[V], at[V];
  run((k0 > 0 ? k0 - 1 : nz - 1) * plane + p, below);
  run(k0 * plane + p, at);
  struct Plane {
    double above[V], south[V], north[V], f[V], west, east;
  };
  auto read = [&](int k, Plane& q) {
    const long long o = k * plane + p;
    run(k < nz - 1 ? o + plane : (long long)p, q.above);
    q.west = phi[o + xl];
    q.east = phi[o + xh];
    run(o + yl, q.south);
    run(o + yh, q.north);
    refine_ld<NT>(f64 + o, 0, q.f);
  };
  Plane cur, nxt;
  read(k0, cur);
  for (int k = k0; k < k1; ++k) {
    const long long o = k * plane + p;
    read(min(k + 1, k1 - 1), nxt);
    const double za = Z.a[k], zb = Z.b[k], zcc = Z.c[k];
    float e[V];
#pragma unroll
    for (int t = 0; t < V; ++t) {
      const double opx = ax[t] * (t > 0 ? at[t - 1] : cur.west) + bx[t] * at[t] +
                         cx[t] * (t < V - 1 ? at[t + 1] : cur.east);
      const double opy = ay * cur.south[t] + by * at[t] + cy * cur.north[t];
      const double opz = za * below[t] + zb * at[t] + zcc * cur.above[t];
      e[t] = (float)(cur.f[t] - ((opx + opy) + opz));
    }
    refine_st<NT>(e32 + o, 0, e);
#pragma unroll
    for (int t = 0; t < V; ++t) {
      below[t] = at[t];
      at[t] = cur.above[t];
    }
    cur = nxt;
  }
}

// ---- kernels for one plan (V points per access: 2 where nx is even, else 1)

// the weighted sums of f; block 0 resets the status block
template <int V>
__global__ __launch_bounds__(REFINE_NT) void refine_wsum_kernel(const double* __restrict__ x,
                                                                 RefineGeom G, int init) {
  __shared__ double sh[REFINE_NT];
  if (init && blockIdx.x == 0) refine_init_body(G.stats);
  refine_wsum_body<V>(x, G, blockIdx.x, gridDim.x, sh);
}

// ... and so does the copy of f of a regular plan
template <bool NT, int V>
__global__ __launch_bounds__(REFINE_NT) void refine_prep_kernel(const double* __restrict__ rhs,
                                                                 double* __restrict__ f64,
                                                                 float* __restrict__ e32,
                                                                 RefineGeom G, int project) {
  __shared__ double sh[REFINE_NT];
  if (!project && blockIdx.x == 0) refine_init_body(G.stats);
  refine_prep_body<NT, V>(rhs, f64, e32, G, project, blockIdx.x, gridDim.x, sh);
}

template <int V>
__global__ __launch_bounds__(REFINE_NT) void refine_shift_kernel(double* __restrict__ x,
                                                                  RefineGeom G, int summed) {
  __shared__ double sh[REFINE_NT];
  refine_shift_body<V>(x, G, summed, blockIdx.x, gridDim.x, sh);
}

// e32 = (float)(f64 - A phi), FP64 arithmetic (see refine_residual_body)
template <bool NT, int V>
__global__ __launch_bounds__(REFINE_NT) void refine_residual_kernel(const double* __restrict__ phi,
                                                                     const double* __restrict__ f64,
                                                                     float* __restrict__ e32,
                                                                     RefineGeom G, ResidualGrid rg) {
  refine_residual_body<NT, V>(phi, f64, e32, G, rg, blockIdx.x);
}

template <bool NT, int V>
__global__ __launch_bounds__(REFINE_NT) void refine_update_kernel(double* __restrict__ phi,
                                                                   const float* __restrict__ e32,
                                                                   RefineGeom G) {
  __shared__ double sh[REFINE_NT];
  refine_update_body<NT, V>(phi, e32, G, blockIdx.x, gridDim.x, sh);
}

__global__ __launch_bounds__(REFINE_NT) void refine_status_kernel(RefineGeom G, int nblocks,
                                                                   int sweep, double tol) {
  __shared__ double sh[REFINE_NT];
  refine_status_body(G, nblocks, sweep, tol, sh);
}

// ---- kernels for a batch: job j owns blocks [first, first + count) of a
// launch (element-wise kernels: nb blocks; residual: rg.blocks, a multiple
// of 8 starting at a multiple of 8, so its XCD order is kept); reductions
// and per-instance steps take one block per job.

struct RefineJob {
  RefineGeom G;
  double* phi;          // the caller's field (Phi, and f on entry)
  double* f64;
  float* e32;
  int singular;
  int vec;              // points per access (2 or 1)
  int nb;               // blocks of the element-wise kernels
  ResidualGrid rg;
  int first_e;          // first block in the element-wise launches
  int first_r;          // first block in the residual launch
  int max_iters;
  double tol;
};

// job of block `b` (jobs sorted by first block, the first one at 0)
template <bool RESIDUAL>
__device__ __forceinline__ int refine_job_of(const RefineJob* __restrict__ jobs, int njobs, int b) {
  int lo = 0, hi = njobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if ((RESIDUAL ? jobs[mid].first_r : jobs[mid].first_e) <= b) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// f(points per access) of an instance, as a constant
template <typename F>
__device__ __forceinline__ void refine_width(const RefineJob& J, F&& f) {
  if (J.vec == 2) f(std::integral_constant<int, 2>{});
  else f(std::integral_constant<int, 1>{});
}

// An instance that ran its first FP32 solve only has no update to take Phi's
// mean from: then Phi is summed.  Read off the status block, since an
// instance's limit and the launch's sweeps may have been set at different times.
__device__ __forceinline__ bool refine_no_update(const double* stats) { return stats[4 + 2] < 0.0; }

// the projection of f and the gauge of Phi touch singular instances only
__global__ __launch_bounds__(REFINE_NT) void refine_batch_wsum(const RefineJob* __restrict__ jobs,
                                                                int njobs, int init) {
  __shared__ double sh[REFINE_NT];
  const RefineJob& J = jobs[refine_job_of<false>(jobs, njobs, blockIdx.x)];
  if (!J.singular || (!init && !refine_no_update(J.G.stats))) return;
  const int block = blockIdx.x - J.first_e;
  if (init && block == 0) refine_init_body(J.G.stats);
  refine_width(J, [&](auto V) { refine_wsum_body<V>(J.phi, J.G, block, J.nb, sh); });
}

__global__ __launch_bounds__(REFINE_NT) void refine_batch_prep(const RefineJob* __restrict__ jobs,
                                                                int njobs) {
  __shared__ double sh[REFINE_NT];
  const RefineJob& J = jobs[refine_job_of<false>(jobs, njobs, blockIdx.x)];
  const int block = blockIdx.x - J.first_e;
  if (!J.singular && block == 0) refine_init_body(J.G.stats);
  refine_width(J, [&](auto V) {
    refine_prep_body<false, V>(J.phi, J.f64, J.e32, J.G, J.singular, block, J.nb, sh);
  });
}

// sweep `sweep`: the residual, or the stop of an instance at its limit
__global__ __launch_bounds__(REFINE_NT) void refine_batch_residual(const RefineJob* __restrict__ jobs,
                                                                    int njobs, int sweep) {
  const RefineJob& J = jobs[refine_job_of<true>(jobs, njobs, blockIdx.x)];
  const int block = blockIdx.x - J.first_r;
  if (sweep >= J.max_iters) {
    if (block == 0 && threadIdx.x == 0) J.G.stats[0] = 1.0;
    return;
  }
  refine_width(J, [&](auto V) { refine_residual_body<false, V>(J.phi, J.f64, J.e32, J.G, J.rg, block); });
}

__global__ __launch_bounds__(REFINE_NT) void refine_batch_update(const RefineJob* __restrict__ jobs,
                                                                  int njobs) {
  __shared__ double sh[REFINE_NT];
  const RefineJob& J = jobs[refine_job_of<false>(jobs, njobs, blockIdx.x)];
  refine_width(J, [&](auto V) {
    refine_update_body<false, V>(J.phi, J.e32, J.G, blockIdx.x - J.first_e, J.nb, sh);
  });
}

__global__ __launch_bounds__(REFINE_NT) void refine_batch_status(const RefineJob* __restrict__ jobs,
                                                                  int sweep) {
  __shared__ double sh[REFINE_NT];
  const RefineJob& J = jobs[blockIdx.x];
  refine_status_body(J.G, J.nb, sweep, J.tol, sh);
}

__global__ __launch_bounds__(REFINE_NT) void refine_batch_shift(const RefineJob* __restrict__ jobs,
                                                                 int njobs) {
  __shared__ double sh[REFINE_NT];
  const RefineJob& J = jobs[refine_job_of<false>(jobs, njobs, blockIdx.x)];
  if (!J.singular) return;
  refine_width(J, [&](auto V) {
    refine_shift_body<V>(J.phi, J.G, refine_no_update(J.G.stats), blockIdx.x - J.first_e, J.nb, sh);
  });
}

}  // namespace poisson_dev
