// tri_line.h - elimination of the reduced systems of Eq. (poi_reduced) for
// lines of any length 17 <= n <= 512 (also those with variants, where the lines
// are strided and nothing was tuned or set): n = RPC P - m rows in P chunks, the
// first m < P chunks one row shorter than the others.
//
// The same chunked elimination as tri_fast.h (tri_line_solve), with a short
// chunk's missing row carried along as an alias of the unknown before it, so
// that every loop bound is still a compile-time constant.  Unlike a line
// padded at its end, the first and the last row stay where the cyclic
// coupling and the pinned unknown need them: periodic and singular lines take
// this form too, and a line of n points costs at most one row per chunk more
// than its own.
//
// The pivots are formed from the row sums a + b + c (tri_line_solve, RAG)
// without cancellation: over 17 lengths, uniform and stretched, four shifts, a
// line's error against extended precision is 0.29 of the size-generic
// kernel's (geometric mean).  Whole solves (P, P, NN, stretched, 512 x 256 x
// 144): 9.6e-14 -> 6.0e-14.
//
// Bound: HBM (16 B per point in FP64) up to 352 rows; beyond, the 128-byte
// rows of its 16-line tiles and the longer reduction.  What makes the
// difference to the other eliminations, on 512 x ny x n fields of 2^25 points:
//  * rows of a chunk in order on one thread, so that no element needs a
//    division or a 64-bit product (n = 144, 16 lanes: 4.4 -> 5.0 TB/s);
//  * the interface reduction ends when its couplings have vanished (pcr,
//    EXIT: n = 144 5.0 -> 6.2, n = 250 4.3 -> 4.8);
//  * few lanes with long chunks, as many rows as registers allow at 2, 3 or 4
//    waves per SIMD: the reduction costs the same for a chunk of any length
//    (n = 50 in 8 lanes 5.1, in 4 lanes 5.9; n = 250 in 32 lanes of 8 rows
//    4.8, in 16 lanes of 16 rows 6.0).
#pragma once
#include "tri_fast.h"

namespace poisson_dev {

// Chunking of lines of n points (p = 0: none): rpc rows per chunk, p chunks
// (lanes) per line, nl lines per tile, nl * p threads, registers for `waves`
// waves per SIMD.  A lane holds its rows, pivots, spikes and the next tile's
// rows: 11 rows fit 128 registers, 12 a third of the 512 (p = 8, p = 4 and
// 16 rows of p = 16 as well).  Lengths 177-192 and 353-512 give up occupancy for
// the wide tile (n = 190: 256-byte rows 5.5-6.1 TB/s, 128-byte rows 5.4-5.7; n =
// 400 on fields past the 256 MB cache: 16 lines 4.0-4.4, 8 lines 3.2-3.5).
struct TriLineShape {
  int rpc, p, nl, waves;
};
constexpr TriLineShape tri_line_shape(int n) {
  const TriLineShape s = n < 17    ? TriLineShape{0, 0, 0, 0}
                         : n <= 48  ? TriLineShape{0, 4, 64, 3}
                         : n <= 96  ? TriLineShape{0, 8, 32, 3}
                         : n <= 176 ? TriLineShape{0, 16, 32, 4}
                         : n <= 192 ? TriLineShape{0, 16, 32, 2}
                         : n <= 256 ? TriLineShape{0, 16, 16, 3}
                         : n <= 352 ? TriLineShape{0, 32, 16, 4}
                         : n <= 512 ? TriLineShape{0, 32, 16, 2}
                                    : TriLineShape{0, 0, 0, 0};
  return TriLineShape{s.p ? (n + s.p - 1) / s.p : 0, s.p, s.nl, s.waves};
}

template <typename T, int RPC, int P, int NL_>
struct TriLineLayout {
  static constexpr int NL = NL_, NT = NL * P, N = RPC * P;
  static constexpr int NLP = NL + 1;          // row pitch
  static constexpr int CP = (RPC * NLP) | 1;  // chunk pitch (odd)
  static constexpr size_t COEF = ((size_t)P * CP * sizeof(T) + 15) / 16 * 16;
  static constexpr size_t BYTES = COEF + (size_t)4 * N * sizeof(double);
};

// Virtual row k (chunk k / RPC, row k mod RPC of it) of a line whose first m
// chunks have no row 0.
struct TriRow {
  int p;         // its point; a missing row repeats a neighbour's
  int k;         // the virtual row that holds that point
  bool missing;
};
// k / RPC for k < 512 (exact: 512 (RPC - 1) < 2^16), with a 24-bit product
template <int RPC>
__device__ __forceinline__ int tri_chunk(int k) {
  return (int)(__umul24((unsigned)k, (65536u + RPC - 1) / RPC) >> 16);
}
template <int RPC>
__device__ __forceinline__ TriRow tri_row(int k, int m) {
  const int ch = tri_chunk<RPC>(k);
  TriRow r;
  r.missing = k == ch * RPC && ch < m;
  r.p = max(k - min(ch + 1, m), 0);
  r.k = r.missing ? (k == 0 ? 1 : k - 1) : k;
  return r;
}

template <typename T, int RPC, int P, int NL_, int WAVES, int LAYOUT>
__global__ __launch_bounds__(NL_ * P, WAVES)
void tri_line_kernel(TriFastArgs<T> A) {
  using L = TriLineLayout<T, RPC, P, NL_>;
  constexpr int N = L::N, NL = L::NL, NT = L::NT;
  if (A.skip && A.skip[0] != 0.0) return;
  __shared__ __align__(16) unsigned char smem_raw[L::BYTES];
  const lptr<T> lds = as_lds(reinterpret_cast<T*>(smem_raw));
  const lptr<double> coef =
      as_lds(reinterpret_cast<double*>(smem_raw + L::COEF));
  const int tid0 = threadIdx.x;
  const int m = N - A.nreal;
  LineGeom g = A.g;
  g.layout = LAYOUT;
  const int nlt = 1 << g.lognl;
  for (int k = tid0; k < N; k += NT) {
    const int ch = k / RPC, i = k - ch * RPC, s = i * P + ch;
    coef[s] = as_global(A.a)[k];
    coef[N + s] = as_global(A.b)[k];
    coef[2 * N + s] = as_global(A.c)[k];
    coef[3 * N + s] = as_global(A.w)[k];
  }
  const gptr<T> data = as_global(A.data);
  const TileRange tr = xcd_tiles(g.ntiles);
  // LDS slot of virtual row k (line 0)
  auto slot = [](int k) {
    const int ch = tri_chunk<RPC>(k);
    return ch * L::CP + (k - ch * RPC) * L::NLP;
  };

  // Lanes past the end of the field repeat a valid line (the same values to
  // the same addresses), and a missing row its neighbour, so no load and no
  // store sits behind a branch, and the compiler can count the operations in
  // flight.
  //
  // Strided: thread tid moves the rows of chunk tid / NL of line tid mod NL in
  // order, so that addresses and LDS slots advance by uniform steps.
  struct Strided {
    gptr<T> row0;     // point of virtual row 0 of the chunk
    long long off0;   // ... moved to the point that a missing row 0 repeats
    lptr<T> col;
    lptr<T> alias;    // slot holding that point
    bool missing;
  };
  auto strided = [&](const TileOrigin& o, int tid) {
    const int l = tid % NL, ch = tid / NL;
    const int lm = l & (nlt - 1);
    const int x = min(o.x0 + (lm & ((1 << g.logtxw) - 1)), g.nx - 1);
    const int b = min(o.b0 + (lm >> g.logtxw), g.nb - 1);
    const int r0 = ch * RPC - min(ch + 1, m);
    Strided t;
    t.row0 = data + (x + (long long)b * g.sb + r0 * g.sp);
    t.col = lds + ch * L::CP + l;
    t.missing = ch < m;
    t.off0 = r0 < 0 ? g.sp : 0;
    t.alias = !t.missing ? t.col : ch == 0 ? t.col + L::NLP : t.col - L::CP + (RPC - 1) * L::NLP;
    return t;
  };
  // Contiguous: thread tid moves the virtual rows c + i P of line tid / P
  // (c = tid mod P): P consecutive points of a line on consecutive lanes.
  struct Contiguous {
    gptr<T> line;
    lptr<T> col;
  };
  auto contiguous = [&](const TileOrigin& o, int tid) {
    const int l = tid / P;
    return Contiguous{data + (long long)min(o.L0 + min(l, nlt - 1), g.nlines - 1) * A.nreal, lds + l};
  };
  // The next tile and its lines' eigenvalue shifts are read before the current
  // tile's stores are issued and placed after them, at the bottom of the loop.
  T buf[RPC];
  double lu = 0.0, lv = 0.0;
  bool sing_n = false;
  auto fetch = [&](int tile, int tid) {
    const TileOrigin o = tile_origin(g, tile);
    if constexpr (LAYOUT == 0) {
      const Strided t = strided(o, tid);
      buf[0] = t.row0[t.off0];
#pragma unroll
      for (int i = 1; i < RPC; ++i) buf[i] = t.row0[i * g.sp];
    } else {
      const Contiguous t = contiguous(o, tid);
#pragma unroll
      for (int i = 0; i < RPC; ++i) buf[i] = t.line[tri_row<RPC>(tid % P + i * P, m).p];
    }
    // the line that this thread helps to eliminate (repeated as above)
    const int l = tid / P;
    int u, v;
    if constexpr (LAYOUT == 0) {
      const int lm = l & (nlt - 1);
      u = min(o.x0 + (lm & ((1 << g.logtxw) - 1)), g.nx - 1);
      v = min(o.b0 + (lm >> g.logtxw), g.nb - 1);
    } else {
      const int line = min(o.L0 + min(l, nlt - 1), g.nlines - 1);
      v = line / A.nu;
      u = line - v * A.nu;
    }
    lu = as_global(A.lamu)[u];
    lv = as_global(A.lamv)[v];
    sing_n = A.singular && u == 0 && v == 0;
  };
  double mu = 0.0;
  bool sing = false;
  auto place = [&](int tile, int tid) {
    const TileOrigin o = tile_origin(g, tile);
    if constexpr (LAYOUT == 0) {
      const Strided t = strided(o, tid);
      t.col[0] = t.missing ? (T)0 : buf[0];
#pragma unroll
      for (int i = 1; i < RPC; ++i) t.col[i * L::NLP] = buf[i];
    } else {
      const Contiguous t = contiguous(o, tid);
#pragma unroll
      for (int i = 0; i < RPC; ++i) {
        const int k = tid % P + i * P;
        t.col[slot(k)] = tri_row<RPC>(k, m).missing ? (T)0 : buf[i];
      }
    }
    mu = lu + lv;
    sing = sing_n;
  };
  if (tr.first < tr.end) {
    fetch(tr.first, tid0);
    place(tr.first, tid0);
  }
  for (int tile = tr.first; tile < tr.end; tile += tr.step) {
    // thread index opaque per step: addresses are recomputed, not held
    int tid = tid0;
    asm volatile("" : "+v"(tid));
    lds_barrier();
    const bool more = tile + tr.step < tr.end;
    if (more) fetch(tile + tr.step, tid);
    asm volatile("" : "+v"(tid));
    const int c = tid % P, l = tid / P;
    const int wave_sing = __any(sing) ? 1 : 0;
    const lptr<T> col = lds + c * L::CP + l;
    double xr[RPC];
#pragma unroll
    for (int i = 0; i < RPC; ++i) xr[i] = (double)col[i * L::NLP];
    // (long chunks: each row's coefficient reads stay in its own step, or
    // they would all be live at once)
    tri_line_solve<RPC, P, (RPC >= 9), true>([&](int i) -> double { return xr[i]; },
                                             [&](int i, double x) { xr[i] = x; }, coef, c, mu,
                                             sing ? 1 : 0, wave_sing, A.periodic, c < m);
#pragma unroll
    for (int i = 0; i < RPC; ++i) col[i * L::NLP] = (T)xr[i];
    lds_barrier();
    asm volatile("" : "+v"(tid));
    {
      const TileOrigin o = tile_origin(g, tile);
      T out[RPC];
      if constexpr (LAYOUT == 0) {
        const Strided t = strided(o, tid);
        out[0] = t.alias[0];
#pragma unroll
        for (int i = 1; i < RPC; ++i) out[i] = t.col[i * L::NLP];
        t.row0[t.off0] = out[0];
#pragma unroll
        for (int i = 1; i < RPC; ++i) t.row0[i * g.sp] = out[i];
      } else {
        const Contiguous t = contiguous(o, tid);
#pragma unroll
        for (int i = 0; i < RPC; ++i) out[i] = t.col[slot(tri_row<RPC>(tid % P + i * P, m).k)];
#pragma unroll
        for (int i = 0; i < RPC; ++i) t.line[tri_row<RPC>(tid % P + i * P, m).p] = out[i];
      }
    }
    lds_barrier();
    asm volatile("" : "+v"(tid));
    if (more) place(tile + tr.step, tid);
  }
}

}  // namespace poisson_dev
