// r2r_line.h - the batched real-to-real transforms (Table 2 / Table 1) for
// every supported length n = 2M with 12 <= M <= 512 (M = 2^a 3^b 5^c) but n =
// 512, each length compiled with its own radices, tile and loop bounds.
//
// Same mathematics as r2r_kernel.h: one complex FFT of length M per line and
// the pre/post steps of the type.  What differs from that size-generic
// kernel, and why:
//  * the next tile's values are read into registers while the current tile is
//    transformed and stored, so the memory system never waits for the FFT;
//  * every step around the FFT runs on data that moves anyway: the inverse
//    real-DFT / DCT-II / DST-II combine as the tile is placed, the DCT-IV
//    pre-twiddle as the first pass reads its inputs, the forward split and
//    the DCT-IV post-twiddle as the tile is stored.  The FFT passes are the
//    only other LDS round trips, two of them up to M = 256 and three beyond;
//  * no lane skips a load or a store: lanes past the end of a line and lines
//    past the end of the field repeat a valid one (the same value to the same
//    address), so the compiler can count the memory operations in flight and
//    its waits for the next tile's loads leave the current tile's stores in
//    flight (the one branch around stores, in the contiguous forward DFT,
//    takes pairs of points on one side and the single ones of k = 0 on the
//    other);
//  * the twiddles live in LDS.
//
// Bound: HBM, like every stage (16 B per point in FP64).  The size-generic
// kernel ran at 1.7-2.4 TB/s (64-bit address arithmetic and run-time
// divisions in every element, each stage a call that drains the loads and
// stores in flight); this one on fields of 2^25 points, the types and both
// directions averaged, along x / y: n = 192 6.3 / 5.8 TB/s, 250 5.9 / 5.6
// (generic 2.2), 288 5.4 / 5.7, 480 6.0 / 5.8 (2.3), 640 5.0 / 4.8 (1.9), 1024
// 4.7 / 4.4 (2.4; its tile leaves room for one block to a CU); on the larger
// field of a 1024 x 640 x 320 solve 640 along y runs at 4.2.  Another
// placement of the field moves a figure by up to 10 %.  Whole solves: 270
// x 150 x 162 281 -> 115 us, 1024 x 640 x 320 8.16 -> 3.80 ms.
//
// Three pipelines: PIPE_FWD (real DFT, DCT-II, DST-II), PIPE_INV (their
// inverses), PIPE_IV (DCT-IV, DST-IV, both directions).  Two layouts: strided
// (lanes run over lines) and contiguous (the x axis: loads and stores run
// over a line's points, the FFT passes over lines as well).
#pragma once
#include <type_traits>
#include "r2r_fast.h"

namespace poisson_dev {

// ---------------------------------------------------------------- composite small DFTs

// cos / sin of 2 pi m / r at compile time (series in an argument reduced to
// [0, pi/4]: twelve terms leave less than one rounding).
constexpr double ct_series(double x, bool sine) {
  double term = sine ? x : 1.0, sum = term;
  for (int k = 1; k < 13; ++k) {
    const int a = sine ? 2 * k : 2 * k - 1;
    term = -term * x * x / ((double)a * (double)(a + 1));
    sum += term;
  }
  return sum;
}
constexpr double ct_trig(int m, int r, bool sine) {
  m %= r;
  // angle 2 pi m / r = (pi/4) (8m / r): octant and remainder exactly
  const int oct = 8 * m / r;
  const int rem = 8 * m - oct * r;                 // (pi/4) rem / r past the octant
  const double pi4 = 0.78539816339744830962;
  const bool odd = oct & 1;
  const double x = odd ? pi4 * (double)(r - rem) / (double)r : pi4 * (double)rem / (double)r;
  const double c = ct_series(x, false), s = ct_series(x, true);
  // octants: cos = c, s, -s, -c, -c, -s, s, c; sin = s, c, c, s, -s, -c, -c, -s
  // (x measured from the nearer axis)
  switch (oct) {
    case 0: return sine ? s : c;
    case 1: return sine ? c : s;
    case 2: return sine ? c : -s;
    case 3: return sine ? s : -c;
    case 4: return sine ? -s : -c;
    case 5: return sine ? -c : -s;
    case 6: return sine ? -c : s;
    default: return sine ? -s : c;
  }
}

constexpr int ct_inverse(int a, int m) {   // a^-1 mod m
  for (int i = 1; i < m; ++i)
    if ((a * i) % m == 1) return i;
  return m == 1 ? 0 : 1;
}
constexpr int ct_gcd(int a, int b) { return b ? ct_gcd(b, a % b) : a; }
// R = first * second, coprime where R allows it
constexpr int small_first(int r) {
  return r == 6 || r == 10 || r == 18 ? 2 : r == 12 || r == 20 ? 4 : r == 15 || r == 9 ? 3 : r == 25 ? 5 : 1;
}

// DFT of length R = R1 R2 from lengths R1 and R2: the Good-Thomas mapping
// (no twiddles) when they are coprime, else R1 x R2 with twiddles.
template <int R, typename T, bool FWD>
struct CompositeDFT {
  static constexpr int R1 = small_first(R), R2 = R / R1;
  static constexpr bool COPRIME = ct_gcd(R1, R2) == 1;
  static __device__ __forceinline__ void run(cplx<T>* v) {
    cplx<T> y[R1][R2];
#pragma unroll
    for (int n2 = 0; n2 < R2; ++n2) {
      cplx<T> c[R1];
#pragma unroll
      for (int n1 = 0; n1 < R1; ++n1) c[n1] = v[COPRIME ? (R2 * n1 + R1 * n2) % R : R2 * n1 + n2];
      SmallDFT<R1, T, FWD>::run(c);
#pragma unroll
      for (int k1 = 0; k1 < R1; ++k1) y[k1][n2] = c[k1];
    }
    if constexpr (!COPRIME) twiddle(y, std::make_integer_sequence<int, R>{});
#pragma unroll
    for (int k1 = 0; k1 < R1; ++k1) {
      SmallDFT<R2, T, FWD>::run(y[k1]);
#pragma unroll
      for (int k2 = 0; k2 < R2; ++k2)
        v[COPRIME ? (k1 * R2 * ct_inverse(R2 % R1, R1) + k2 * R1 * ct_inverse(R1 % R2, R2)) % R
                  : k1 + R1 * k2] = y[k1][k2];
    }
  }
  template <int I>
  static __device__ __forceinline__ void twiddle_one(cplx<T> (&y)[R1][R2]) {
    constexpr int k1 = I / R2, n2 = I % R2;
    if constexpr (k1 > 0 && n2 > 0) {
      constexpr double c = ct_trig(k1 * n2, R, false), s = ct_trig(k1 * n2, R, true);
      y[k1][n2] = cmul(y[k1][n2], cplx<T>{(T)c, FWD ? (T)-s : (T)s});
    }
  }
  template <int... I>
  static __device__ __forceinline__ void twiddle(cplx<T> (&y)[R1][R2], std::integer_sequence<int, I...>) {
    (twiddle_one<I>(y), ...);
  }
};
#define POISSON_COMPOSITE(R_) \
  template <typename T, bool FWD> struct SmallDFT<R_, T, FWD> : CompositeDFT<R_, T, FWD> {};
POISSON_COMPOSITE(6) POISSON_COMPOSITE(9) POISSON_COMPOSITE(10) POISSON_COMPOSITE(12)
POISSON_COMPOSITE(15) POISSON_COMPOSITE(18) POISSON_COMPOSITE(20) POISSON_COMPOSITE(25)
#undef POISSON_COMPOSITE

// ---------------------------------------------------------------- radix plan

constexpr bool line_radix(int r) {
  return r == 2 || r == 3 || r == 4 || r == 5 || r == 6 || r == 8 || r == 9 || r == 10 || r == 12 ||
         r == 15 || r == 16 || r == 18 || r == 20 || r == 25;
}
// thread slots of one pass of radix r with qt threads per line
constexpr int line_pass_cost(int m, int r, int qt) { return (m / r + qt - 1) / qt * qt * r; }

// As few passes as the radices allow (one LDS round trip and two barriers
// each), then the fewest idle thread slots; the largest radix first, since
// the first pass needs no twiddles.
// rmax: the largest radix whose values fit the registers.
constexpr RadixPlan line_plan(int m, int qt, int rmax) {
  RadixPlan best{0, {0}};
  int cost = 1 << 30;
  for (int r1 = rmax; r1 >= 2; --r1)
    if (line_radix(r1) && m % r1 == 0 && line_radix(m / r1) && m / r1 <= r1) {
      const int c = line_pass_cost(m, r1, qt) + line_pass_cost(m, m / r1, qt) + 4 * r1;
      if (c < cost) { cost = c; best = RadixPlan{2, {r1, m / r1}}; }
    }
  if (best.count) return best;
  for (int r1 = 16; r1 >= 2; --r1)
    for (int r2 = r1; r2 >= 2; --r2)
      if (line_radix(r1) && line_radix(r2) && m % (r1 * r2) == 0 && line_radix(m / (r1 * r2)) &&
          m / (r1 * r2) <= r2) {
        const int r3 = m / (r1 * r2);
        const int c = line_pass_cost(m, r1, qt) + line_pass_cost(m, r2, qt) +
                      line_pass_cost(m, r3, qt) + 4 * r1;
        if (c < cost) { cost = c; best = RadixPlan{3, {r1, r2, r3}}; }
      }
  return best;
}

// Tile: NL lines, NT threads, QT = NT / NL threads per line.
template <int M_, int NL_, int NT_, int RMAX_>
struct LineCfg {
  static constexpr int M = M_, NL = NL_, NT = NT_, QT = NT_ / NL_;
  static constexpr RadixPlan plan = line_plan(M_, QT, RMAX_);
  static_assert(plan.count > 0, "length without a radix plan");
  static_assert(QT * NL == NT && (NL & (NL - 1)) == 0, "whole threads per line");
};

enum LinePipe { PIPE_FWD = 0, PIPE_INV = 1, PIPE_IV = 2 };

template <typename T, typename C>
struct LineLayout {
  static constexpr int M = C::M, N = 2 * M, NL = C::NL, NT = C::NT, QT = C::QT;
  static constexpr int NLP = NL + 1;                        // odd LDS row pitch
  static constexpr int TILE = N * NLP;
  static constexpr int EP = (N + QT - 1) / QT;              // points per thread
  static constexpr int EC = (M + QT - 1) / QT;              // complex values per thread
  // wavenumber pairs (k, M - k) of a line, 0 <= k <= M/2, and per thread; for
  // the DCT-IV types the pairs (k, M - 1 - k).  The contiguous layout deals
  // out the pairs of all lines over the block (line-major), so that the lanes
  // of a wave run along a line however few threads a line has.
  static constexpr int NP = M / 2 + 1, NQ = (M + 1) / 2;
  static constexpr int per_thread(int pairs, int layout) {
    return layout == 0 ? (pairs + QT - 1) / QT : (pairs * NL + NT - 1) / NT;
  }
  static constexpr int SPLIT = M / 2 + 1;
  static constexpr size_t lds_bytes(int pipe) {
    return (size_t)TILE * sizeof(T) +
           (size_t)(M + (pipe == PIPE_IV ? 2 * M : SPLIT + M + 1)) * sizeof(cplx<T>);
  }
};

// a b with its fused operations spelled out.  The placement below is compiled
// twice (for a block's first tile, and in its loop); left to the compiler the
// two copies may fuse differently, and a tile's bits would depend on which
// block ran it.
template <typename T>
__device__ __forceinline__ cplx<T> cmul_fixed(cplx<T> a, cplx<T> b) {
#pragma clang fp contract(off)
  const T p = a.im * b.im, q = a.im * b.re;
  if constexpr (sizeof(T) == 8) return {__builtin_fma(a.re, b.re, -p), __builtin_fma(a.re, b.im, q)};
  else return {__builtin_fmaf(a.re, b.re, -p), __builtin_fmaf(a.re, b.im, q)};
}

// ---------------------------------------------------------------- FFT passes

template <typename T, typename C, int R, int NS, bool FWD, bool PRE>
__device__ __forceinline__ void line_pass(lptr<T> lds, lptr<const cplx<T>> tw,
                                          lptr<const cplx<T>> pre, int l, int q) {
  using L = LineLayout<T, C>;
  constexpr int M = L::M, B = M / R, SB = (B + L::QT - 1) / L::QT, TS = M / (NS * R);
  cplx<T> v[SB][R];
#pragma unroll
  for (int s = 0; s < SB; ++s) {
    const int j = q + s * L::QT;
    if (B % L::QT == 0 || j < B) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int idx = j + r * B;
        v[s][r] = {lds[(2 * idx) * L::NLP + l], lds[(2 * idx + 1) * L::NLP + l]};
        if constexpr (PRE) v[s][r] = cmul(v[s][r], ldc(pre, idx));
      }
      if constexpr (NS > 1) {
        const int k = j % NS;
#pragma unroll
        for (int r = 1; r < R; ++r) {
          cplx<T> w = ldc(tw, r * k * TS);
          if (!FWD) w.im = -w.im;
          v[s][r] = cmul(v[s][r], w);
        }
      }
    }
  }
  lds_barrier();
#pragma unroll
  for (int s = 0; s < SB; ++s) {
    const int j = q + s * L::QT;
    if (B % L::QT == 0 || j < B) {
      SmallDFT<R, T, FWD>::run(v[s]);
      const int k = NS > 1 ? j % NS : 0;
      const int base = (j - k) * R + k;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int idx = base + r * NS;
        lds[(2 * idx) * L::NLP + l] = v[s][r].re;
        lds[(2 * idx + 1) * L::NLP + l] = v[s][r].im;
      }
    }
  }
  lds_barrier();
}

template <typename T, typename C, bool FWD, bool PRE, int P = 0>
__device__ __forceinline__ void line_passes(lptr<T> lds, lptr<const cplx<T>> tw,
                                            lptr<const cplx<T>> pre, int l, int q) {
  if constexpr (P < C::plan.count) {
    line_pass<T, C, C::plan.r[P], plan_ns(C::plan, P), FWD, PRE && P == 0>(lds, tw, pre, l, q);
    line_passes<T, C, FWD, PRE, P + 1>(lds, tw, pre, l, q);
  }
}

// ---------------------------------------------------------------- kernel

template <typename T, typename C, int PIPE, int LAYOUT, int WAVES>
__global__ __launch_bounds__(C::NT, WAVES)
void r2r_line_kernel(R2RFastArgs<T> A) {
  using L = LineLayout<T, C>;
  constexpr int M = L::M, N = L::N, NL = L::NL, NT = L::NT, QT = L::QT, NLP = L::NLP;
  constexpr int H = M / 2;
  using T2 = T __attribute__((ext_vector_type(2)));
  using T2u = T __attribute__((ext_vector_type(2), aligned(sizeof(T))));   // at any element
  if (A.skip && A.skip[0] != 0.0) return;
  __shared__ __align__(16) unsigned char raw[L::lds_bytes(PIPE)];
  const lptr<T> tile_lds = as_lds(reinterpret_cast<T*>(raw));
  const lptr<cplx<T>> twf = as_lds(reinterpret_cast<cplx<T>*>(reinterpret_cast<T*>(raw) + L::TILE));
  const lptr<cplx<T>> twa = twf + M;                                  // pre or split
  const lptr<cplx<T>> twb = twa + (PIPE == PIPE_IV ? M : L::SPLIT);   // post or quarter
  const int tid0 = threadIdx.x;
  const int kind = A.kind;
  LineGeom g = A.g;
  g.layout = LAYOUT;

  for (int i = tid0; i < M; i += NT) stc(twf, i, ldg(A.tw_fft, i));
  if constexpr (PIPE == PIPE_IV) {
    for (int i = tid0; i < M; i += NT) {
      stc(twa, i, ldg(A.tw_pre, i));
      stc(twb, i, ldg(A.tw_post, i));
    }
  } else {
    for (int i = tid0; i < L::SPLIT; i += NT) stc(twa, i, ldg(A.tw_split, i));
    for (int i = tid0; i <= M; i += NT) stc(twb, i, ldg(A.tw_quarter, i));
  }

  // Line `l` of a tile (strided: one column, repeated for lanes past the
  // field; contiguous: one run of N values).  off(p): element offset of
  // point p from the tile's first point.  24-bit products: a stride is at
  // most 2^20 and a point index below 2^10.
  const unsigned sp = LAYOUT == 0 ? (unsigned)g.sp : 1u;
  const gptr<const T> src = as_global(static_cast<const T*>(A.data));
  struct Tile {
    long long base;
    int lines;
    TileOrigin o;
  };
  auto tile_at = [&](int tile) {
    Tile t;
    t.o = tile_origin(g, tile);
    if constexpr (LAYOUT == 0) {
      t.base = t.o.x0 + (long long)t.o.b0 * g.sb;
      t.lines = 0;
    } else {
      t.base = (long long)t.o.L0 * N;
      t.lines = g.nlines - t.o.L0;
    }
    return t;
  };
  auto line_off = [&](const Tile& t, int l) -> unsigned {
    if constexpr (LAYOUT == 0) {
      const int lm = l & ((1 << g.lognl) - 1);
      const int x = min(t.o.x0 + (lm & ((1 << g.logtxw) - 1)), g.nx - 1);
      const int b = min(t.o.b0 + (lm >> g.logtxw), g.nb - 1);
      return (unsigned)(x - t.o.x0) + (unsigned)((long long)(b - t.o.b0) * g.sb);
    } else {
      return (unsigned)min(l, t.lines - 1) * (unsigned)N;
    }
  };
  auto at = [&](unsigned lo, int p) -> unsigned { return lo + __umul24((unsigned)p, sp); };

  // registers of the next tile: PIPE_INV holds the four rows of each of the
  // thread's wavenumber pairs, the others the thread's points in order
  constexpr int SP = L::per_thread(L::NP, LAYOUT), SQ = L::per_thread(L::NQ, LAYOUT);
  constexpr int NBUF = PIPE == PIPE_INV ? 4 * SP : LAYOUT == 0 ? L::EP : 2 * L::EC;
  T buf[NBUF];
  // pair s of the thread: its line of the tile and k (past the end: the last
  // pair again)
  struct Pair {
    int ln, k;
  };
  auto pair_at = [&](int s, int pairs, int l, int q, int tid) -> Pair {
    if constexpr (LAYOUT == 0) {
      const int k = q + s * QT;
      return Pair{l, pairs % QT == 0 ? k : min(k, pairs - 1)};
    } else {
      int e = tid + s * NT;
      if ((pairs * NL) % NT != 0) e = min(e, pairs * NL - 1);
      const int ln = e / pairs;
      return Pair{ln, e - ln * pairs};
    }
  };

  auto fetch = [&](int tile, int l, int q, int tid) {
    const Tile t = tile_at(tile);
    const gptr<const T> tb = src + t.base;
    if constexpr (PIPE == PIPE_INV) {
      // rows of wavenumber k and M - k (combine below); those that k = 0
      // does not have repeat another
      auto rows = [&](auto f) {
#pragma unroll
        for (int s = 0; s < SP; ++s) {
          const Pair pr = pair_at(s, L::NP, l, q, tid);
          const unsigned lo = line_off(t, pr.ln);
          int r[4];
          f(pr.k, r);
#pragma unroll
          for (int a = 0; a < 4; ++a) buf[4 * s + a] = tb[at(lo, r[a])];
        }
      };
      if (kind == K_P) {
        if constexpr (LAYOUT == 0) {
          rows([&](int k, int (&r)[4]) {
            r[0] = max(2 * k - 1, 0);
            r[1] = 2 * k;
            r[2] = N - 1 - 2 * k;
            r[3] = min(N - 2 * k, N - 1);
          });
        } else {   // two adjacent points per load
#pragma unroll
          for (int s = 0; s < SP; ++s) {
            const Pair pr = pair_at(s, L::NP, l, q, tid);
            const int k = pr.k;
            const gptr<const T> row = tb + line_off(t, pr.ln);
            const T2u lo = *reinterpret_cast<const gptr<const T2u>>(row + max(2 * k - 1, 0));
            const T2u hi = *reinterpret_cast<const gptr<const T2u>>(row + min(N - 1 - 2 * k, N - 2));
            buf[4 * s] = lo.x;
            buf[4 * s + 1] = lo.y;
            buf[4 * s + 2] = k == 0 ? hi.y : hi.x;
            buf[4 * s + 3] = hi.y;
          }
        }
      } else if (kind == K_NN)
        rows([&](int k, int (&r)[4]) {
          r[0] = k;
          r[1] = min(N - k, N - 1);
          r[2] = M - k;
          r[3] = M + k;
        });
      else
        rows([&](int k, int (&r)[4]) {
          r[0] = N - 1 - k;
          r[1] = max(k - 1, 0);
          r[2] = M - 1 + k;
          r[3] = M - 1 - k;
        });
    } else if constexpr (LAYOUT == 0) {
      const unsigned lo = line_off(t, l);
#pragma unroll
      for (int i = 0; i < L::EP; ++i) {
        const int p = q + i * QT;
        buf[i] = tb[at(lo, N % QT == 0 ? p : min(p, N - 1))];
      }
    } else {
#pragma unroll
      for (int i = 0; i < L::EC; ++i) {
        int e = tid + i * NT;                       // pair of points: line e / M, points 2j, 2j + 1
        if constexpr (M % QT != 0) e = min(e, M * NL - 1);
        const int ll = e / M, j = e - ll * M;
        const T2 v = *reinterpret_cast<const gptr<const T2>>(tb + line_off(t, ll) + 2 * j);
        buf[2 * i] = v.x;
        buf[2 * i + 1] = v.y;
      }
    }
  };

  auto place = [&](int l, int q, int tid) {
    if constexpr (PIPE == PIPE_INV) {
      // Z'_k = (X_k + conj X_{M-k}) + i (X_k - conj X_{M-k}) e^{2 pi i k/n}
      auto put = [&](int ln, int k, cplx<T> xk, cplx<T> xj) {
        const cplx<T> sk = ldc(twa, k);
        const cplx<T> s1 = cadd(xk, cconj(xj)), d = csub(xk, cconj(xj));
        const cplx<T> d1 = cmul_fixed(d, cconj(sk));
        tile_lds[(2 * k) * NLP + ln] = s1.re - d1.im;
        tile_lds[(2 * k + 1) * NLP + ln] = s1.im + d1.re;
        // (k = M/2 is its own partner: lanes past the last pair repeat it, and
        // only one formula may write it)
        if (k > 0 && 2 * k != M) {
          const int j = M - k;
          tile_lds[(2 * j) * NLP + ln] = s1.re + d1.im;
          tile_lds[(2 * j + 1) * NLP + ln] = -s1.im + d1.re;
        }
      };
#pragma unroll
      for (int s = 0; s < SP; ++s) {
        const Pair pr = pair_at(s, L::NP, l, q, tid);
        const int k = pr.k;
        cplx<T> xk, xj;
        if (kind == K_P) {
          xk = {buf[4 * s], k == 0 ? (T)0 : -buf[4 * s + 1]};
          xj = {buf[4 * s + 2], k == 0 ? (T)0 : -buf[4 * s + 3]};
        } else {
          xk = cmul_fixed(cconj(ldc(twb, k)), cplx<T>{(T)0.5 * buf[4 * s], k == 0 ? (T)0 : (T)-0.5 * buf[4 * s + 1]});
          xj = cmul_fixed(cconj(ldc(twb, M - k)), cplx<T>{(T)0.5 * buf[4 * s + 2], (T)-0.5 * buf[4 * s + 3]});
        }
        put(pr.ln, k, xk, xj);
      }
    } else if constexpr (LAYOUT == 0) {
#pragma unroll
      for (int i = 0; i < L::EP; ++i) {
        const int p = q + i * QT;
        if (N % QT == 0 || p < N) {
          bool neg;
          const int r = load_row(kind, 0, p, N, neg);
          tile_lds[r * NLP + l] = neg ? -buf[i] : buf[i];
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < L::EC; ++i) {
        const int e = tid + i * NT;
        if (M % QT == 0 || e < M * NL) {
          const int ll = e / M, j = e - ll * M;
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            bool neg;
            const int r = load_row(kind, 0, 2 * j + h, N, neg);
            tile_lds[r * NLP + ll] = neg ? -buf[2 * i + h] : buf[2 * i + h];
          }
        }
      }
    }
  };

  // the transformed tile to the field (O: the element type written)
  auto store = [&](auto* field, int tile, int l, int q, int tid) {
    using O = std::remove_pointer_t<decltype(field)>;
    const Tile t = tile_at(tile);
    const gptr<O> tb = as_global(field) + t.base;
    const T scale = A.scale;
    if constexpr (PIPE == PIPE_FWD) {
#pragma unroll
      for (int s = 0; s < SP; ++s) {
        const Pair pr = pair_at(s, L::NP, l, q, tid);
        const int ln = pr.ln, k = pr.k;
        const unsigned lo = line_off(t, ln);
        const int j = M - k, kc = k == 0 ? 0 : j;
        const cplx<T> z = {tile_lds[(2 * k) * NLP + ln], tile_lds[(2 * k + 1) * NLP + ln]};
        const cplx<T> zc = {tile_lds[(2 * kc) * NLP + ln], -tile_lds[(2 * kc + 1) * NLP + ln]};
        const cplx<T> E = {(T)0.5 * (z.re + zc.re), (T)0.5 * (z.im + zc.im)};
        const cplx<T> D = csub(z, zc);
        const cplx<T> O_ = {(T)0.5 * D.im, (T)-0.5 * D.re};
        const cplx<T> wO = cmul(ldc(twa, k), O_);
        const cplx<T> X = cadd(E, wO);
        const cplx<T> Y = cconj(csub(E, wO));
        // four outputs; where k = 0 or k = M - k has two, they are repeated
        int r[4];
        T v[4];
        const bool one = k == j;
        if (kind == K_P) {
          const bool zero = k == 0;
          r[0] = zero ? 0 : 2 * k - 1;
          r[1] = zero ? N - 1 : 2 * k;
          v[0] = X.re;
          v[1] = zero ? Y.re : -X.im;
          r[2] = zero ? 0 : 2 * j - 1;
          r[3] = zero ? N - 1 : 2 * j;
          v[2] = zero || one ? v[0] : Y.re;
          v[3] = zero || one ? v[1] : -Y.im;
        } else {
          // DCT-II: y_k = 2 Re(q_k X_k), y_{n-k} = -2 Im(q_k X_k); DST-II reversed
          const bool zero = k == 0;
          const cplx<T> u = cmul(ldc(twb, k), X);
          const cplx<T> u2 = cmul(ldc(twb, j), Y);
          r[0] = k;
          r[1] = zero ? 0 : N - k;
          r[2] = j;
          r[3] = zero ? j : N - j;
          v[0] = (T)2 * u.re;
          v[1] = zero ? v[0] : (T)-2 * u.im;
          v[2] = one ? v[0] : (T)2 * u2.re;
          v[3] = one ? v[1] : zero ? v[2] : (T)-2 * u2.im;
          if (kind == K_DD) {
#pragma unroll
            for (int a = 0; a < 4; ++a) r[a] = N - 1 - r[a];
          }
        }
        if (LAYOUT == 1 && kind == K_P && k > 0) {   // adjacent points 2k-1, 2k and 2j-1, 2j
          using O2u = O __attribute__((ext_vector_type(2), aligned(sizeof(O))));
          *reinterpret_cast<gptr<O2u>>(tb + lo + r[0]) = O2u{(O)(v[0] * scale), (O)(v[1] * scale)};
          *reinterpret_cast<gptr<O2u>>(tb + lo + r[2]) = O2u{(O)(v[2] * scale), (O)(v[3] * scale)};
        } else {
#pragma unroll
          for (int a = 0; a < 4; ++a) tb[at(lo, r[a])] = (O)(v[a] * scale);
        }
      }
    } else if constexpr (PIPE == PIPE_IV) {
      const T so = kind == K_ND ? (T)-2 : (T)2;   // the DST-IV negates odd points
      // V_k = Z_k times the post-twiddle: point 2k = 2 Re V_k, point n-1-2k =
      // -2 Im V_k; k and M-1-k together give the adjacent points 2k, 2k+1
      // and n-2-2k, n-1-2k
#pragma unroll
      for (int s = 0; s < SQ; ++s) {
        const Pair pr = pair_at(s, L::NQ, l, q, tid);
        const int ln = pr.ln, k = pr.k;
        const unsigned lo = line_off(t, ln);
        const int j = M - 1 - k;
        const cplx<T> V = cmul(cplx<T>{tile_lds[(2 * k) * NLP + ln], tile_lds[(2 * k + 1) * NLP + ln]},
                               ldc(twb, k));
        const cplx<T> W = cmul(cplx<T>{tile_lds[(2 * j) * NLP + ln], tile_lds[(2 * j + 1) * NLP + ln]},
                               ldc(twb, j));
        const T a0 = ((T)2 * V.re) * scale, a1 = (so * W.im) * scale;
        T b0 = ((T)2 * W.re) * scale, b1 = (so * V.im) * scale;
        if constexpr (M % 2 == 1) {   // the middle element is its own partner
          b0 = k == j ? a0 : b0;
          b1 = k == j ? a1 : b1;
        }
        if constexpr (LAYOUT == 0) {
          tb[at(lo, 2 * k)] = (O)a0;
          tb[at(lo, 2 * k + 1)] = (O)a1;
          tb[at(lo, 2 * j)] = (O)b0;
          tb[at(lo, 2 * j + 1)] = (O)b1;
        } else {
          using O2 = O __attribute__((ext_vector_type(2)));
          *reinterpret_cast<gptr<O2>>(tb + lo + 2 * k) = O2{(O)a0, (O)a1};
          *reinterpret_cast<gptr<O2>>(tb + lo + 2 * j) = O2{(O)b0, (O)b1};
        }
      }
    } else if constexpr (LAYOUT == 0) {
      const unsigned lo = line_off(t, l);
#pragma unroll
      for (int i = 0; i < L::EP; ++i) {
        const int p = N % QT == 0 ? q + i * QT : min(q + i * QT, N - 1);
        bool neg;
        const int r = store_row(kind, 1, p, N, neg);
        const T v = tile_lds[r * NLP + l] * scale;
        tb[at(lo, p)] = (O)(neg ? -v : v);
      }
    } else {
      using O2 = O __attribute__((ext_vector_type(2)));
#pragma unroll
      for (int i = 0; i < L::EC; ++i) {
        int e = tid + i * NT;
        if constexpr (M % QT != 0) e = min(e, M * NL - 1);
        int ll = e / M;
        const int j = e - ll * M;
        bool n0, n1;
        const int r0 = store_row(kind, 1, 2 * j, N, n0), r1 = store_row(kind, 1, 2 * j + 1, N, n1);
        const T v0 = tile_lds[r0 * NLP + ll] * scale, v1 = tile_lds[r1 * NLP + ll] * scale;
        *reinterpret_cast<gptr<O2>>(tb + line_off(t, ll) + 2 * j) =
            O2{(O)(n0 ? -v0 : v0), (O)(n1 ? -v1 : v1)};
      }
    }
  };

  const TileRange tr = xcd_tiles(g.ntiles);
  if (tr.first < tr.end) {
    fetch(tr.first, tid0 % NL, tid0 / NL, tid0);
    lds_barrier();   // the twiddles (read by the combine)
    place(tid0 % NL, tid0 / NL, tid0);
  }
  // the next tile is placed at the bottom of the loop, after the current
  // tile's stores, so that the waits for its loads count those stores
  for (int tile = tr.first; tile < tr.end; tile += tr.step) {
    // thread index opaque per tile, and with 128 registers per step:
    // addresses are recomputed instead of being held (or spilled) across the
    // loop.  With 256 registers the steps are faster with them held (n = 640
    // along x 5.24 against 4.99 TB/s).
    int tid = tid0;
    asm volatile("" : "+v"(tid));
    auto step = [&] {
      if constexpr (WAVES > 2) asm volatile("" : "+v"(tid));
    };
    lds_barrier();
    const bool more = tile + tr.step < tr.end;
    if (more) fetch(tile + tr.step, tid % NL, tid / NL, tid);
    step();
    line_passes<T, C, PIPE != PIPE_INV, PIPE == PIPE_IV>(tile_lds, twf, twa, tid % NL, tid / NL);
    step();
    bool widened = false;
    if constexpr (sizeof(T) == 4 && PIPE != PIPE_FWD) {
      if (A.out64) {   // last pass of an FP32 solve: the widened result
        store(A.out64, tile, tid % NL, tid / NL, tid);
        widened = true;
      }
    }
    if (!widened) store(A.data, tile, tid % NL, tid / NL, tid);
    lds_barrier();
    step();
    if (more) place(tid % NL, tid / NL, tid);
  }
}

}  // namespace poisson_dev
