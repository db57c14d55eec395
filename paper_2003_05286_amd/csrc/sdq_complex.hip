// sdq_complex.hip -- complex UDT of independent matrices (Sec. 4.2.2 over the
// complex numbers, as the complex slices of App. B need it):
//   W P = Q R (column-pivoted Householder QR), U = Q, D = |diag R|,
//   T = D^{-1} R P^T.
// One workgroup (four wave64s) per matrix, n <= 64, held in registers while
// it is factored (lane = column, the rows dealt to the waves) and in LDS, as
// interleaved (re, im) pairs, for what follows.  Reflector convention: for
// x = A[i:, i] with alpha = x_0, beta = -sign(Re alpha) ||x|| is real, tau =
// (beta - alpha) / beta, v = x / (alpha - beta); H = I - tau v v^H, H^H x =
// beta e_0, so the diagonal of R is real.  Pivot: the first column of largest
// remaining norm, norms downdated with an exact recompute when cancellation
// threatens (Drmac & Bujanovic).  Q is formed from the reflectors by backward
// accumulation, Q = H_0 H_1 ... H_{n-1}.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "sdq_internal.h"

namespace sdq {
namespace {

constexpr int kCN = 64;         // largest n
constexpr int kCThreads = 256;  // four waves: wave w takes rows w, w+4, ...

// The kernels are built for NT = 1 .. 4 tiles of 16 (n <= 16 NT): registers,
// LDS and the padding of the products follow the size.
template <int NT>
struct Dim {
  static constexpr int cn = 16 * NT;  // padded n
  static constexpr int ld = cn + 1;   // LDS row stride (in complex entries)
  // workgroups of a CU: what LDS and 512 registers a SIMD lane hold of them
  static constexpr int udt_groups = NT == 4 ? 2 : NT == 3 ? 3 : NT == 2 ? 4 : 6;
  static constexpr int chain_groups = NT >= 3 ? 1 : 2;
};

struct cplx {
  double x, y;
};
__device__ __forceinline__ cplx cmul(cplx a, cplx b) { return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }
// conj(a) * b
__device__ __forceinline__ cplx cjmul(cplx a, cplx b) { return {a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x}; }

// Cross-lane reductions over the wave on the DPP paths of the VALU (no LDS
// round trips): swap neighbours (quad_perm 1,0,3,2 and 2,3,0,1), mirror
// within 8 and 16 lanes, then broadcast lane 15 of each row into the next
// and lane 31 into the upper half; lane 63 then holds the result, which
// readlane makes uniform.  A lane outside a step's row mask keeps `old`.
constexpr int kDppSteps[6] = {0xB1, 0x4E, 0x141, 0x140, 0x142, 0x143};
constexpr int kDppRows[6] = {0xf, 0xf, 0xf, 0xf, 0xa, 0xc};

template <int S>
__device__ __forceinline__ double dpp_d(double old, double v) {
  const long long o = __double_as_longlong(old), x = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp((int)o, (int)x, kDppSteps[S], kDppRows[S], 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp((int)(o >> 32), (int)(x >> 32), kDppSteps[S], kDppRows[S], 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
template <int S>
__device__ __forceinline__ int dpp_i(int old, int v) {
  return __builtin_amdgcn_update_dpp(old, v, kDppSteps[S], kDppRows[S], 0xf, false);
}
__device__ __forceinline__ double lane63(double v) {
  const long long x = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)x, 63), hi = __builtin_amdgcn_readlane((int)(x >> 32), 63);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

template <int S = 0>
__device__ __forceinline__ double wave_sum_(double v) {
  if constexpr (S == 6) {
    return lane63(v);
  } else {
    return wave_sum_<S + 1>(v + dpp_d<S>(0.0, v));
  }
}
__device__ __forceinline__ double wave_sum(double v) { return wave_sum_<0>(v); }

// LDS work space of the factorization and of applying its Q.
struct QrScratch {
  cplx sc[kCN];         // the reflectors' factors
  union {
    cplx row[2][kCN];       // a row of a solution
    double norms[4][kCN];   // per wave: sums of squares of the columns
  };
  cplx red[2][5][kCN];  // per wave: partial column products; [4]: row i
  double beta[kCN];     // diag R
};

// A matrix in registers: lane = column, wave w holds the rows 16 q + 4 t + w.
// Every register index is static: a loop over the steps is one loop for each
// 16 rows, which leaves out the rows that its steps don't touch.
template <int NT>
struct RegMat {
  cplx a[NT][4];
};
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }
template <int NT, class F>
__device__ __forceinline__ void each_row(F f) {
  const int w = wave_id();
#pragma unroll
  for (int q = 0; q < NT; ++q)
#pragma unroll
    for (int t = 0; t < 4; ++t) f(q, t, 16 * q + 4 * t + w);
}

// f(q, i) for the steps i of 0 .. n-1 upwards (or n-1 .. 0), q = i / 16 a
// constant
template <int Q>
struct TileNo {
  static constexpr int q = Q;
};
template <int NT, int Q = 0, class F>
__device__ __forceinline__ void steps_up(int n, F f) {
  if constexpr (Q < NT) {
    for (int i = 16 * Q; i < min(n, 16 * Q + 16); ++i) f(TileNo<Q>{}, i);
    steps_up<NT, Q + 1>(n, f);
  }
}
template <int NT, int Q = NT - 1, class F>
__device__ __forceinline__ void steps_down(int n, F f) {
  if constexpr (Q >= 0) {
    for (int i = min(n, 16 * Q + 16) - 1; i >= 16 * Q; --i) f(TileNo<Q>{}, i);
    steps_down<NT, Q - 1>(n, f);
  }
}

// A uniform value as one per lane, for conditions that select instead of
// branch: a taken branch costs more than the four selects of a value.
__device__ __forceinline__ int per_lane(int x) {
  asm("" : "+v"(x));
  return x;
}
__device__ __forceinline__ cplx select(bool c, cplx a, cplx b) { return {c ? a.x : b.x, c ? a.y : b.y}; }

__device__ __forceinline__ double lane_of(double v, int l) {
  const long long x = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)x, l), hi = __builtin_amdgcn_readlane((int)(x >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// A column as the wave's own rows use it: lane l < 4 NT holds row 4 l + w, and the rows are handed to the products as uniform values.
// Sixteen broadcast reads of every wave instead would keep LDS busy longer
// than the products take.
template <int NT>
__device__ __forceinline__ int own_row(int lane, int w) {
  return 4 * min(lane & 15, 4 * NT - 1) + w;
}
__device__ __forceinline__ cplx row_of(cplx v, int q, int t) { return {lane_of(v.x, 4 * q + t), lane_of(v.y, 4 * q + t)}; }

// Sums of the squares of the rows >= r0 of every column (lane = column),
// 16 Q0 <= r0; the same in every wave.  One barrier inside, none after the
// reads: `buf` is an array of its own (QrScratch::norms), since the next step
// writes either half of `red` before a barrier, and its own next use comes
// after that step's barrier.
template <int NT, int Q0>
__device__ __forceinline__ double col_squares(double (*buf)[kCN], const RegMat<NT>& A, int r0) {
  const int lane = threadIdx.x & 63, w = wave_id();
  const int w0 = per_lane(16 * Q0 + w - r0);  // row 16 Q0 + w + d counts if w0 + d >= 0
  double s = 0.0;
#pragma unroll
  for (int q = Q0; q < NT; ++q)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int d = 16 * (q - Q0) + 4 * t;
      const cplx x = d >= 16 ? A.a[q][t] : select(w0 + d >= 0, A.a[q][t], cplx{0.0, 0.0});
      s = fma(x.x, x.x, fma(x.y, x.y, s));
    }
  buf[w][lane] = s;
  __syncthreads();
  return (buf[0][lane] + buf[1][lane]) + (buf[2][lane] + buf[3][lane]);
}

// Largest real or imaginary part in the rows >= r0 of every column, as
// col_squares; with a barrier before it writes.
template <int NT, int Q0>
__device__ __forceinline__ double col_max(double (*buf)[kCN], const RegMat<NT>& A, int r0) {
  const int lane = threadIdx.x & 63, w = wave_id();
  const int w0 = per_lane(16 * Q0 + w - r0);
  double m = 0.0;
#pragma unroll
  for (int q = Q0; q < NT; ++q)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int d = 16 * (q - Q0) + 4 * t;
      if (d >= 16 || w0 + d >= 0) m = fmax(m, fmax(fabs(A.a[q][t].x), fabs(A.a[q][t].y)));
    }
  __syncthreads();
  buf[w][lane] = m;
  __syncthreads();
  return fmax(fmax(buf[0][lane], buf[1][lane]), fmax(buf[2][lane], buf[3][lane]));
}

// What remains of a column is scaled up, the whole column with it, once its
// squares sum to less than kSmallSquares (they would soon underflow, and the
// reflector with them); by 2^kMaxShift in all at most, so that the finished
// rows, at most 8 in size, do not overflow.
constexpr double kSmallSquares = 1e-200;
constexpr int kMaxShift = 1000;

// sqrt(c) and 1 / sqrt(c) (Goldschmidt from v_rsq_f64), 1 / c (Newton from
// v_rcp_f64) to the last place or two, for c in 1e-285 .. 1e285: what the
// library adds for the other arguments is a third of a step's scalar chain.
__device__ __forceinline__ double sqrt_mid(double c, double* inv) {
  const double y = __builtin_amdgcn_rsq(c);
  double g = c * y, h = 0.5 * y;
  double r = fma(-h, g, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  r = fma(-h, g, 0.5);
  h = fma(h, r, h);
  *inv = 2.0 * h;
  return fma(fma(-g, g, c), h, g);
}
__device__ __forceinline__ double rcp_mid(double c) {
  double y = __builtin_amdgcn_rcp(c);
  y = fma(fma(-c, y, 1.0), y, y);
  return fma(fma(-c, y, 1.0), y, y);
}

// lane of the largest key (keys >= 0, or -1 for none), among equal ones the
// one of lowest `pos`.  The high words first: their maximum takes one DPP
// operation a step and nearly always belongs to one lane.
__device__ __forceinline__ int max_lane(double key, int pos) {
  const long long k = __double_as_longlong(key);
  const int hi = (int)(k >> 32);
  int m = hi;
#define SDQ_MAX_STEP(S) m = max(m, dpp_i<S>(m, m))
  SDQ_MAX_STEP(0);
  SDQ_MAX_STEP(1);
  SDQ_MAX_STEP(2);
  SDQ_MAX_STEP(3);
  SDQ_MAX_STEP(4);
  SDQ_MAX_STEP(5);
#undef SDQ_MAX_STEP
  m = __builtin_amdgcn_readlane(m, 63);
  unsigned long long bl = __ballot(hi == m);
  int best = __ffsll((long long)bl) - 1;
#pragma unroll 1
  while ((bl &= bl - 1) != 0) {
    const int l = __ffsll((long long)bl) - 1;
    const unsigned a = __builtin_amdgcn_readlane((int)k, l), b = __builtin_amdgcn_readlane((int)k, best);
    if (a > b || (a == b && __builtin_amdgcn_readlane(pos, l) < __builtin_amdgcn_readlane(pos, best))) best = l;
  }
  return best;
}

// Column-pivoted Householder QR of M (n x n in LDS, zero below row n): on
// return M holds R on and above the diagonal, columns permuted, and the
// reflectors below it, tau the reflector scalars, jpvt the original column
// of each position.  Ends with a barrier.
//
// A serial chain of n steps, bound by the instructions one step issues.  The
// matrix is held in registers (lane = column) and a column keeps its lane
// (its place in the order is a number), so a step passes over LDS only for
// the pivot column and the products with it, with two barriers.  The products
// are taken with the column itself: the pivot lane's own is its squared norm,
// and every wave works out the reflector's scalars and the norms that remain
// for itself from the same numbers.  Norms are kept as c2 = (norm / norm at
// the last recompute)^2, so that a downdate is a subtraction; c2 is also what
// Drmac & Bujanovic's test of a downdate asks for.
//
// 64 x 64 complex matrices, one / 4096 of them factored with Q and T: 0.34 ->
// 0.16 ms / 3.23 -> 1.65 ms against the matrix in LDS with one wave choosing
// pivots while three wait (three barriers a step); a step takes about 2900
// cycles, and one of apply_q 1300.  At n = 16 the tile-sized variants take
// 4096 matrices from 0.50 to 0.21 ms.
template <int NT>
__device__ __forceinline__ void cpqr_lds(cplx* M, QrScratch& X, cplx* tau, int* jpvt, int n) {
  const int lane = threadIdx.x & 63, w = wave_id();
  const double tol3z = sqrt(2.220446049250313e-16);
  RegMat<NT> A;
  const int lc = min(lane, Dim<NT>::cn - 1);
  each_row<NT>([&](int q, int t, int r) {
    const cplx v = M[r * Dim<NT>::ld + lc];
    A.a[q][t] = r < n && lane < n ? v : cplx{0.0, 0.0};
  });
  // every column to entries of at most 1 by a power of two, undone in R: a
  // reflector does not depend on its column's scale and no square overflows
  // (what remains of a column is scaled up again where its squares would vanish)
  double mx = 0.0;
  each_row<NT>([&](int q, int t, int r) { mx = fmax(mx, fmax(fabs(A.a[q][t].x), fabs(A.a[q][t].y))); });
  X.red[0][w][lane].x = mx;
  __syncthreads();
#pragma unroll
  for (int v = 0; v < 4; ++v) mx = fmax(mx, X.red[0][v][lane].x);
  int e = __builtin_amdgcn_frexp_exp(mx), shifted = 0;
  each_row<NT>([&](int q, int t, int r) { A.a[q][t] = cplx{ldexp(A.a[q][t].x, -e), ldexp(A.a[q][t].y, -e)}; });
  int pos = lane;  // place of this lane's column
  // squared norm at its last computation, its inverse, and what is left of it
  double s0 = col_squares<NT, 0>(X.norms, A, 0), c2 = 1.0;
  double r0 = s0 > 1e-280 ? 1.0 / s0 : 0.0;
  steps_up<NT>(n, [&](auto tile, int i) {
    constexpr int iq = decltype(tile)::q;
    const bool mine = w == (i & 3);  // this wave holds row i
    // the column of largest remaining norm, the first among equals
    double inv;
    const double nk = r0 != 0.0 ? ldexp(sqrt_mid(s0 * c2, &inv), e) : 0.0;
    const int lp = max_lane(pos >= i && lane < n ? (nk >= 0.0 ? nk : 0.0) : -1.0, pos);
    const int p = __builtin_amdgcn_readlane(pos, lp);
    if (pos == i) pos = p;
    if (lane == lp) pos = i;
    const int below = 16 * iq + w - i;  // row 16 iq + w + d is i + below + d
    cplx row = {0.0, 0.0};
    if (mine) {
      const int b = per_lane(below);
#pragma unroll
      for (int t = 0; t < 4; ++t) row = select(b + 4 * t == 0, A.a[iq][t], row);
    }
    cplx v[NT][4];  // uniform: the rows of the column that are this wave's
    cplx part = {0.0, 0.0};
#pragma unroll
    for (int q = iq; q < NT; ++q)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const cplx x = {lane_of(A.a[q][t].x, lp), lane_of(A.a[q][t].y, lp)};
        v[q][t] = q > iq || below + 4 * t > 0 ? x : cplx{0.0, 0.0};
        const cplx z = cjmul(v[q][t], A.a[q][t]);
        part.x += z.x;
        part.y += z.y;
      }
    if (lane == lp) {
#pragma unroll
      for (int q = iq; q < NT; ++q)
#pragma unroll
        for (int t = 0; t < 4; ++t)
          M[(16 * q + 4 * t + w) * Dim<NT>::ld + i] = A.a[q][t];
    }
    auto& red = X.red[i & 1];
    red[w][lane] = part;
    if (mine) red[4][lane] = row;
    __syncthreads();
    cplx g = {(red[0][lane].x + red[1][lane].x) + (red[2][lane].x + red[3][lane].x),
              (red[0][lane].y + red[1][lane].y) + (red[2][lane].y + red[3][lane].y)};
    cplx ri = red[4][lane];
    // the reflector I - tau u u^H, u = (1, sc x), of (al, x): with
    // dn = al - beta, tau = -dn / beta and sc = 1 / dn
    const cplx al = {lane_of(ri.x, lp), lane_of(ri.y, lp)};
    const double ss = lane_of(g.x, lp);
    double beta = al.x, rb = 0.0;
    cplx dn = {0.0, 0.0}, sc = {0.0, 0.0};
    const double tot = ss + (al.x * al.x + al.y * al.y);
    if (tot > 1e-280 && (ss != 0.0 || al.y != 0.0)) {
      beta = -copysign(sqrt_mid(tot, &rb), al.x);
      rb = -copysign(rb, al.x);
      dn = cplx{al.x - beta, al.y};
      const double rd = rcp_mid(fma(dn.x, dn.x, dn.y * dn.y));
      sc = cplx{dn.x * rd, -dn.y * rd};
    }
    const cplx ti = {-dn.x * rb, -dn.y * rb};
    // A -= conj(tau) u u^H A
    const cplx ug = cjmul(sc, g);
    g = cjmul(ti, cplx{ri.x + ug.x, ri.y + ug.y});
    ri = cplx{ri.x - g.x, ri.y - g.y};
    const cplx f = cmul(sc, g);
#pragma unroll
    for (int q = iq; q < NT; ++q) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const cplx z = cmul(v[q][t], f);
        A.a[q][t].x -= z.x;
        A.a[q][t].y -= z.y;
      }
    }
    // row i's wave keeps the row and the reflector's scalars
    if (mine) {
      const int b = per_lane(below);
#pragma unroll
      for (int t = 0; t < 4; ++t) A.a[iq][t] = select(b + 4 * t == 0, ri, A.a[iq][t]);
      if (lane == 0) {
        tau[i] = ti;
        X.sc[i] = sc;
        X.beta[i] = beta;
        jpvt[i] = lp;
      }
    }
    // the norms that remain, downdated by row i; recomputed where the
    // difference has lost too many digits (the same lanes in every wave)
    bool again = false;
    if (pos > i && lane < n && r0 != 0.0) {
      c2 -= fma(ri.x, ri.x, ri.y * ri.y) * r0;
      again = !(c2 > tol3z);
    }
    if (__any(again)) {
      double sn = col_squares<NT, iq>(X.norms, A, i + 1);
      const bool small = again && sn < kSmallSquares && shifted < kMaxShift;
      if (__any(small)) {
        const double m = col_max<NT, iq>(X.norms, A, i + 1);
        const int s = small && m > 0.0 ? min(-__builtin_amdgcn_frexp_exp(m), kMaxShift - shifted) : 0;
        each_row<NT>([&](int q, int t, int r) { A.a[q][t] = cplx{ldexp(A.a[q][t].x, s), ldexp(A.a[q][t].y, s)}; });
        e -= s;
        shifted += s;
        __syncthreads();  // the maxima are read
        sn = col_squares<NT, iq>(X.norms, A, i + 1);
      }
      if (again) {
        s0 = sn;
        r0 = sn > 1e-280 ? 1.0 / sn : 0.0;
        c2 = 1.0;
      }
    }
  });
  // R to the places of the columns; a lane's rows below its place are rounding
  each_row<NT>([&](int q, int t, int r) {
    if (lane < n && r < pos) M[r * Dim<NT>::ld + pos] = cplx{ldexp(A.a[q][t].x, e), ldexp(A.a[q][t].y, e)};
  });
  __syncthreads();
  if (w == 0 && lane < n) {
    const double b = ldexp(X.beta[pos], e);
    X.beta[pos] = b;
    M[pos * Dim<NT>::ld + pos] = cplx{b, 0.0};
  }
  __syncthreads();
}

// A <- Q A (or Q^H A) for Q = H_0 H_1 ... H_{n-1} from the reflectors
// cpqr_lds left below the diagonal of M, A in registers: one barrier per
// reflector, every wave with its own rows.  M is zero below row n.
template <int NT, bool ADJ>
__device__ __forceinline__ void apply_q(const cplx* M, QrScratch& X, const cplx* tau, int n, RegMat<NT>& A) {
  const int lane = threadIdx.x & 63, w = wave_id();
  auto step = [&](auto tile, int i) {
    constexpr int iq = decltype(tile)::q;
    const int own = own_row<NT>(lane, w);
    const cplx vl = select(own > i, cmul(M[own * Dim<NT>::ld + i], X.sc[i]), cplx{own == i ? 1.0 : 0.0, 0.0});
    cplx part = {0.0, 0.0};
#pragma unroll
    for (int q = iq; q < NT; ++q)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const cplx z = cjmul(row_of(vl, q, t), A.a[q][t]);
        part.x += z.x;
        part.y += z.y;
      }
    auto& red = X.red[i & 1];
    red[w][lane] = part;
    cplx ti = tau[i];
    if (ADJ) ti.y = -ti.y;
    __syncthreads();
    const cplx g = cmul(ti, cplx{(red[0][lane].x + red[1][lane].x) + (red[2][lane].x + red[3][lane].x),
                                 (red[0][lane].y + red[1][lane].y) + (red[2][lane].y + red[3][lane].y)});
#pragma unroll
    for (int q = iq; q < NT; ++q) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const cplx z = cmul(row_of(vl, q, t), g);
        A.a[q][t].x -= z.x;
        A.a[q][t].y -= z.y;
      }
    }
  };
  if constexpr (ADJ)
    steps_up<NT>(n, step);
  else
    steps_down<NT>(n, step);
}

// Q of the reflectors in M into M itself; what is outside n x n becomes zero.
// Ends with a barrier.
template <int NT>
__device__ __forceinline__ void form_q_lds(cplx* M, QrScratch& X, const cplx* tau, int n) {
  const int lane = threadIdx.x & 63;
  RegMat<NT> A;
  each_row<NT>([&](int q, int t, int r) { A.a[q][t] = cplx{r == lane && r < n ? 1.0 : 0.0, 0.0}; });
  apply_q<NT, false>(M, X, tau, n, A);
  __syncthreads();
  if (lane < Dim<NT>::cn) each_row<NT>([&](int q, int t, int r) { M[r * Dim<NT>::ld + lane] = A.a[q][t]; });
  __syncthreads();
}

// det Q, the product of det H_j = -tau_j / conj(tau_j), by every wave on its
// own (lane = reflector).
__device__ __forceinline__ cplx det_q(const cplx* tau, int n) {
  const int lane = threadIdx.x & 63;
  cplx h = {1.0, 0.0};
  if (lane < n) {
    const cplx t = tau[lane];
    if (t.x != 0.0 || t.y != 0.0) {
      const double a2 = t.x * t.x + t.y * t.y;
      h = cplx{-(t.x * t.x - t.y * t.y) / a2, -(2.0 * t.x * t.y) / a2};
    }
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) h = cmul(h, cplx{__shfl_xor(h.x, d), __shfl_xor(h.y, d)});
  return h;
}

template <int NT>
struct CSmem {
  cplx a[Dim<NT>::cn * Dim<NT>::ld];
  QrScratch x;
  cplx tau[kCN];
  int jpvt[kCN], ipiv[kCN];
};

template <int NT>
__global__ __launch_bounds__(kCThreads, Dim<NT>::udt_groups) void k_udt_complex(int n, int count, const double* __restrict__ w,
                                                           double* __restrict__ u, double* __restrict__ d,
                                                           double* __restrict__ t) {
  __shared__ CSmem<NT> S;
  constexpr int CN = Dim<NT>::cn, LD = Dim<NT>::ld;
  const int tid = threadIdx.x;
  for (int b = blockIdx.x; b < count; b += gridDim.x) {
    const size_t off = (size_t)b * n * n;
    const cplx* W = reinterpret_cast<const cplx*>(w) + off;
    for (int e = tid; e < CN * CN; e += kCThreads) {
      const int r = e / CN, c = e % CN;
      S.a[r * LD + c] = r < n && c < n ? W[r * n + c] : cplx{0.0, 0.0};
    }
    __syncthreads();
    cpqr_lds<NT>(S.a, S.x, S.tau, S.jpvt, n);
    // D = |diag R| (real), T = D^{-1} R P^T (rows with D = 0 undivided)
    if (tid < n) {
      d[(size_t)b * n + tid] = fabs(S.a[tid * LD + tid].x);
      S.ipiv[S.jpvt[tid]] = tid;
    }
    __syncthreads();
    cplx* T = reinterpret_cast<cplx*>(t) + off;
    for (int e = tid; e < n * n; e += kCThreads) {
      const int r = e / n, col = e % n, c = S.ipiv[col];
      cplx v = {0.0, 0.0};
      if (c >= r) {
        const double dr = fabs(S.a[r * LD + r].x);
        const double sc = dr > 0.0 ? 1.0 / dr : 1.0;
        v = {S.a[r * LD + c].x * sc, S.a[r * LD + c].y * sc};
      }
      T[e] = v;
    }
    __syncthreads();
    form_q_lds<NT>(S.a, S.x, S.tau, n);
    cplx* U = reinterpret_cast<cplx*>(u) + off;
    for (int e = tid; e < n * n; e += kCThreads) U[e] = S.a[(e / n) * LD + e % n];
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Chains of complex slices (App. B): G = (1 + B_m ... B_1)^{-1} for complex
// dense slices, with log|det(1 + B_m ... B_1)| and its phase.  One workgroup
// per chain, everything resident in LDS (n <= 64):
//   chain (Sec. 4.1): per block of k slices W <- B_q W on FP64 MFMA (a
//     complex product is four real ones), then W <- W D, the complex pivoted
//     QR of W (Sec. 4.2.2), D <- |diag R|, T <- D^{-1} R P^T T on MFMA, and
//     U = Q formed in place;
//   inversion (Sec. 5.1, Loh's split, in the mirror form of the real path):
//     1 + U D T = U D_p (D_p^{-1} U^H + D_m T), so G = M^{-1} D_p^{-1} U^H
//     with M = D_p^{-1} U^H + D_m T, solved through the same pivoted QR, Q^H
//     applied to the right-hand sides in registers, and back substitution;
//   determinant: det(1 + B) = det U prod(D_p) det M, det U the product of
//     det H_j = -tau_j / conj(tau_j) over the reflectors of the last QR, det M
//     that of its own, the diagonal of R and the sign of the permutation.
// 128 chains of 200 slices, k = 10, n = 64: 10.5 -> 5.6 ms, of which the
// slice products take 2.3 (1.4 at the FP64 matrix rate of the 128 CUs in use),
// 21 factorizations 3; the elimination in LDS that the QR replaced took 0.6.
template <int NT>
struct CCSmem {
  cplx a[Dim<NT>::cn * Dim<NT>::ld];  // W, then R and the reflectors, then U = Q, then the right-hand sides / G
  cplx t[Dim<NT>::cn * Dim<NT>::ld];  // T, then M
  QrScratch x;
  cplx tau[kCN];
  double d[kCN];  // D of the current factorization
  int jpvt[kCN];
};

typedef double cd4 __attribute__((ext_vector_type(4)));

// C = A X for the n x n (padded to 16 NT) complex matrices A (by a callable:
// A(i, k) for the calling lane) and X in LDS (X(k, c) callable): wave w
// (w < NT) produces the output columns 16 w .. 16 w + 15, all row tiles, into
// cr / ci in the FP64 MFMA 16x16x4 accumulator layout (lane l: rows
// 16 ti + l / 16 + 4 r of column 16 w + l % 16).
template <int NT, class AF, class XF>
__device__ __forceinline__ void cgemm(AF A, XF X, cd4 (&cr)[NT], cd4 (&ci)[NT]) {
  const int lane = threadIdx.x & 63, w = wave_id();
  if (NT < 4 && w >= NT) return;
  const int g = lane >> 4, cl = lane & 15;
#pragma unroll
  for (int ti = 0; ti < NT; ++ti) cr[ti] = ci[ti] = cd4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int tk = 0; tk < NT; ++tk) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int kk = 16 * tk + g + 4 * r;
      const cplx b = X(kk, 16 * w + cl);
#pragma unroll
      for (int ti = 0; ti < NT; ++ti) {
        const cplx a = A(16 * ti + cl, kk);
        cr[ti] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, cr[ti], 0, 0, 0);
        cr[ti] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b.y, cr[ti], 0, 0, 0);
        ci[ti] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.y, ci[ti], 0, 0, 0);
        ci[ti] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.x, ci[ti], 0, 0, 0);
      }
    }
  }
}

// C = B X as cgemm, with B the row-major n x n complex matrix at Bq in device
// memory.  The sixteen B entries of a k tile are loaded at once, from
// clamped in-range addresses (entries outside n x n zeroed after the load),
// and the next tile's loads are in flight while the current tile's MFMAs
// run: a load behind a per-entry branch would be waited for before the
// next one.
template <int NT, class XF>
__device__ __forceinline__ void cgemm_hbm(const cplx* Bq, int n, XF X, cd4 (&cr)[NT], cd4 (&ci)[NT]) {
  const int lane = threadIdx.x & 63, w = wave_id();
  if (NT < 4 && w >= NT) return;
  const int g = lane >> 4, cl = lane & 15;
  const auto* gB = (const __attribute__((address_space(1))) double*)Bq;
#pragma unroll
  for (int ti = 0; ti < NT; ++ti) cr[ti] = ci[ti] = cd4{0.0, 0.0, 0.0, 0.0};
  cplx a[2][4][NT];  // [buffer][r][ti]
  auto load = [&](int tk, cplx (&dst)[4][NT]) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int ti = 0; ti < NT; ++ti) {
        const int i = 16 * ti + cl, kk = 16 * tk + g + 4 * r;
        const size_t off = 2 * ((size_t)min(i, n - 1) * n + min(kk, n - 1));
        dst[r][ti] = cplx{gB[off], gB[off + 1]};
      }
  };
  load(0, a[0]);
#pragma unroll
  for (int tk = 0; tk < NT; ++tk) {
    if (tk + 1 < NT) load(tk + 1, a[(tk + 1) & 1]);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int kk = 16 * tk + g + 4 * r;
      const cplx b = X(kk, 16 * w + cl);
#pragma unroll
      for (int ti = 0; ti < NT; ++ti) {
        const bool ok = 16 * ti + cl < n && kk < n;
        const cplx av = a[tk & 1][r][ti];
        const double ax = ok ? av.x : 0.0, ay = ok ? av.y : 0.0;
        cr[ti] = __builtin_amdgcn_mfma_f64_16x16x4f64(ax, b.x, cr[ti], 0, 0, 0);
        cr[ti] = __builtin_amdgcn_mfma_f64_16x16x4f64(-ay, b.y, cr[ti], 0, 0, 0);
        ci[ti] = __builtin_amdgcn_mfma_f64_16x16x4f64(ax, b.y, ci[ti], 0, 0, 0);
        ci[ti] = __builtin_amdgcn_mfma_f64_16x16x4f64(ay, b.x, ci[ti], 0, 0, 0);
      }
    }
  }
}

// write the accumulators of cgemm to an LDS matrix, each column scaled by
// cs(c) and each row by rs(i)
template <int NT, class CS, class RS>
__device__ __forceinline__ void cstore(cplx* M, const cd4 (&cr)[NT], const cd4 (&ci)[NT], CS cs, RS rs) {
  const int lane = threadIdx.x & 63, w = wave_id();
  if (NT < 4 && w >= NT) return;
  const int g = lane >> 4, c = 16 * w + (lane & 15);
  const double sc = cs(c);
#pragma unroll
  for (int ti = 0; ti < NT; ++ti)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * ti + g + 4 * r;
      const double f = sc * rs(i);
      M[i * Dim<NT>::ld + c] = cplx{cr[ti][r] * f, ci[ti][r] * f};
    }
}

template <int NT>
__global__ __launch_bounds__(kCThreads, Dim<NT>::chain_groups) void k_greens_complex(const CChain* __restrict__ tab, int count) {
  __shared__ CCSmem<NT> S;
  constexpr int CN = Dim<NT>::cn, LD = Dim<NT>::ld;
  const int tid = threadIdx.x, lane = tid & 63, wv = wave_id();
  for (int b = blockIdx.x; b < count; b += gridDim.x) {
    const CChain C = tab[b];
    const int n = C.n, m = C.m, k = C.k;
    const cplx* Bs = reinterpret_cast<const cplx*>(C.slices);
    // W = U = 1, T = 1, D = 1; the padding of both matrices zero
    for (int e = tid; e < CN * LD; e += kCThreads) {
      const int i = e / LD, j = e % LD;
      const cplx one = {(i == j && i < n) ? 1.0 : 0.0, 0.0};
      S.a[e] = one;
      S.t[e] = one;
    }
    if (tid < CN) S.d[tid] = 1.0;
    __syncthreads();
    for (int q0 = 1; q0 <= m; q0 += k) {
      const int q1 = q0 + k - 1 < m ? q0 + k - 1 : m;
      // W <- B_q W for q = q0 .. q1; after the last, W <- W D
      for (int q = q0; q <= q1; ++q) {
        const cplx* Bq = Bs + (size_t)(q - 1) * n * n;
        cd4 cr[NT], ci[NT];
        cgemm_hbm<NT>(Bq, n, [&](int kk, int c) -> cplx { return S.a[kk * LD + c]; }, cr, ci);
        __syncthreads();
        const bool last = q == q1;
        cstore<NT>(S.a, cr, ci, [&](int c) { return last ? S.d[c] : 1.0; }, [](int) { return 1.0; });
        __syncthreads();
      }
      // pivoted QR, D <- |diag R|
      cpqr_lds<NT>(S.a, S.x, S.tau, S.jpvt, n);
      __syncthreads();
      if (tid < n) S.d[tid] = fabs(S.a[tid * LD + tid].x);
      if (tid >= n && tid < CN) S.jpvt[tid] = tid;
      __syncthreads();
      // T <- D^{-1} R P^T T: row i of the result is sum_{j >= i} R[i][j] T[jpvt[j]][:] / D_i
      {
        cd4 cr[NT], ci[NT];
        cgemm<NT>([&](int i, int j) -> cplx { return (i < n && j < n && j >= i) ? S.a[i * LD + j] : cplx{0.0, 0.0}; },
              [&](int j, int c) -> cplx { return S.t[S.jpvt[j] * LD + c]; }, cr, ci);
        __syncthreads();
        cstore<NT>(S.t, cr, ci, [](int) { return 1.0; },
               [&](int i) { return (i < n && S.d[i] > 0.0) ? 1.0 / S.d[i] : 1.0; });
        __syncthreads();
      }
      // U = Q in place
      form_q_lds<NT>(S.a, S.x, S.tau, n);
    }
    const cplx phu = det_q(S.tau, n);  // phase of det U: the reflectors of the last QR
    // M = D_p^{-1} U^H + D_m T into S.t (reads U, writes T's own entry)
    for (int e = tid; e < n * n; e += kCThreads) {
      const int i = e / n, j = e % n;
      const double di = S.d[i], dp = di > 1.0 ? di : 1.0, dm = di > 1.0 ? 1.0 : di;
      const cplx u = S.a[j * LD + i];
      const cplx t = S.t[i * LD + j];
      S.t[i * LD + j] = cplx{u.x / dp + dm * t.x, -u.y / dp + dm * t.y};
    }
    __syncthreads();
    // G = M^{-1} D_p^{-1} U^H through the pivoted QR of M: the right-hand
    // sides in registers (lane = column), Q^H applied by reflectors, then
    // back substitution with the rows of the result passed over LDS
    RegMat<NT> Y;
    each_row<NT>([&](int q, int t, int r) {
      const cplx u = S.a[min(lane, CN - 1) * LD + r];
      const double dp = r < n && S.d[r] > 1.0 ? S.d[r] : 1.0;
      Y.a[q][t] = r < n && lane < n ? cplx{u.x / dp, -u.y / dp} : cplx{0.0, 0.0};
    });
    __syncthreads();  // det_q has read tau
    cpqr_lds<NT>(S.t, S.x, S.tau, S.jpvt, n);
    apply_q<NT, true>(S.t, S.x, S.tau, n, Y);
    __syncthreads();
    if (tid < n) S.x.beta[tid] = 1.0 / S.x.beta[tid];
    __syncthreads();
    steps_down<NT>(n, [&](auto tile, int j) {
      constexpr int jq = decltype(tile)::q;
      cplx* row = S.x.row[j & 1];
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (16 * jq + 4 * t + wv == j) {
          const double rb = S.x.beta[j];
          Y.a[jq][t] = cplx{Y.a[jq][t].x * rb, Y.a[jq][t].y * rb};
          row[lane] = Y.a[jq][t];
        }
      __syncthreads();
      const cplx y = row[lane];
#pragma unroll
      for (int q = 0; q <= jq; ++q) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int r = 16 * q + 4 * t + wv;
          const cplx z = cmul(r < j ? S.t[r * LD + j] : cplx{0.0, 0.0}, y);
          Y.a[q][t].x -= z.x;
          Y.a[q][t].y -= z.y;
        }
      }
    });
    // det M: the diagonal of R, det Q and the sign of the permutation
    cplx phm = det_q(S.tau, n);
    double ldm = 0.0;
    if (wv == 0) {
      const double rb = lane < n ? S.x.beta[lane] : 1.0;
      ldm = wave_sum(-log(fabs(rb)));
      unsigned long long inv = __ballot(lane < n && rb < 0.0);
      int odd = __popcll(inv) & 1;
      const int pj = lane < n ? S.jpvt[lane] : lane;
      for (int j = 0; j < n; ++j) odd ^= __popcll(__ballot(lane > j && pj < __builtin_amdgcn_readlane(pj, j))) & 1;
      if (odd) phm = cplx{-phm.x, -phm.y};
    }
    // outputs
    int bad = 0;
    if (C.g) {
      cplx* G = reinterpret_cast<cplx*>(C.g);
      each_row<NT>([&](int q, int t, int r) {
        if (r >= n || lane >= n) return;
        const cplx x = Y.a[q][t];
        G[S.jpvt[r] * n + lane] = x;
        if (!isfinite(x.x) || !isfinite(x.y)) bad = 1;
      });
    }
    if (tid == 0) {
      double ldp = 0.0;
      for (int i = 0; i < n; ++i) ldp += log(S.d[i] > 1.0 ? S.d[i] : 1.0);
      const double ld = ldp + ldm;
      const double fr = phu.x * phm.x - phu.y * phm.y, fi = phu.x * phm.y + phu.y * phm.x;
      if (C.logdet) *C.logdet = ld;
      if (C.phase) {
        C.phase[0] = fr;
        C.phase[1] = fi;
      }
      if (!isfinite(ld) || !isfinite(fr) || !isfinite(fi)) bad = 1;
    }
    for (int i = tid; i < n; i += kCThreads)
      if (!isfinite(S.d[i]) || !(S.d[i] > 0.0)) bad = 1;
    if (__any(bad) && lane == 0 && C.status) atomicOr(C.status, kStatusRange);
    __syncthreads();
  }
}

}  // namespace

int complex_udt_max_n() { return kCN; }

// The variant of the smallest padded size; grid-stride over at most the
// workgroups that `cus` compute units hold.
template <class F>
hipError_t by_tiles(int n, F go) {
  if (n <= 16)
    go(TileNo<1>{});
  else if (n <= 32)
    go(TileNo<2>{});
  else if (n <= 48)
    go(TileNo<3>{});
  else
    go(TileNo<4>{});
  return hipGetLastError();
}

hipError_t launch_greens_complex(const CChain* tab, int count, int nmax, int cus, hipStream_t s) {
  if (count < 1 || cus < 1 || nmax < 1 || nmax > kCN) return hipErrorInvalidValue;
  return by_tiles(nmax, [&](auto tiles) {
    constexpr int NT = decltype(tiles)::q;
    const int grid = std::min(count, Dim<NT>::chain_groups * cus);
    hipLaunchKernelGGL(k_greens_complex<NT>, dim3(grid), dim3(kCThreads), 0, s, tab, count);
  });
}

hipError_t launch_udt_complex(int n, int count, const double* w, double* u, double* d, double* t, int cus,
                              hipStream_t s) {
  if (n < 1 || n > kCN || count < 1 || cus < 1) return hipErrorInvalidValue;
  return by_tiles(n, [&](auto tiles) {
    constexpr int NT = decltype(tiles)::q;
    const int grid = std::min(count, Dim<NT>::udt_groups * cus);
    hipLaunchKernelGGL(k_udt_complex<NT>, dim3(grid), dim3(kCThreads), 0, s, n, count, w, u, d, t);
  });
}

}  // namespace sdq
