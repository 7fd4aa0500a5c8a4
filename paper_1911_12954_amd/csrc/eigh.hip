// FP64 symmetric eigendecomposition of the HOSVD Gram matrices (Fig. 1B of
// the paper: the isometries are the leading eigenvectors of the two-site
// environment) and the selection of the truncated isometry.
//
// Eigensolver up to order 160: cyclic two-sided Jacobi in parallel (round-robin)
// order.  Each round rotates n/2 disjoint index pairs (A <- J^T A J, V <- V J); the
// workgroups of a matrix all rotate A and share the rows of V.  A sweep is n-1
// rounds; sweeps repeat until the off-diagonal Frobenius norm falls below
// 1e-14 of the matrix norm, plus one final sweep.  Above order 160:
// Householder reduction, with QL or with multisection and inverse iteration.
// Everything is deterministic: fixed pairing order, fixed reduction trees.
#include <algorithm>
#include <cmath>

#include "internal.h"

namespace trg {
namespace {

constexpr int MAX_N = 1024;
constexpr int MAX_SWEEPS = 40;

__device__ inline double wave_sum(double v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
__device__ inline double wave_max(double v) {
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}
// over the NW waves of a workgroup, in a fixed order; sh: NW doubles, free again after the next barrier
template <int NW, bool MAX>
__device__ inline double wg_reduce(double v, double *sh) {
  v = MAX ? wave_max(v) : wave_sum(v);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = sh[0];
  for (int i = 1; i < NW; ++i) r = MAX ? fmax(r, sh[i]) : r + sh[i];
  return r;
}

// 1 / sqrt(x) for x in a range where nothing overflows: the hardware estimate
// and two Newton steps
__device__ inline double jac_rsqrt(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = y * __builtin_fma(-0.5 * x * y, y, 1.5);
  return y * __builtin_fma(-0.5 * x * y, y, 1.5);
}

// Rotation (c, s), t = s / c that takes a_pq of [[app, apq], [apq, aqq]] to
// zero: t = x sgn(d) / (|d| + sqrt(d^2 + x^2)), d = aqq - app, x = 2 apq, both
// scaled by the power of two that brings the larger into [1, 2).  One chain
// of multiplications from hardware estimates instead of two square roots and
// three divisions; the last correction brings c^2 + s^2 back to 1 to a rounding, so
// that the vectors' norms do not drift over a run's thousands of rotations.
__device__ inline void jac_rotation(double app, double aqq, double apq, double &c, double &s, double &t) {
  double d = aqq - app, x = 2.0 * apq;
  int ex;
  (void)frexp(fmax(fabs(d), fabs(x)), &ex);
  d = ldexp(d, -ex);
  x = ldexp(x, -ex);
  const double hh = __builtin_fma(d, d, x * x);
  const double den = __builtin_fma(hh, jac_rsqrt(hh), fabs(d));
  double r = __builtin_amdgcn_rcp(den);
  r = __builtin_fma(r, __builtin_fma(-den, r, 1.0), r);
  r = __builtin_fma(r, __builtin_fma(-den, r, 1.0), r);
  x = copysign(1.0, d) * x;
  t = x * r;
  t = __builtin_fma(__builtin_fma(-den, t, x), r, t);
  c = jac_rsqrt(__builtin_fma(t, t, 1.0));
  s = t * c;
  const double e = 0.5 * __builtin_fma(-s, s, __builtin_fma(-c, c, 1.0));
  c = __builtin_fma(e, c, c);
  s = __builtin_fma(e, s, s);
}

// LDS of one workgroup: A over np players (its lower triangle, or all of it),
// rl rows of V (column by column), two sets of rotations, the reductions
constexpr int JAC_LDS = 160 * 1024;
constexpr size_t jac_fixed(int np, bool tri) {
  return size_t(np) * (tri ? np + 1 : 2 * np) / 2 * 8 + size_t(np) * 16 + 512;
}
static_assert(jac_fixed(JACOBI_MAX_N, true) + size_t(JACOBI_MAX_N) * 8 * 8 <= JAC_LDS, "eight rows of V fit");
static_assert(jac_fixed(JACOBI_SQUARE_N, false) + size_t(JACOBI_SQUARE_N) * 8 <= JAC_LDS, "a row of V fits");
__device__ inline int jac_tri(int x, int y) {   // x >= y
  return int(__umul24(x, x + 1) >> 1) + y;
}

// What bounds it: a round is a chain (three entries of A, the rotation, then
// every entry of A moves once), and there are n - 1 rounds a sweep.  Hence A's
// lower triangle in LDS, each 2 x 2 block of it taking both rotations in one
// visit; and V by rows over blockIdx.x: every workgroup of a matrix repeats the
// rotations of A (the same operations, the same bits) and applies them to its
// own rows of V, while its first waves work out the next round's rotations.
// Measured, six Gram-like and random matrices (square; triangle): order 16 0.14
// ms, 36 0.26, 64 1.7; 1.2, 100 4.0; 2.6, 144 7.3 (triangle), against 0.26, 0.7,
// 16.5, 46.6 and 180 ms with A and V in L2, rows and columns of all of A
// rotated in turn by one workgroup; |V^T V - 1| of order 100 1.2e-13 (square,
// as before), 5e-15 (triangle).
//
// TRI false keeps all of A and, operation for operation, the rotations of that
// slower form (hypot, two square roots, three divisions).  In a mixed-precision
// HOTRG run the sign and the pick among near-degenerate vectors hang on the
// last bits of the Grams' eigensystems, so a run that is continued from a state
// written by a library with the slower form would part from it after a few
// steps if the bits differed.  They agree as long as both forms stop at the
// same sweep: the norm that decides it is summed in another order, so one
// that falls within a rounding of the threshold may not.  HOTRG asks for this
// form up to order JACOBI_SQUARE_N; the matrices above it fit LDS as triangles only.
template <int NT, bool TRI>
__global__ void __launch_bounds__(NT)
jacobi_kernel(const double *Aall, double *wall, double *Vall, int *sweeps_out, int n, int rl, FastDiv by_n,
              FastDiv by_rl, FastDiv by_half) {
  extern __shared__ __attribute__((aligned(16))) double lds[];
  __shared__ double red[4][NT / 64];
  typedef double d2 __attribute__((ext_vector_type(2)));
  const int b = blockIdx.y, t = threadIdx.x, n2 = n * n;
  const double *Ag = Aall + size_t(b) * n2;
  double *Vg = Vall + size_t(b) * n2, *w = wall + size_t(b) * n;
  const int np = (n + 1) & ~1;   // even number of players; index n is a dummy of zeros
  const int half = np / 2, cyc = np - 1;
  const int row0 = blockIdx.x * rl, rows = n - row0 < rl ? n - row0 : rl;
  d2 *cs = reinterpret_cast<d2 *>(lds);   // rotations (16-byte aligned): set u, pair j at cs[u half + j]
  double *A = lds + 2 * np;
  const int elems = TRI ? np * (np + 1) / 2 : np * np;
  double *V = A + elems;
  // entry (x, y); the triangle needs x >= y
  auto at = [&](int x, int y) { return TRI ? jac_tri(x, y) : x * np + y; };
  for (int i = t; i < elems; i += NT) A[i] = 0.0;
  for (int i = t; i < np * rl; i += NT) {
    const int col = int(fast_div(i, by_rl));
    V[i] = col == row0 + i - col * rl ? 1.0 : 0.0;
  }
  __syncthreads();
  double fro = 0.0;
  for (int i = t; i < n2; i += NT) {
    const int x = int(fast_div(i, by_n)), y = i - x * n;
    const double v = Ag[i];
    if (!TRI || x >= y) A[at(x, y)] = v;
    fro += v * v;
  }
  const double norm2 = wg_reduce<NT / 64, false>(fro, red[0]);   // its barrier: A is complete

  // pairs of round r: player np - 1 against r, r + j against r - j (mod np - 1)
  auto players = [&](int r, int j, int &p, int &q) {
    int x = r + j < cyc ? r + j : r + j - cyc;
    int y = j == 0 ? cyc : (r - j >= 0 ? r - j : r - j + cyc);
    p = x < y ? x : y;
    q = x < y ? y : x;
  };
  auto rotate = [](d2 g, double &x, double &y) {
    const double nx = __builtin_fma(g.x, x, -(g.y * y));
    y = __builtin_fma(g.y, x, g.x * y);
    x = nx;
  };
  auto offdiag = [&](double *sh) {
    double v = 0.0;
    for (int x = 1 + (t >> 6); x < n; x += NT / 64)
      for (int y = t & 63; y < x; y += 64) {
        const double a = A[at(x, y)];
        v += a * a;
      }
    return 2.0 * wg_reduce<NT / 64, false>(v, sh);
  };
  // rotations of round r into set u, the 2 x 2 blocks on the diagonal included
  auto pivots = [&](int r, int u) {
    for (int j = t; j < half; j += NT) {
      int p, q;
      players(r, j, p, q);
      double c = 1.0, s = 0.0;
      const int iq = TRI ? jac_tri(q, p) : p * np + q;
      const double apq = A[iq];
      if constexpr (!TRI) {
        if (apq != 0.0) {
          const double tau = (A[q * np + q] - A[p * np + p]) / (2.0 * apq);
          const double tt = copysign(1.0, tau) / (fabs(tau) + hypot(1.0, tau));
          c = 1.0 / sqrt(1.0 + tt * tt);
          s = tt * c;
        }
      } else if (apq != 0.0) {
        const int ip = jac_tri(p, p), id = jac_tri(q, q);
        const double app = A[ip], aqq = A[id];
        double tt;
        jac_rotation(app, aqq, apq, c, s, tt);
        A[ip] = __builtin_fma(-tt, apq, app);
        A[id] = __builtin_fma(tt, apq, aqq);
        A[iq] = 0.0;
      }
      cs[u * half + j] = d2{c, s};
    }
  };
  // the blocks of pairs j1 < j2: rows j1 = i and half - 1 - i of the triangle of pairs side by side
  const int width = half - 1, lines = half / 2;   // half - 1 blocks in each of half / 2 lines (+ half a line)
  auto blocks = [&](int r, int u) {
    if constexpr (!TRI) {   // every block, the ones on the diagonal too
      for (int e = t; e < half * half; e += NT) {
        const int j1 = int(fast_div(e, by_half)), j2 = e - j1 * half;
        int p1, q1, p2, q2;
        players(r, j1, p1, q1);
        players(r, j2, p2, q2);
        const d2 g1 = cs[u * half + j1], g2 = cs[u * half + j2];
        double *x = A + p1 * np, *y = A + q1 * np;
        double a00 = x[p2], a01 = x[q2], a10 = y[p2], a11 = y[q2];
        rotate(g1, a00, a10);
        rotate(g1, a01, a11);
        rotate(g2, a00, a01);
        rotate(g2, a10, a11);
        x[p2] = a00;
        x[q2] = a01;
        y[p2] = a10;
        y[q2] = a11;
      }
      return;
    }
    for (int l = t >> 6; l < lines + (half & 1); l += NT / 64)
      for (int e = t & 63; e < width; e += 64) {
        const int first = half - 1 - l;           // blocks of row l: j2 = l + 1 ..
        int j1 = l, j2 = l + 1 + e;
        if (e >= first) {
          if (l == lines) continue;               // the middle row of an odd triangle stands alone
          j1 = half - 1 - l;
          j2 = j1 + 1 + e - first;
        }
        int p1, q1, p2, q2;
        players(r, j1, p1, q1);
        players(r, j2, p2, q2);
        const d2 g1 = cs[u * half + j1], g2 = cs[u * half + j2];
        double *e00 = A + (p1 > p2 ? jac_tri(p1, p2) : jac_tri(p2, p1));
        double *e01 = A + (p1 > q2 ? jac_tri(p1, q2) : jac_tri(q2, p1));
        double *e10 = A + (q1 > p2 ? jac_tri(q1, p2) : jac_tri(p2, q1));
        double *e11 = A + (q1 > q2 ? jac_tri(q1, q2) : jac_tri(q2, q1));
        double a00 = *e00, a01 = *e01, a10 = *e10, a11 = *e11;
        rotate(g1, a00, a10);
        rotate(g1, a01, a11);
        rotate(g2, a00, a01);
        rotate(g2, a10, a11);
        *e00 = a00;
        *e01 = a01;
        *e10 = a10;
        *e11 = a11;
      }
  };
  // this workgroup's rows of V, by the threads from t0 on
  auto vectors = [&](int r, int u, int t0) {
    for (int e = t - t0; e < half * rl; e += NT - t0) {
      const int j = int(fast_div(e, by_rl)), i = e - j * rl;
      int p, q;
      players(r, j, p, q);
      rotate(cs[u * half + j], V[p * rl + i], V[q * rl + i]);
    }
  };
  const int t0 = half <= 64 ? 64 : 128;   // threads below it compute rotations

  // converged once the off-diagonal norm is below 1e-14 of the matrix norm;
  // one more sweep then brings it to the rounding level
  int used = -1;
  bool last = false;
  for (int sweep = 0; sweep <= MAX_SWEEPS; ++sweep) {
    if (last) {
      used = sweep;
      break;
    }
    const double offs = offdiag(red[1 + (sweep & 1)]);
    if (offs == 0.0 || norm2 == 0.0) {
      used = sweep;
      break;
    }
    if (offs <= 1e-28 * norm2) last = true;
    if (sweep == MAX_SWEEPS) break;
    pivots(0, 0);
    __syncthreads();
    for (int r = 0; r < cyc; ++r) {
      const int u = r & 1;
      blocks(r, u);
      __syncthreads();
      if (t >= t0)
        vectors(r, u, t0);
      else if (r + 1 < cyc)
        pivots(r + 1, u ^ 1);
      __syncthreads();
    }
  }
  if (blockIdx.x == 0 && t == 0) sweeps_out[b] = used;

  // sort descending (ties by index): rank of each eigenvalue
  double *wdiag = lds;
  int *rank = reinterpret_cast<int *>(lds + np);
  __syncthreads();
  for (int i = t; i < n; i += NT) wdiag[i] = A[at(i, i)];
  __syncthreads();
  for (int i = t; i < n; i += NT) {
    const double v = wdiag[i];
    int rk = 0;
    for (int j = 0; j < n; ++j) rk += (wdiag[j] > v) || (wdiag[j] == v && j < i);
    rank[i] = rk;
    if (blockIdx.x == 0) w[rk] = v;
  }
  __syncthreads();
  for (int i = t; i < rows * n; i += NT) {
    const int x = int(fast_div(i, by_n)), col = i - x * n;
    Vg[(row0 + x) * n + rank[col]] = V[col * rl + x];
  }
}

template <int NT, bool TRI>
void launch_jacobi_as(const double *A, double *w, double *V, int *sweeps, int n, int batch, hipStream_t st) {
  static const bool attr = [] {   // dynamic LDS above 64 KB must be allowed per kernel
    TRG_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void *>(&jacobi_kernel<NT, TRI>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, JAC_LDS - 512));
    return true;
  }();
  (void)attr;
  // rows of V per workgroup: what LDS leaves, and as few as eight while the
  // matrices of the batch leave CUs idle
  const int np = (n + 1) & ~1;
  const int fit = int((JAC_LDS - jac_fixed(np, TRI)) / (size_t(np) * 8));
  const int groups = std::max(1, 256 / batch);
  const int rl = std::max(1, std::min(std::min(fit, n), std::max(8, (n + groups - 1) / groups)));
  const size_t lds = jac_fixed(np, TRI) - 512 + size_t(np) * rl * 8;
  hipLaunchKernelGGL((jacobi_kernel<NT, TRI>), dim3(uint32_t((n + rl - 1) / rl), uint32_t(batch)), dim3(NT), lds, st, A,
                     w, V, sweeps, n, rl, make_fastdiv(uint32_t(n)), make_fastdiv(uint32_t(rl)),
                     make_fastdiv(uint32_t(np / 2)));
}

// Two waves up to order 20, where a round has no more than 100 blocks.  The
// triangle from order 56 on unless the caller asks for the square: half the
// LDS traffic against more address arithmetic (six matrices: order 16 0.14 ms
// square, 0.24 triangle; 49 0.51, 0.65; 64 1.74, 1.18; 100 4.0, 2.6).
constexpr int JAC_TRI_N = 56;

void launch_jacobi(const double *A, double *w, double *V, int *sweeps, int n, int batch, bool square, hipStream_t st) {
  if (n < JAC_TRI_N || (square && n <= JACOBI_SQUARE_N)) {
    if (n <= 20)
      launch_jacobi_as<128, false>(A, w, V, sweeps, n, batch, st);
    else
      launch_jacobi_as<512, false>(A, w, V, sweeps, n, batch, st);
  } else {
    launch_jacobi_as<512, true>(A, w, V, sweeps, n, batch, st);
  }
}

// ------------------------------------------ tridiagonalisation + QL (large n) ---
// For larger orders a sweep-based Jacobi streams the whole matrix through one
// CU thousands of times.  This solver reduces A to tridiagonal form with
// Householder reflections (A <- H A H, H = I - 2 v v^T / v^T v, one column at
// a time), accumulates Q = H_0 H_1 ..., then diagonalises the tridiagonal
// matrix by implicit QL iterations with Wilkinson-type shifts; the QL step
// follows the order of the published tql2 procedure (Bowdler, Martin, Reinsch
// and Wilkinson, Numer. Math. 11 (1968) 293-306).  Thread 0 runs
// the scalar QL recurrence and records the Givens rotations of one sweep in
// LDS; all threads then apply the sweep to their rows of the eigenvector
// matrix.  Deterministic (fixed order everywhere).
constexpr int TQ_THREADS = 1024;
constexpr int TQ_MAX = 1024;
constexpr int TQ_CHUNK = 16;

__device__ inline double tq_max(double v, double *sh) {
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int s = TQ_THREADS / 2; s > 0; s >>= 1) {
    if (t < s) sh[t] = fmax(sh[t], sh[t + s]);
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

__device__ inline double tq_sum(double v, double *sh) {
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int s = TQ_THREADS / 2; s > 0; s >>= 1) {
    if (t < s) sh[t] += sh[t + s];
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

// out[j] = sum_i v[i] B[i][j] for the m x m block B (row stride ld) of a
// matrix in global memory, j < m: column j is summed by one thread, or by
// two (the upper and the lower half of the rows, added through w2) when 2 m
// fits the workgroup; loads go out eight at a time so that several are in
// flight per thread.  Ends with a barrier.
__device__ inline void tq_colvec(const double *B, int ld, int m, const double *v, double *out, double *w2, int t) {
  const bool split = 2 * m <= TQ_THREADS;
  const int half = split ? t / (TQ_THREADS / 2) : 0;
  const int j0 = split ? t % (TQ_THREADS / 2) : t;
  const int stride = split ? TQ_THREADS / 2 : TQ_THREADS;
  const int i0 = split ? half * (m / 2) : 0, i1 = split ? (half ? m : m / 2) : m;
  for (int j = j0; j < m; j += stride) {
    double a0 = 0.0, a1 = 0.0;
    int i = i0;
    for (; i + 8 <= i1; i += 8) {
      double x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = B[size_t(i + u) * ld + j];
#pragma unroll
      for (int u = 0; u < 8; u += 2) {
        a0 += x[u] * v[i + u];
        a1 += x[u + 1] * v[i + u + 1];
      }
    }
    for (; i < i1; ++i) a0 += B[size_t(i) * ld + j] * v[i];
    if (half) w2[j] = a0 + a1;
    else out[j] = a0 + a1;
  }
  __syncthreads();
  if (split)
    for (int j = t; j < m; j += TQ_THREADS) out[j] += w2[j];
  __syncthreads();
}

// Householder reduction of the symmetric n x n matrix A (global memory) to
// tridiagonal form, diagonal in dd and subdiagonal in ee (LDS); reflector k
// is left in column k of V (rows k+1..n-1), scaled so that H_k = I - u u^T.
// A is overwritten.  Every thread of the workgroup calls it.
__device__ void tq_tridiagonalise(double *A, double *V, int n, double *sh, double *vv, double *ww, double *w2,
                                  double *dd, double *ee) {
  const int t = threadIdx.x;
  for (int i = t; i < n * n; i += TQ_THREADS) V[i] = 0.0;
  __syncthreads();
  for (int k = 0; k + 2 < n; ++k) {
    const int m = n - k - 1;              // length of the column below the diagonal
    // The reflector is built from the column scaled by a power of two that
    // brings its largest entry into [1, 2): H = I - 2 v v^T / v^T v does not
    // depend on the scale of v, and sums of squares of columns far below
    // the matrix's scale (a parity block of a Gram whose weights are
    // 1e-150 of the other block's) neither underflow nor make tau overflow.
    double amax = 0.0;
    for (int i = t; i < m; i += TQ_THREADS) {
      const double x = A[(k + 1 + i) * n + k];
      vv[i] = x;
      amax = fmax(amax, fabs(x));
    }
    amax = tq_max(amax, sh);
    if (amax == 0.0) continue;           // column already reduced: H = I
    int ex;
    (void)frexp(amax, &ex);
    double s2 = 0.0;
    for (int i = t; i < m; i += TQ_THREADS) {
      const double x = ldexp(vv[i], -ex);
      vv[i] = x;
      s2 += x * x;
    }
    const double nrm2 = tq_sum(s2, sh);
    const double x0 = vv[0];
    const double alpha = x0 >= 0.0 ? -sqrt(nrm2) : sqrt(nrm2);
    const double vtv = nrm2 - 2.0 * alpha * x0 + alpha * alpha;  // |x - alpha e1|^2
    __syncthreads();
    if (t == 0) vv[0] = x0 - alpha;
    __syncthreads();
    if (!(vtv > 0.0)) continue;          // column already reduced: H = I
    const double tau = 2.0 / vtv;
    // p = tau A_sub v  (A symmetric: column access, coalesced across threads)
    tq_colvec(A + (k + 1) * n + (k + 1), n, m, vv, ww, w2, t);
    for (int j = t; j < m; j += TQ_THREADS) ww[j] *= tau;
    __syncthreads();
    double pv = 0.0;
    for (int i = t; i < m; i += TQ_THREADS) pv += ww[i] * vv[i];
    const double K = 0.5 * tau * tq_sum(pv, sh);
    for (int j = t; j < m; j += TQ_THREADS) ww[j] -= K * vv[j];   // w = p - K v
    __syncthreads();
    // A_sub <- A_sub - v w^T - w v^T (TQ_CHUNK independent elements per
    // thread loaded before any is stored, so their loads overlap)
    for (int base = t; base < m * m; base += TQ_THREADS * TQ_CHUNK) {
      double a[TQ_CHUNK];
#pragma unroll
      for (int u = 0; u < TQ_CHUNK; ++u) {
        const int idx = base + u * TQ_THREADS;
        if (idx < m * m) a[u] = A[(k + 1 + idx / m) * n + (k + 1 + idx % m)];
      }
#pragma unroll
      for (int u = 0; u < TQ_CHUNK; ++u) {
        const int idx = base + u * TQ_THREADS;
        if (idx < m * m) {
          const int i = idx / m, j = idx % m;
          A[(k + 1 + i) * n + (k + 1 + j)] = a[u] - (vv[i] * ww[j] + ww[i] * vv[j]);
        }
      }
    }
    for (int i = t; i < m; i += TQ_THREADS) {
      const double val = i == 0 ? ldexp(alpha, ex) : 0.0;
      A[(k + 1 + i) * n + k] = val;
      A[k * n + (k + 1 + i)] = val;
      V[(k + 1 + i) * n + k] = vv[i] * sqrt(tau);   // scaled: H = I - u u^T
    }
    __syncthreads();
  }
  for (int i = t; i < n; i += TQ_THREADS) {
    dd[i] = A[i * n + i];
    ee[i] = i + 1 < n ? A[(i + 1) * n + i] : 0.0;
  }
  __syncthreads();
}

__global__ void __launch_bounds__(TQ_THREADS)
tridiag_ql_kernel(double *Aall, double *wall, double *Vall, int *status, int n) {
  __shared__ double sh[TQ_THREADS];
  __shared__ double vv[TQ_MAX], ww[TQ_MAX], w2[TQ_MAX];
  __shared__ double dd[TQ_MAX], ee[TQ_MAX];
  __shared__ double rc[TQ_MAX], rs[TQ_MAX];
  __shared__ int rank[TQ_MAX];
  __shared__ int sweep_lo, sweep_hi, done_flag, iters_total;
  const int b = blockIdx.x;
  double *A = Aall + size_t(b) * n * n;
  double *V = Vall + size_t(b) * n * n;   // Householder vectors, then Q, then eigenvectors
  double *w = wall + size_t(b) * n;
  const int t = threadIdx.x;

  // ---- Householder tridiagonalisation; v_k stored in column k of V (rows k+1..n-1)
  tq_tridiagonalise(A, V, n, sh, vv, ww, w2, dd, ee);
  // ---- Q = H_0 H_1 ... H_{n-3}, built backwards in A (Q_k = H_k Q_{k+1})
  for (int i = t; i < n * n; i += TQ_THREADS) A[i] = (i / n == i % n) ? 1.0 : 0.0;
  __syncthreads();
  for (int k = n - 3; k >= 0; --k) {
    const int m = n - k - 1;
    for (int i = t; i < m; i += TQ_THREADS) vv[i] = V[(k + 1 + i) * n + k];
    __syncthreads();
    // ww[j] = sum_i u_i Q[k+1+i][k+1+j]; then Q_sub -= u ww^T
    tq_colvec(A + (k + 1) * n + (k + 1), n, m, vv, ww, w2, t);
    __syncthreads();
    for (int base = t; base < m * m; base += TQ_THREADS * TQ_CHUNK) {
      double a[TQ_CHUNK];
#pragma unroll
      for (int u = 0; u < TQ_CHUNK; ++u) {
        const int idx = base + u * TQ_THREADS;
        if (idx < m * m) a[u] = A[(k + 1 + idx / m) * n + (k + 1 + idx % m)];
      }
#pragma unroll
      for (int u = 0; u < TQ_CHUNK; ++u) {
        const int idx = base + u * TQ_THREADS;
        if (idx < m * m) {
          const int i = idx / m, j = idx % m;
          A[(k + 1 + i) * n + (k + 1 + j)] = a[u] - vv[i] * ww[j];
        }
      }
    }
    __syncthreads();
  }
  // ---- Z = Q^T into V (the Householder vectors are no longer needed), so
  // that a rotation of columns (i, i+1) of Q reads and writes two contiguous
  // rows of Z across the threads
  for (int idx = t; idx < n * n; idx += TQ_THREADS) {
    const int r = idx / n, c = idx % n;
    V[c * n + r] = A[idx];
  }
  __syncthreads();
  // ---- implicit QL on (dd, ee) with rotations applied to the columns of Q.
  // An off-diagonal entry deflates when it is at the rounding level of its
  // neighbours or of the whole matrix (anorm): next to rounding-level zero
  // diagonals (rank-deficient Grams) a purely relative test never fires.
  __shared__ double anorm;
  if (t == 0) {
    iters_total = 0;
    done_flag = 0;
    double md = 0.0, me = 0.0;
    for (int i = 0; i < n; ++i) {
      md = fmax(md, fabs(dd[i]));
      me = fmax(me, fabs(ee[i]));
    }
    anorm = md + me;
  }
  __syncthreads();
  for (int l = 0; l < n; ++l) {
    int iter = 0;
    while (true) {
      // Thread 0's sweep is one dependent chain of FP64 operations per
      // rotation, so each Givens rotation takes r, c, s from one reciprocal
      // square root refined by two Newton steps (y <- y (3 - x y^2) / 2
      // doubles the correct bits of the hardware estimate) instead of hypot
      // and two divisions; f and g are first scaled by the power of two that
      // brings the larger into [1, 2), so that f^2 + g^2 neither underflows
      // nor overflows (f = g = 0 is the zero rotation).
      if (t == 0) {
        int mm = l;
        for (; mm < n - 1; ++mm) {
          const double s = fabs(dd[mm]) + fabs(dd[mm + 1]);
          if (fabs(ee[mm]) <= 2.220446049250313e-16 * (s + anorm)) break;
        }
        done_flag = (mm == l) || iter >= 60;
        if (iter >= 60) iters_total = -1000000;
        sweep_lo = l;
        sweep_hi = l - 1;   // empty rotation list unless a sweep runs
        if (!done_flag) {
          double g = (dd[l + 1] - dd[l]) / (2.0 * ee[l]);
          double r = hypot(g, 1.0);
          g = dd[mm] - dd[l] + ee[l] / (g + (g >= 0.0 ? fabs(r) : -fabs(r)));
          double s = 1.0, c = 1.0, p = 0.0;
          int i = mm - 1;
          bool underflow = false;
          for (; i >= l; --i) {
            const double f = s * ee[i], bb = c * ee[i];
            const double a = fmax(fabs(f), fabs(g));
            if (a == 0.0) {
              ee[i + 1] = 0.0;
              dd[i + 1] -= p;
              ee[mm] = 0.0;
              underflow = true;
              break;
            }
            int ex;
            (void)frexp(a, &ex);
            const double fs = ldexp(f, -ex), gs = ldexp(g, -ex);
            const double x = fma(fs, fs, gs * gs);   // in [1/4, 2)
            double y = __builtin_amdgcn_rsq(x);
            y = y * fma(-0.5 * x * y, y, 1.5);
            y = y * fma(-0.5 * x * y, y, 1.5);
            r = ldexp(x * y, ex);
            ee[i + 1] = r;
            s = fs * y;
            c = gs * y;
            g = dd[i + 1] - p;
            r = (dd[i] - g) * s + 2.0 * c * bb;
            p = s * r;
            dd[i + 1] = g + p;
            g = c * r - bb;
            rc[i] = c;
            rs[i] = s;
          }
          sweep_hi = mm - 1;
          sweep_lo = underflow ? i + 1 : l;
          if (!underflow) {
            dd[l] -= p;
            ee[l] = g;
            ee[mm] = 0.0;
          }
          ++iters_total;
        }
      }
      __syncthreads();
      if (done_flag) break;
      // rotations i = hi down to lo act on columns (i, i+1) of every row of
      // Q, i.e. on rows (i, i+1) of Z; the new entry i is carried in a
      // register into the next rotation.  Entries are read TQ_CHUNK at a
      // time before any of them is written back (each rotation reads entry
      // i and writes entry i + 1, so a chunk's reads all precede its
      // writes), which keeps TQ_CHUNK loads in flight instead of one.
      const int lo = sweep_lo, hi = sweep_hi;
      if (hi >= lo) {
        for (int row = t; row < n; row += TQ_THREADS) {
          double *z = V + row;
          double carry = z[size_t(hi + 1) * n];
          for (int i0 = hi; i0 >= lo; i0 -= TQ_CHUNK) {
            const int cnt = i0 - lo + 1 < TQ_CHUNK ? i0 - lo + 1 : TQ_CHUNK;
            double v[TQ_CHUNK];
#pragma unroll
            for (int u = 0; u < TQ_CHUNK; ++u)
              if (u < cnt) v[u] = z[size_t(i0 - u) * n];
#pragma unroll
            for (int u = 0; u < TQ_CHUNK; ++u)
              if (u < cnt) {
                const int i = i0 - u;
                const double zi = v[u], f = carry;
                v[u] = rs[i] * zi + rc[i] * f;      // new entry i + 1
                carry = rc[i] * zi - rs[i] * f;
              }
#pragma unroll
            for (int u = 0; u < TQ_CHUNK; ++u)
              if (u < cnt) z[size_t(i0 - u + 1) * n] = v[u];
          }
          z[size_t(lo) * n] = carry;
        }
      }
      ++iter;
      __syncthreads();
    }
  }
  if (t == 0) status[b] = iters_total >= 0 ? iters_total : -1;
  // ---- sort descending (ties by index) and write w, V
  for (int i = t; i < n; i += TQ_THREADS) {
    const double v = dd[i];
    int rk = 0;
    for (int j = 0; j < n; ++j) rk += (dd[j] > v) || (dd[j] == v && j < i);
    rank[i] = rk;
  }
  __syncthreads();
  for (int i = t; i < n; i += TQ_THREADS) w[rank[i]] = dd[i];
  // eigenvector col = row col of Z, sorted into column rank[col] of V
  for (int i = t; i < n * n; i += TQ_THREADS) {
    const int col = i / n, row = i % n;
    A[row * n + rank[col]] = V[i];
  }
  __syncthreads();
  for (int i = t; i < n * n; i += TQ_THREADS) V[i] = A[i];
}

// ------------------------------------------ leading eigenpairs (large n) ---
// The isometry selection needs every eigenvalue (the discarded weight, the
// degenerate-cut flag, the spectrum record) but the eigenvectors only of the
// kept indices and of the rest of a cluster of near-degenerate eigenvalues
// that the cut splits.  No serial QL sweeps, no n x n rotation accumulation:
//   1. Householder reduction to tridiagonal T: one launch per column while
//      more than TD_LDS columns remain (td_column_kernel, many workgroups per
//      matrix), the rest in LDS (td_finish_kernel, one workgroup);
//   2. T splits into blocks where an off-diagonal is negligible against its
//      neighbours or exactly zero (as between the parity sectors of a
//      sector-ordered matrix); every eigenvalue of every block by
//      multisection on Sturm counts (td_values_kernel);
//   3. sorted descending; the number kk of vectors needed: k, extended while
//      the next eigenvalue continues a cluster (gap <= cluster_rel *
//      lambda_max);
//   4. inverse iteration for the kk vectors at once, one lane per vector: LU
//      with partial pivoting of T_b - lambda I (pivots below eps ||T_b||
//      raised to that size), three solves from fixed start vectors, each
//      followed by Gram-Schmidt in descending order (td_vectors_kernel;
//      Wilkinson, The Algebraic Eigenvalue Problem, 1965, ch. 5 and 9);
//   5. back-transformation by the reflectors, one wave per vector
//      (td_back_kernel); V gets the kk vectors as its leading columns (zeros
//      elsewhere), w every eigenvalue, status the number of vectors computed.
// What bounds it is latency: a column's reflector needs the whole previous
// update, and each recurrence along T is a chain of divisions.  Measured:
// 9.4 ms for six matrices of order 576 with 24 vectors (448 columns of 10 us,
// 0.6 ms in LDS, values 1.1, vectors 1.6) and 2.0 ms for two of order 196 (68
// columns of 7 us, 0.6 in LDS, 0.4, 0.4), against 81 and 11.2 ms with one
// workgroup per matrix for all of it (140 us a column at order 576: 2.6 MB
// through one CU and 33 barriers).  Columns that are zero already (diagonal and
// block-diagonal matrices) change nothing and are passed over; what they leave
// is their launch (order 576, two matrices: diagonal 2.4 ms, blocks of 8 5.2, zero
// with all 576 vectors 6.0; 5.5, 5.7 and 71 with every column worked through and
// every pair of vectors orthogonalised).  The column and finish kernels hold the
// pointers of TdScratch in private memory (120 bytes per lane), because p and v
// are indexed by the parity of the column.
constexpr int TD_THREADS = 256, TD_WAVES = TD_THREADS / 64;
constexpr int TD_LDS = 128;          // order from which the trailing matrix lives in LDS
constexpr int TD_FIN = 1024;         // threads of td_finish_kernel and td_vectors_kernel
constexpr int TOP_ITERS = 3;
constexpr int TD_CHUNK = 64;         // vectors solved together: lanes of a wave
constexpr int TD_MS = 16;            // multisection points per eigenvalue
// doubles of scratch per n beside two n x n matrices; td_scratch uses 77 of them
constexpr int TOP_SCRATCH = 96;

constexpr double TD_ZERO = -1.0;     // tau of a column with nothing below the diagonal

// fixed start vector of inverse iteration: entries in [-1, 1) from a hash of
// the vector's rank and the entry's index
__device__ inline double top_start(int r, int i) {
  uint32_t x = uint32_t(r) * 0x9E3779B1u ^ (uint32_t(i) + 0x7F4A7C15u) * 0x85EBCA77u;
  x ^= x >> 15;
  x *= 0x2C1B3C6Du;
  x ^= x >> 12;
  x *= 0x297A2D39u;
  x ^= x >> 15;
  return double(x) * (2.0 / 4294967296.0) - 1.0;
}

// scratch of one matrix (offsets in units of n doubles from its end of work)
struct TdScratch {
  double *dd, *ee, *lam, *p[2], *v[2];         // diagonal, subdiagonal, eigenvalues by slot, A v and v of a column
  double *tau;                                 // of each reflector, or TD_ZERO
  double *eb;                                  // subdiagonal with zeros between the blocks
  int *s0, *e0, *kk;                           // block of each slot, vectors needed
  unsigned long long *piv;                     // row swaps of the LU, one bit per lane
  double *X;                                   // iterates of a chunk, [entry][lane]
};
__device__ inline TdScratch td_scratch(double *scr, int n) {
  TdScratch t;
  t.dd = scr;
  t.ee = scr + n;
  t.lam = scr + 2 * n;
  t.p[0] = scr + 3 * n;
  t.p[1] = scr + 4 * n;
  t.v[0] = scr + 5 * n;
  t.v[1] = scr + 6 * n;
  t.tau = scr + 7 * n;
  t.eb = scr + 8 * n;
  t.s0 = reinterpret_cast<int *>(scr + 9 * n);
  t.e0 = reinterpret_cast<int *>(scr + 10 * n);
  t.kk = reinterpret_cast<int *>(scr + 11 * n);
  t.piv = reinterpret_cast<unsigned long long *>(scr + 12 * n);
  t.X = scr + 13 * n;                          // 64 n
  return t;
}
__device__ inline double *td_work(double *work, int n, int b) {
  return work + size_t(b) * (size_t(2) * n * n + size_t(TOP_SCRATCH) * n);
}

// Reflector of the column x (entries k+1.. of length m, in vv), scaled by a
// power of two that brings its largest entry into [1, 2): H = I - tau v v^T
// does not depend on the scale of v, and sums of squares of columns far below
// the matrix's scale (a parity block of a Gram whose weights are 1e-150 of
// the other block's) neither underflow nor make tau overflow.  vv becomes v
// (zero and tau = 0 for a column that is reduced already); returns the new
// subdiagonal entry.  zero: every entry is exactly 0 (a NaN among them is not),
// so that nothing of the trailing matrix changes.  Every thread calls it; vv is
// complete after it.
template <int NT>
__device__ inline double td_reflector(double *vv, int m, double &tau, bool &zero, double *sh0, double *sh1) {
  const int t = threadIdx.x;
  double amax = 0.0;
  for (int i = t; i < m; i += NT) amax = fmax(amax, fabs(vv[i]));
  amax = wg_reduce<NT / 64, true>(amax, sh0);
  int ex = 0;
  if (amax > 0.0) (void)frexp(amax, &ex);
  double s2 = 0.0;
  for (int i = t; i < m; i += NT) {
    const double x = ldexp(vv[i], -ex);
    s2 += x * x;
  }
  const double raw0 = vv[0];
  const double nrm2 = wg_reduce<NT / 64, false>(s2, sh1);   // its barrier: raw0 is read everywhere
  zero = nrm2 == 0.0;
  const double x0 = ldexp(raw0, -ex);
  const double alpha = x0 >= 0.0 ? -sqrt(nrm2) : sqrt(nrm2);
  const double vtv = nrm2 - 2.0 * alpha * x0 + alpha * alpha;  // |x - alpha e1|^2
  const bool on = amax > 0.0 && vtv > 0.0;
  tau = on ? 2.0 / vtv : 0.0;
  for (int i = t; i < m; i += NT) vv[i] = on ? (i == 0 ? x0 - alpha : ldexp(vv[i], -ex)) : 0.0;
  __syncthreads();
  return on ? ldexp(alpha, ex) : raw0;
}

// Column k: every workgroup of a matrix rebuilds w of column k - 1 from its
// product p = A v, brings row k up to date and forms the reflector of column
// k; then each wave updates its rows of the trailing matrix with column k - 1
// and multiplies them by the new v in the same pass, so the matrix is read and
// written once per column, and not at all when both columns are zero.
__global__ void __launch_bounds__(TD_THREADS)
td_column_kernel(double *Aall, double *workall, int n, int k) {
  __shared__ double vo[MAX_N], wo[MAX_N], vn[MAX_N];
  __shared__ double sh[3][TD_WAVES];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  double *A = Aall + size_t(blockIdx.y) * n * n;
  double *work = td_work(workall, n, blockIdx.y);
  TdScratch T = td_scratch(work + size_t(2) * n * n, n);
  const int m = n - k - 1;                 // trailing order; entry i of vn is row k + 1 + i
  const double *p = T.p[(k + 1) & 1], *vp = T.v[(k + 1) & 1];
  const double tau_o = k > 0 ? T.tau[k - 1] : TD_ZERO;
  const bool still = tau_o < 0.0;          // column k - 1 leaves the matrix as it is
  if (!still) {
    // vo, wo: entries of rows k .. n - 1
    double pv = 0.0;
    for (int i = t; i <= m; i += TD_THREADS) {
      vo[i] = vp[i];
      wo[i] = tau_o * p[i];
      pv += wo[i] * vo[i];
    }
    const double K = 0.5 * tau_o * wg_reduce<TD_WAVES, false>(pv, sh[0]);
    for (int i = t; i <= m; i += TD_THREADS) wo[i] -= K * vo[i];
  } else {
    for (int i = t; i <= m; i += TD_THREADS) vo[i] = wo[i] = 0.0;
  }
  __syncthreads();
  const double v0 = vo[0], w0 = wo[0];
  const double *row = A + size_t(k) * n + k;
  for (int i = t; i < m; i += TD_THREADS) vn[i] = row[1 + i] - (v0 * wo[1 + i] + w0 * vo[1 + i]);
  __syncthreads();
  double tau;
  bool zero;
  const double sub = td_reflector<TD_THREADS>(vn, m, tau, zero, sh[1], sh[2]);
  if (blockIdx.x == 0) {
    double *u = work + size_t(k) * n;      // reflector k, scaled: H = I - u u^T
    const double st = sqrt(tau);
    for (int i = t; i < n; i += TD_THREADS) u[i] = i > k ? vn[i - k - 1] * st : 0.0;
    double *vk = T.v[k & 1];
    for (int i = t; i < m; i += TD_THREADS) vk[i] = vn[i];
    if (t == 0) {
      T.dd[k] = row[0] - 2.0 * v0 * w0;
      T.ee[k] = sub;
      T.tau[k] = zero ? TD_ZERO : tau;
    }
  }
  if (still && zero) return;
  // rows of this wave, two at a time
  const int nw = gridDim.x * TD_WAVES;
  double *pk = T.p[k & 1];
  for (int i0 = (blockIdx.x * TD_WAVES + wave) * 2; i0 < m; i0 += 2 * nw) {
    const bool two = i0 + 1 < m;
    double *r0 = A + size_t(k + 1 + i0) * n + k + 1, *r1 = two ? r0 + n : r0;
    const double a0 = vo[1 + i0], b0 = wo[1 + i0], a1 = two ? vo[2 + i0] : a0, b1 = two ? wo[2 + i0] : b0;
    double s0 = 0.0, s1 = 0.0;
#pragma unroll 4
    for (int j = lane; j < m; j += 64) {
      const double wj = wo[1 + j], vj = vo[1 + j], nj = vn[j];
      const double x0 = r0[j] - (a0 * wj + b0 * vj), x1 = r1[j] - (a1 * wj + b1 * vj);
      r0[j] = x0;
      if (two) r1[j] = x1;
      s0 += x0 * nj;
      s1 += x1 * nj;
    }
    s0 = wave_sum(s0);
    s1 = wave_sum(s1);
    if (lane == 0) {
      pk[i0] = s0;
      if (two) pk[i0 + 1] = s1;
    }
  }
}

// The last columns (trailing order q = n - k0 <= TD_LDS) with the matrix in LDS
constexpr int TD_LD = TD_LDS + 1;

__global__ void __launch_bounds__(TD_FIN)
td_finish_kernel(const double *Aall, double *workall, int n, int k0) {
  extern __shared__ double L[];            // TD_LDS x TD_LD
  __shared__ double vo[TD_LDS], wo[TD_LDS], part[8][TD_LDS];
  __shared__ double sh[3][TD_FIN / 64];
  const int t = threadIdx.x;
  const double *A = Aall + size_t(blockIdx.x) * n * n;
  double *work = td_work(workall, n, blockIdx.x);
  TdScratch T = td_scratch(work + size_t(2) * n * n, n);
  const int q = n - k0;
  {
    const double *p = T.p[(k0 + 1) & 1], *vp = T.v[(k0 + 1) & 1];
    const double tau_o = k0 > 0 ? T.tau[k0 - 1] : TD_ZERO;
    const bool still = tau_o < 0.0;
    const double tau = still ? 0.0 : tau_o;
    double pv = 0.0;
    if (t < q) {
      vo[t] = still ? 0.0 : vp[t];
      wo[t] = still ? 0.0 : tau * p[t];
      pv = wo[t] * vo[t];
    }
    const double K = 0.5 * tau * wg_reduce<TD_FIN / 64, false>(pv, sh[0]);
    if (t < q) wo[t] -= K * vo[t];
    __syncthreads();
    bool off = false;
    for (int idx = t; idx < q * q; idx += TD_FIN) {
      const int i = idx / q, j = idx - i * q;
      const double x = A[size_t(k0 + i) * n + k0 + j] - (vo[i] * wo[j] + wo[i] * vo[j]);
      L[i * TD_LD + j] = x;
      off = off || (i != j && !(x == 0.0));
    }
    if (!__syncthreads_or(off)) {          // diagonal: no reflector, and td_back_kernel reads none
      if (t < q) {
        T.dd[k0 + t] = L[t * TD_LD + t];
        T.ee[k0 + t] = 0.0;
        T.tau[k0 + t] = TD_ZERO;
      }
      return;
    }
  }
  // thread (g, c) of 8 x 128: column c, every eighth row
  const int c = t & (TD_LDS - 1), g = t / TD_LDS;
  for (int s = 0; s + 2 < q; ++s) {
    const int m = q - s - 1, k = k0 + s;
    double *sub = L + (s + 1) * TD_LD + s + 1;   // trailing m x m
    if (t < m) vo[t] = L[s * TD_LD + s + 1 + t];
    __syncthreads();
    double tau;
    bool zero;
    const double off = td_reflector<TD_FIN>(vo, m, tau, zero, sh[0], sh[1]);
    if (!zero) {
      double a = 0.0;
      if (c < m)
        for (int i = g; i < m; i += 8) a += sub[i * TD_LD + c] * vo[i];
      part[g][c] = a;
      __syncthreads();
      double pv = 0.0;
      if (t < m) {
        double x = part[0][t];
        for (int u = 1; u < 8; ++u) x += part[u][t];
        wo[t] = tau * x;
        pv = wo[t] * vo[t];
      }
      const double K = 0.5 * tau * wg_reduce<TD_FIN / 64, false>(pv, sh[2]);
      if (t < m) wo[t] -= K * vo[t];
      __syncthreads();
      if (c < m) {
        const double vc = vo[c], wc = wo[c];
        for (int i = g; i < m; i += 8) sub[i * TD_LD + c] -= vo[i] * wc + wo[i] * vc;
      }
    }
    double *u = work + size_t(k) * n;
    const double st = sqrt(tau);
    for (int i = t; i < n; i += TD_FIN) u[i] = i > k ? vo[i - k - 1] * st : 0.0;
    if (t == 0) {
      T.dd[k] = L[s * TD_LD + s];
      T.ee[k] = off;
      T.tau[k] = zero ? TD_ZERO : tau;
    }
    __syncthreads();
  }
  if (t == 0) {
    const int e = q - 2;
    T.dd[n - 2] = L[e * TD_LD + e];
    T.ee[n - 2] = L[(e + 1) * TD_LD + e];
    T.dd[n - 1] = L[(e + 1) * TD_LD + e + 1];
    T.ee[n - 1] = 0.0;
  }
}

// Eigenvalues of T, TD_MS lanes each: every lane counts the eigenvalues of
// its slot's block below one of TD_MS equally spaced points, so a pass
// shrinks the interval 17-fold (14 passes to the rounding level instead of 55
// halvings, each a chain of n divisions).
__global__ void __launch_bounds__(TD_THREADS)
td_values_kernel(double *workall, int n) {
  __shared__ double dd[MAX_N], ee[MAX_N], ee2[MAX_N];
  __shared__ int s0s[MAX_N], e0s[MAX_N];
  const int t = threadIdx.x, lane = t & 63;
  double *work = td_work(workall, n, blockIdx.y);
  TdScratch T = td_scratch(work + size_t(2) * n * n, n);
  const double eps = 2.220446049250313e-16;
  for (int i = t; i < n; i += TD_THREADS) {
    dd[i] = T.dd[i];
    ee[i] = T.ee[i];
  }
  __syncthreads();
  for (int i = t; i < n; i += TD_THREADS) {
    // negligible against its neighbours or exactly zero: a block ends at i
    double e = ee[i];
    if (i + 1 < n && fabs(e) <= eps * sqrt(fabs(dd[i])) * sqrt(fabs(dd[i + 1]))) e = 0.0;
    ee2[i] = i + 1 < n ? e : 0.0;
  }
  __syncthreads();
  if (t < 64) {   // block bounds of every slot, 64 slots at a time
    int start = 0;
    for (int base = 0; base < n; base += 64) {
      const int i = base + lane;
      const unsigned long long ends = __ballot(i > 0 && i < n && ee2[i > 0 ? i - 1 : 0] == 0.0);
      const unsigned long long upto = ends & (~0ull >> (63 - lane));
      if (i < n) s0s[i] = upto ? base + 63 - __clzll(upto) : start;
      if (ends) start = base + 63 - __clzll(ends);
    }
    int stop = n;
    for (int base = (n - 1) / 64 * 64; base >= 0; base -= 64) {
      const int i = base + lane;
      const unsigned long long ends = __ballot(i < n && ee2[i < n ? i : 0] == 0.0);
      const unsigned long long from = ends & (~0ull << lane);
      if (i < n) e0s[i] = from ? base + __ffsll(from) : stop;
      if (ends) stop = base + __ffsll(ends);
    }
  }
  __syncthreads();
  for (int i = t; i < n; i += TD_THREADS) {
    const double e = ee2[i];
    if (blockIdx.x == 0) {
      T.eb[i] = e;   // not over T.ee, which other workgroups may still be reading
      T.s0[i] = s0s[i];
      T.e0[i] = e0s[i];
    }
    ee[i] = e;
    ee2[i] = e * e;
  }
  __syncthreads();
  const int slot = (blockIdx.x * TD_THREADS + t) / TD_MS, l = t % TD_MS;
  if (slot >= n) return;   // whole groups of TD_MS lanes
  const int s0 = s0s[slot], e0 = e0s[slot];
  if (e0 - s0 == 1 && isfinite(dd[s0])) {   // a block of one entry is its own eigenvalue
    if (l == 0) T.lam[slot] = dd[s0];
    return;
  }
  const int target = e0 - slot;   // (slot - s0 + 1)-th largest = target-th smallest
  double lo = 0.0, hi = 0.0, emax2 = 0.0;
  for (int i = s0 + l; i < e0; i += TD_MS) {
    const double r = (i > s0 ? fabs(ee[i - 1]) : 0.0) + (i + 1 < e0 ? fabs(ee[i]) : 0.0);
    lo = i == s0 + l ? dd[i] - r : fmin(lo, dd[i] - r);
    hi = i == s0 + l ? dd[i] + r : fmax(hi, dd[i] + r);
    if (i + 1 < e0) emax2 = fmax(emax2, ee2[i]);
  }
  const bool any = s0 + l < e0;
  if (!any) {
    lo = 1.7976931348623157e308;
    hi = -1.7976931348623157e308;
  }
  for (int off = TD_MS / 2; off > 0; off >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, off, 64));
    hi = fmax(hi, __shfl_xor(hi, off, 64));
    emax2 = fmax(emax2, __shfl_xor(emax2, off, 64));
  }
  const double bn = fmax(fabs(lo), fabs(hi));
  const double pivmin = 2.2250738585072014e-308 * fmax(1.0, emax2);
  lo -= 2.0 * eps * bn + pivmin;
  hi += 2.0 * eps * bn + pivmin;
  for (int it = 0; it < 120; ++it) {
    const double mid = 0.5 * (lo + hi);
    if (!(mid > lo && mid < hi) || hi - lo <= 2.0 * eps * fmax(fabs(lo), fabs(hi)) + pivmin) break;
    double x = lo + (hi - lo) * (double(l + 1) * (1.0 / (TD_MS + 1)));
    x = fmin(fmax(x, lo), hi);
    // Sturm count: eigenvalues of the block below x
    int cnt = 0;
    double q = dd[s0] - x;
    if (fabs(q) < pivmin) q = -pivmin;
    cnt += q < 0.0;
    for (int i = s0 + 1; i < e0; ++i) {
      q = (dd[i] - x) - ee2[i - 1] / q;
      if (fabs(q) < pivmin) q = -pivmin;
      cnt += q < 0.0;
    }
    // the first point with enough eigenvalues below it bounds the slot's from above
    const unsigned mine = unsigned(__ballot(cnt >= target) >> (lane & ~(TD_MS - 1))) & ((1u << TD_MS) - 1);
    const int f = mine ? __ffs(mine) - 1 : TD_MS;
    const double xf = __shfl(x, (lane & ~(TD_MS - 1)) + (f < TD_MS ? f : TD_MS - 1), 64);
    const double xb = __shfl(x, (lane & ~(TD_MS - 1)) + (f > 0 ? f - 1 : 0), 64);
    const double nhi = f < TD_MS ? xf : hi, nlo = f > 0 ? xb : lo;
    if (nlo == lo && nhi == hi) break;     // the points no longer separate the ends
    lo = nlo;
    hi = nhi;
  }
  if (l == 0) T.lam[slot] = 0.5 * (lo + hi);
}

// Sorting, the number of vectors and the inverse iteration of one matrix.
// A and V (n x n each, free by now) hold the LU factors of a chunk.
__global__ void __launch_bounds__(TD_FIN)
td_vectors_kernel(double *Aall, double *wall, double *Vall, int *status, int n, int k, double cluster_rel,
                  double *workall) {
  __shared__ double dd[MAX_N], ee[MAX_N], lam[MAX_N], w[MAX_N];
  __shared__ int slot_of[MAX_N], s0_of[MAX_N], e0_of[MAX_N];   // by rank: slot, bounds of its block
  __shared__ int kk_s;
  const int b = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = t >> 6;
  double *work = td_work(workall, n, b);
  TdScratch T = td_scratch(work + size_t(2) * n * n, n);
  double *Zv = work + size_t(n) * n;       // vector of rank r in row r
  double *D = Aall + size_t(b) * n * n, *DL = D + size_t(TD_CHUNK) * n;
  double *DU = Vall + size_t(b) * n * n, *DU2 = DU + size_t(TD_CHUNK) * n;
  const double eps = 2.220446049250313e-16;
  for (int i = t; i < n; i += TD_FIN) {
    dd[i] = T.dd[i];
    ee[i] = T.eb[i];
    const double v = T.lam[i];
    lam[i] = v == v ? v : INFINITY;
  }
  __syncthreads();
  // ---- sort descending (ties by slot).  NaN, the spectrum of a matrix that is
  // not finite, sorts as infinity: the ranks are a permutation of the slots
  // whatever the matrix holds, so every slot_of that is read has been written
  // and every block bound taken from it lies inside the matrix.
  for (int slot = t; slot < n; slot += TD_FIN) {
    const double key = lam[slot], v = T.lam[slot];
    int rk = 0;
    for (int u = 0; u < n; ++u) rk += (lam[u] > key) || (lam[u] == key && u < slot);
    w[rk] = v;
    slot_of[rk] = slot;
    s0_of[rk] = T.s0[slot];
    e0_of[rk] = T.e0[slot];
    wall[size_t(b) * n + rk] = v;
  }
  __syncthreads();
  if (t == 0) {
    const double tol = cluster_rel * fmax(w[0], 0.0);
    int bnd = k < n ? k : n;
    while (bnd < n && w[bnd - 1] - w[bnd] <= tol) ++bnd;
    kk_s = bnd;
    status[b] = bnd;
    *T.kk = bnd;
  }
  __syncthreads();
  const int kk = kk_s;
  const int chunks = (kk + TD_CHUNK - 1) / TD_CHUNK;
  for (int it = 0; it < TOP_ITERS; ++it) {
    for (int ch = 0; ch < chunks; ++ch) {
      const int r0 = ch * TD_CHUNK, nr = kk - r0 < TD_CHUNK ? kk - r0 : TD_CHUNK;
      // iterates of the chunk, transposed: X[i][lane] = entry i of the lane's block
      for (int idx = t; idx < nr * n; idx += TD_FIN) {
        const int r = idx / n, i = idx - r * n, s = slot_of[r0 + r], s0 = T.s0[s], e0 = T.e0[s];
        if (i < e0 - s0) T.X[size_t(i) * TD_CHUNK + r] = it == 0 ? top_start(r0 + r, i) : Zv[size_t(r0 + r) * n + s0 + i];
        if (it == 0 && (i < s0 || i >= e0)) Zv[size_t(r0 + r) * n + i] = 0.0;
      }
      __syncthreads();
      if (wave == 0 && lane < nr) {
        const int s = slot_of[r0 + lane], s0 = T.s0[s], nb = T.e0[s] - s0;
        const double sigma = w[r0 + lane];
        double bnorm = 0.0;
        for (int i = s0; i < s0 + nb; ++i)
          bnorm = fmax(bnorm, fabs(dd[i]) + (i > s0 ? fabs(ee[i - 1]) : 0.0) + (i + 1 < s0 + nb ? fabs(ee[i]) : 0.0));
        const double ptol = fmax(eps * bnorm, 2.2250738585072014e-308);
        auto inverse = [&](double piv) {
          if (fabs(piv) < ptol) piv = piv >= 0.0 ? ptol : -ptol;
          return 1.0 / piv;
        };
        double *X = T.X + lane, *d = D + lane, *dl = DL + lane, *du = DU + lane, *du2 = DU2 + lane;
        // LU with partial pivoting of T_b - sigma I and the forward sweep
        // together; d holds inverse pivots.  The pivots that a chunk leaves
        // serve its later solves while they are still there (one chunk).
        double xc = X[0];
        if (it == 0 || chunks > 1) {
          double dc = dd[s0] - sigma, uc = nb > 1 ? ee[s0] : 0.0;
          for (int i = 0; i + 1 < nb; ++i) {
            const size_t o = size_t(i) * TD_CHUNK;
            const double e = ee[s0 + i], dn = dd[s0 + i + 1] - sigma, un = i + 2 < nb ? ee[s0 + i + 1] : 0.0;
            const double xn = X[o + TD_CHUNK];
            const bool swap = !(fabs(dc) >= fabs(e));
            const double num = swap ? dc : e, den = swap ? e : dc;
            const double f = den != 0.0 ? num / den : 0.0;
            d[o] = inverse(den);
            dl[o] = f;
            du[o] = swap ? dn : uc;
            du2[o] = swap ? un : 0.0;
            const unsigned long long mask = __ballot(swap);
            if (lane == __ffsll(__ballot(1)) - 1) T.piv[i] = mask;
            dc = swap ? uc - f * dn : dn - f * uc;
            uc = swap ? -f * un : un;
            X[o] = swap ? xn : xc;
            xc = swap ? xc - f * xn : xn - f * xc;
          }
          d[size_t(nb - 1) * TD_CHUNK] = inverse(dc);
        } else {
#pragma unroll 4
          for (int i = 0; i + 1 < nb; ++i) {
            const size_t o = size_t(i) * TD_CHUNK;
            const double xn = X[o + TD_CHUNK], f = dl[o];
            const bool swap = (T.piv[i] >> lane) & 1;
            X[o] = swap ? xn : xc;
            xc = swap ? xc - f * xn : xn - f * xc;
          }
        }
        double x1 = xc * d[size_t(nb - 1) * TD_CHUNK], x2 = 0.0;
        X[size_t(nb - 1) * TD_CHUNK] = x1;
#pragma unroll 4
        for (int i = nb - 2; i >= 0; --i) {
          const size_t o = size_t(i) * TD_CHUNK;
          const double x = (X[o] - du[o] * x1 - du2[o] * x2) * d[o];
          X[o] = x;
          x2 = x1;
          x1 = x;
        }
      }
      __syncthreads();
      for (int idx = t; idx < nr * n; idx += TD_FIN) {
        const int r = idx / n, i = idx - r * n, s = slot_of[r0 + r], s0 = T.s0[s], e0 = T.e0[s];
        if (i < e0 - s0) Zv[size_t(r0 + r) * n + s0 + i] = T.X[size_t(i) * TD_CHUNK + r];
      }
      __syncthreads();
    }
    // Gram-Schmidt in descending order: vector r, normalised, is taken out of
    // the later ones of its block (vectors of different blocks have disjoint
    // entries).  Lane l of a wave holds the entries l mod 64 whatever the block.
    for (int r = 0; r < kk; ++r) {
      double *z = Zv + size_t(r) * n;
      const int s0 = s0_of[r], i0 = (s0 & ~63) + lane, i1 = e0_of[r];
      double amax = 0.0;
      for (int i = i0; i < i1; i += 64) amax = fmax(amax, fabs(z[i]));
      amax = wave_max(amax);
      int ex = 0;
      if (amax > 0.0) (void)frexp(amax, &ex);
      double nrm = 0.0;
      for (int i = i0; i < i1; i += 64) {
        const double x = ldexp(z[i], -ex);
        nrm += x * x;
      }
      nrm = wave_sum(nrm);
      const double inv = nrm > 0.0 ? 1.0 / sqrt(nrm) : 0.0;
      // this wave's later vectors, every TD_FIN / 64-th, 64 of them looked at together
      for (int base = r + 1 + wave; base < kk; base += TD_FIN) {
        const int mine = base + lane * (TD_FIN / 64);
        for (unsigned long long same = __ballot(mine < kk && s0_of[mine < kk ? mine : r] == s0); same; same &= same - 1) {
          double *y = Zv + size_t(base + (__ffsll(same) - 1) * (TD_FIN / 64)) * n;
          double dot = 0.0;
          for (int i = i0; i < i1; i += 64) dot += ldexp(z[i], -ex) * inv * y[i];
          dot = wave_sum(dot);
          if (dot != 0.0)
            for (int i = i0; i < i1; i += 64) y[i] -= dot * (ldexp(z[i], -ex) * inv);
        }
      }
      __syncthreads();
      if (wave == r % (TD_FIN / 64))   // nobody reads z in this pass any more
        for (int i = i0; i < i1; i += 64) z[i] = ldexp(z[i], -ex) * inv;
    }
    __syncthreads();
  }
}

// Back-transformation z <- H_0 ... H_{n-3} z, one wave per vector, z in
// registers (entry lane + 64 u), the next reflector loaded during the sum.  The
// reflectors before the first and after the last that is one are left out.
template <int R>
__global__ void __launch_bounds__(TD_THREADS)
td_back_kernel(double *workall, int n) {
  const int lane = threadIdx.x & 63, r = blockIdx.x * TD_WAVES + (threadIdx.x >> 6);
  double *work = td_work(workall, n, blockIdx.y);
  const TdScratch T = td_scratch(work + size_t(2) * n * n, n);
  if (r >= *T.kk) return;
  int first = n, last = -1;
  for (int base = 0; base < n - 2; base += 64) {
    const unsigned long long on = __ballot(base + lane < n - 2 && !(T.tau[base + lane] < 0.0));
    if (on) {
      if (last < 0) first = base + __ffsll(on) - 1;
      last = base + 63 - __clzll(on);
    }
  }
  if (last < 0) return;
  double *zg = work + size_t(n) * n + size_t(r) * n;
  double z[R], u[R], un[R];
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int i = lane + 64 * q;
    z[q] = i < n ? zg[i] : 0.0;
    un[q] = i < n ? work[size_t(last) * n + i] : 0.0;
  }
  for (int j = last; j >= first; --j) {
#pragma unroll
    for (int q = 0; q < R; ++q) u[q] = un[q];
    const double *next = work + size_t(j > first ? j - 1 : first) * n;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int i = lane + 64 * q;
      un[q] = i < n ? next[i] : 0.0;
    }
    double dot = 0.0;
#pragma unroll
    for (int q = 0; q < R; ++q) dot += u[q] * z[q];
    dot = wave_sum(dot);
#pragma unroll
    for (int q = 0; q < R; ++q) z[q] -= u[q] * dot;
  }
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int i = lane + 64 * q;
    if (i < n) zg[i] = z[q];
  }
}

__global__ void __launch_bounds__(TD_THREADS)
td_output_kernel(double *Vall, double *workall, int n) {
  double *work = td_work(workall, n, blockIdx.y);
  const TdScratch T = td_scratch(work + size_t(2) * n * n, n);
  const double *Zv = work + size_t(n) * n;
  const int kk = *T.kk;
  for (int idx = blockIdx.x * TD_THREADS + threadIdx.x; idx < n * n; idx += gridDim.x * TD_THREADS) {
    const int i = idx / n, c = idx - i * n;
    Vall[size_t(blockIdx.y) * n * n + idx] = c < kk ? Zv[size_t(c) * n + i] : 0.0;
  }
}

void launch_tridiag_top(double *A, double *w, double *V, int *sweeps, int n, int batch, int k, double cluster_rel,
                        double *work, hipStream_t st) {
  const size_t lds = size_t(TD_LDS) * TD_LD * 8;
  static const bool attr = [&] {
    TRG_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void *>(&td_finish_kernel),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)));
    return true;
  }();
  (void)attr;
  const int k0 = n > TD_LDS ? n - TD_LDS : 0;
  for (int col = 0; col < k0; ++col) {
    // about two workgroups per CU over the batch, at least two rows per wave
    const int rows = n - col - 1;
    const int want = (512 + batch - 1) / batch, most = (rows + 2 * TD_WAVES - 1) / (2 * TD_WAVES);
    hipLaunchKernelGGL(td_column_kernel, dim3(uint32_t(want < most ? want : most), uint32_t(batch)), dim3(TD_THREADS), 0,
                       st, A, work, n, col);
  }
  hipLaunchKernelGGL(td_finish_kernel, dim3(batch), dim3(TD_FIN), lds, st, A, work, n, k0);
  hipLaunchKernelGGL(td_values_kernel, dim3(uint32_t((n * TD_MS + TD_THREADS - 1) / TD_THREADS), uint32_t(batch)),
                     dim3(TD_THREADS), 0, st, work, n);
  hipLaunchKernelGGL(td_vectors_kernel, dim3(batch), dim3(TD_FIN), 0, st, A, w, V, sweeps, n, k, cluster_rel, work);
  const dim3 bg(uint32_t((n + TD_WAVES - 1) / TD_WAVES), uint32_t(batch));
  // up to order 256 the 12 registers that would hold nothing cost 10 % (order 196
  // 120 against 132 us, 256 163 against 190); from 300 on 9 for 16 gained 1 %
  if (n <= 256)
    hipLaunchKernelGGL((td_back_kernel<4>), bg, dim3(TD_THREADS), 0, st, work, n);
  else
    hipLaunchKernelGGL((td_back_kernel<16>), bg, dim3(TD_THREADS), 0, st, work, n);
  hipLaunchKernelGGL(td_output_kernel, dim3(uint32_t((n * n + 4 * TD_THREADS - 1) / (4 * TD_THREADS)), uint32_t(batch)),
                     dim3(TD_THREADS), 0, st, V, work, n);
  TRG_HIP_CHECK(hipGetLastError());
}

// ------------------------------------------------------------- selection ---
constexpr int SEL_THREADS = 256;
constexpr double TIE_REL = 1e-10;      // side rule: backward only if clearly better
constexpr double SIGN_REL = 1e-9;      // "largest" coordinate within this relative window
constexpr double DEGEN_REL = 1e-8;     // degenerate-cut flag

__device__ inline double sel_reduce(double v, double *sh, bool is_max) {
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int s = SEL_THREADS / 2; s > 0; s >>= 1) {
    if (t < s) sh[t] = is_max ? fmax(sh[t], sh[t + s]) : (sh[t] + sh[t + s]);
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

__device__ inline int sel_min_index(int v, int *sh) {
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int s = SEL_THREADS / 2; s > 0; s >>= 1) {
    if (t < s) sh[t] = min(sh[t], sh[t + s]);
    __syncthreads();
  }
  const int r = sh[0];
  __syncthreads();
  return r;
}

// w2/V2: the two sides' sorted eigensystems (side 0 backward, 1 forward).
__global__ void __launch_bounds__(SEL_THREADS)
select_kernel(const double *w2, const double *V2, const int *sweeps2, int n, int k, int force_side,
              double cluster_rel, double *U, double *rec_eps, int *rec_int, double *spectrum) {
  __shared__ double sh[SEL_THREADS];
  __shared__ int shi[SEL_THREADS];
  __shared__ double diag[MAX_N];
  __shared__ double col[MAX_N];
  const int t = threadIdx.x;

  double eps[2];
  for (int side = 0; side < 2; ++side) {
    double s = 0.0;
    for (int j = k + t; j < n; j += SEL_THREADS) s += fmax(w2[side * n + j], 0.0);
    eps[side] = sel_reduce(s, sh, false);
  }
  int side = (eps[0] < (1.0 - TIE_REL) * eps[1]) ? 0 : 1;
  if (force_side == 0 || force_side == 1) side = force_side;
  const double *w = w2 + side * n;
  const double *V = V2 + size_t(side) * n * n;
  for (int j = t; j < n; j += SEL_THREADS) spectrum[j] = w[j];

  // neighbouring eigenvalues within cluster_rel lambda_max form one
  // eigenspace, kept in its canonical basis; every larger gap is resolved by
  // the leading eigenvectors (plain truncated HOSVD)
  const double tol = cluster_rel * fmax(w[0], 0.0);
  int a = 0;
  while (a < k) {
    int bnd = a + 1;
    while (bnd < n && w[bnd - 1] - w[bnd] <= tol) ++bnd;  // cluster [a, bnd)
    const int stop = bnd < k ? bnd : k;
    for (int j = a; j < stop; ++j) {
      // remaining weight of each coordinate in the cluster's projector
      double mx = 0.0;
      for (int i = t; i < n; i += SEL_THREADS) {
        double dg = 0.0;
        for (int c = a; c < bnd; ++c) dg += V[i * n + c] * V[i * n + c];
        for (int c = a; c < j; ++c) dg -= U[i * k + c] * U[i * k + c];
        diag[i] = dg;
        mx = fmax(mx, dg);
      }
      mx = sel_reduce(mx, sh, true);
      int first = n;
      for (int i = t; i < n; i += SEL_THREADS)
        if (diag[i] >= (1.0 - SIGN_REL) * mx && i < first) first = i;
      // no coordinate qualifies when the vectors are NaN: the last one then, whose
      // entries are as good as any, for n is past the end of V, U and col
      const int found = sel_min_index(first, shi), r = found < n ? found : n - 1;
      // column of the remaining projector at coordinate r
      for (int i = t; i < n; i += SEL_THREADS) {
        double v = 0.0;
        for (int c = a; c < bnd; ++c) v += V[i * n + c] * V[r * n + c];
        for (int c = a; c < j; ++c) v -= U[i * k + c] * U[r * k + c];
        col[i] = v;
      }
      __syncthreads();
      const double inv = 1.0 / sqrt(col[r]);
      for (int i = t; i < n; i += SEL_THREADS) U[i * k + j] = col[i] * inv;
      __syncthreads();
    }
    a = bnd;
  }
  if (t == 0) {
    rec_eps[0] = eps[0];
    rec_eps[1] = eps[1];
    const int degenerate = (k < n && w[k - 1] > 0.0 && (w[k - 1] - w[k]) <= DEGEN_REL * w[k - 1]) ? 1 : 0;
    rec_int[0] = side;
    rec_int[1] = k;
    rec_int[2] = degenerate;
    rec_int[3] = sweeps2[side];
  }
}

}  // namespace

// Jacobi up to order JACOBI_MAX_N (accurate, and cheap while the matrix is
// small), tridiagonalisation + QL above.

namespace {
// The solvers' matrices are grid.y (a workgroup index of a matrix is grid.x),
// which ends at 65535: larger batches go in pieces, f(first matrix, count).
constexpr int MAX_GRID_Y = 65535;
template <class F>
void each_piece(int batch, F &&f) {
  for (int b0 = 0; b0 < batch;) {
    const int nb = std::min(batch - b0, MAX_GRID_Y);
    f(size_t(b0), nb);
    b0 += nb;
  }
}
}  // namespace

void eigh_batched(double *A, double *w, double *V, int *sweeps, int n, int batch, hipStream_t st) {
  TRG_REQUIRE(n >= 1 && n <= MAX_N && batch >= 1, "eigh: order must be in [1, 1024]");
  const size_t n2 = size_t(n) * n;
  if (n <= JACOBI_MAX_N)
    each_piece(batch, [&](size_t b, int nb) {
      launch_jacobi(A + b * n2, w + b * n, V + b * n2, sweeps + b, n, nb, false, st);
    });
  else
    hipLaunchKernelGGL(tridiag_ql_kernel, dim3(batch), dim3(TQ_THREADS), 0, st, A, w, V, sweeps, n);
  TRG_HIP_CHECK(hipGetLastError());
}

size_t eigh_top_work_doubles(int n, int batch) {
  return size_t(batch) * (size_t(2) * n * n + size_t(TOP_SCRATCH) * n);
}

void eigh_top_batched(double *A, double *w, double *V, int *sweeps, int n, int batch, int k, double cluster_rel,
                      double *work, hipStream_t st, bool square) {
  TRG_REQUIRE(n >= 1 && n <= MAX_N && batch >= 1 && k >= 1, "eigh_top: bad sizes");
  TRG_REQUIRE(work != nullptr || n <= JACOBI_MAX_N, "eigh_top: workspace missing");
  const size_t n2 = size_t(n) * n;
  each_piece(batch, [&](size_t b, int nb) {
    if (n <= JACOBI_MAX_N)
      launch_jacobi(A + b * n2, w + b * n, V + b * n2, sweeps + b, n, nb, square, st);
    else
      launch_tridiag_top(A + b * n2, w + b * n, V + b * n2, sweeps + b, n, nb, k, cluster_rel,
                         work + eigh_top_work_doubles(n, 1) * b, st);
  });
  TRG_HIP_CHECK(hipGetLastError());
}

void select_isometry(const double *w2, const double *V2, const int *sweeps2, int n, int k,
                     int force_side, double cluster_rel, SelectOut out, hipStream_t st) {
  TRG_REQUIRE(n >= 1 && n <= MAX_N && k >= 1 && k <= n, "select: bad sizes");
  TRG_REQUIRE(cluster_rel >= 0.0 && cluster_rel < 1.0, "select: bad degeneracy window");
  hipLaunchKernelGGL(select_kernel, dim3(1), dim3(SEL_THREADS), 0, st, w2, V2, sweeps2, n, k, force_side,
                     cluster_rel, out.U, out.rec_eps, out.rec_int, out.spectrum);
  TRG_HIP_CHECK(hipGetLastError());
}

}  // namespace trg
