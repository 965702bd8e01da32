// Symmetric tridiagonal eigen-solver pieces (FP64), one GPU thread each.
//
//  * sturm_count: number of eigenvalues of T below x (LDL^T pivot signs);
//  * tri_lu / tri_solve: LU factors of T - sI with partial pivoting and
//    solves with them, the step of inverse iteration for one eigenvector
//    (vectors of a cluster are re-orthogonalised by the caller, as LAPACK's
//    dstein does).
// T has diagonal d[0..n) and off-diagonal e[0..n-1). Divisions use the
// hardware reciprocal refined by two Newton steps (error of a few ulps), so
// that the sequential recurrences carry five dependent operations per step
// instead of a full division.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>

namespace dg {

__device__ __forceinline__ double recip(double q) {
  double r = __builtin_amdgcn_rcp(q);
  double t = fma(-q, r, 1.0);
  r = fma(r, t, r);
  t = fma(-q, r, 1.0);
  return fma(r, t, r);
}

__device__ inline int sturm_count(const double* d, const double* e, int n, double x, double pivmin) {
  int cnt = 0;
  double q = d[0] - x;
  if (fabs(q) < pivmin) q = -pivmin;
  cnt += q < 0.0;
  for (int i = 1; i < n; ++i) {
    const double e2 = e[i - 1] * e[i - 1];
    q = fma(-e2, recip(q), d[i] - x);
    if (fabs(q) < pivmin) q = -pivmin;
    cnt += q < 0.0;
  }
  return cnt;
}

// strided views (per-thread arrays interleaved across the threads of a block)
struct StridedD {
  double* p;
  int s;
  __device__ double& operator[](int i) const { return p[(size_t)i * s]; }
};
struct StridedB {
  unsigned char* p;
  int s;
  __device__ unsigned char& operator[](int i) const { return p[(size_t)i * s]; }
};

// deterministic start vector entries in (-1, 1)
__device__ inline double hash_unit(unsigned a, unsigned b) {
  unsigned long long x = (unsigned long long)a * 0x9E3779B97F4A7C15ull ^ ((unsigned long long)b + 0x632BE59BD9B4E019ull);
  x ^= x >> 31;
  x *= 0xBF58476D1CE4E5B9ull;
  x ^= x >> 29;
  x *= 0x94D049BB133111EBull;
  x ^= x >> 32;
  return (double)(x & 0xFFFFFFFFull) / 2147483648.0 - 1.0;
}

// Blocks of 8 consecutive indices 0..n-1, then the remainder one by one: f(i, width) with
// the width as a compile-time constant, so that a block's loads can be issued together
// before its serial part (the compiler keeps loads behind stores that may alias).
template <int N>
struct Width {
  static constexpr int value = N;
};
#define CVN(u) (decltype(u)::value)
template <typename F>
__device__ __forceinline__ void strided_blocks(int n, F f) {
  int i = 0;
  for (; i + 8 <= n; i += 8) f(i, Width<8>{});
  for (; i < n; ++i) f(i, Width<1>{});
}
template <int N, typename F>
__device__ __forceinline__ void for_n(Width<N>, F f) {
#pragma unroll
  for (int k = 0; k < N; ++k) f(k);
}

// Factor T - s I = P L U with partial pivoting: on return ai (reciprocal of the
// diagonal of U), b (first super-diagonal), u2 (second), l (multipliers), piv
// (row swaps). A zero pivot is replaced by tiny. The running diagonal entry and
// the next super-diagonal are carried in registers.
template <typename DA, typename BA>
__device__ inline void tri_lu(const double* d, const double* e, int n, double s, double tiny, DA ai, DA b,
                              DA u2, DA l, BA piv) {
  double ak = d[0] - s;            // current diagonal of row k
  double bk = n > 1 ? e[0] : 0.0;  // current first super-diagonal of row k
  strided_blocks(n - 1, [&](int k0, auto w) {
    double c[CVN(w)], an[CVN(w)], bn[CVN(w)];
    for_n(w, [&](int q) {
      const int k = k0 + q;
      c[q] = e[k];                                 // sub-diagonal below the pivot
      an[q] = d[k + 1] - s;                        // row k+1 diagonal
      bn[q] = (k + 1 < n - 1) ? e[k + 1] : 0.0;    // row k+1 super-diagonal
    });
    for_n(w, [&](int q) {
      const int k = k0 + q;
      const bool keep = fabs(ak) >= fabs(c[q]);
      // the pivot: row k's diagonal, or row k+1's (the sub-diagonal entry)
      const double a0 = keep ? (ak != 0.0 ? ak : tiny) : c[q];
      const double r = recip(a0);
      const double m = (keep ? c[q] : ak) * r;
      piv[k] = keep ? 0 : 1;
      l[k] = m;
      ai[k] = r;
      b[k] = keep ? bk : an[q];
      u2[k] = keep ? 0.0 : bn[q];
      ak = keep ? fma(-m, bk, an[q]) : fma(-m, an[q], bk);
      bk = keep ? bn[q] : -m * bn[q];
    });
  });
  ai[n - 1] = recip(ak != 0.0 ? ak : tiny);
}

// solve (T - s I) x = y in place with the factors of tri_lu
template <typename DA, typename BA>
__device__ inline void tri_solve(int n, DA ai, DA b, DA u2, DA l, BA piv, DA y) {
  double cur = y[0];
  strided_blocks(n - 1, [&](int k0, auto w) {
    double nx[CVN(w)], lk[CVN(w)], out[CVN(w)];
    bool pk[CVN(w)];
    for_n(w, [&](int q) {
      nx[q] = y[k0 + q + 1];
      lk[q] = l[k0 + q];
      pk[q] = piv[k0 + q] != 0;
    });
    for_n(w, [&](int q) {
      const double top = pk[q] ? nx[q] : cur, below = pk[q] ? cur : nx[q];
      out[q] = top;
      cur = fma(-lk[q], top, below);
    });
    for_n(w, [&](int q) { y[k0 + q] = out[q]; });
  });
  // back substitution with U (diagonal 1/ai, super-diagonals b and u2)
  double y1 = cur * ai[n - 1];   // y[k+1]
  y[n - 1] = y1;
  double y2 = 0.0;               // y[k+2]
  strided_blocks(n - 1, [&](int i0, auto w) {
    double yk[CVN(w)], bk[CVN(w)], uk[CVN(w)], ak[CVN(w)];
    for_n(w, [&](int q) {
      const int k = n - 2 - i0 - q;
      yk[q] = y[k];
      bk[q] = b[k];
      uk[q] = u2[k];
      ak[q] = ai[k];
    });
    for_n(w, [&](int q) {
      const double v = (yk[q] - bk[q] * y1 - uk[q] * y2) * ak[q];
      yk[q] = v;
      y2 = y1;
      y1 = v;
    });
    for_n(w, [&](int q) { y[n - 2 - i0 - q] = yk[q]; });
  });
}

}  // namespace dg
