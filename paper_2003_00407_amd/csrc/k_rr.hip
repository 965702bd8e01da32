// Rayleigh-Ritz on the small projected problem (FP64): the generalised eigenproblem of
// (S^T H S, S^T S) for S = [X W P] (Eq. (4); Algorithm 1 step 5, Algorithm 2 step 4), and
// the eigen-decomposition and Cholesky-QR passes of the ALB orthonormalisation.
//
//   scaled overlap -> Cholesky with column dropping    (k_rr_chol, one workgroup per element)
//   -> U^{-1} = Z                                      (k_rr_zinv_*, a wave or a quad of lanes per row)
//   -> A^ = Z^T A~ Z                                   (k_rr_prod, a wave per 16x16 tile)
//   -> Householder tridiagonal T                       (k_rr_tri, one workgroup per element)
//   -> eigenvalues of T by multisection                (k_rr_eig, a workgroup per eigenvalue)
//   -> eigenvectors of T by inverse iteration          (k_rr_inv, a lane per vector)
//   -> in-order Gram-Schmidt                           (k_rr_mgs, one workgroup per element)
//   -> back-transformation                             (k_rr_back, a wave or eight lanes per vector)
//   -> coefficients C = D Z V                          (k_rr_coef, a wave per 16x16 tile)
//
// The steps are separate launches so that each takes the split that suits it: a launch
// has one to a few dozen elements, and one workgroup per element for all of it leaves
// most of the 256 compute units idle behind serial sweeps.
#include "dense_ops.h"
#include "tridiag.h"

#include <algorithm>
#include <cstdio>

namespace dg {

struct RRArgs {
  const ElemDev* elems;
  const int* active;
  int nb;              // K3 = nb * E.K (RR_GEN); RR_SVD: K3 = kfix
  int kfix;            // RR_SVD: matrix order
  int nkeep;           // columns of C to produce (<= 0: E.K)
  int mode;
  int* status;         // per element: 0 ok, 2 breakdown of the X block
  long long* phase_clk;  // optional: 16 timestamps per element (diagnostics)
  double* work;          // per element work region: the overlap factorisation's matrix, and the
                         // tridiagonalisation's where an order is above kRRLdsOrder
  long long work_stride;
  double pivot_tol;      // X-column overlap pivots below this (after unit-diagonal scaling) = breakdown
  double drop_tol;       // W/P columns whose scaled pivot is below this are left out of the basis
  double* minpiv;        // optional: smallest scaled pivot, its column, dropped count (diagnostics)
  double ortol;          // eigenvalues closer than ortol * ||T|| are treated as one cluster
  int mgs_lds;           // dynamic LDS bytes of the Gram-Schmidt launch
  int* hp_flag;          // optional, per element: 1 when the smallest scaled pivot is below hp_tol
                         // (the rotated H P' would carry cancellation error), 0 otherwise and
                         // for inactive elements
  double hp_tol;
};


constexpr int kRRThreads = 512;     // LDS variant (orders up to kRRLdsOrder)
constexpr int kRRThreadsL2 = 1024;  // L2-resident variant: more loads in flight for its latency-bound sweeps
constexpr int kTriMax = 272;   // largest projected problem handled (3 x 88 + pad)
constexpr int kOrthMax = 88;   // most eigenvectors (J + guards)

constexpr int kLdsPerCU = 163840;                 // 160 KB of LDS per compute unit
constexpr int kRRStaticLds = 21504;               // bound on k_rr_tri's static LDS
constexpr int kRRLdsBytes = kLdsPerCU - kRRStaticLds;
constexpr int kRRLdsOrder = 132;                  // np * np doubles fit in kRRLdsBytes

// where the steps leave their matrices (leading dimension np); the inputs are S^T S in
// slot G and S^T H S in slot A (leading dimension n), the result C is in slot C
enum RRSlot { kSlotUt, kSlotZ, kSlotT, kSlotAhat, kSlotAhatT, kSlotRefl, kSlotVec };
__device__ __forceinline__ long long rr_slot(RRSlot w, int KP) {
  switch (w) {
    case kSlotZ: return SmallLayout::G(KP);      // S^T S is done with once it is factored
    case kSlotT: return SmallLayout::V(KP);
    case kSlotAhat:                              // S^T H S is done with once T is formed
    case kSlotRefl: return SmallLayout::A(KP);   // A^ is read before the reflectors are written
    default: return SmallLayout::U(KP);          // U^T until Z is formed, (A^)^T, then the eigenvectors
  }
}

struct RRShape {
  int n, np;      // order, and rounded up to even (leading dimension)
  int kx;         // leading columns that are never left out
  int nkeep;      // columns of C
  int nwant;      // eigenpairs computed
  int KP;
  bool gen, svd;
};

__device__ __forceinline__ RRShape rr_shape(const RRArgs& A, const ElemDev& E) {
  RRShape s;
  s.gen = A.mode == RR_GEN;
  s.svd = A.mode == RR_SVD;
  s.n = s.gen ? A.nb * E.K : kcode(A.kfix, E);
  s.np = s.n + (s.n & 1);
  s.kx = s.gen ? E.K : s.n;
  s.nkeep = kcode(A.nkeep, E);
  s.nwant = s.svd ? s.n : min(s.nkeep, s.n);
  s.KP = E.kmax3 + 2;
  return s;
}

// element e takes part: active, and its overlap factorisation did not break down
__device__ __forceinline__ bool rr_on(const RRArgs& A, int e) {
  if (A.active && !A.active[e]) return false;
  return A.mode == RR_SVD || A.status[e] != 2;
}

__device__ __forceinline__ void rr_stamp(const RRArgs& A, int e, int k, int block) {
  if (A.phase_clk && block == 0 && threadIdx.x == 0) A.phase_clk[e * 16 + k] = wall_clock64();
}

// ---------------------------------------------------------------------------
// scaled overlap -> Cholesky with column dropping: U (upper, U^T U = D S^T S D), written
// transposed (column j of U contiguous at Ut + j np), 1 / U_jj, the scaling D.
//
// One workgroup per element, right-looking in panels of 16 rows.  Every wave factors the
// panel's diagonal block for itself (a lane per column, multipliers broadcast by lane
// reads), carrying one trailing column per lane along, so a panel needs two barriers;
// the trailing update is FP64 MFMA tiles.  v_mfma_f64_16x16x4f64 adds its four products
// as a chain of fused multiply-adds in ascending k (checked on the device), so every
// entry is updated by the same chain, one fused operation per row in ascending order, as
// by rank-1 updates.  Nearly dependent W/P columns leave the basis.
// Order 264: 252 us; 1870 us as 264 rank-1 updates of the L2-resident matrix, a barrier
// each, before.
// ---------------------------------------------------------------------------
constexpr int kCholThreads = 1024;
constexpr int kCholPitch = 280;                                        // doubles per staged row
constexpr int kCholLds = 3 * 16 * kCholPitch * (int)sizeof(double);    // panel rows (twice), multipliers

__device__ __forceinline__ void no_basis_change(double* C, int n, int nkeep) {
  for (int idx = threadIdx.x; idx < n * nkeep; idx += blockDim.x) {
    const int i = idx / nkeep, j = idx % nkeep;
    C[idx] = (i == j) ? 1.0 : 0.0;
  }
}

__global__ void __launch_bounds__(kCholThreads) k_rr_chol(RRArgs A) {
  const int e = blockIdx.x;
  const ElemDev& E = A.elems[e];
  if (A.active && !A.active[e]) {
    if (A.hp_flag && threadIdx.x == 0) A.hp_flag[e] = 0;
    return;
  }
  const RRShape s = rr_shape(A, E);
  rr_stamp(A, e, 0, 0);
  const int n = s.n, np = s.np;
  const double* G = E.small + SmallLayout::G(s.KP);
  double* Ut = E.small + rr_slot(kSlotUt, s.KP);
  double* vec = E.small + SmallLayout::vec(s.KP);
  double* d = vec + VS_D * s.KP;
  double* rinv = vec + VS_T0 * s.KP;
  double* W = A.work + (size_t)e * A.work_stride;   // working matrix, upper part
  extern __shared__ double dyn[];
  double* P = dyn;                       // the panel's rows as the trailing update left them
  double* Pf = dyn + 16 * kCholPitch;    // factored
  double* F = dyn + 32 * kCholPitch;     // -(row / pivot): multipliers of the trailing update
  __shared__ double sd[kTriMax], sdiag[kTriMax], su[kTriMax];
  __shared__ int brk;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  constexpr int nw = kCholThreads / 64;
  if (tid == 0) brk = 0;
  __syncthreads();
  for (int i = tid; i < n; i += kCholThreads) {
    const double gii = G[(size_t)i * n + i];
    if (!(gii > 0.0) && i < s.kx) brk = 1;
    sd[i] = gii > 0.0 ? 1.0 / sqrt(gii) : 0.0;
  }
  __syncthreads();
  for (int idx = tid; idx < n * n; idx += kCholThreads) {
    const int i = idx / n, j = idx % n;
    if (j < i) continue;
    const double s2 = sd[i] * sd[j];
    W[(size_t)i * np + j] = G[idx] * s2;
  }
  const int l16 = lane & 15, kl = lane >> 4;
  double pmin = 1.0;
  int jmin = -1, ndrop = 0;
  __syncthreads();
  // the first panel's rows; later ones are left in P by the trailing update
  for (int idx = tid; idx < 16 * n; idx += kCholThreads) {
    const int r = idx / n, k = idx % n;
    P[r * kCholPitch + k] = (r < n && k >= r) ? W[(size_t)r * np + k] : 0.0;
  }
  for (int j0 = 0; j0 < n; j0 += 16) {
    const int nr = min(16, n - j0);
    __syncthreads();
    // this lane's columns: j0 + l16 of the diagonal block, and trailing column k
    const int k = j0 + 16 + tid;
    if (wv == 0 || j0 + 16 + 64 * wv < n) {
      double c[16], t[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        c[r] = (r < nr && l16 < nr && l16 >= r) ? P[r * kCholPitch + j0 + l16] : 0.0;
        t[r] = (r < nr && k < n) ? P[r * kCholPitch + k] : 0.0;
      }
      unsigned dropped = 0;   // rows of this panel that leave the basis
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        double f = 0.0;
        if (j < nr) {
          const double piv = lane_read(c[j], j);
          if (piv < pmin) {
            pmin = piv;
            jmin = j0 + j;
          }
          if (j0 + j >= s.kx && !(piv > A.drop_tol)) {
            dropped |= 1u << j;
            ++ndrop;
            t[j] = 0.0;
          } else {
            if (!(piv > A.pivot_tol) && tid == 0) brk = 1;
            const double pinv = 1.0 / fmax(piv, 1e-300);
            const double fj = c[j] * pinv;
            f = -(t[j] * pinv);
#pragma unroll
            for (int i = j + 1; i < 16; ++i) {
              const double fi = lane_read(fj, i);
              c[i] = fma(-fi, c[j], c[i]);
              t[i] = fma(-fi, t[j], t[i]);
            }
          }
        }
        if (k < n) F[j * kCholPitch + k] = f;
      }
      // rows j0 .. j0 + nr - 1, not yet divided by the square roots of their pivots
      if (k < n) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          Pf[r * kCholPitch + k] = r < nr ? t[r] : 0.0;
          if (r < nr) gstore(Ut + (size_t)k * np + j0 + r, t[r]);
        }
      }
      if (wv == 0 && lane < nr) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (r <= l16 && r < nr) {
            const bool on = !((dropped >> r) & 1);
            if (r < l16) gstore(Ut + (size_t)(j0 + l16) * np + j0 + r, on ? c[r] : 0.0);
            else sdiag[j0 + r] = on ? fmax(c[r], 1e-300) : -1.0;   // -1: left out
          }
      }
    }
    lds_barrier();
    // trailing update, upper tiles; the first tile row is the next panel
    const int b0 = j0 + 16, nb = (n - b0 + 15) >> 4;
    for (int tl = wv; b0 < n && tl < nb * (nb + 1) / 2; tl += nw) {
      int ti = 0, tk = tl;
      while (tk >= nb - ti) {
        tk -= nb - ti;
        ++ti;
      }
      tk += ti;
      const int i0 = b0 + 16 * ti, kc = b0 + 16 * tk + l16;
      const int ia = min(i0 + l16, n - 1), kb = min(kc, n - 1);   // beyond the matrix: results not stored
      double a[4], b[4];
      d4v acc;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        acc[q] = gload<double>(W + (size_t)min(i0 + kl + 4 * q, n - 1) * np + kb);
        a[q] = F[(4 * q + kl) * kCholPitch + ia];
        b[q] = Pf[(4 * q + kl) * kCholPitch + kb];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) acc = mfma16x16x4(a[q], b[q], acc);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = i0 + kl + 4 * q;
        if (i >= n || kc >= n) continue;
        if (ti == 0) P[(kl + 4 * q) * kCholPitch + kc] = acc[q];
        else gstore(W + (size_t)i * np + kc, acc[q]);
      }
    }
  }
  __syncthreads();
  // U: rows divided by the square roots of the pivots; a left-out row or column is zero
  // beside its unit diagonal
  for (int j = tid; j < n; j += kCholThreads) {
    const double p = sdiag[j];
    const double u = p < 0.0 ? 1.0 : sqrt(p);
    su[j] = u;
    rinv[j] = 1.0 / u;
    if (p < 0.0) sd[j] = 0.0;
  }
  __syncthreads();
  for (int k = wv; k < n; k += nw) {
    const bool out = sd[k] == 0.0;
    for (int j = lane; j <= k; j += 64) {
      double* p = Ut + (size_t)k * np + j;
      *p = j == k ? su[k] : (out ? 0.0 : *p / su[j]);
    }
  }
  for (int i = tid; i < n; i += kCholThreads) d[i] = sd[i];
  if (tid == 0) {
    if (A.hp_flag) A.hp_flag[e] = (brk || !(pmin >= A.hp_tol)) ? 1 : 0;
    if (A.minpiv) {
      A.minpiv[3 * e] = pmin;
      A.minpiv[3 * e + 1] = jmin;
      A.minpiv[3 * e + 2] = ndrop;
    }
    A.status[e] = brk ? 2 : 0;
  }
  // X itself is not positive definite: keep X (C = [I; 0; 0]) and report it
  if (brk) no_basis_change(E.small + SmallLayout::C(s.KP), n, s.nkeep);
}

// ---------------------------------------------------------------------------
// Z = U^{-1}, row by row: Z[i][j] = -(1/U[j][j]) sum_{k=i}^{j-1} Z[i][k] U[k][j].  The rows
// are independent chains over j, so each has lanes of its own, spread over the chip: a
// wave (kWave: Z[i][k] on lane (k - i) % 64, the columns of U prefetched) or, for the
// orders that fit in LDS as a matrix, a quad of lanes (the k sum split four ways).
// RR_CHOLQR: the coefficients C = D Z.
// Order 264: 93 us; 1070 us in the element's one workgroup, two barriers a column, before.
// ---------------------------------------------------------------------------
constexpr int kZinvRows = 4;   // rows per workgroup, kWave

__global__ void __launch_bounds__(64 * kZinvRows) k_rr_zinv_wave(RRArgs A) {
  const int e = blockIdx.y;
  const ElemDev& E = A.elems[e];
  if (!rr_on(A, e)) return;
  const RRShape s = rr_shape(A, E);
  rr_stamp(A, e, 1, blockIdx.x);
  const int n = s.n, np = s.np;
  const int lane = threadIdx.x & 63;
  const int i = blockIdx.x * kZinvRows + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const double* Ut = E.small + rr_slot(kSlotUt, s.KP);
  double* Z = E.small + rr_slot(kSlotZ, s.KP);
  const double* vec = E.small + SmallLayout::vec(s.KP);
  const double* gr = vec + VS_T0 * s.KP;
  __shared__ double rinv[kTriMax];
  for (int x = threadIdx.x; x < n; x += blockDim.x) rinv[x] = gr[x];
  __syncthreads();
  if (i >= n) return;
  constexpr int NQ = (kTriMax + 63) / 64, NC = 4;
  double z[NQ], u[NC][NQ], un[NC][NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) z[q] = 0.0;
  if (lane == 0) z[0] = rinv[i];
  // columns jb .. jb + 3 of U, rows i + lane + 64 q above the diagonal
  auto load = [&](int jb, double (&dst)[NC][NQ]) {
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        // on and past the diagonal (where Z is still zero): the diagonal
        const int j = min(jb + c, n - 1), k = min(i + lane + 64 * q, j);
        if (64 * q < jb + NC - i) dst[c][q] = gload<double>(Ut + (size_t)j * np + k);
      }
  };
  if (i + 1 < n) load(i + 1, un);
  for (int jb = i + 1; jb < n; jb += NC) {
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int q = 0; q < NQ; ++q) u[c][q] = un[c][q];
    if (jb + NC < n) load(jb + NC, un);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int j = jb + c;
      if (j >= n) continue;
      double t = 0.0;
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        if (64 * q < j - i) t = fma(z[q], u[c][q], t);
      t = wave_sum_dpp(t);
      const double zj = -rinv[j] * t;
      const int off = j - i;
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        if ((off >> 6) == q && lane == (off & 63)) z[q] = zj;
    }
  }
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int k = i + lane + 64 * q;
    if (k < n) Z[(size_t)i * np + k] = z[q];
  }
  if (!s.gen) {
    const double di = vec[VS_D * s.KP + i];
    double* C = E.small + SmallLayout::C(s.KP) + (size_t)i * s.nkeep;
    for (int k = lane; k < i && k < s.nkeep; k += 64) C[k] = 0.0;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int k = i + lane + 64 * q;
      if (k < s.nkeep) C[k] = k < n ? di * z[q] : 0.0;
    }
  }
}

__global__ void __launch_bounds__(64) k_rr_zinv_quad(RRArgs A) {
  const int e = blockIdx.y;
  const ElemDev& E = A.elems[e];
  if (!rr_on(A, e)) return;
  const RRShape s = rr_shape(A, E);
  const int n = s.n, np = s.np;
  const int i0 = blockIdx.x * 16;
  if (i0 >= n) return;
  rr_stamp(A, e, 1, blockIdx.x);
  const int tid = threadIdx.x, ql = tid & 3, r = tid >> 2, i = i0 + r;
  const double* Ut = E.small + rr_slot(kSlotUt, s.KP);
  double* Z = E.small + rr_slot(kSlotZ, s.KP);
  const double* vec = E.small + SmallLayout::vec(s.KP);
  const double* rinv = vec + VS_T0 * s.KP;
  constexpr int kPitch = kRRLdsOrder + 1;
  __shared__ double zl[16][kPitch], ul[16][kPitch], ri[kPitch];
  for (int x = tid; x < n; x += 64) ri[x] = rinv[x];
  for (int x = tid; x < 16 * kPitch; x += 64) zl[x / kPitch][x % kPitch] = 0.0;
  __syncthreads();
  if (ql == 0 && i < n) zl[r][i] = ri[i];
  constexpr int NS = (16 * kRRLdsOrder + 63) / 64;
  double pre[NS];
  // columns j0 .. j0 + 15 of U from row i0 on
  auto fetch = [&](int j0) {
#pragma unroll
    for (int x = 0; x < NS; ++x) {
      const int c = (tid + 64 * x) & 15, k = i0 + ((tid + 64 * x) >> 4);
      pre[x] = (j0 + c < n && k < j0 + c) ? gload<double>(Ut + (size_t)(j0 + c) * np + k) : 0.0;
    }
  };
  fetch(i0);
  for (int j0 = i0; j0 < n; j0 += 16) {
    __syncthreads();
#pragma unroll
    for (int x = 0; x < NS; ++x) {
      const int c = (tid + 64 * x) & 15, k = i0 + ((tid + 64 * x) >> 4);
      if (k < kRRLdsOrder) ul[c][k] = pre[x];
    }
    __syncthreads();
    if (j0 + 16 < n) fetch(j0 + 16);
    for (int j = max(j0, i0 + 1); j < min(n, j0 + 16); ++j) {
      double t = 0.0;
      if (j > i) {
        const double* zr = zl[r];
        const double* uc = ul[j - j0];
#pragma unroll 4
        for (int k = i + ql; k < j; k += 4) t = fma(zr[k], uc[k], t);
      }
      t += dpp_mov<0xB1>(t);   // quad_perm [1,0,3,2]
      t += dpp_mov<0x4E>(t);   // quad_perm [2,3,0,1]
      if (ql == 0 && j > i) zl[r][j] = -ri[j] * t;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }
  __syncthreads();
  const int nrow = min(16, n - i0);
  for (int x = tid; x < nrow * n; x += 64) {
    const int rr = x / n, k = x % n;
    if (k >= i0 + rr) Z[(size_t)(i0 + rr) * np + k] = zl[rr][k];
  }
  if (!s.gen) {
    double* C = E.small + SmallLayout::C(s.KP);
    for (int x = tid; x < nrow * s.nkeep; x += 64) {
      const int rr = x / s.nkeep, k = x % s.nkeep;
      C[(size_t)(i0 + rr) * s.nkeep + k] =
          (k >= i0 + rr && k < n) ? vec[VS_D * s.KP + i0 + rr] * zl[rr][k] : 0.0;
    }
  }
}

// ---------------------------------------------------------------------------
// standard form: T = A~ Z (kSecond = false; A~ = D S^T H S D, symmetrised as it is read),
// then A^ = Z^T T, as 16x16 FP64 MFMA tiles, one wave each.  Order 264: 33 us for both;
// 640 us in the element's one workgroup before.
// ---------------------------------------------------------------------------
template <bool kSecond>
__global__ void __launch_bounds__(256) k_rr_prod(RRArgs A) {
  const int e = blockIdx.y;
  const ElemDev& E = A.elems[e];
  if (!rr_on(A, e)) return;
  const RRShape s = rr_shape(A, E);
  if (!kSecond) rr_stamp(A, e, 2, blockIdx.x);
  const int n = s.n, np = s.np;
  const double* Am = E.small + SmallLayout::A(s.KP);
  const double* Z = E.small + rr_slot(kSlotZ, s.KP);
  const double* d = E.small + SmallLayout::vec(s.KP) + VS_D * s.KP;
  double* T = E.small + rr_slot(kSlotT, s.KP);
  double* Ah = E.small + rr_slot(kSlotAhat, s.KP);
  double* AhT = E.small + rr_slot(kSlotAhatT, s.KP);
  const int lane = threadIdx.x & 63;
  const int nt16 = (n + 15) >> 4, kst = (n + 3) >> 2;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= nt16 * nt16) return;
  const int ti = t / nt16, tj = t % nt16;
  const int ia = ti * 16 + (lane & 15), jb = tj * 16 + (lane & 15);
  d4v acc = {0.0, 0.0, 0.0, 0.0};
  const int tz = kSecond ? ti : tj;
  const int kmax = min(kst, (tz * 16 + 16 + 3) >> 2);   // Z[k][j] = 0 for k > j
  const int ic = min(ia, n - 1), jc = min(jb, n - 1);   // beyond the matrix: results not stored
  const double di = kSecond ? 0.0 : d[ic];
  constexpr int U = 8;   // k-steps whose loads are in flight together
  for (int k0 = 0; k0 < kmax; k0 += U) {
    double av[U], bv[U], aw[U], dk[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = min((k0 + u) * 4 + (lane >> 4), n - 1);
      if constexpr (!kSecond) {
        av[u] = gload<double>(Am + (size_t)ic * n + k);
        aw[u] = gload<double>(Am + (size_t)k * n + ic);
        dk[u] = gload<double>(d + k);
        bv[u] = gload<double>(Z + (size_t)min(k, jc) * np + jc);
      } else {
        av[u] = gload<double>(Z + (size_t)min(k, ic) * np + ic);
        bv[u] = gload<double>(T + (size_t)k * np + jc);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (k0 + u >= kmax) continue;
      const int k = (k0 + u) * 4 + (lane >> 4);
      double a, b;
      if constexpr (!kSecond) {
        // left-out columns have d = 0: their rows and columns are zero
        const double s2 = di * dk[u];
        a = (k < n && s2 != 0.0) ? 0.5 * (av[u] + aw[u]) * s2 : 0.0;
        b = k <= jc ? bv[u] : 0.0;
      } else {
        a = k <= ic ? av[u] : 0.0;
        b = k < n ? bv[u] : 0.0;
      }
      acc = mfma16x16x4(a, b, acc);
    }
  }
  double* out = kSecond ? Ah : T;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = ti * 16 + (lane >> 4) + 4 * q;
    if (i < n && jb < n) {
      out[(size_t)i * np + jb] = acc[q];
      if (kSecond) AhT[(size_t)jb * np + i] = acc[q];   // for the symmetrisation
    }
  }
}

// ---------------------------------------------------------------------------
// Householder tridiagonalisation of A^ (RR_SVD: of the Gram matrix itself), one workgroup
// per element.
//
// Per step: the rank-2 update of the step before, the product with the new reflector, and
// a serial part on one wave that forms w from the product and, ahead of the update, the
// next column and reflector.  In LDS (odd pitch) the update spreads rows over the waves
// and the product columns and NS row ranges over the threads (a chain each); while the
// trailing matrix is too large for LDS it is in L2 and one pass does both, so that an
// entry is read and written once per step.  The steps in LDS hand on through barriers
// that order LDS only: __syncthreads() would wait for the reflector's global stores.
// Bound by the latency of a step (L2 accesses while in L2, then the serial part).  Order
// 264: 2270 us, 3430 us with two passes and four barriers a step on the L2-resident matrix
// before; order 132, in LDS: 371 us, 507 us before; order 36: 57 us, 59 us.
// ---------------------------------------------------------------------------
// t = v_i w_j + w_i v_j of row i and column j.  Which product is rounded first differs
// between the two size classes and is fixed, so that results do not hang on the
// compiler's choice.
template <bool kLds>
__device__ __forceinline__ double tri_t(double vi, double wi, double vj, double wj) {
  return kLds ? fma(vi, wj, wi * vj) : fma(wi, vj, vi * wj);
}

constexpr int kTriPitch = 133;                                            // LDS pitch (odd)
constexpr int kTriLdsRows = kRRLdsBytes / (kTriPitch * (int)sizeof(double));   // 133
static_assert(kRRLdsOrder < kTriPitch && kTriLdsRows >= kTriPitch, "LDS matrix of the tridiagonalisation");

// In LDS: M -= v w^T + w v^T, rows over the waves (NW of them), lanes over columns.
template <bool kLds, int NW>
__device__ __forceinline__ void tri_update(double* M, int mr, const double* v, const double* w) {
  constexpr int NC = (kTriPitch + 63) / 64;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double vj[NC], wj[NC];
  int c[NC];   // columns past the end repeat the last one: the same value is stored again
#pragma unroll
  for (int u = 0; u < NC; ++u) {
    c[u] = min(lane + 64 * u, mr - 1);
    vj[u] = v[c[u]];
    wj[u] = w[c[u]];
  }
  for (int j = wv; j < mr; j += NW) {
    const double vi = v[j], wi = w[j];
    double* row = M + j * kTriPitch;
#pragma unroll
    for (int u = 0; u < NC; ++u)
      if (64 * u < mr) row[c[u]] -= tri_t<kLds>(vi, wi, vj[u], wj[u]);
  }
}

// In LDS: pq[q][i] = sum over row range q of M[j][i] v[j], a chain per thread.
template <int NS>
__device__ __forceinline__ void tri_product(const double* M, int mr, const double* v, double (*pq)[kTriMax]) {
  const int q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
  const int qn = (mr + NS - 1) / NS;
  const int j0 = q * qn, j1 = min(mr, j0 + qn);
  const int w0 = __builtin_amdgcn_readfirstlane(threadIdx.x & 192);
  if (w0 >= mr) return;   // mr <= 256: a wave has at most one range of columns
  const int i = min(w0 + (int)(threadIdx.x & 63), mr - 1);
  double acc = 0.0;
  constexpr int B = 8;
  int j = j0;
  for (; j + B <= j1; j += B) {
    double m[B], x[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      m[u] = M[(j + u) * kTriPitch + i];
      x[u] = v[j + u];
    }
#pragma unroll
    for (int u = 0; u < B; ++u) acc = fma(m[u], x[u], acc);
  }
  for (; j < j1; ++j) acc = fma(M[j * kTriPitch + i], v[j], acc);
  pq[q][i] = acc;
}

// From L2: the update and the product in one pass over the mr x mr matrix at src (pitch
// sp), into dst (in place, or into LDS).  A thread owns a column and one of NS row
// ranges; the row's values of v, w and the new reflector come by lane reads.
// col: the updated first column.
template <bool kLds, int NS, bool kToLds>
__device__ __forceinline__ void tri_pass(const double* src, int sp, double* dst, int mr, const double* vo,
                                         const double* wo, const double* vn, double* col, double (*pq)[kTriMax]) {
  constexpr int B = 8;   // rows in flight
  const int lane = threadIdx.x & 63;
  const int q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
  const int w0 = __builtin_amdgcn_readfirstlane(threadIdx.x & 192);
  const int qn = (mr + NS - 1) / NS;
  const int j0 = q * qn, j1 = min(mr, j0 + qn);
  const int dp = kToLds ? kTriPitch : sp;
  // this range's row values, 64 rows a register
  double rv[2], rw[2], rn[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int j = min(j0 + lane + 64 * h, mr - 1);
    rv[h] = vo[j];
    rw[h] = wo[j];
    rn[h] = vn[j];
  }
  for (int i0 = w0; i0 < mr; i0 += 256) {
    // whole waves, so that every lane is there for the lane reads; lanes past the last
    // column repeat it (and store the same values again)
    const int i = min(i0 + lane, mr - 1);
    const double vj = vo[i], wj = wo[i];
    double acc = 0.0;
    auto rows = [&](int jb, int je, double av, double aw, double an) {
      auto one = [&](double x, int j) {
        const int l = (j - j0) & 63;
        const double b = x - tri_t<kLds>(lane_read(av, l), lane_read(aw, l), vj, wj);
        acc = fma(b, lane_read(an, l), acc);
        if (kToLds) dst[j * dp + i] = b;
        else gstore(dst + (size_t)j * dp + i, b);
        if (!kToLds && i0 == 0 && lane == 0) col[j] = b;
      };
      int j = jb;
      double nx[B];
      if (j + B <= je) {
#pragma unroll
        for (int u = 0; u < B; ++u) nx[u] = gload<double>(src + (size_t)(j + u) * sp + i);
      }
      for (; j + B <= je; j += B) {
        double cu[B];
#pragma unroll
        for (int u = 0; u < B; ++u) cu[u] = nx[u];
        if (j + 2 * B <= je) {
#pragma unroll
          for (int u = 0; u < B; ++u) nx[u] = gload<double>(src + (size_t)(j + B + u) * sp + i);
        }
#pragma unroll
        for (int u = 0; u < B; ++u) one(cu[u], j + u);
      }
      for (; j < je; ++j) one(gload<double>(src + (size_t)j * sp + i), j);
    };
    rows(j0, min(j1, j0 + 64), rv[0], rw[0], rn[0]);
    if (j0 + 64 < j1) rows(j0 + 64, j1, rv[1], rw[1], rn[1]);
    pq[q][i] = acc;
  }
}

template <bool kLds>
__global__ void __launch_bounds__(kLds ? kRRThreads : kRRThreadsL2) k_rr_tri(RRArgs A) {
  const int e = blockIdx.x;
  const ElemDev& E = A.elems[e];
  if (!rr_on(A, e)) return;
  const RRShape s = rr_shape(A, E);
  rr_stamp(A, e, 3, 0);
  const int m = s.n, np = s.np, KP = s.KP;
  double* vec = E.small + SmallLayout::vec(KP);
  const double* d = vec + VS_D * KP;
  double* gd = vec + VS_T0 * KP;
  double* ge = vec + VS_T1 * KP;
  double* gtau = vec + VS_T2 * KP;
  double* Rf = E.small + rr_slot(kSlotRefl, KP);
  constexpr int NT = kLds ? kRRThreads : kRRThreadsL2;
  constexpr int NS = NT / 256;
  constexpr int NR = ((kLds ? kRRLdsOrder : kTriMax) + 63) / 64;   // rows per lane of wave 0
  extern __shared__ double lm[];
  __shared__ double vb[2][kTriMax], ws[kTriMax], col[kTriMax], pq[NS][kTriMax];
  __shared__ double sh[16];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the matrix: in LDS from the start, or in L2 until the trailing part fits
  double* const gm = A.work + (size_t)e * A.work_stride;
  bool in_lds = kLds;
  int base = 0;   // LDS: row and column of the first entry
  {
    const double* G = E.small + SmallLayout::G(KP);
    const double* Ah = E.small + rr_slot(kSlotAhat, KP);
    const double* AhT = E.small + rr_slot(kSlotAhatT, KP);
    double* M = kLds ? lm : gm;
    const int mp = kLds ? kTriPitch : np;
    for (int idx = tid; idx < m * np; idx += NT) {
      const int i = idx / np, j = idx % np;
      if (j >= m) continue;
      M[(size_t)i * mp + j] = s.svd ? G[(size_t)i * m + j] : 0.5 * (Ah[idx] + AhT[idx]);
    }
    for (int i = tid; i < kTriMax; i += NT) vb[0][i] = ws[i] = 0.0;
    int left = 0;
    if (!s.svd)
      for (int i = tid; i < m; i += NT) left |= d[i] == 0.0;
    if (__syncthreads_or(left)) {
      // left-out columns get an eigenvalue above the whole spectrum (Gershgorin bound;
      // the matrix is symmetric, so a row's sum is read down its column)
      double rmax = 0.0;
      for (int i = tid; i < m; i += NT) {
        double sacc = 0.0;
        for (int k = 0; k < m; ++k) sacc += fabs(M[(size_t)k * mp + i]);
        rmax = fmax(rmax, sacc);
      }
      rmax = block_max(rmax, sh);
      for (int j = tid; j < m; j += NT)
        if (d[j] == 0.0) M[(size_t)j * mp + j] = 2.0 * rmax + 1.0;
      __syncthreads();
    }
    if (!kLds)
      for (int i = tid; i < m; i += NT) col[i] = M[(size_t)i * mp];
    __syncthreads();
  }
  int cur = 0;   // buffer of the last reflector
  for (int kk = 0; kk < m - 2; ++kk) {
    const int mr = m - kk - 1;
    double tau = 0.0;
    if (wv == 0) {
      // column kk after the last update, and the reflector that annihilates it below
      // row kk + 1: v in vb[cur ^ 1]
      const double* vo = vb[cur];
      double* vn = vb[cur ^ 1];
      auto entry = [&](int r) {
        const double x = in_lds ? lm[(r - base) * kTriPitch + kk - base] : col[r];
        return x - tri_t<kLds>(vo[r], ws[r], vo[kk], ws[kk]);
      };
      double x[NR], part = 0.0;
#pragma unroll
      for (int u = 0; u < NR; ++u) {
        x[u] = 0.0;
        if (64 * u < mr) {   // uniform; lanes past the end add zero
          const int i = lane + 64 * u;
          const double y = entry(kk + 1 + min(i, mr - 1));
          x[u] = i < mr ? y : 0.0;
          part += x[u] * x[u];
        }
      }
      const double ss = wave_sum_dpp(part);
      const double x0 = lane_read(x[0], 0);
      const double root = sqrt(ss);
      const double alpha = x0 >= 0.0 ? -root : root;
      const double dx = x0 - alpha;
      const bool zero = !(ss > 0.0);
      x[0] = lane == 0 ? dx : x[0];
#pragma unroll
      for (int u = 0; u < NR; ++u)
        if (64 * u < mr) {
          if (zero) x[u] = 0.0;
          if (lane + 64 * u < mr) vn[kk + 1 + lane + 64 * u] = x[u];
        }
      const double vv = fma(dx, dx, fma(-x0, x0, ss));
      tau = zero ? 0.0 : 2.0 / vv;
      const double dk = entry(kk);
      if (lane == 0) {
        gstore(gd + kk, dk);
        gstore(ge + kk, zero ? 0.0 : alpha);
        gstore(gtau + kk, tau);
      }
#pragma unroll
      for (int u = 0; u < NR; ++u)
        if (64 * u < mr && lane + 64 * u < mr) gstore(Rf + (size_t)kk * np + kk + 1 + lane + 64 * u, x[u]);
    }
    lds_barrier();
    {
      const double* vo = vb[cur] + kk + 1;
      const double* wo = ws + kk + 1;
      const double* vn = vb[cur ^ 1] + kk + 1;
      if (in_lds) {
        double* M = lm + (kk + 1 - base) * kTriPitch + kk + 1 - base;
        if (kk > 0) tri_update<kLds, NT / 64>(M, mr, vo, wo);
        lds_barrier();
        tri_product<NS>(M, mr, vn, pq);
      } else if constexpr (!kLds) {
        double* M = gm + (size_t)(kk + 1) * np + kk + 1;
        if (mr <= kTriLdsRows) {
          in_lds = true;
          base = kk + 1;
          tri_pass<kLds, NS, true>(M, np, lm, mr, vo, wo, vn, nullptr, pq);
        } else {
          tri_pass<kLds, NS, false>(M, np, M, mr, vo, wo, vn, col + kk + 1, pq);
        }
      }
    }
    // (the matrix moves between threads from pass to pass: in L2 its stores are waited for)
    if (in_lds) lds_barrier();
    else __syncthreads();
    cur ^= 1;
    if (wv == 0) {
      // w = tau A v - (tau / 2) (tau v^T A v) v
      const double* v = vb[cur] + kk + 1;
      double p[NR], vi[NR], kp = 0.0;
#pragma unroll
      for (int u = 0; u < NR; ++u)
        if (64 * u < mr) {
          const int i = min(lane + 64 * u, mr - 1);
          double t = 0.0;
#pragma unroll
          for (int q = 0; q < NS; ++q) t += pq[q][i];
          const double y = v[i];
          const bool on = lane + 64 * u < mr;
          p[u] = on ? t * tau : 0.0;
          vi[u] = on ? y : 0.0;
          kp += vi[u] * p[u];
        }
      const double Kc = 0.5 * tau * wave_sum_dpp(kp);
#pragma unroll
      for (int u = 0; u < NR; ++u)
        if (64 * u < mr && lane + 64 * u < mr)
          ws[kk + 1 + lane + 64 * u] = tau == 0.0 ? 0.0 : fma(-Kc, vi[u], p[u]);
      // the next reflector's lanes read rows that other lanes wrote
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }
  __syncthreads();
  if (tid < 3) {
    // the last 2 x 2 block: (m-2, m-2), (m-1, m-2), (m-1, m-1)
    const int r = m - 2 + (tid > 0), c = m - 2 + (tid > 1);
    if (c >= 0 && r >= 0) {
      const double x = in_lds ? lm[(r - base) * kTriPitch + c - base] : gm[(size_t)r * np + c];
      const double y = x - tri_t<kLds>(vb[cur][r], ws[r], vb[cur][c], ws[c]);
      if (tid == 1) ge[m - 2] = y;
      else gd[r] = y;
      if (tid == 0) gtau[m - 2] = 0.0;
    }
    if (tid == 2) ge[m - 1] = gtau[m - 1] = 0.0;
  }
}

// ---------------------------------------------------------------------------
// eigenvalues 0..nwant-1 (ascending) of the tridiagonal T by multisection on Sturm
// counts.  One round takes the counts at the 8 interior points of the bracket, which
// shrinks 9-fold; it keeps count(lo) <= j < count(hi) and stops below 2 eps ||T|| or a
// few ulps of its end points (FP64: about 17 rounds).
// Bound by the serial count (a reciprocal and five fused operations per row, about 100
// cycles), so a workgroup of two waves owns one eigenvalue and takes two rounds per
// count: lanes 0..7 the round's points, 72 more lanes the points of each of the nine
// brackets it may leave.  Order 264, 88 eigenvalues: 140 us; 490 us in the element's one
// workgroup, eight lanes per eigenvalue, before.
// ---------------------------------------------------------------------------
constexpr int kEigThreads = 128;

__global__ void __launch_bounds__(kEigThreads) k_rr_eig(RRArgs A) {
  const int e = blockIdx.y;
  const ElemDev& E = A.elems[e];
  if (!rr_on(A, e)) return;
  const RRShape s = rr_shape(A, E);
  const int j = blockIdx.x;
  if (j >= s.nwant) return;
  rr_stamp(A, e, 4, blockIdx.x);
  const int m = s.n;
  double* vec = E.small + SmallLayout::vec(s.KP);
  const double* gd = vec + VS_T0 * s.KP;
  const double* ge = vec + VS_T1 * s.KP;
  double* lam = vec + VS_FLAGS * s.KP;
  __shared__ double sd[kTriMax], se[kTriMax];
  __shared__ double sh[16];
  __shared__ unsigned long long bits[2][2];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int i = tid; i < m; i += kEigThreads) {
    sd[i] = gd[i];
    se[i] = ge[i];
  }
  __syncthreads();
  // Gershgorin bounds
  double lo = 1e300, hi = -1e300, nrm = 0.0;
  for (int i = tid; i < m; i += kEigThreads) {
    const double r = (i > 0 ? fabs(se[i - 1]) : 0.0) + (i < m - 1 ? fabs(se[i]) : 0.0);
    lo = fmin(lo, sd[i] - r);
    hi = fmax(hi, sd[i] + r);
    nrm = fmax(nrm, fabs(sd[i]) + r);
  }
  const double onenorm = fmax(block_max(nrm, sh), 1e-300);
  lo = -block_max(-lo, sh);
  hi = block_max(hi, sh);
  lo = lo - 1e-12 * onenorm - 1e-300;
  hi = hi + 1e-12 * onenorm + 1e-300;
  const double pivmin = 1e-300 + 1e-30 * onenorm * onenorm;
  const double abstol = 2.0 * 2.2204460492503131e-16 * onenorm;
  // a round's update from the flags of its 8 points (count > j)
  auto shrink = [](unsigned b, double step, double& l, double& h) {
    if (b == 0) {
      l = l + step * 8.0;
    } else {
      const int f = __ffs(b) - 1;   // first point whose count exceeds j
      const double nlo = f > 0 ? l + step * (double)f : l;
      h = l + step * (double)(f + 1);
      l = nlo;
    }
  };
  auto wide = [&](double l, double h) {
    return h - l > fmax(abstol, 4.0 * 2.2204460492503131e-16 * fmax(fabs(l), fabs(h)));
  };
  // this lane's point: of the current bracket (tid < 8), or of the bracket that the
  // round leaves when its first exceeding point is f (8: none)
  const int f = (tid - 8) >> 3, t = tid & 7;
  for (int r = 0; r < 80; r += 2) {
    if (!wide(lo, hi)) break;
    const double step = (hi - lo) * (1.0 / 9.0);
    int cnt = 0;
    if (tid < 80) {
      double pl = lo, ph = hi, ps = step;
      if (tid >= 8) {
        shrink(f < 8 ? 1u << f : 0u, step, pl, ph);
        ps = (ph - pl) * (1.0 / 9.0);
      }
      cnt = sturm_count(sd, se, m, pl + ps * (double)(t + 1), pivmin);
    }
    const unsigned long long bl = __ballot(tid < 80 && cnt > j);
    const int buf = (r >> 1) & 1;   // two buffers: one barrier per count
    if (lane == 0) bits[buf][wv] = bl;
    __syncthreads();
    const unsigned long long b0 = bits[buf][0], b1 = bits[buf][1];
    const unsigned first = (unsigned)(b0 & 0xFF);
    const int at = 8 + 8 * (first ? __ffs(first) - 1 : 8);   // the second round's flags
    const unsigned second = (unsigned)((at < 64 ? b0 >> at : b1 >> (at - 64)) & 0xFF);
    shrink(first, step, lo, hi);
    if (!wide(lo, hi)) break;
    shrink(second, (hi - lo) * (1.0 / 9.0), lo, hi);
  }
  if (tid == 0) {
    lam[j] = 0.5 * (lo + hi);
    if (j == 0) lam[s.KP - 1] = onenorm;   // for the eigenvectors
  }
}

// ---------------------------------------------------------------------------
// eigenvectors of T by inverse iteration.  Eigenvalues closer than ortol ||T|| form a
// cluster, whose vectors are computed in order, each re-orthogonalised against the
// earlier ones; a lane owns the clusters that start at its index.  Serial per vector
// (LU with partial pivoting, two or four solves), so the vectors are spread over the
// chip, four clusters per one-wave workgroup, with the factors in LDS.
// Order 264, 88 vectors: 115 us; 1020 us in the element's one workgroup (factors in L2)
// before.
// ---------------------------------------------------------------------------
constexpr int kInvPerWg = 4;

__host__ __device__ constexpr size_t inv_lds(int np) { return (size_t)np * kInvPerWg * (5 * sizeof(double) + 1); }

__global__ void __launch_bounds__(64) k_rr_inv(RRArgs A) {
  const int e = blockIdx.y;
  const ElemDev& E = A.elems[e];
  if (!rr_on(A, e)) return;
  const RRShape s = rr_shape(A, E);
  const int j0 = blockIdx.x * kInvPerWg;
  if (j0 >= s.nwant) return;
  rr_stamp(A, e, 5, blockIdx.x);
  const int m = s.n, np = s.np, nwant = s.nwant;
  const double* vec = E.small + SmallLayout::vec(s.KP);
  const double* gd = vec + VS_T0 * s.KP;
  const double* ge = vec + VS_T1 * s.KP;
  const double* lam = vec + VS_FLAGS * s.KP;
  double* Zv = E.small + rr_slot(kSlotVec, s.KP);
  extern __shared__ double dyn[];
  __shared__ double sd[kTriMax], se[kTriMax], slam[kTriMax];
  const int lane = threadIdx.x;
  for (int i = lane; i < m; i += 64) {
    sd[i] = gd[i];
    se[i] = ge[i];
  }
  for (int i = lane; i < nwant; i += 64) slam[i] = lam[i];
  __syncthreads();
  const double onenorm = lam[s.KP - 1];
  const double ortol = A.ortol * onenorm, pertol = 10.0 * 2.2e-16 * onenorm;
  const int c = j0 + lane;
  if (lane >= kInvPerWg || c >= nwant) return;
  if (c > 0 && slam[c] - slam[c - 1] <= ortol) return;   // not the first of its cluster
  constexpr int R = kInvPerWg;
  StridedD ta{dyn + 0 * (size_t)np * R + lane, R};
  StridedD tb{dyn + 1 * (size_t)np * R + lane, R};
  StridedD tu{dyn + 2 * (size_t)np * R + lane, R};
  StridedD tl{dyn + 3 * (size_t)np * R + lane, R};
  StridedD z{dyn + 4 * (size_t)np * R + lane, R};
  StridedB pv{reinterpret_cast<unsigned char*>(dyn + 5 * (size_t)np * R) + lane, R};
  double shift = slam[c];
  for (int j = c; j < nwant; ++j) {
    if (j > c) {
      if (!(slam[j] - slam[j - 1] <= ortol)) break;
      double sj = slam[j];
      if (sj < shift + pertol) sj = shift + pertol;
      shift = sj;
    }
    tri_lu(sd, se, m, shift, 2.2e-16 * onenorm, ta, tb, tu, tl, pv);
    for (int i = 0; i < m; ++i) z[i] = hash_unit(j, i);
    // an isolated eigenvalue needs no re-orthogonalisation: two solves (growth
    // at most ~1/(eps ||T||) each, far from overflow), one normalisation
    const bool single = j == c && (j + 1 >= nwant || !(slam[j + 1] - slam[j] <= ortol));
    const int n_it = single ? 2 : 4;
    for (int it = 0; it < n_it; ++it) {
      tri_solve(m, ta, tb, tu, tl, pv, z);
      if (single && it + 1 < n_it) continue;
      for (int q = c; q < j; ++q) {
        const double* zq = Zv + (size_t)q * np;
        double dot = 0.0;
        strided_blocks(m, [&](int i, auto u) {
          double a[CVN(u)], b[CVN(u)];
          for_n(u, [&](int k) { a[k] = zq[i + k]; b[k] = z[i + k]; });
          for_n(u, [&](int k) { dot += a[k] * b[k]; });
        });
        strided_blocks(m, [&](int i, auto u) {
          double a[CVN(u)], b[CVN(u)];
          for_n(u, [&](int k) { a[k] = zq[i + k]; b[k] = z[i + k]; });
          for_n(u, [&](int k) { b[k] -= dot * a[k]; });
          for_n(u, [&](int k) { z[i + k] = b[k]; });
        });
      }
      double nn = 0.0;
      strided_blocks(m, [&](int i, auto u) {
        double b[CVN(u)];
        for_n(u, [&](int k) { b[k] = z[i + k]; });
        for_n(u, [&](int k) { nn += b[k] * b[k]; });
      });
      nn = 1.0 / sqrt(nn);
      strided_blocks(m, [&](int i, auto u) {
        double b[CVN(u)];
        for_n(u, [&](int k) { b[k] = z[i + k]; });
        for_n(u, [&](int k) { z[i + k] = b[k] * nn; });
      });
    }
    strided_blocks(m, [&](int i, auto u) {
      double b[CVN(u)];
      for_n(u, [&](int k) { b[k] = z[i + k]; });
      for_n(u, [&](int k) { Zv[(size_t)j * np + i + k] = b[k]; });
    });
    if (np > m) Zv[(size_t)j * np + m] = 0.0;
  }
}

// ---------------------------------------------------------------------------
// in-order Gram-Schmidt on the eigenvectors, one workgroup per element: each vector
// against all earlier ones (dot products a wave each, the update a quad of lanes per row
// with the sum over vectors split four ways), then its norm.  A serial chain over the
// vectors, so the vectors stay in LDS, as many as fit (the later ones are read from L2).
// NT threads set the order of the norm's sum: 512 for orders that fit in LDS as a
// matrix, 1024 above.  Order 264, 88 vectors: 310 us; 751 us with all vectors in L2 before.
// ---------------------------------------------------------------------------
constexpr int kMgsLds = kLdsPerCU - 8192;   // dynamic LDS limit

template <int NT>
__global__ void __launch_bounds__(NT) k_rr_mgs(RRArgs A) {
  const int e = blockIdx.x;
  const ElemDev& E = A.elems[e];
  if (!rr_on(A, e)) return;
  const RRShape s = rr_shape(A, E);
  rr_stamp(A, e, 6, 0);
  const int m = s.n, np = s.np, nwant = s.nwant;
  double* Zv = E.small + rr_slot(kSlotVec, s.KP);
  extern __shared__ double dyn[];
  __shared__ double ps[kOrthMax];
  __shared__ double sh[16];
  constexpr int nw = NT / 64;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  double* zj = dyn;                 // the current vector
  double* zl = dyn + np;            // vectors 0 .. cap - 1
  const int cap = min(nwant, A.mgs_lds / (np * (int)sizeof(double)) - 1);
  for (int idx = tid; idx < cap * np; idx += NT) zl[idx] = Zv[idx];
  __syncthreads();
  for (int j = 1; j < nwant; ++j) {
    // (vector 0 stays as inverse iteration left it)
    for (int i = tid; i < np; i += NT) zj[i] = j < cap ? zl[j * np + i] : Zv[(size_t)j * np + i];
    lds_barrier();
    for (int q = wv; q < j; q += nw) {
      double dot = 0.0;
      if (q < cap) {
        const double* zq = zl + q * np;
        for (int i = lane; i < m; i += 64) dot += zq[i] * zj[i];
      } else {
        const double* zq = Zv + (size_t)q * np;
        for (int i = lane; i < m; i += 64) dot += zq[i] * zj[i];
      }
      dot = wave_sum_dpp(dot);
      if (lane == 0) ps[q] = dot;
    }
    lds_barrier();
    // z_j -= sum_q (z_q . z_j) z_q; per-wave sums of squares for the norm
    const int ql = tid & 3;
    double part = 0.0;
    for (int i = tid >> 2; i < m; i += NT >> 2) {
      double t = 0.0;
      const int jl = min(j, cap);
      int q = ql;
#pragma unroll 8
      for (; q < jl; q += 4) t += ps[q] * zl[q * np + i];
      for (; q < j; q += 4) t += ps[q] * Zv[(size_t)q * np + i];
      t += dpp_mov<0xB1>(t);   // quad_perm [1,0,3,2]
      t += dpp_mov<0x4E>(t);   // quad_perm [2,3,0,1]
      if (ql == 0) {
        const double v = zj[i] - t;
        zj[i] = v;
        part += v * v;
      }
    }
    part = wave_sum_dpp(part);
    if (lane == 0) sh[wv] = part;
    lds_barrier();
    double nn2 = 0.0;
    for (int q = 0; q < nw; ++q) nn2 += sh[q];
    const double nn = 1.0 / sqrt(nn2);
    for (int i = tid; i < m; i += NT) {
      const double v = zj[i] * nn;
      if (j < cap) zl[j * np + i] = v;
      gstore(Zv + (size_t)j * np + i, v);
    }
    if (j < cap) lds_barrier();   // read back from LDS only
    else __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// back-transformation z <- H_0 ... H_{m-3} z of the eigenvectors, in place.  A vector's
// reflectors are a serial chain (dot product, reduction, update), so every vector has
// lanes of its own and the vectors are spread over the chip: a wave per vector (kWave),
// or eight lanes for the orders that fit in LDS as a matrix.  The vectors sit in LDS and
// the reflectors stream through it, kBackChunk at a time, the next ones in flight.
// Order 264, 88 vectors: 127 us; 1766 us in the element's one workgroup, both in L2, before.
// ---------------------------------------------------------------------------
constexpr int kBackThreads = 256;
constexpr int kBackChunk = 16;
constexpr int kBackStage = (kBackChunk * kTriMax + kBackThreads - 1) / kBackThreads;
template <bool kWave>
constexpr int kBackVecs = kWave ? kBackThreads / 64 : kBackThreads / 8;   // vectors per workgroup

template <bool kWave>
constexpr size_t back_lds(int np) { return (size_t)(kBackVecs<kWave> + kBackChunk) * np * sizeof(double); }

template <bool kWave>
__global__ void __launch_bounds__(kBackThreads) k_rr_back(RRArgs A) {
  const int e = blockIdx.y;
  const ElemDev& E = A.elems[e];
  if (!rr_on(A, e)) return;
  const RRShape s = rr_shape(A, E);
  constexpr int NV = kBackVecs<kWave>;
  const int j0 = blockIdx.x * NV;
  if (j0 >= s.nwant) return;
  rr_stamp(A, e, 7, blockIdx.x);
  const int m = s.n, np = s.np, nwant = s.nwant;
  const double* gtau = E.small + SmallLayout::vec(s.KP) + VS_T2 * s.KP;
  const double* Rf = E.small + rr_slot(kSlotRefl, s.KP);
  double* V = E.small + rr_slot(kSlotVec, s.KP);
  extern __shared__ double dyn[];
  __shared__ double stau[kTriMax];
  double* rl = dyn;                            // reflectors of the chunk
  double* zl = dyn + (size_t)kBackChunk * np;  // vectors
  const int tid = threadIdx.x;
  constexpr int LPV = kWave ? 64 : 8;          // lanes per vector
  const int l = tid % LPV, slot = tid / LPV;
  const int nv = min(NV, nwant - j0);
  for (int i = tid; i < m; i += kBackThreads) stau[i] = gtau[i];
  for (int idx = tid; idx < nv * np; idx += kBackThreads) zl[idx] = V[(size_t)j0 * np + idx];
  const int nrefl = max(0, m - 2);
  const int nchunk = (nrefl + kBackChunk - 1) / kBackChunk;
  double pre[kBackStage];
  auto fetch = [&](int c) {
    const int cnt = min(kBackChunk, nrefl - c * kBackChunk) * np;
    const double* src = Rf + (size_t)c * kBackChunk * np;
#pragma unroll
    for (int u = 0; u < kBackStage; ++u) {
      const int idx = tid + kBackThreads * u;
      if (idx < cnt) pre[u] = gload<double>(src + idx);
    }
  };
  if (nchunk > 0) fetch(nchunk - 1);
  for (int c = nchunk - 1; c >= 0; --c) {
    const int k0 = c * kBackChunk, nk = min(kBackChunk, nrefl - k0), cnt = nk * np;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kBackStage; ++u) {
      const int idx = tid + kBackThreads * u;
      if (idx < cnt) rl[idx] = pre[u];
    }
    __syncthreads();
    if (c > 0) fetch(c - 1);
    if (slot < nv) {
      for (int k = nk - 1; k >= 0; --k) {
        const int kk = k0 + k;
        const double tau = stau[kk];
        if (tau == 0.0) continue;
        const double* v = rl + k * np + kk + 1;   // rows kk + 1 .. m - 1
        double* z = zl + slot * np + kk + 1;
        const int len = m - 1 - kk;
        if constexpr (kWave) {
          constexpr int NQ = (kTriMax + 63) / 64;
          double vq[NQ], zq[NQ], dot = 0.0;
#pragma unroll
          for (int q = 0; q < NQ; ++q)
            if (64 * q < len) {
              const int i = l + 64 * q;
              vq[q] = i < len ? v[i] : 0.0;
              zq[q] = i < len ? z[i] : 0.0;
            }
#pragma unroll
          for (int q = 0; q < NQ; ++q)
            if (64 * q < len && l + 64 * q < len) dot += vq[q] * zq[q];
          dot = wave_sum_dpp(dot) * tau;
#pragma unroll
          for (int q = 0; q < NQ; ++q)
            if (64 * q < len && l + 64 * q < len) z[l + 64 * q] = zq[q] - dot * vq[q];
        } else {
          constexpr int NQ = (kRRLdsOrder + 7) / 8;
          double vq[NQ], zq[NQ], dot = 0.0;
#pragma unroll
          for (int q = 0; q < NQ; ++q)
            if (8 * q < len) {
              const int i = l + 8 * q;
              vq[q] = i < len ? v[i] : 0.0;
              zq[q] = i < len ? z[i] : 0.0;
            }
#pragma unroll
          for (int q = 0; q < NQ; ++q)
            if (8 * q < len && l + 8 * q < len) dot += vq[q] * zq[q];
          dot = group8_sum(dot) * tau;
#pragma unroll
          for (int q = 0; q < NQ; ++q)
            if (8 * q < len && l + 8 * q < len) z[l + 8 * q] = zq[q] - dot * vq[q];
        }
        // the next reflector's lanes read rows that other lanes of the group wrote
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
  __syncthreads();
  for (int idx = tid; idx < nv * np; idx += kBackThreads) V[(size_t)j0 * np + idx] = zl[idx];
}

// ---------------------------------------------------------------------------
// coefficients: C = D Z V (RR_GEN, 16x16 FP64 MFMA tiles, one wave each; Z[i][k] = 0 for
// k < i, so a tile's k range starts at its first row; left-out rows are zero, d = 0), or
// the singular vectors over their singular values, descending (RR_SVD)
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_rr_coef(RRArgs A) {
  const int e = blockIdx.y;
  const ElemDev& E = A.elems[e];
  if (!rr_on(A, e)) return;
  const RRShape s = rr_shape(A, E);
  const int n = s.n, np = s.np, nkeep = s.nkeep, nwant = s.nwant;
  double* vec = E.small + SmallLayout::vec(s.KP);
  const double* d = vec + VS_D * s.KP;
  const double* lam = vec + VS_FLAGS * s.KP;
  double* theta = vec + VS_THETA * s.KP;
  const double* Z = E.small + rr_slot(kSlotZ, s.KP);
  const double* V = E.small + rr_slot(kSlotVec, s.KP);
  double* C = E.small + SmallLayout::C(s.KP);
  if (s.svd) {
    for (int idx = blockIdx.x * 256 + threadIdx.x; idx < n * nkeep; idx += gridDim.x * 256) {
      const int i = idx / nkeep, j = idx % nkeep;
      const int col = n - 1 - j;
      const double sg = (col >= 0) ? sqrt(fmax(lam[col], 0.0)) : 0.0;
      C[idx] = (col >= 0 && sg > 0.0) ? V[(size_t)col * np + i] / sg : 0.0;
    }
    if (blockIdx.x == 0)
      for (int j = threadIdx.x; j < nkeep; j += 256)
        theta[j] = (n - 1 - j >= 0) ? sqrt(fmax(lam[n - 1 - j], 0.0)) : 0.0;
    return;
  }
  rr_stamp(A, e, 8, blockIdx.x);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int nti = (n + 15) >> 4, ntj = (nkeep + 15) >> 4;
  const int kst = (n + 3) >> 2;
  const int tile = blockIdx.x * 4 + wv;
  if (tile < nti * ntj) {
    const int ti = tile / ntj, tj = tile % ntj;
    const int ia = ti * 16 + (lane & 15), jb = tj * 16 + (lane & 15);
    d4v acc = {0.0, 0.0, 0.0, 0.0};
    for (int ks = ti * 4; ks < kst; ++ks) {
      const int k = ks * 4 + (lane >> 4);
      const double av = (ia < n && k < n && k >= ia) ? Z[(size_t)ia * np + k] : 0.0;
      const double bv = (jb < nwant && k < n) ? V[(size_t)jb * np + k] : 0.0;
      acc = mfma16x16x4(av, bv, acc);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = ti * 16 + (lane >> 4) + 4 * q;
      if (i < n && jb < nkeep) C[(size_t)i * nkeep + jb] = jb < nwant ? d[i] * acc[q] : 0.0;
    }
  }
  if (blockIdx.x == 0)
    for (int j = threadIdx.x; j < nkeep; j += 256) theta[j] = j < nwant ? lam[j] : 0.0;
}

// ---------------------------------------------------------------------------
// launcher
// ---------------------------------------------------------------------------
void init_rr_attributes() {
  static const bool done = [] {
    auto lds = [](const void* fn, int bytes) {
      (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    };
    lds((const void*)k_rr_chol, kCholLds);
    lds((const void*)k_rr_tri<true>, kRRLdsBytes);
    lds((const void*)k_rr_tri<false>, kRRLdsBytes);
    lds((const void*)k_rr_inv, (int)inv_lds(kTriMax));
    lds((const void*)k_rr_mgs<512>, kMgsLds);
    lds((const void*)k_rr_mgs<1024>, kMgsLds);
    lds((const void*)k_rr_back<true>, (int)back_lds<true>(kTriMax));
    lds((const void*)k_rr_back<false>, (int)back_lds<false>(kRRLdsOrder));
    return true;
  }();
  (void)done;
}

int launch_rr(Ctx& c, int nb, int kfix, int nkeep, int mode, const int* active) {
  // algorithmic flop estimate: Cholesky + inverse (n^3/3 each), two n^3 products,
  // tridiagonalisation (4n^3/3), back-transformation and coefficients (4 n^2 k)
  double flops = 0.0;
  int npmax = 0;
  size_t need = 0;   // bytes of the working matrix
  int nmax = 0, nwmax = 0, nkmax = 0;
  for (int e = 0; e < c.n_elem; ++e) {
    const int n = mode == RR_GEN ? nb * c.K[e] : (kfix > 0 ? kfix : (kfix == 0 ? c.K[e] : c.J[e]));
    const int npe = n + (n & 1);
    const int nk = nkeep > 0 ? nkeep : (nkeep == 0 ? c.K[e] : c.J[e]);
    nmax = std::max(nmax, n);
    nkmax = std::max(nkmax, nk);
    nwmax = std::max(nwmax, mode == RR_SVD ? n : std::min(nk, n));
    npmax = std::max(npmax, npe);
    need = std::max(need, (size_t)npe * npe * sizeof(double));
    if (active && !c.active_host.empty() && !c.active_host[e]) continue;
    flops += (mode == RR_GEN ? 2.0 / 3.0 + 2.0 : 0.0) * (double)n * n * n + 4.0 / 3.0 * (double)n * n * n +
             4.0 * (double)n * n * nk;
  }
  if (npmax > kTriMax) {
    set_error("projected problem of order " + std::to_string(npmax) + " above the limit " +
              std::to_string(kTriMax));
    return DG_ERR_SHAPE;
  }
  // the tridiagonalisation works in LDS when the orders allow it, else (and the overlap
  // factorisation always) in the element's slice of the Gram partial-sum area (free
  // between the Gram reduction and the rotation)
  const bool in_lds = npmax <= kRRLdsOrder && need <= (size_t)kRRLdsBytes;
  if (need > (size_t)c.gram_part_stride * sizeof(double)) {
    set_error("Rayleigh-Ritz work region of " + std::to_string(need) + " bytes above the partial-sum slice");
    return DG_ERR_SHAPE;
  }
  RRArgs a{c.elems_dev, active, nb, kfix, nkeep, mode, c.dev_status,
           c.log_level >= 2 ? c.dev_phase : nullptr, c.gram_part, c.gram_part_stride,
           c.rr_pivot_tol, c.rr_drop_tol, c.log_level >= 3 ? c.dev_minpiv : nullptr, c.rr_ortol,
           0, mode == RR_GEN ? c.dev_hpflag : nullptr, c.hp_tol};
  TimedScope ts(c, TC_RR, flops);
  auto over = [](int n, int per) { return (unsigned)((n + per - 1) / per); };
  const unsigned ne = (unsigned)c.n_elem;
  if (mode != RR_SVD) {
    hipLaunchKernelGGL(k_rr_chol, dim3(ne), dim3(kCholThreads), kCholLds, c.stream, a);
    if (in_lds) hipLaunchKernelGGL(k_rr_zinv_quad, dim3(over(nmax, 16), ne), dim3(64), 0, c.stream, a);
    else hipLaunchKernelGGL(k_rr_zinv_wave, dim3(over(nmax, kZinvRows), ne), dim3(64 * kZinvRows), 0, c.stream, a);
  }
  if (mode == RR_GEN) {
    const unsigned nt = over(nmax, 16);
    hipLaunchKernelGGL(k_rr_prod<false>, dim3(over(nt * nt, 4), ne), dim3(256), 0, c.stream, a);
    hipLaunchKernelGGL(k_rr_prod<true>, dim3(over(nt * nt, 4), ne), dim3(256), 0, c.stream, a);
  }
  if (mode != RR_CHOLQR) {
    if (in_lds) {
      hipLaunchKernelGGL(k_rr_tri<true>, dim3(ne), dim3(kRRThreads), (size_t)npmax * kTriPitch * sizeof(double), c.stream, a);
    } else {
      hipLaunchKernelGGL(k_rr_tri<false>, dim3(ne), dim3(kRRThreadsL2), kRRLdsBytes, c.stream, a);
    }
    hipLaunchKernelGGL(k_rr_eig, dim3(nwmax, ne), dim3(kEigThreads), 0, c.stream, a);
    hipLaunchKernelGGL(k_rr_inv, dim3(over(nwmax, kInvPerWg), ne), dim3(64), inv_lds(npmax), c.stream, a);
    // as many vectors as fit, and the current one
    const size_t mgs = std::min((size_t)kMgsLds, (size_t)(nwmax + 1) * npmax * sizeof(double));
    a.mgs_lds = (int)mgs;
    if (in_lds) {
      hipLaunchKernelGGL(k_rr_mgs<512>, dim3(ne), dim3(512), mgs, c.stream, a);
      hipLaunchKernelGGL(k_rr_back<false>, dim3(over(nwmax, kBackVecs<false>), ne), dim3(kBackThreads),
                         back_lds<false>(npmax), c.stream, a);
    } else {
      hipLaunchKernelGGL(k_rr_mgs<1024>, dim3(ne), dim3(1024), mgs, c.stream, a);
      hipLaunchKernelGGL(k_rr_back<true>, dim3(over(nwmax, kBackVecs<true>), ne), dim3(kBackThreads),
                         back_lds<true>(npmax), c.stream, a);
    }
    hipLaunchKernelGGL(k_rr_coef, dim3(over(over(nmax, 16) * over(nkmax, 16), 4), ne), dim3(256), 0, c.stream, a);
  }
  DG_HIP(hipGetLastError());
  return DG_OK;
}


}  // namespace dg
