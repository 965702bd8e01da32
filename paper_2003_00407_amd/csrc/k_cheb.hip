// Chebyshev filter coefficients and the band-energy adjoint (elementwise / reduction
// kernels).
//
// Algorithm 2 step 2 with Eq. (8)'s three-term recurrence, scaled as in Zhou &
// Saad (2007): with e = (b - a)/2, c = (b + a)/2, sigma_1 = e / (a0 - c),
//   Y_1     = (sigma_1 / e) (H - c) Y_0
//   Y_{k+1} = (2 sigma_{k+1} / e) (H - c) Y_k - sigma_k sigma_{k+1} Y_{k-1},
//   sigma_{k+1} = 1 / (2 / sigma_1 - sigma_k).
// The step coefficients are computed on the device from each element's bounds, once per
// filter; the steps themselves are part of the H*psi passes (FilterStep).
#include "dg_internal.h"

#include <algorithm>

namespace dg {

// bounds of element e: from the context (ChFSI: a = largest Ritz value of the
// block, a0 = smallest, b = upper spectral bound) or from a caller array
__device__ __forceinline__ void elem_bounds(const ElemDev& E, const double* bounds, int e, double& a, double& b,
                                            double& a0) {
  if (bounds) {
    a = bounds[3 * e];
    b = bounds[3 * e + 1];
    a0 = bounds[3 * e + 2];
  } else {
    const int KP = E.kmax3 + 2;
    const double* th = E.small + SmallLayout::vec(KP) + VS_THETA * KP;
    a = th[E.K - 1];
    a0 = th[0];
    b = E.bup;
  }
}

// coef[e stride + 3 k + {0, 1, 2}] = alpha, c, beta of step k < m:
// Y_{k+1} = alpha (H Y_k - c Y_k) - beta Y_{k-1}.  The adjoint step takes beta of k + 1:
// A_k = alpha_k (H A_{k+1} - c A_{k+1}) - beta_{k+1} A_{k+2}.
__global__ void __launch_bounds__(64) k_cheb_coef(const ElemDev* elems, const double* bounds, int m, double* coef,
                                                  long long stride, int n_elem) {
  const int e = blockIdx.x * 64 + threadIdx.x;
  if (e >= n_elem) return;
  double a, b, a0;
  elem_bounds(elems[e], bounds, e, a, b, a0);
  const double h = 0.5 * (b - a), c = 0.5 * (b + a);
  const double s1 = h / (a0 - c);
  double s = s1;
  double* o = coef + e * stride;
  for (int k = 0; k < m; ++k, o += 3) {
    const double sn = k == 0 ? s1 : 1.0 / (2.0 / s1 - s);
    o[0] = k == 0 ? s1 / h : 2.0 * sn / h;
    o[1] = c;
    o[2] = k == 0 ? 0.0 : s * sn;
    s = sn;
  }
}

// partial[e][j][q] = sum over row range q of u_j(r) w_j(r) (FP64 accumulation, fixed
// order).  Bound by memory once the row ranges fill the GPU: with one workgroup per
// column, 40 columns of 48x48x64 took 177 us, with 36 ranges 15 us.
constexpr int kDotRows = 4096;   // rows of a range
template <typename T>
__global__ void __launch_bounds__(256) k_coldot(const ElemDev* elems, int u_blk, int w_blk, int ncols,
                                               double* partial, int pstride) {
  const int e = blockIdx.z, j = blockIdx.y;
  const ElemDev& E = elems[e];
  if (j >= ncols) return;
  const T* u = reinterpret_cast<const T*>(E.blk[u_blk]) + (size_t)j * E.ld;
  const T* w = reinterpret_cast<const T*>(E.blk[w_blk]) + (size_t)j * E.ld;
  const int r0 = blockIdx.x * kDotRows, r1 = min(E.N, r0 + kDotRows);
  double s = 0.0;
#pragma unroll 4
  for (int r = r0 + threadIdx.x; r < r1; r += 256) s += double(u[r]) * double(w[r]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  __shared__ double sh[4];
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0)
    partial[(size_t)e * pstride + j * gridDim.x + blockIdx.x] = sh[0] + sh[1] + sh[2] + sh[3];
}

// E[e] = scale * sum_j f_j sum_q partial[e][j][q], a wave per element
__global__ void __launch_bounds__(64) k_wsum(const double* partial, int pstride, const double* f, int ncols, int nq,
                                             double scale, double* E) {
  const int e = blockIdx.x;
  double s = 0.0;
  for (int i = threadIdx.x; i < ncols * nq; i += 64) s += f[i / nq] * partial[(size_t)e * pstride + i];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if (threadIdx.x == 0) E[e] = scale * s;
}

// vbar[e][r] = beta * vbar[e][r] + sum_j wt_j * u_j(r) y_j(r), wt_j = coef_e * (f ? f_j : 1)
// coef_e: the filter step's alpha, or the caller's scale
struct VbarArgs {
  const ElemDev* elems;
  int u_blk, y_blk;
  int ncols;
  const double* f;
  const double* scale;        // per element multiplier (dE), may be nullptr
  FilterStep step;            // coef: multiply by the step's alpha
  double beta;                // 0: overwrite
  double* vbar;               // FP64, packed N per element
  const long long* off;       // packed offsets (N per element)
};

template <typename T>
__global__ void __launch_bounds__(256) k_vbar(VbarArgs A) {
  const int e = blockIdx.y;
  const ElemDev& E = A.elems[e];
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= E.N) return;
  double coef = A.scale ? A.scale[e] : 1.0;
  if (A.step.coef) coef *= A.step.coef[e * A.step.stride];
  const T* u = reinterpret_cast<const T*>(E.blk[A.u_blk]);
  const T* y = reinterpret_cast<const T*>(E.blk[A.y_blk]);
  double s = 0.0;
  for (int j = 0; j < A.ncols; ++j) {
    const double w = A.f ? A.f[j] : 1.0;
    s += w * double(u[(size_t)j * E.ld + r]) * double(y[(size_t)j * E.ld + r]);
  }
  double* v = A.vbar + A.off[e] + r;
  *v = (A.beta != 0.0 ? A.beta * *v : 0.0) + coef * s;
}

// out[:, j] = s_e * f_j * in[:, j]
template <typename T>
__global__ void __launch_bounds__(256) k_scale_cols(const ElemDev* elems, int in_blk, int out_blk, int ncols,
                                                    const double* f, const double* scale, double mult) {
  const int e = blockIdx.z, j = blockIdx.y;
  const ElemDev& E = elems[e];
  if (j >= ncols) return;
  const double s = mult * (scale ? scale[e] : 1.0) * (f ? f[j] : 1.0);
  const T* in = reinterpret_cast<const T*>(E.blk[in_blk]) + (size_t)j * E.ld;
  T* out = reinterpret_cast<T*>(E.blk[out_blk]) + (size_t)j * E.ld;
  for (int r = blockIdx.x * 256 + threadIdx.x; r < E.N; r += gridDim.x * 256) out[r] = T(s * double(in[r]));
}

// block copy (same precision); blocks may live outside E.blk (checkpoints)
template <typename T>
__global__ void __launch_bounds__(256) k_copy_cols(const ElemDev* elems, const void* const* src_tab,
                                                   void* const* dst_tab, int src_blk, int dst_blk, int ncols) {
  const int e = blockIdx.z, j = blockIdx.y;
  const ElemDev& E = elems[e];
  if (j >= (ncols > 0 ? ncols : E.K)) return;
  const T* s = reinterpret_cast<const T*>(src_tab ? src_tab[e] : E.blk[src_blk]) + (size_t)j * E.ld;
  T* d = reinterpret_cast<T*>(dst_tab ? dst_tab[e] : E.blk[dst_blk]) + (size_t)j * E.ld;
  for (int r = blockIdx.x * 256 + threadIdx.x; r < E.N; r += gridDim.x * 256) d[r] = s[r];
}

// new V_eff (packed FP64, N per element) into the element arrays
__global__ void __launch_bounds__(256) k_set_potential(const ElemDev* elems, const double* v, const long long* off) {
  const int e = blockIdx.y;
  const ElemDev& E = elems[e];
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= E.N) return;
  const double x = v[off[e] + r];
  const_cast<double*>(E.v64)[r] = x;
  const_cast<float*>(E.v32)[r] = float(x);
}

// spectral upper bound after a potential update: bup = bup_base + max(max V, 0),
// a NaN in V propagates into bup (fmax would drop it)
__global__ void __launch_bounds__(1024) k_update_bounds(ElemDev* elems) {
  const int e = blockIdx.x;
  ElemDev& E = elems[e];
  double m = -1e300;
  bool nan = false;
  for (int r = threadIdx.x; r < E.N; r += 1024) {
    const double x = E.v64[r];
    nan |= !(x == x);
    m = fmax(m, x);
  }
  __shared__ double sh[16];
  __shared__ int snan;
  if (threadIdx.x == 0) snan = 0;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
  if (nan) atomicOr(&snan, 1);
  __syncthreads();
  if (threadIdx.x == 0) {
    double mm = sh[0];
    for (int w = 1; w < 16; ++w) mm = fmax(mm, sh[w]);
    E.bup = snan ? __builtin_nan("") : E.bup_base + fmax(mm, 0.0);
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static int maxN(Ctx& c) {
  int m = 0;
  for (int e = 0; e < c.n_elem; ++e) m = std::max(m, c.N[e]);
  return m;
}

static dim3 col_grid(Ctx& c, int ncols) {
  const int gx = std::min(64, (maxN(c) + 255) / 256);
  return dim3(gx, ncols, c.n_elem);
}

// the coefficients of a filter of degree m for every element, in the Gram partials'
// memory (no Gram runs during a filter; 3 m doubles of an element's part); bounds:
// nullptr for the context's
int launch_cheb_coef(Ctx& c, int m, const double* bounds) {
  if (3LL * m > c.gram_part_stride) {
    set_error("filter degree above the coefficient table");
    return DG_ERR_ARG;
  }
  hipLaunchKernelGGL(k_cheb_coef, dim3((c.n_elem + 63) / 64), dim3(64), 0, c.stream, c.elems_dev, bounds, m,
                     c.gram_part, c.gram_part_stride, c.n_elem);
  DG_HIP(hipGetLastError());
  return DG_OK;
}

int launch_weighted_dot(Ctx& c, int prec, int u_blk, int w_blk, int ncols, const double* f, double scale,
                        double* E) {
  double* partial = c.gram_part;   // n_elem x ncols x row ranges
  const int pstride = (int)std::min<long long>(c.gram_part_stride, 1 << 20);
  const int nq = (maxN(c) + kDotRows - 1) / kDotRows;
  if ((long long)ncols * nq > pstride) {
    set_error("weighted dot: the partial sums exceed their scratch");
    return DG_ERR_SHAPE;
  }
  dim3 g(nq, ncols, c.n_elem);
  if (prec == DG_FP64) hipLaunchKernelGGL(k_coldot<double>, g, dim3(256), 0, c.stream, c.elems_dev, u_blk, w_blk, ncols, partial, pstride);
  else hipLaunchKernelGGL(k_coldot<float>, g, dim3(256), 0, c.stream, c.elems_dev, u_blk, w_blk, ncols, partial, pstride);
  hipLaunchKernelGGL(k_wsum, dim3(c.n_elem), dim3(64), 0, c.stream, partial, pstride, f, ncols, nq, scale, E);
  DG_HIP(hipGetLastError());
  return DG_OK;
}

int launch_vbar(Ctx& c, int prec, int u_blk, int y_blk, int ncols, const double* f, const double* scale,
                const FilterStep& step, double beta, double* vbar) {
  VbarArgs a{c.elems_dev, u_blk, y_blk, ncols, f, scale, step, beta, vbar, c.dev_off_grid};
  dim3 g((maxN(c) + 255) / 256, c.n_elem);
  if (prec == DG_FP64) hipLaunchKernelGGL(k_vbar<double>, g, dim3(256), 0, c.stream, a);
  else hipLaunchKernelGGL(k_vbar<float>, g, dim3(256), 0, c.stream, a);
  DG_HIP(hipGetLastError());
  return DG_OK;
}

int launch_scale_cols(Ctx& c, int prec, int in_blk, int out_blk, int ncols, const double* f, const double* scale,
                      double mult) {
  if (prec == DG_FP64) hipLaunchKernelGGL(k_scale_cols<double>, col_grid(c, ncols), dim3(256), 0, c.stream, c.elems_dev, in_blk, out_blk, ncols, f, scale, mult);
  else hipLaunchKernelGGL(k_scale_cols<float>, col_grid(c, ncols), dim3(256), 0, c.stream, c.elems_dev, in_blk, out_blk, ncols, f, scale, mult);
  DG_HIP(hipGetLastError());
  return DG_OK;
}

int launch_copy_cols(Ctx& c, int prec, const void* const* src_tab, void* const* dst_tab, int src_blk, int dst_blk,
                     int ncols) {
  int gcols = ncols;
  if (gcols <= 0)
    for (int e = 0; e < c.n_elem; ++e) gcols = std::max(gcols, c.K[e]);
  if (prec == DG_FP64) hipLaunchKernelGGL(k_copy_cols<double>, col_grid(c, gcols), dim3(256), 0, c.stream, c.elems_dev, src_tab, dst_tab, src_blk, dst_blk, ncols);
  else hipLaunchKernelGGL(k_copy_cols<float>, col_grid(c, gcols), dim3(256), 0, c.stream, c.elems_dev, src_tab, dst_tab, src_blk, dst_blk, ncols);
  DG_HIP(hipGetLastError());
  return DG_OK;
}

int set_potential(Ctx& c, const double* v) {
  if (!v) {
    set_error("v_dev is NULL");
    return DG_ERR_ARG;
  }
  dim3 g((maxN(c) + 255) / 256, c.n_elem);
  hipLaunchKernelGGL(k_set_potential, g, dim3(256), 0, c.stream, c.elems_dev, v, c.dev_off_grid);
  DG_HIP(hipGetLastError());
  int st;
  if ((st = launch_update_bounds(c))) return st;
  // the eigenvectors stay as a warm start, but are no solution of the new H
  c.solved = false;
  // a band energy taken at the old potential can no longer be differentiated
  c.be_valid = false;
  return DG_OK;
}

int launch_update_bounds(Ctx& c) {
  hipLaunchKernelGGL(k_update_bounds, dim3(c.n_elem), dim3(1024), 0, c.stream, c.elems_dev);
  DG_HIP(hipGetLastError());
  return DG_OK;
}

}  // namespace dg
