// CheFSI on the DG Hamiltonian (Algorithm 2 with the block-row product of Eq. (8)).
//
// The global problem H^DG C = C Lambda is one more "element" to the subspace-iteration
// machinery: a single block of N_b = sum_k J_k rows (the ALBs of every element,
// element-major) and n_vec columns.  Filter steps, Gram matrices, the Cholesky /
// projected eigenproblem and the rotations are the element solver's own kernels; two
// pieces are specific to H^DG:
//   * k_dg_bsr: Y = H^DG X for a block of columns, one workgroup per (element row k, 16
//     or 32 columns), a wave per 16 x 16 tile: Y_k = sum over the nonzero blocks (k, k')
//     of H_{k,k'} X_{k'} (Eq. (8)) on FP64 matrix cores, both staged through LDS;
//   * the upper bound b_up by a k-step Lanczos run (Algorithm 2, step 1): seeded start,
//     H v by k_dg_bsr, one single-workgroup update kernel per step, and the largest
//     eigenvalue of the Lanczos tridiagonal (Sturm bisection) plus the last residual
//     norm, written straight into the device-side bound the filter reads.
// The lower bounds are the previous Ritz values (largest and smallest of the block),
// as in the element solver.
#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#include "dense_ops.h"

namespace dg {

int run_chfsi(Ctx& c, int prec, double tol, int max_iter, int degree, int* iters, int* n_done);

constexpr int kBsrWaves = 8;
constexpr int kBsrThreads = 64 * kBsrWaves;
constexpr int kBsrCols = 32;      // columns of X a workgroup stages at most
constexpr int kBsrChunk = 40;     // block columns staged at a time at most,
constexpr int kBsrEntries = 2048; // and their entries
constexpr int kLanczosMax = 64;

// H^DG X (or the filter step on it) of block in_blk into out_blk: workgroup (k, y) forms the rows of element k in
// 16-column tiles y, or 2 y and 2 y + 1 where the rows leave waves for both (J_k <= 64).
//
// The operator (some MB) comes from beyond L2 at each product, so what counts is the
// latency along a row's blocks and the number of load instructions per CU (operand
// fragments straight from memory: 30 us at any prefetch depth).  A chunk of up to 40 columns of a block is
// one contiguous range: the workgroup stages it and its rows of X in LDS, with three
// chunks in flight in registers and one barrier a chunk.  The block list is read 64
// blocks at a time, one a lane.  An entry's products are summed in the order of the
// blocks and of their columns.  8x8 elements of 40 functions, 13 blocks a row, 86
// columns: 24 us; 96 us with a thread per row and two barriers per block before.
__global__ void __launch_bounds__(kBsrThreads) k_dg_bsr(const ElemDev* elems, DgOp op, int in_blk, int out_blk,
                                                        int ncols, const int* active, FilterStep f) {
  // the loads that the block list hangs on go out together, before any test
  const ElemDev& E = elems[0];
  const int k = blockIdx.x;
  const int Jk = op.J[k];
  const long long b0 = op.row_ptr[k], b1 = op.row_ptr[k + 1], y0 = op.roff[k], ld = E.ld;
  const double* const X = reinterpret_cast<const double*>(E.blk[in_blk]);
  double* const Y = reinterpret_cast<double*>(E.blk[out_blk]);
  const int EK = E.K;
  const bool run = !active || active[0];
  const int K = ncols > 0 ? ncols : EK;
  const int nrt = (Jk + 15) / 16;                 // row tiles, at most 6
  const int nct = 2 * nrt <= kBsrWaves ? 2 : 1;   // column tiles
  const int c0 = 16 * nct * blockIdx.y;
  if (!run || Jk == 0 || c0 >= K) return;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kq = lane >> 4, l16 = lane & 15;
  const int ct = w / nrt, r0 = 16 * (w - ct * nrt);
  const bool on = ct < nct && c0 + 16 * ct < K;
  constexpr int XP = kBsrChunk + 1;   // odd pitch
  __shared__ double hs[2][kBsrEntries], xs[2][kBsrCols][XP];
  // rows past the end repeat the last one and are not stored
  const int i = min(r0 + l16, Jk - 1);
  const int chunk = min(kBsrChunk, (kBsrEntries / Jk) & ~3);
  // staged per thread: entries tid + kBsrThreads u of the chunk, and of X rows xr of
  // columns xc (columns past the end repeat the last one and are not stored)
  constexpr int NH = kBsrEntries / kBsrThreads;
  constexpr int NX = (kBsrCols * kBsrChunk + kBsrThreads - 1) / kBsrThreads;
  int xr[NX], xc[NX];
  const double* xcol[NX];
#pragma unroll
  for (int u = 0; u < NX; ++u) {
    const int idx = min(tid + kBsrThreads * u, 16 * nct * kBsrChunk - 1);
    xr[u] = idx % kBsrChunk;
    xc[u] = idx / kBsrChunk;
    xcol[u] = X + (long long)min(c0 + xc[u], K - 1) * ld;
  }
  d4v acc = {0.0, 0.0, 0.0, 0.0};
  int buf = 0;
  for (long long g = b0; g < b1; g += 64) {
    const int ng = (int)(b1 - g < 64 ? b1 - g : 64);
    const long long bl = g + min(lane, ng - 1);
    const int nbl = op.col_idx[bl];
    const int Jl = op.J[nbl];
    const long long hl = op.boff[bl], xl = op.roff[nbl];
    auto lane64 = [](long long v, int u) {
      const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)v, u);
      const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(v >> 32), u);
      return (long long)(((unsigned long long)hi << 32) | lo);
    };
    // the next chunk: columns l .. of block blk
    int blk = -1, l = 0, Jn = 0;
    const double* hp = op.H;
    long long xo = 0;
    auto next_block = [&] {
      do {
        if (++blk >= ng) {   // past the end the same entry is loaded, so that the count of loads in flight is fixed
          Jn = l = 0;
          hp = op.H;
          xo = 0;
          return;
        }
        Jn = __builtin_amdgcn_readlane(Jl, blk);
      } while (Jn == 0);
      l = 0;
      hp = op.H + lane64(hl, blk);
      xo = lane64(xl, blk);
    };
    struct Staged {
      double h[NH], x[NX];
      int cols;   // 0: past the end
    };
    auto fetch = [&](Staged& f) {
      f.cols = min(chunk, Jn - l);
      const int last = max(f.cols, 1) - 1, n1 = max(f.cols * Jk, 1) - 1;
#pragma unroll
      for (int u = 0; u < NH; ++u) f.h[u] = gload<double>(hp + min(tid + kBsrThreads * u, n1));
#pragma unroll
      for (int u = 0; u < NX; ++u) f.x[u] = gload<double>(xcol[u] + xo + min(xr[u], last));
      l += chunk;
      hp += chunk * Jk;
      xo += chunk;
      if (l >= Jn) next_block();
    };
    auto step = [&](Staged& f) {
      const int cols = f.cols, n1 = cols * Jk - 1;
      const double* hb = hs[buf];
#pragma unroll
      for (int u = 0; u < NH; ++u) hs[buf][min(tid + kBsrThreads * u, n1)] = f.h[u];
#pragma unroll
      for (int u = 0; u < NX; ++u) xs[buf][xc[u]][xr[u]] = f.x[u];
      lds_barrier();
      fetch(f);
      constexpr int H = kBsrChunk / 8;   // k-steps of half a chunk, without branches between
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (!on || 4 * H * h >= cols) continue;
        double a[H], b[H];
#pragma unroll
        for (int s = 0; s < H; ++s) {
          const int j = 4 * (H * h + s) + kq;
          a[s] = hb[min(j, cols - 1) * Jk + i];
          b[s] = xs[buf][16 * ct + l16][j];
        }
#pragma unroll
        for (int s = 0; s < H; ++s) {
          const bool in = 4 * (H * h + s) + kq < cols;
          acc = mfma16x16x4(in ? a[s] : 0.0, in ? b[s] : 0.0, acc);
        }
      }
      buf ^= 1;
    };
    next_block();
    Staged f0, f1, f2;   // by name: a copy from one to the next would wait for its loads
    if (blk >= ng) continue;
    fetch(f0);
    fetch(f1);
    fetch(f2);
    for (;;) {
      if (f0.cols <= 0) break;
      step(f0);
      if (f1.cols <= 0) break;
      step(f1);
      if (f2.cols <= 0) break;
      step(f2);
    }
  }
  const int c = c0 + 16 * ct + l16;
  if (!on || c >= K) return;
  const long long o = y0 + (long long)c * ld + r0 + kq;
  const double* pv = f.prev_blk >= 0 ? reinterpret_cast<const double*>(E.blk[f.prev_blk]) : nullptr;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (r0 + kq + 4 * q >= Jk) continue;
    double v = acc[q];
    if (f.coef) {
      v = f.coef[0] * (v - f.coef[1] * gload<double>(X + o + 4 * q));
      if (pv) v -= f.coef[f.beta_at] * gload<double>(pv + o + 4 * q);
    }
    gstore(Y + o + 4 * q, v);
  }
}

int launch_dg_bsr(Ctx& c, int in_blk, int out_blk, int ncols, const int* active, const FilterStep& f) {
  const int K = ncols > 0 ? ncols : c.K[0];
  TimedScope ts(c, TC_OTHER);
  hipLaunchKernelGGL(k_dg_bsr, dim3(c.dg_op.M, (K + 15) / 16), dim3(kBsrThreads), 0, c.stream,
                     c.elems_dev, c.dg_op, in_blk, out_blk, ncols, active, f);
  DG_HIP(hipGetLastError());
  return DG_OK;
}

// ---------------------------------------------------------------------------
// Lanczos upper bound
// ---------------------------------------------------------------------------
__device__ double lz_block_sum(double v, double* sh) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  __syncthreads();
  if (l == 0) sh[w] = v;
  __syncthreads();
  double s = 0.0;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) s += sh[i];
  return s;
}

// state lz: [0, 64) alpha, [64, 128) beta, 128 steps done, 129 stopped (invariant subspace)
// v = column 0 of blk_v, v_prev = column 1 of blk_v, w = H v = column 0 of blk_w.
// step < 0: normalise the start vector and clear v_prev.
__global__ void __launch_bounds__(1024) k_lz_step(const ElemDev* elems, int blk_v, int blk_w, int step, double* lz) {
  const ElemDev& E = elems[0];
  __shared__ double sh[16];
  double* v = reinterpret_cast<double*>(E.blk[blk_v]);
  double* vp = v + E.ld;
  const double* w = reinterpret_cast<const double*>(E.blk[blk_w]);
  const int N = E.N;
  if (step < 0) {
    double s = 0.0;
    for (int r = threadIdx.x; r < N; r += blockDim.x) s += v[r] * v[r];
    const double nrm = sqrt(lz_block_sum(s, sh));
    for (int r = threadIdx.x; r < N; r += blockDim.x) {
      v[r] = nrm > 0.0 ? v[r] / nrm : 0.0;
      vp[r] = 0.0;
    }
    if (threadIdx.x == 0) {
      lz[128] = 0.0;
      lz[129] = nrm > 0.0 ? 0.0 : 1.0;
    }
    return;
  }
  if (lz[129] != 0.0) return;   // uniform: every thread reads the same flag
  double s = 0.0;
  for (int r = threadIdx.x; r < N; r += blockDim.x) s += v[r] * w[r];
  const double alpha = lz_block_sum(s, sh);
  const double beta_prev = step > 0 ? lz[64 + step - 1] : 0.0;
  double f2 = 0.0;
  for (int r = threadIdx.x; r < N; r += blockDim.x) {
    const double f = w[r] - alpha * v[r] - beta_prev * vp[r];
    f2 += f * f;
  }
  const double beta = sqrt(lz_block_sum(f2, sh));
  for (int r = threadIdx.x; r < N; r += blockDim.x) {
    const double f = w[r] - alpha * v[r] - beta_prev * vp[r];
    vp[r] = v[r];
    v[r] = beta > 0.0 ? f / beta : 0.0;
  }
  if (threadIdx.x == 0) {
    lz[step] = alpha;
    lz[64 + step] = beta;
    lz[128] = step + 1;
    if (!(beta > 0.0)) lz[129] = 1.0;
  }
}

// Sturm count: eigenvalues of the m x m tridiagonal (d, e) below x
__device__ int lz_count_below(const double* d, const double* e, int m, double x) {
  int cnt = 0;
  double q = 1.0;
  for (int i = 0; i < m; ++i) {
    const double off = i > 0 ? e[i - 1] * e[i - 1] : 0.0;
    q = d[i] - x - (i > 0 ? off / q : 0.0);
    if (q == 0.0) q = -1e-300;
    if (q < 0.0) ++cnt;
  }
  return cnt;
}

// b_up = lambda_max(T_m) + |beta_m| into the element's filter bound
__global__ void k_lz_bound(ElemDev* elems, const double* lz) {
  if (threadIdx.x != 0) return;
  const int m = (int)lz[128];
  if (m <= 0) return;
  const double* d = lz;
  const double* e = lz + 64;
  double lo = 1e300, hi = -1e300;
  for (int i = 0; i < m; ++i) {
    const double r = (i > 0 ? fabs(e[i - 1]) : 0.0) + (i + 1 < m ? fabs(e[i]) : 0.0);
    lo = fmin(lo, d[i] - r);
    hi = fmax(hi, d[i] + r);
  }
  for (int it = 0; it < 200 && hi - lo > 1e-13 * fmax(fabs(lo), fabs(hi)); ++it) {
    const double mid = 0.5 * (lo + hi);
    if (lz_count_below(d, e, m, mid) == m) hi = mid;
    else lo = mid;
  }
  elems[0].bup = hi + fabs(e[m - 1]);
}

// ---------------------------------------------------------------------------
// host driver
// ---------------------------------------------------------------------------
namespace {
size_t al256(size_t x) { return (x + 255) / 256 * 256; }

struct ChefsiLayout {
  int M = 0, Nb = 0, K = 0, ld = 0, Kpad = 0, part_ld = 0, nsplit = 16;
  size_t part_stride = 0;
  size_t off_elem = 0, off_blk[kMaxBlocks] = {}, off_small = 0, off_part = 0, off_ints = 0, off_dbl = 0,
         off_phase = 0, off_rowptr = 0, off_col = 0, off_boff = 0, off_roff = 0, off_J = 0, off_lz = 0,
         off_offkall = 0, off_v64 = 0, off_v32 = 0, total = 0;
};

ChefsiLayout chefsi_layout(int M, int Nb, int K, int n_blocks) {
  ChefsiLayout L;
  L.M = M;
  L.Nb = Nb;
  L.K = K;
  L.ld = (Nb + 63) / 64 * 64;
  L.Kpad = K + (K & 1);
  L.part_ld = 3 * K;
  L.part_stride = std::max((size_t)L.nsplit * L.part_ld * L.part_ld, (size_t)6 * (L.part_ld + 2) * 512);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = al256(off + bytes);
    return o;
  };
  L.off_elem = take(sizeof(ElemDev));
  for (int b = 0; b < kMaxBlocks; ++b) L.off_blk[b] = take(sizeof(double) * (size_t)L.ld * L.Kpad);
  L.off_small = take(sizeof(double) * SmallLayout::total(3 * K + 2));
  L.off_part = take(sizeof(double) * L.part_stride);
  L.off_ints = take(sizeof(int) * 16);
  L.off_dbl = take(sizeof(double) * 16);
  L.off_phase = take(sizeof(long long) * 16);
  L.off_rowptr = take(sizeof(long long) * (M + 1));
  L.off_col = take(sizeof(int) * std::max(1, n_blocks));
  L.off_boff = take(sizeof(long long) * std::max(1, n_blocks));
  L.off_roff = take(sizeof(long long) * (M + 1));
  L.off_J = take(sizeof(int) * M);
  L.off_lz = take(sizeof(double) * 136);
  L.off_offkall = take(sizeof(long long) * 2);
  // a zero potential: the residual kernel also forms x^T V x for the element solver's
  // preconditioner energy, which the DG iteration does not use
  L.off_v64 = take(sizeof(double) * (size_t)L.ld);
  L.off_v32 = take(sizeof(float) * (size_t)L.ld);
  L.total = off + 256;
  return L;
}
}  // namespace

size_t chefsi_work_bytes(int M, int Nb, int K, int n_blocks) { return chefsi_layout(M, Nb, K, n_blocks).total; }

int chefsi(hipStream_t stream, const std::vector<int>& Js, const dg_chefsi_params& p, int n_blocks,
           const int64_t* row_ptr, const int32_t* col_idx, const int64_t* block_off, const double* hdg,
           double* x, double* eig, double* resid, void* work, size_t work_bytes, int* iters_out) {
  const int M = (int)Js.size();
  std::vector<long long> roff(M + 1, 0);
  for (int k = 0; k < M; ++k) roff[k + 1] = roff[k] + Js[k];
  const int Nb = (int)roff[M];
  const int K = p.n_vec;
  // layout of the blocks: ascending rows, columns in range, sizes J_k x J_col
  if (row_ptr[0] != 0 || row_ptr[M] != n_blocks || block_off[0] != 0) {
    set_error("row_ptr must start at 0 and end at n_blocks; block_off must start at 0");
    return DG_ERR_ARG;
  }
  for (int k = 0; k < M; ++k) {
    if (row_ptr[k + 1] < row_ptr[k]) {
      set_error("row_ptr must be non-decreasing");
      return DG_ERR_ARG;
    }
    for (long long b = row_ptr[k]; b < row_ptr[k + 1]; ++b) {
      if (col_idx[b] < 0 || col_idx[b] >= M) {
        set_error("col_idx out of range in row " + std::to_string(k));
        return DG_ERR_ARG;
      }
      if (block_off[b + 1] - block_off[b] != (long long)Js[k] * Js[col_idx[b]]) {
        set_error("block " + std::to_string(b) + " is not J_k x J_col");
        return DG_ERR_ARG;
      }
    }
  }
  for (int k = 0; k < M; ++k)
    if (Js[k] > 88) {
      set_error("J_k above 88");
      return DG_ERR_SHAPE;
    }
  if (p.n_want < 1 || K < p.n_want || K > 88 || 2 * K > Nb) {
    set_error("need 1 <= n_want <= n_vec <= min(88, N_b / 2); N_b = " + std::to_string(Nb));
    return DG_ERR_SHAPE;
  }
  if (!(p.tol > 0.0) || p.max_iter < 1 || p.degree < 1 || p.degree > 64 || p.lanczos_steps < 0 ||
      p.lanczos_steps > kLanczosMax) {
    set_error("tol > 0, max_iter >= 1, degree in [1, 64], lanczos_steps in [0, 64] (0: 10)");
    return DG_ERR_ARG;
  }
  const ChefsiLayout L = chefsi_layout(M, Nb, K, n_blocks);
  if (work_bytes < L.total) {
    set_error("work_bytes below " + std::to_string(L.total));
    return DG_ERR_OOM;
  }
  char* A = (char*)work;
  // the one-"element" context
  Ctx c;
  c.stream = stream;
  c.n_elem = 1;
  c.J = {p.n_want};
  c.G = {K - p.n_want};
  c.K = {K};
  c.N = {Nb};
  c.ld = {L.ld};
  for (int a = 0; a < 3; ++a) {
    c.elo[a] = {0};
    c.en[a] = {a == 0 ? Nb : 1};
  }
  c.kmax = K;
  c.gram_part = (double*)(A + L.off_part);
  c.gram_part_stride = (long long)L.part_stride;
  c.gram_part_ld = L.part_ld;
  c.gram_max_split = L.nsplit;
  int* ints = (int*)(A + L.off_ints);
  c.dev_active = ints;
  c.dev_status = ints + 1;
  c.dev_count = ints + 4;
  c.dev_iters = ints + 8;
  c.iota_dev = ints + 9;
  double* dbl = (double*)(A + L.off_dbl);
  c.dev_maxres = dbl;
  c.dev_minpiv = dbl + 1;
  c.dev_bounds = dbl + 4;
  c.dev_de = dbl + 7;
  c.dev_phase = (long long*)(A + L.off_phase);
  c.dev_off_kall = (long long*)(A + L.off_offkall);
  ElemDev E{};
  E.nx = Nb;
  E.ny = 1;
  E.nz = 1;
  E.N = Nb;
  E.ld = L.ld;
  E.K = K;
  E.J = p.n_want;
  E.en[0] = Nb;
  E.en[1] = 1;
  E.en[2] = 1;
  for (int b = 0; b < kMaxBlocks; ++b) E.blk[b] = A + L.off_blk[b];
  E.v64 = (const double*)(A + L.off_v64);
  E.v32 = (const float*)(A + L.off_v32);
  E.small = (double*)(A + L.off_small);
  E.kmax3 = 3 * K;
  E.bup = 0.0;
  c.elems_host = {E};
  c.elems_dev = (ElemDev*)(A + L.off_elem);
  c.dg_op.M = M;
  c.dg_op.H = hdg;
  c.dg_op.row_ptr = (const long long*)(A + L.off_rowptr);
  c.dg_op.col_idx = (const int*)(A + L.off_col);
  c.dg_op.boff = (const long long*)(A + L.off_boff);
  c.dg_op.roff = (const long long*)(A + L.off_roff);
  c.dg_op.J = (const int*)(A + L.off_J);
  c.dg_op.active = true;
  std::vector<long long> rp(row_ptr, row_ptr + M + 1), bo(block_off, block_off + std::max(1, n_blocks));
  std::vector<int> ci(col_idx, col_idx + std::max(0, n_blocks));
  if (ci.empty()) ci.push_back(0);
  const long long kall[2] = {0, K};
  const int iota0 = 0;
  auto put = [&](size_t off, const void* src, size_t bytes) -> int {
    DG_HIP(hipMemcpyAsync(A + off, src, bytes, hipMemcpyHostToDevice, stream));
    return DG_OK;
  };
  int st;
  if ((st = put(L.off_elem, &E, sizeof(ElemDev)))) return st;
  if ((st = put(L.off_rowptr, rp.data(), sizeof(long long) * rp.size()))) return st;
  if ((st = put(L.off_col, ci.data(), sizeof(int) * ci.size()))) return st;
  if ((st = put(L.off_boff, bo.data(), sizeof(long long) * bo.size()))) return st;
  if ((st = put(L.off_roff, roff.data(), sizeof(long long) * roff.size()))) return st;
  if ((st = put(L.off_J, Js.data(), sizeof(int) * M))) return st;
  if ((st = put(L.off_offkall, kall, sizeof(kall)))) return st;
  for (int b = 0; b < kMaxBlocks; ++b)
    DG_HIP(hipMemsetAsync(A + L.off_blk[b], 0, sizeof(double) * (size_t)L.ld * L.Kpad, stream));
  // flags, counters, status, iteration counts, the Lanczos state and the zero potential
  DG_HIP(hipMemsetAsync(A + L.off_ints, 0, sizeof(int) * 16, stream));
  DG_HIP(hipMemsetAsync(A + L.off_dbl, 0, sizeof(double) * 16, stream));
  DG_HIP(hipMemsetAsync(A + L.off_lz, 0, sizeof(double) * 136, stream));
  DG_HIP(hipMemsetAsync(A + L.off_v64, 0, sizeof(double) * (size_t)L.ld, stream));
  DG_HIP(hipMemsetAsync(A + L.off_v32, 0, sizeof(float) * (size_t)L.ld, stream));
  if ((st = put(L.off_ints + 9 * sizeof(int), &iota0, sizeof(int)))) return st;
  // start block
  if ((st = launch_copy_ext(c, DG_FP64, B_X, x, 0, 0, 0, Nb))) return st;
  // b_up by Lanczos from a seeded start (T0 column 0)
  const int steps = p.lanczos_steps > 0 ? p.lanczos_steps : 10;
  double* lz = (double*)(A + L.off_lz);
  if ((st = launch_random_block(c, DG_FP64, B_T0, (unsigned long long)p.seed))) return st;
  hipLaunchKernelGGL(k_lz_step, dim3(1), dim3(1024), 0, stream, c.elems_dev, (int)B_T0, (int)B_T1, -1, lz);
  for (int j = 0; j < steps; ++j) {
    if ((st = launch_dg_bsr(c, B_T0, B_T1, 1, nullptr))) return st;
    hipLaunchKernelGGL(k_lz_step, dim3(1), dim3(1024), 0, stream, c.elems_dev, (int)B_T0, (int)B_T1, j, lz);
  }
  hipLaunchKernelGGL(k_lz_bound, dim3(1), dim3(64), 0, stream, c.elems_dev, lz);
  DG_HIP(hipGetLastError());
  // Algorithm 2 iterations
  int it = 0, done = 0;
  st = run_chfsi(c, DG_FP64, p.tol, p.max_iter, p.degree, &it, &done);
  if (st < 0) return st;
  if ((st = launch_extract_kall(c, eig, resid))) return st;
  if ((st = launch_copy_ext(c, DG_FP64, B_X, x, 0, 0, 1, Nb))) return st;
  DG_HIP(hipStreamSynchronize(stream));
  if (iters_out) *iters_out = it;
  return done == 1 ? DG_OK : DG_WARN_NOT_CONVERGED;
}

}  // namespace dg
