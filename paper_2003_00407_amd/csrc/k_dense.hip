// Subspace linear algebra for the batched eigensolvers on gfx950.
//
//  * Gram matrices S^T S and S^T (H S) (the projected matrices of Eq. (4),
//    Algorithm 1 step 5; and Y^T Y, Y^T H Y of Algorithm 2 steps 3-4):
//    tall-skinny TN products, split over the grid dimension N, FP64 partial
//    tiles, then a fixed-order reduction (deterministic).
//  * Rotations X <- S C (Eq. (2), Algorithm 1 steps 6-7; Algorithm 2 step 5).
//  * Residual norms ||H x_i - theta_i x_i|| and the preconditioner energy.
#include "dense_ops.h"

#include <algorithm>
#include <cstdio>
#include <type_traits>

namespace dg {

// ---------------------------------------------------------------------------
// virtual column access: column c of the concatenation of nb blocks of K cols
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ const T* vcol(const ElemDev& E, const ColSet& s, int c, int K) {
  const int b = c / K;
  return reinterpret_cast<const T*>(E.blk[s.blk[b]]) + (size_t)(c - b * K) * E.ld;
}

// ---------------------------------------------------------------------------
// Gram: part[e][split][i][j] = sum_{r in split} S[r,i] T[r,j]
//
// Tiled row-panel design.  The 16x16 output blocks form a grid (bi x bj, the
// upper triangle when the result is symmetric); it is cut into square tiles of
// tb x tb blocks.  A workgroup owns one element, one tile and one contiguous
// range of grid rows: per step it stages GP_R rows of only the columns its tile
// touches (S columns of the tile's block rows, T columns of its block columns)
// in LDS and accumulates the tile's blocks in MFMA registers.  In pair mode a
// tile also holds the same blocks of S^T S, whose columns are S's (staged once
// on the diagonal).  With tb >= bi there is one tile: every column is staged
// once and read from HBM once per Gram.  Partial sums of the row ranges are
// reduced in a fixed order afterwards (deterministic).
// ---------------------------------------------------------------------------
struct GramArgs {
  const ElemDev* elems;
  const int* active;
  ColSet S, T;
  int kS, kT;          // columns per block (per element: <=0 -> E.K) -- multiplied by nb
  int nsplit;
  int rows_e;          // 1: reduce over the first |E_k| rows only
  int sym;             // 1: the result is symmetric, only 16x16 blocks with p <= q are computed
  int same;            // 1: T is the same column set as S
  int tb;              // tile side in 16x16 blocks
  int ntile;           // tiles of the largest element (work items per row range)
  int n_elem;          // elements in the launch
  double* part;        // per element region of part_stride doubles
  long long part_stride;
  int part_ld;         // leading dim of a partial matrix
  int pair;            // 1: also S^T S (symmetric) from the same staged S columns
  long long part_pair; // offset (doubles) of the S^T S partials inside an element's region
};

constexpr int GP_THREADS = 512;
constexpr int GP_R = 16;        // grid rows staged per step
constexpr int GP_MAXCOL = 384;  // staged columns per workgroup (tiles are chosen to fit)

// 16x16 output block number b -> (p, q): row-major over p <= q when sym, else over all
__host__ __device__ __forceinline__ void gram_block(int b, int bi, int bj, int sym, int& p, int& q) {
  if (!sym) {
    p = b / bj;
    q = b - p * bj;
    return;
  }
  p = 0;
  while (b >= bj - p) {
    b -= bj - p;
    ++p;
  }
  q = p + b;
}

// One tile of a Gram launch, for an element with bi x bj output blocks.
struct GramTile {
  int P0, P1, Q0, Q1;   // block rows / columns
  bool diag;            // symmetric result, tile on the diagonal: blocks p <= q only
  int ncA, ncB, ncC;    // staged columns: S rows-range, T cols-range, S cols-range (pair, off-diagonal)
  int nloc;             // blocks per product
};

__host__ __device__ __forceinline__ int gram_ntiles(int bi, int bj, int tb, int sym) {
  const int ti = (bi + tb - 1) / tb, tj = (bj + tb - 1) / tb;
  return sym ? ti * (ti + 1) / 2 : ti * tj;
}

__host__ __device__ __forceinline__ GramTile gram_tile(int tile, int bi, int bj, int tb, int sym, int same,
                                                       int pair) {
  const int ti = (bi + tb - 1) / tb, tj = (bj + tb - 1) / tb;
  int I, J;
  gram_block(tile, ti, tj, sym, I, J);
  GramTile g;
  g.P0 = I * tb;
  g.P1 = min(bi, g.P0 + tb);
  g.Q0 = J * tb;
  g.Q1 = min(bj, g.Q0 + tb);
  g.diag = sym && I == J;
  const int np = g.P1 - g.P0, nq = g.Q1 - g.Q0;
  g.ncA = 16 * np;
  g.ncB = (same && g.diag) ? 0 : 16 * nq;
  g.ncC = (pair && !g.diag) ? 16 * nq : 0;
  g.nloc = g.diag ? np * (np + 1) / 2 : np * nq;
  return g;
}

// Block b of a tile's list (blocks nloc .. 2 nloc - 1 are those of S^T S in pair
// mode): LDS columns of its A and B operands, and its output position packed as
// (row block << 16) | (column block << 1) | second product.
__host__ __device__ __forceinline__ void gram_tile_block(const GramTile& g, int b, int offB, int offC, int& acol,
                                                         int& bcol, int& pos) {
  const int np = g.P1 - g.P0, nq = g.Q1 - g.Q0;
  const int second = b >= g.nloc;
  const int lb = b - second * g.nloc;
  int dp, dq;
  if (g.diag) {
    gram_block(lb, np, np, 1, dp, dq);
  } else {
    dp = lb / nq;
    dq = lb - dp * nq;
  }
  acol = dp * 16;
  bcol = (second ? offC : offB) + dq * 16;
  pos = ((g.P0 + dp) << 16) | ((g.Q0 + dq) << 1) | second;
}

// Work item of a Gram workgroup on the 1D grid (ntile x row ranges, the row ranges
// padded to a multiple of 8).  Workgroup p is dispatched to XCD p % 8; its item is
// chosen so that each XCD runs every tile of its row ranges (split, element) back
// to back: the tiles of one row range stage overlapping columns, which that XCD's
// L2 then serves, and the row ranges are interleaved over the XCDs for balance.
struct GramItem {
  int tile, split, e;
  bool valid;
};

__device__ __forceinline__ GramItem gram_item(const GramArgs& A) {
  const int p = blockIdx.x;
  const int xcd = p & 7, slot = p >> 3;
  const int tile = slot % A.ntile, j = slot / A.ntile;
  const int rr = j * 8 + xcd;
  GramItem it;
  it.tile = tile;
  it.split = rr % A.nsplit;
  it.e = rr / A.nsplit;
  it.valid = it.e < A.n_elem;
  return it;
}

// FP64 staging: column-major panels, GP_RP doubles per staged column (16 rows + 2 pad), two
// panels (at most 110 KB, 55 KB for the 192 columns of the usual tiles).  Lane l reads
// rows 4 (l / 16) .. 4 (l / 16) + 3 of column (l % 16) of a 16-column fragment as two
// 16-byte loads.  MFMA k-step j takes row 4 (l / 16) + j from every lane group: the four
// k-steps cover the 16 rows of the panel, the same assignment for both operands (a Gram
// sums over rows in any order).
// Bound by the matrix cores, where their waits are covered: with at most 6 output blocks
// per wave (<= 128 VGPRs) two workgroups share a CU and one's barrier overlaps the other's
// matrix work, the next panel's loads are in flight during this one's products, and a
// block's fragments are read during the products of the one before.  Order 144, both
// products, 16 elements of 48x48x64: 2350 us, 41.9 TFLOP/s by N n (n + 1) (2580 us with the prefetched
// panel waited for at once, since its loads were behind branches, and two barriers a
// panel); twelve uneven elements up to order 264: 3160 us, 3720 us; order 36, one element
// of 16^3: 16 us, 21 us.
constexpr int GP_RP = GP_R + 2;
constexpr int GP_LDS_LIMIT = 120000;

// Block b' of a wave's contiguous run: in pair mode the two products of one (p, q)
// are adjacent (they share the A operand, S's column block p); blocks follow the
// tile's row-major order, so runs share p as well.
__device__ __forceinline__ void gram_run_block(const GramTile& g, int bprime, int pair, int offB, int offC,
                                               int& acol, int& bcol, int& pos) {
  const int lb = pair ? (bprime >> 1) : bprime;
  const int second = pair ? (bprime & 1) : 0;
  gram_tile_block(g, lb + second * g.nloc, offB, offC, acol, bcol, pos);
}

// PF: 16-byte pieces staged per thread and step (64 columns per pass of the workgroup)
template <int MAXB, int PF>
__global__ void __launch_bounds__(GP_THREADS, 4) k_gram(GramArgs A) {
  const GramItem item = gram_item(A);
  if (!item.valid) return;
  const int e = item.e;
  const ElemDev& E = A.elems[e];
  if (A.active && !A.active[e]) return;
  const int kS = kcode(A.kS, E);
  const int kT = kcode(A.kT, E);
  const int ni = A.S.nb * kS, nj = A.T.nb * kT;
  const int bi = (ni + 15) >> 4, bj = (nj + 15) >> 4;
  if (item.tile >= gram_ntiles(bi, bj, A.tb, A.sym)) return;
  const GramTile g = gram_tile(item.tile, bi, bj, A.tb, A.sym, A.same, A.pair);
  const int nblk_all = A.pair ? 2 * g.nloc : g.nloc;
  const int split = item.split;
  const int nrows = nrows_of(E, A.rows_e);
  const int rows_per = ((nrows + A.nsplit - 1) / A.nsplit + GP_R - 1) / GP_R * GP_R;
  const int r0 = split * rows_per;
  const int r1 = min(nrows, r0 + rows_per);
  const int nc = g.ncA + g.ncB + g.ncC;
  // LDS column of the B operand's first staged column, per product
  const int offB = (A.same && g.diag) ? 0 : g.ncA;
  const int offC = g.diag ? 0 : g.ncA + g.ncB;
  extern __shared__ __align__(16) double gsm[];   // two panels of [nc][GP_RP]
  // the wave index is uniform: the block bookkeeping below stays in scalar registers.
  // Wave w owns the contiguous run [w cs, (w + 1) cs) of the tile's blocks; bp, bq: LDS
  // columns of the A and B operands, bo: output position (row block, column block)
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cs = (nblk_all + 7) >> 3;
  int bp[MAXB], bq[MAXB], bo[MAXB];
  bool bv[MAXB];
#pragma unroll
  for (int t = 0; t < MAXB; ++t) {
    const int b = w * cs + t;
    bv[t] = t < cs && b < nblk_all;
    bp[t] = bq[t] = bo[t] = 0;
    if (bv[t]) gram_run_block(g, b, A.pair, offB, offC, bp[t], bq[t], bo[t]);
  }
  const int l16 = lane & 15;
  const int lrow = (lane >> 4) * (GP_R / 4);
  d4v acc[MAXB];
#pragma unroll
  for (int t = 0; t < MAXB; ++t) acc[t] = d4v{0.0, 0.0, 0.0, 0.0};
  // staging map: thread -> rows srow, srow + 1 of columns tid / 8 + 64 u.  Columns past the
  // matrix's (in its last blocks) repeat its first one, and those past the tile's the
  // tile's last; neither reaches an entry that is stored.
  constexpr int kCPP = GP_THREADS / (GP_R / 2);   // columns per pass of the workgroup
  const int srow = 2 * (threadIdx.x & (GP_R / 2 - 1)), scol = threadIdx.x / (GP_R / 2);
  const double* cp[PF];
#pragma unroll
  for (int u = 0; u < PF; ++u) {
    const int c = min(scol + kCPP * u, nc - 1);
    const bool inT = c >= g.ncA && c < g.ncA + g.ncB && !A.same;
    const int v = c < g.ncA ? 16 * g.P0 + c : 16 * g.Q0 + c - g.ncA - (c < g.ncA + g.ncB ? 0 : g.ncB);
    cp[u] = (inT ? vcol<double>(E, A.T, v < nj ? v : 0, kT) : vcol<double>(E, A.S, v < ni ? v : 0, kS)) + srow;
  }
  double2 pre[PF];
  auto load = [&](int r) {
#pragma unroll
    for (int u = 0; u < PF; ++u) pre[u] = gload2(cp[u] + r);
  };
  constexpr int KF = GP_R / 4;   // k-steps per panel = values per lane and fragment
  // two panels in LDS and one barrier a step: a panel is overwritten two steps later,
  // when every wave has passed the barrier after its reads
  int buf = 0;
  auto stage = [&] {
    double* st = gsm + buf * nc * GP_RP;
#pragma unroll
    for (int u = 0; u < PF; ++u)
      *reinterpret_cast<double2*>(st + (size_t)min(scol + kCPP * u, nc - 1) * GP_RP + srow) = pre[u];
    lds_barrier();
  };
  const int full = r0 < r1 ? (r1 - r0) / GP_R : 0, rl = r0 + full * GP_R;
  // the whole row range with n blocks per wave in a straight line: with a branch per
  // block, its fragment reads would be waited for before the next one's are issued.  (The
  // last waves' missing blocks multiply block 0 and are not stored.)
  auto run = [&](auto n) {
    constexpr int N = decltype(n)::value;
    auto multiply = [&] {
      const double* sm = gsm + buf * nc * GP_RP + l16 * GP_RP + lrow;
      auto frag = [&](int col, double (&f)[KF]) {
        const double2* q = reinterpret_cast<const double2*>(sm + col * GP_RP);
#pragma unroll
        for (int m = 0; m < KF / 2; ++m) {
          const double2 x = q[m];
          f[2 * m] = x.x;
          f[2 * m + 1] = x.y;
        }
      };
      double fa[2][KF], fb[2][KF];
      frag(bp[0], fa[0]);
      frag(bq[0], fb[0]);
#pragma unroll
      for (int t = 0; t < N; ++t) {
        if (t + 1 < N) {
          frag(bp[t + 1], fa[(t + 1) & 1]);
          frag(bq[t + 1], fb[(t + 1) & 1]);
        }
        __builtin_amdgcn_sched_barrier(0);   // one block ahead, not all of them: registers
#pragma unroll
        for (int j = 0; j < KF; ++j) acc[t] = mfma16x16x4(fa[t & 1][j], fb[t & 1][j], acc[t]);
        __builtin_amdgcn_sched_barrier(0);
      }
      buf ^= 1;
    };
    if (full > 0) {
      // the loads of the next panel are unconditional (the last step repeats its own):
      // behind a branch they would be waited for at its end, before the products
      load(r0);
      for (int r = r0; r < rl; r += GP_R) {
        stage();
        load(min(r + GP_R, rl - GP_R));
        multiply();
      }
    }
    if (rl < r1) {
      // the last rows: zero past the end (a lone last row's partner lies inside the leading
      // dimension, which is even)
      const bool in0 = rl + srow < r1, in1 = rl + srow + 1 < r1;
#pragma unroll
      for (int u = 0; u < PF; ++u) {
        const double2 x = gload2(cp[u] + (in0 ? rl : -srow));
        pre[u] = double2{in0 ? x.x : 0.0, in1 ? x.y : 0.0};
      }
      stage();
      multiply();
    }
  };
  switch (cs) {   // cs <= MAXB: the launch's plan covers every element shape (gram_blocks_per_wave)
    case 1: run(std::integral_constant<int, 1>()); break;
    case 2: if constexpr (MAXB >= 2) run(std::integral_constant<int, 2>()); break;
    case 3: if constexpr (MAXB >= 3) run(std::integral_constant<int, 3>()); break;
    case 4: if constexpr (MAXB >= 4) run(std::integral_constant<int, 4>()); break;
    case 5: if constexpr (MAXB >= 5) run(std::integral_constant<int, 5>()); break;
    default: if constexpr (MAXB >= 6) run(std::integral_constant<int, 6>());
  }
  double* out = A.part + (size_t)e * A.part_stride + (size_t)split * A.part_ld * A.part_ld;
#pragma unroll
  for (int t = 0; t < MAXB; ++t) {
    if (!bv[t]) continue;
    const bool second = bo[t] & 1;
    double* o = second ? out + A.part_pair : out;
    const int i0 = (bo[t] >> 16) * 16, j = ((bo[t] >> 1) & 0x7FFF) * 16 + l16;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = i0 + (lane >> 4) + 4 * q;
      if (i < ni && j < (second ? ni : nj)) gstore(o + (size_t)i * A.part_ld + j, acc[t][q]);
    }
  }
}

// ---------------------------------------------------------------------------
// Gram of FP32 blocks on FP32 matrix cores (the FP32 parts of the mixed path).
// Same tiles, work items, pair mode and partial sums as k_gram.  A workgroup stages
// 32-row panels of FP32 values column-major in LDS (pitch 36 floats: the sixteen
// columns of a fragment start on distinct 4-bank groups, so the 16-byte fragment
// reads are conflict-free); per panel and output block the eight k-steps of
// v_mfma_f32_16x16x4f32 are summed in FP32 and the panel's sum is added to FP64
// accumulators, so rounding grows with the 32 products of a panel, not with N.
// v_mfma_f32_16x16x4f32 (checked on the device): lane l supplies A[l%16][l/16] and
// B[l/16][l%16]; result register q of lane l is D[4 (l/16) + q][l%16].
// ---------------------------------------------------------------------------
constexpr int G3_R = 32;            // grid rows staged per step
constexpr int G3_RP = G3_R + 4;     // floats per staged column
constexpr int G3_MAXCOL = 384;

__device__ __forceinline__ f4v mfma32_16x16x4(float a, float b, f4v c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Six uneven elements up to order 264: 1187 us, 1624 us with a value a thread, loads behind
// branches and two barriers a panel.
// PF: 16-byte pieces staged per thread and step (64 columns per pass of the workgroup)
template <int MAXB, int PF>
__global__ void __launch_bounds__(GP_THREADS, 4) k_gram32(GramArgs A) {
  const GramItem item = gram_item(A);
  if (!item.valid) return;
  const int e = item.e;
  const ElemDev& E = A.elems[e];
  if (A.active && !A.active[e]) return;
  const int kS = kcode(A.kS, E);
  const int kT = kcode(A.kT, E);
  const int ni = A.S.nb * kS, nj = A.T.nb * kT;
  const int bi = (ni + 15) >> 4, bj = (nj + 15) >> 4;
  if (item.tile >= gram_ntiles(bi, bj, A.tb, A.sym)) return;
  const GramTile g = gram_tile(item.tile, bi, bj, A.tb, A.sym, A.same, A.pair);
  const int nblk_all = A.pair ? 2 * g.nloc : g.nloc;
  const int split = item.split;
  const int nrows = nrows_of(E, A.rows_e);
  const int rows_per = ((nrows + A.nsplit - 1) / A.nsplit + G3_R - 1) / G3_R * G3_R;
  const int r0 = split * rows_per;
  const int r1 = min(nrows, r0 + rows_per);
  const int nc = g.ncA + g.ncB + g.ncC;
  const int offB = (A.same && g.diag) ? 0 : g.ncA;
  const int offC = g.diag ? 0 : g.ncA + g.ncB;
  extern __shared__ __align__(16) double gsm[];
  float* const sm0 = reinterpret_cast<float*>(gsm);   // two panels of [nc][G3_RP]
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cs = (nblk_all + 7) >> 3;
  int bp[MAXB], bq[MAXB], bo[MAXB];
  bool bv[MAXB];
#pragma unroll
  for (int t = 0; t < MAXB; ++t) {
    const int b = w * cs + t;
    bv[t] = t < cs && b < nblk_all;
    bp[t] = bq[t] = bo[t] = 0;
    if (bv[t]) gram_run_block(g, b, A.pair, offB, offC, bp[t], bq[t], bo[t]);
  }
  const int l16 = lane & 15;
  const int lrow = (lane >> 4) * (G3_R / 4);
  d4v acc[MAXB];
#pragma unroll
  for (int t = 0; t < MAXB; ++t) acc[t] = d4v{0.0, 0.0, 0.0, 0.0};
  // staging and the straight line of blocks as in k_gram: thread -> rows srow .. srow + 3 of
  // columns tid / 8 + 64 u
  constexpr int kCPP = GP_THREADS / (G3_R / 4);   // columns per pass of the workgroup
  const int srow = 4 * (threadIdx.x & (G3_R / 4 - 1)), scol = threadIdx.x / (G3_R / 4);
  const float* cp[PF];
#pragma unroll
  for (int u = 0; u < PF; ++u) {
    const int c = min(scol + kCPP * u, nc - 1);
    const bool inT = c >= g.ncA && c < g.ncA + g.ncB && !A.same;
    const int v = c < g.ncA ? 16 * g.P0 + c : 16 * g.Q0 + c - g.ncA - (c < g.ncA + g.ncB ? 0 : g.ncB);
    cp[u] = (inT ? vcol<float>(E, A.T, v < nj ? v : 0, kT) : vcol<float>(E, A.S, v < ni ? v : 0, kS)) + srow;
  }
  f4v pre[PF];
  auto load = [&](int r) {
#pragma unroll
    for (int u = 0; u < PF; ++u) pre[u] = gload<f4v>(cp[u] + r);
  };
  constexpr int KF = G3_R / 4;   // k-steps per panel = values per lane and fragment
  int buf = 0;
  auto stage = [&] {
    float* st = sm0 + buf * nc * G3_RP;
#pragma unroll
    for (int u = 0; u < PF; ++u)
      *reinterpret_cast<f4v*>(st + (size_t)min(scol + kCPP * u, nc - 1) * G3_RP + srow) = pre[u];
    lds_barrier();
  };
  auto run = [&](auto n) {
    constexpr int N = decltype(n)::value;
    auto multiply = [&] {
      const float* sm = sm0 + buf * nc * G3_RP + l16 * G3_RP + lrow;
      auto frag = [&](int col, float (&f)[KF]) {
        const f4v* q = reinterpret_cast<const f4v*>(sm + col * G3_RP);
#pragma unroll
        for (int m = 0; m < KF / 4; ++m) {
          const f4v x = q[m];
#pragma unroll
          for (int i = 0; i < 4; ++i) f[4 * m + i] = x[i];
        }
      };
      float fa[2][KF], fb[2][KF];
      frag(bp[0], fa[0]);
      frag(bq[0], fb[0]);
#pragma unroll
      for (int t = 0; t < N; ++t) {
        if (t + 1 < N) {
          frag(bp[t + 1], fa[(t + 1) & 1]);
          frag(bq[t + 1], fb[(t + 1) & 1]);
        }
        __builtin_amdgcn_sched_barrier(0);
        f4v s = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < KF; ++j) s = mfma32_16x16x4(fa[t & 1][j], fb[t & 1][j], s);
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[t][q] += (double)s[q];
        __builtin_amdgcn_sched_barrier(0);
      }
      buf ^= 1;
    };
    if (r0 < r1) {   // a whole number of panels: every FP32 block has a multiple of G3_R rows
      load(r0);
      for (int r = r0; r < r1; r += G3_R) {
        stage();
        load(min(r + G3_R, r1 - G3_R));
        multiply();
      }
    }
  };
  switch (cs) {
    case 1: run(std::integral_constant<int, 1>()); break;
    case 2: if constexpr (MAXB >= 2) run(std::integral_constant<int, 2>()); break;
    case 3: if constexpr (MAXB >= 3) run(std::integral_constant<int, 3>()); break;
    case 4: if constexpr (MAXB >= 4) run(std::integral_constant<int, 4>()); break;
    case 5: if constexpr (MAXB >= 5) run(std::integral_constant<int, 5>()); break;
    default: if constexpr (MAXB >= 6) run(std::integral_constant<int, 6>());
  }
  double* out = A.part + (size_t)e * A.part_stride + (size_t)split * A.part_ld * A.part_ld;
#pragma unroll
  for (int t = 0; t < MAXB; ++t) {
    if (!bv[t]) continue;
    const bool second = bo[t] & 1;
    double* o = second ? out + A.part_pair : out;
    const int i0 = (bo[t] >> 16) * 16, j = ((bo[t] >> 1) & 0x7FFF) * 16 + l16;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = i0 + 4 * (lane >> 4) + q;
      if (i < ni && j < (second ? ni : nj)) gstore(o + (size_t)i * A.part_ld + j, acc[t][q]);
    }
  }
}

// ---------------------------------------------------------------------------
// Gram of FP32 blocks with BF16 matrix cores (the FP32 stage of the mixed path):
// every FP32 value is split into three BF16 pieces x = x0 + x1 + x2 (24 significant
// bits), the six products x_a y_b with a + b <= 2 of a 32-row stage are summed by
// v_mfma_f32_16x16x32_bf16 in FP32, and each stage's sum is added to FP64
// accumulators.  Same row-panel structure as k_gram: a workgroup stages 32 rows of
// every column (three BF16 planes, column-major in LDS) and owns all output blocks.
// v_mfma_f32_16x16x32_bf16 (checked on the device): lane l supplies A[l%16][k] and
// B[k][l%16] for eight k that A and B share; result register q is D[4(l/16)+q][l%16].
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int GB_R = 32;          // rows per stage (the MFMA's k)
constexpr int GB_PITCH = 40;      // BF16 per staged column (32 rows + pad)

__device__ __forceinline__ unsigned short bf16_bits_rn(float x) {
  const unsigned u = __float_as_uint(x);
  return (unsigned short)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ float bf16_to_float(unsigned short h) { return __uint_as_float((unsigned)h << 16); }

// PF: staged values per thread and stage (16 columns per pass of the workgroup)
template <int MAXB, int PF>
__global__ void __launch_bounds__(GP_THREADS, MAXB <= 6 && PF <= 8 ? 4 : 2) k_gram_bf16(GramArgs A) {
  const GramItem item = gram_item(A);
  if (!item.valid) return;
  const int e = item.e;
  const ElemDev& E = A.elems[e];
  if (A.active && !A.active[e]) return;
  const int kS = kcode(A.kS, E);
  const int kT = kcode(A.kT, E);
  const int ni = A.S.nb * kS, nj = A.T.nb * kT;
  const int bi = (ni + 15) >> 4, bj = (nj + 15) >> 4;
  if (item.tile >= gram_ntiles(bi, bj, A.tb, A.sym)) return;
  const GramTile g = gram_tile(item.tile, bi, bj, A.tb, A.sym, A.same, A.pair);
  const int nblk_all = A.pair ? 2 * g.nloc : g.nloc;
  const int split = item.split;
  const int nrows = nrows_of(E, A.rows_e);
  const int rows_per = ((nrows + A.nsplit - 1) / A.nsplit + GB_R - 1) / GB_R * GB_R;
  const int r0 = split * rows_per;
  const int r1 = min(nrows, r0 + rows_per);
  const int nc = g.ncA + g.ncB + g.ncC;
  const int offB = (A.same && g.diag) ? 0 : g.ncA;
  const int offC = g.diag ? 0 : g.ncA + g.ncB;
  extern __shared__ double gsm[];
  unsigned short* sm = reinterpret_cast<unsigned short*>(gsm);          // [3][nc][GB_PITCH]
  const float** cp = reinterpret_cast<const float**>(sm + 3 * nc * GB_PITCH);   // [nc]
  for (int c = threadIdx.x; c < nc; c += GP_THREADS) {
    const float* ptr = nullptr;
    if (c < g.ncA) {
      const int v = 16 * g.P0 + c;
      if (v < ni) ptr = vcol<float>(E, A.S, v, kS);
    } else if (c < g.ncA + g.ncB) {
      const int v = 16 * g.Q0 + c - g.ncA;
      if (A.same) {
        if (v < ni) ptr = vcol<float>(E, A.S, v, kS);
      } else if (v < nj) {
        ptr = vcol<float>(E, A.T, v, kT);
      }
    } else {
      const int v = 16 * g.Q0 + c - g.ncA - g.ncB;
      if (v < ni) ptr = vcol<float>(E, A.S, v, kS);
    }
    cp[c] = ptr;
  }
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int bp[MAXB], bq[MAXB], bo[MAXB];
  bool bv[MAXB];
#pragma unroll
  for (int t = 0; t < MAXB; ++t) {
    const int b = w + 8 * t;
    bv[t] = b < nblk_all;
    bp[t] = bq[t] = bo[t] = 0;
    if (bv[t]) gram_tile_block(g, b, offB, offC, bp[t], bq[t], bo[t]);
  }
  double acc[MAXB][4];
#pragma unroll
  for (int t = 0; t < MAXB; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[t][q] = 0.0;
  __syncthreads();
  // staging map: thread -> grid row (tid % 32) of columns tid / 32 + 16 u
  const int srow = threadIdx.x & (GB_R - 1), scol = threadIdx.x >> 5;
  float pre[PF];
  auto load = [&](int rbase) {
    const int rr = rbase + srow;
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      const int c = scol + 16 * u;
      float v = 0.f;
      if (c < nc) {
        const float* ptr = cp[c];
        if (ptr && rr < r1) v = ptr[rr];
      }
      pre[u] = v;
    }
  };
  const int plane = nc * GB_PITCH;
  const int koff = 8 * (lane >> 4);
  if (r0 < r1) load(r0);
  for (int r = r0; r < r1; r += GB_R) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      const int c = scol + 16 * u;
      if (c < nc) {
        const float x = pre[u];
        const unsigned short h0 = bf16_bits_rn(x);
        const float x1 = x - bf16_to_float(h0);
        const unsigned short h1 = bf16_bits_rn(x1);
        const unsigned short h2 = bf16_bits_rn(x1 - bf16_to_float(h1));
        const int o = c * GB_PITCH + srow;
        sm[o] = h0;
        sm[plane + o] = h1;
        sm[2 * plane + o] = h2;
      }
    }
    __syncthreads();
    if (r + GB_R < r1) load(r + GB_R);
#pragma unroll
    for (int t = 0; t < MAXB; ++t) {
      if (!bv[t]) continue;
      const int ca = (bp[t] + (lane & 15)) * GB_PITCH + koff;
      const int cb = (bq[t] + (lane & 15)) * GB_PITCH + koff;
      const bf16x8 a0 = *reinterpret_cast<const bf16x8*>(sm + ca);
      const bf16x8 a1 = *reinterpret_cast<const bf16x8*>(sm + plane + ca);
      const bf16x8 a2 = *reinterpret_cast<const bf16x8*>(sm + 2 * plane + ca);
      const bf16x8 c0 = *reinterpret_cast<const bf16x8*>(sm + cb);
      const bf16x8 c1 = *reinterpret_cast<const bf16x8*>(sm + plane + cb);
      const bf16x8 c2 = *reinterpret_cast<const bf16x8*>(sm + 2 * plane + cb);
      f4v sacc = {0.f, 0.f, 0.f, 0.f};
      sacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, c1, sacc, 0, 0, 0);
      sacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, c2, sacc, 0, 0, 0);
      sacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a2, c0, sacc, 0, 0, 0);
      sacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, c1, sacc, 0, 0, 0);
      sacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, c0, sacc, 0, 0, 0);
      sacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, c0, sacc, 0, 0, 0);
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[t][q] += (double)sacc[q];
    }
  }
  double* out = A.part + (size_t)e * A.part_stride + (size_t)split * A.part_ld * A.part_ld;
#pragma unroll
  for (int t = 0; t < MAXB; ++t) {
    if (!bv[t]) continue;
    const bool second = bo[t] & 1;
    double* o = second ? out + A.part_pair : out;
    const int j = ((bo[t] >> 1) & 0x7FFF) * 16 + (lane & 15);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = (bo[t] >> 16) * 16 + 4 * (lane >> 4) + q;
      if (i < ni && j < (second ? ni : nj)) o[(size_t)i * A.part_ld + j] = acc[t][q];
    }
  }
}

struct GramReduceArgs {
  const ElemDev* elems;
  const int* active;
  int sym;
  int nbS, nbT, kS, kT;
  int nsplit;
  const double* part;
  long long part_stride;
  int part_ld;
  long long out_off;   // doubles, inside E.small
  int out_ld;          // <= 0: ni
};

__global__ void __launch_bounds__(256) k_gram_reduce(GramReduceArgs A) {
  const int e = blockIdx.y;
  const ElemDev& E = A.elems[e];
  if (A.active && !A.active[e]) return;
  const int kS = kcode(A.kS, E);
  const int kT = kcode(A.kT, E);
  const int ni = A.nbS * kS, nj = A.nbT * kT;
  const int ld = A.out_ld > 0 ? A.out_ld : nj;
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= ni * nj) return;
  const int i = idx / nj, j = idx % nj;
  const bool mirror = A.sym && (i >> 4) > (j >> 4);
  const double* p = A.part + (size_t)e * A.part_stride +
                    (mirror ? (size_t)j * A.part_ld + i : (size_t)i * A.part_ld + j);
  double s = 0.0;
  for (int q = 0; q < A.nsplit; ++q) s += p[(size_t)q * A.part_ld * A.part_ld];
  E.small[soff(A.out_off, E) + (size_t)i * ld + j] = s;
}

// ---------------------------------------------------------------------------
// rotation: out_o[:, j] = beta_o out_o[:, j] + alpha sum_{c in [c0_o, c1_o)} S[:, c] C[c, j]
// ---------------------------------------------------------------------------
constexpr int RT_THREADS = 512;
constexpr int RT_RT = 2;                            // 16-row tiles per wave
constexpr int RT_ROWS = (RT_THREADS / 64) * RT_RT * 16;   // rows per workgroup (256)
constexpr int RT_CC = 32;     // C rows staged per step
constexpr int RT_MAXC = 96;   // max output columns (6 MFMA column tiles)
constexpr int RT_NCT = RT_MAXC / 16;

// out_o[:, j] = beta_o out_o[:, j] + alpha sum_c S[:, c] C[c, j] with FP64 MFMA.
// The product is formed transposed, out^T = C^T S^T, so that each lane's
// results are 16 consecutive grid rows of one column (128-byte stores).
// With two outputs whose C row ranges nest (range 1 is a suffix of range 0),
// the suffix is accumulated first, stored as output 1, then completed.
// C rows of a chunk are staged transposed: for each output column n, its RT_CC
// coefficients contiguous (pitch RT_CP doubles).  Lane l takes the 8 coefficients
// k = 8 (l / 16) .. 8 (l / 16) + 7 of column (l % 16) of a 16-column tile with four
// 16-byte LDS loads (pitch 272 bytes: 8 or 16 consecutive lanes on distinct banks);
// MFMA k-step ks uses k = 8 (l / 16) + ks, and the S operand follows the same
// assignment.  The two 16-row tiles of a wave interleave (lane row 2 (l % 16) + u), so
// a lane's two S values of a column, and its two outputs, are adjacent in memory and
// move as one 16-byte access.
constexpr int RT_CP = RT_CC + 2;

// with three column tiles three workgroups of 256 threads share a CU (<= 168 VGPRs; at 512
// threads one does, or with 128 VGPRs two that spill), with six one of 512
constexpr int rt_threads(int nct) { return nct <= 3 ? 256 : 512; }
constexpr int rt_rows(int nct) { return rt_threads(nct) / 64 * RT_RT * 16; }

// Bound by memory with few columns, by the matrix cores with many; in between by how well
// the two overlap.  A lane's S values of a chunk are two halves (k-steps 0..3, 4..7): each
// half of the next chunk is loaded as soon as this one's is used, without a branch, so
// that no wait comes before its use.  C chunks alternate
// between two LDS buffers with one barrier each.
// 16 elements of 48x48x64, 144 to 2 x 48 columns: 998 us, 4.5 TB/s (1275 us with a copy of
// the prefetched chunk and one workgroup of 512 threads per CU); twelve uneven elements up
// to 264 to 2 x 88 columns: 1380 us, 1475 us; one of 16^3, 36 to 2 x 12: 8.4 us, 9.3 us.
template <int NCT>
__global__ void __launch_bounds__(rt_threads(NCT), NCT <= 3 ? 3 : 2) k_rotate(RotArgs A) {
  static_assert(RT_RT == 2, "two interleaved row tiles per lane");
  constexpr int TH = rt_threads(NCT);
  const int e = blockIdx.y;
  const ElemDev& E = A.elems[e];
  if (A.active && !A.active[e]) return;
  const int kS = kcode(A.kS, E);
  const int ncol = kcode(A.ncol, E);
  const int cld = A.c_ld > 0 ? A.c_ld : ncol;
  const int nrows = nrows_of(E, A.rows_e);
  const int r0 = blockIdx.x * rt_rows(NCT);
  if (r0 >= nrows) return;
  int c0[2], c1[2];
  for (int o = 0; o < 2; ++o) {
    c0[o] = A.c_blockrows > 0 ? A.c0[o] * kS : A.c0[o];
    c1[o] = A.c_blockrows > 0 ? A.c1[o] * kS : A.c1[o];
  }
  __shared__ double sc[2][NCT * 16][RT_CP];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int kl = lane >> 4;
  // rows of this lane: rr0, rr0 + 1 (u = 0, 1)
  const int rr0 = r0 + w * RT_RT * 16 + 2 * (lane & 15);
  const bool in0 = rr0 < nrows, in1 = rr0 + 1 < nrows;
  const int nct = (ncol + 15) / 16;
  const double* Cm = E.small + soff(A.c_off, E);
  d4v acc[RT_RT][NCT];
#pragma unroll
  for (int u = 0; u < RT_RT; ++u)
#pragma unroll
    for (int t = 0; t < NCT; ++t) acc[u][t] = d4v{0.0, 0.0, 0.0, 0.0};
  const int nseg = A.nout > 1 ? 2 : 1;
  int buf = 0;
  for (int sg = 0; sg < nseg; ++sg) {
    // segment bounds
    int lo, hi;
    if (A.nout > 1) {
      lo = sg == 0 ? c0[1] : c0[0];
      hi = sg == 0 ? c1[1] : c0[1];
    } else {
      lo = c0[0];
      hi = c1[0];
    }
    // The (at most three) block bases of S are resolved once: a per-column lookup of
    // the block table would put a dependent pointer load before every column load.
    const double* sb0 = reinterpret_cast<const double*>(E.blk[A.S.blk[0]]);
    const long long d1 = A.S.nb > 1 ? reinterpret_cast<const double*>(E.blk[A.S.blk[1]]) - sb0 : 0;
    const long long d2 = A.S.nb > 2 ? reinterpret_cast<const double*>(E.blk[A.S.blk[2]]) - sb0 : 0;
    const long long ldS = E.ld;
    auto scol = [&](int c) -> const double* {
      const bool in1 = c >= kS, in2 = c >= 2 * kS;
      const long long off = (in2 ? d2 : (in1 ? d1 : 0LL)) + (long long)(c - (in2 ? 2 * kS : (in1 ? kS : 0))) * ldS;
      return sb0 + off;
    };
    constexpr int KH = RT_CC / 8;   // k-steps of half a chunk
    double2 s0[KH], s1[KH];
    // every lane loads one 16-byte pair from a valid address (the column clamped to lo, the
    // row pair to 0; a lone last row's partner lies inside the leading dimension, which is
    // even and at least N + 1 for odd N): rows past the end are not stored, columns past
    // the segment are multiplied as zero
    const int rv = in0 ? rr0 : 0;
    auto load_s = [&](int cb, int h, double2 (&dst)[KH]) {
#pragma unroll
      for (int ks = 0; ks < KH; ++ks) {
        const int c = cb + kl * (RT_CC / 4) + h * KH + ks;
        dst[ks] = gload2(scol(c < hi ? c : lo) + rv);
      }
    };
    constexpr int CPT = (RT_CC * NCT * 16 + TH - 1) / TH;
    double cn[CPT];
    auto load_c = [&](int cb) {
#pragma unroll
      for (int u = 0; u < CPT; ++u) {
        const int idx = threadIdx.x + u * TH;
        const int c = cb + idx / (NCT * 16), j = idx % (NCT * 16);
        cn[u] = gload<double>(Cm + (c < hi && j < ncol ? (size_t)c * cld + j : 0));
      }
    };
    if (lo < hi) {
      load_c(lo);
      load_s(lo, 0, s0);
      load_s(lo, 1, s1);
    }
    auto chunk = [&](int cb, auto more) {
#pragma unroll
      for (int u = 0; u < CPT; ++u) {
        const int idx = threadIdx.x + u * TH;
        const int cc = idx / (NCT * 16), j = idx % (NCT * 16);
        if (idx < RT_CC * NCT * 16) sc[buf][j][cc] = cb + cc < hi && j < ncol ? cn[u] : 0.0;
      }
      lds_barrier();
      if (decltype(more)::value) load_c(cb + RT_CC);
      auto half = [&](int h, double2 (&sv)[KH]) {
        double av[KH][RT_RT];
#pragma unroll
        for (int ks = 0; ks < KH; ++ks) {
          const bool in = cb + kl * (RT_CC / 4) + h * KH + ks < hi;
          av[ks][0] = in ? sv[ks].x : 0.0;
          av[ks][1] = in ? sv[ks].y : 0.0;
        }
        double cf[2][KH];
        auto coef = [&](int t) {
          const double2* q = reinterpret_cast<const double2*>(&sc[buf][t * 16 + (lane & 15)][kl * (RT_CC / 4) + h * KH]);
#pragma unroll
          for (int m = 0; m < KH / 2; ++m) {
            const double2 v = q[m];
            cf[t & 1][2 * m] = v.x;
            cf[t & 1][2 * m + 1] = v.y;
          }
        };
        coef(0);
#pragma unroll
        for (int t = 0; t < NCT; ++t) {
          if (t + 1 < NCT) coef(t + 1);   // one tile ahead (zeros past the last)
          __builtin_amdgcn_sched_barrier(0);
          if (t < nct) {
#pragma unroll
            for (int ks = 0; ks < KH; ++ks)
#pragma unroll
              for (int u = 0; u < RT_RT; ++u) acc[u][t] = mfma16x16x4(cf[t & 1][ks], av[ks][u], acc[u][t]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      half(0, s0);
      if (decltype(more)::value) load_s(cb + RT_CC, 0, s0);
      half(1, s1);
      if (decltype(more)::value) load_s(cb + RT_CC, 1, s1);
      buf ^= 1;
    };
    // (all but the last chunk load ahead without a branch)
    if (lo < hi) {
      const int last = lo + (hi - lo - 1) / RT_CC * RT_CC;
      for (int cb = lo; cb < last; cb += RT_CC) chunk(cb, std::true_type());
      chunk(last, std::false_type());
    }
    // store the output this segment completes: lane holds out[rows rr0, rr0 + 1][col 16 t + kl + 4 q]
    const int o = (A.nout > 1 && sg == 0) ? 1 : 0;
    double* out = reinterpret_cast<double*>(E.blk[A.out_blk[o]]);
    const double beta = A.beta[o];
#pragma unroll
    for (int t = 0; t < NCT; ++t) {
      if (t >= nct) continue;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = t * 16 + kl + 4 * q;
        if (j >= ncol) continue;
        double* p = out + (size_t)j * E.ld + rr0;
        // the beta term: the output's own values, or those of an FP32 block
        const float* p32 = A.add32 ? reinterpret_cast<const float*>(E.blk[A.add32_blk[o]]) + (size_t)j * E.ld + rr0
                                   : nullptr;
        if (in1) {
          double2 v = {A.alpha * acc[0][t][q], A.alpha * acc[1][t][q]};
          if (beta != 0.0) {
            double2 prev;
            if (p32) {
              const float2 f = gload2f(p32);
              prev = double2{(double)f.x, (double)f.y};
            } else {
              prev = gload2(p);
            }
            v.x += beta * prev.x;
            v.y += beta * prev.y;
          }
          gstore2(p, v.x, v.y);
        } else if (in0) {
          const double prev = beta != 0.0 ? beta * (p32 ? (double)*p32 : double(*p)) : 0.0;
          *p = prev + A.alpha * acc[0][t][q];
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// The same rotation for FP32 blocks on FP32 matrix cores (v_mfma_f32_16x16x4f32,
// FP32 sums): C chunks of 32 rows staged transposed as FP32 (pitch 36 floats, the
// eight coefficients of a lane two 16-byte reads), each lane's two row tiles are
// adjacent rows, so S loads and output stores move 8 bytes per column.  Lane l's
// result q of column tile t is output column 16 t + 4 (l / 16) + q.
// ---------------------------------------------------------------------------
constexpr int R3_CP = RT_CC + 4;

template <int NCT>
__global__ void __launch_bounds__(RT_THREADS, NCT <= 3 ? 4 : 2) k_rotate32(RotArgs A) {
  const int e = blockIdx.y;
  const ElemDev& E = A.elems[e];
  if (A.active && !A.active[e]) return;
  const int kS = kcode(A.kS, E);
  const int ncol = kcode(A.ncol, E);
  const int cld = A.c_ld > 0 ? A.c_ld : ncol;
  const int nrows = nrows_of(E, A.rows_e);
  const int r0 = blockIdx.x * RT_ROWS;
  if (r0 >= nrows) return;
  int c0[2], c1[2];
  for (int o = 0; o < 2; ++o) {
    c0[o] = A.c_blockrows > 0 ? A.c0[o] * kS : A.c0[o];
    c1[o] = A.c_blockrows > 0 ? A.c1[o] * kS : A.c1[o];
  }
  __shared__ __attribute__((aligned(16))) float sc[2][NCT * 16][R3_CP];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int kl = lane >> 4;
  const int rr0 = r0 + w * RT_RT * 16 + 2 * (lane & 15);
  const bool in0 = rr0 < nrows, in1 = rr0 + 1 < nrows;
  const int nct = (ncol + 15) / 16;
  const double* Cm = E.small + soff(A.c_off, E);
  f4v acc[RT_RT][NCT];
#pragma unroll
  for (int u = 0; u < RT_RT; ++u)
#pragma unroll
    for (int t = 0; t < NCT; ++t) acc[u][t] = f4v{0.f, 0.f, 0.f, 0.f};
  const int nseg = A.nout > 1 ? 2 : 1;
  int buf = 0;
  for (int sg = 0; sg < nseg; ++sg) {
    int lo, hi;
    if (A.nout > 1) {
      lo = sg == 0 ? c0[1] : c0[0];
      hi = sg == 0 ? c1[1] : c0[1];
    } else {
      lo = c0[0];
      hi = c1[0];
    }
    const float* sb0 = reinterpret_cast<const float*>(E.blk[A.S.blk[0]]);
    const long long d1 = A.S.nb > 1 ? reinterpret_cast<const float*>(E.blk[A.S.blk[1]]) - sb0 : 0;
    const long long d2 = A.S.nb > 2 ? reinterpret_cast<const float*>(E.blk[A.S.blk[2]]) - sb0 : 0;
    const long long ldS = E.ld;
    auto scol = [&](int c) -> const float* {
      const bool b1 = c >= kS, b2 = c >= 2 * kS;
      const long long off = (b2 ? d2 : (b1 ? d1 : 0LL)) + (long long)(c - (b2 ? 2 * kS : (b1 ? kS : 0))) * ldS;
      return sb0 + off;
    };
    // as in k_rotate: halves of the next chunk loaded as this one's are used, coefficients in
    // two LDS buffers
    constexpr int KH = RT_CC / 8;
    float2 s0[KH], s1[KH];
    const int rv = in0 ? rr0 : 0;
    auto load_s = [&](int cb, int h, float2 (&dst)[KH]) {
#pragma unroll
      for (int ks = 0; ks < KH; ++ks) {
        const int c = cb + kl * (RT_CC / 4) + h * KH + ks;
        dst[ks] = gload2f(scol(c < hi ? c : lo) + rv);
      }
    };
    constexpr int CPT = (RT_CC * NCT * 16 + RT_THREADS - 1) / RT_THREADS;
    double cn[CPT];
    auto load_c = [&](int cb) {
#pragma unroll
      for (int u = 0; u < CPT; ++u) {
        const int idx = threadIdx.x + u * RT_THREADS;
        const int c = cb + idx / (NCT * 16), j = idx % (NCT * 16);
        cn[u] = gload<double>(Cm + (c < hi && j < ncol ? (size_t)c * cld + j : 0));
      }
    };
    if (lo < hi) {
      load_c(lo);
      load_s(lo, 0, s0);
      load_s(lo, 1, s1);
    }
    auto chunk = [&](int cb, auto more) {
#pragma unroll
      for (int u = 0; u < CPT; ++u) {
        const int idx = threadIdx.x + u * RT_THREADS;
        const int cc = idx / (NCT * 16), j = idx % (NCT * 16);
        if (idx < RT_CC * NCT * 16) sc[buf][j][cc] = cb + cc < hi && j < ncol ? (float)cn[u] : 0.f;
      }
      lds_barrier();
      if (decltype(more)::value) load_c(cb + RT_CC);
      auto half = [&](int h, float2 (&sv)[KH]) {
        float av[KH][RT_RT];
#pragma unroll
        for (int ks = 0; ks < KH; ++ks) {
          const bool in = cb + kl * (RT_CC / 4) + h * KH + ks < hi;
          av[ks][0] = in ? sv[ks].x : 0.f;
          av[ks][1] = in ? sv[ks].y : 0.f;
        }
        f4v cf[2];
        static_assert(KH == 4, "a half chunk's coefficients are one 16-byte piece");
        auto coef = [&](int t) {
          cf[t & 1] = *reinterpret_cast<const f4v*>(&sc[buf][t * 16 + (lane & 15)][kl * (RT_CC / 4) + h * KH]);
        };
        coef(0);
#pragma unroll
        for (int t = 0; t < NCT; ++t) {
          if (t + 1 < NCT) coef(t + 1);   // one tile ahead (zeros past the last)
          __builtin_amdgcn_sched_barrier(0);
          if (t < nct) {
#pragma unroll
            for (int ks = 0; ks < KH; ++ks)
#pragma unroll
              for (int u = 0; u < RT_RT; ++u) acc[u][t] = mfma32_16x16x4(cf[t & 1][ks], av[ks][u], acc[u][t]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      half(0, s0);
      if (decltype(more)::value) load_s(cb + RT_CC, 0, s0);
      half(1, s1);
      if (decltype(more)::value) load_s(cb + RT_CC, 1, s1);
      buf ^= 1;
    };
    if (lo < hi) {
      const int last = lo + (hi - lo - 1) / RT_CC * RT_CC;
      for (int cb = lo; cb < last; cb += RT_CC) chunk(cb, std::true_type());
      chunk(last, std::false_type());
    }
    // store the output this segment completes: lane holds out[rows rr0, rr0 + 1][col 16 t + 4 kl + q]
    const int o = (A.nout > 1 && sg == 0) ? 1 : 0;
    float* out = reinterpret_cast<float*>(E.blk[A.out_blk[o]]);
    const double beta = A.beta[o];
#pragma unroll
    for (int t = 0; t < NCT; ++t) {
      if (t >= nct) continue;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = t * 16 + 4 * kl + q;
        if (j >= ncol) continue;
        float* p = out + (size_t)j * E.ld + rr0;
        if (in1) {
          double v0 = A.alpha * (double)acc[0][t][q], v1 = A.alpha * (double)acc[1][t][q];
          if (beta != 0.0) {
            const float2 prev = gload2f(p);
            v0 += beta * (double)prev.x;
            v1 += beta * (double)prev.y;
          }
          gstore2f(p, (float)v0, (float)v1);
        } else if (in0) {
          const double prev = beta != 0.0 ? beta * (double)*p : 0.0;
          *p = (float)(prev + A.alpha * (double)acc[0][t][q]);
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// The same rotation for FP32 blocks on BF16 matrix cores (the FP32 stage of the
// mixed path): S values and C coefficients are split into three BF16 pieces each
// (24 significant bits), and the six products s_a c_b with a + b <= 2 of every
// 32-row step of C go to v_mfma_f32_16x16x32_bf16, smallest first, summed in FP32.
// out^T = C^T S^T as in k_rotate: the A operand is a 16-column tile of C^T (staged
// as three BF16 planes in LDS, the 32 C rows of a step contiguous per column), the
// B operand 32 S columns of 16 grid rows (eight per lane, split in registers).
// ---------------------------------------------------------------------------
constexpr int RB_K = 32;        // C rows per MFMA step
constexpr int RB_PITCH = 40;    // BF16 per staged C column (32 rows + pad)

typedef unsigned short us8v __attribute__((ext_vector_type(8)));

template <int NCT>
__global__ void __launch_bounds__(RT_THREADS, 2) k_rotate_bf16(RotArgs A) {
  const int e = blockIdx.y;
  const ElemDev& E = A.elems[e];
  if (A.active && !A.active[e]) return;
  const int kS = kcode(A.kS, E);
  const int ncol = kcode(A.ncol, E);
  const int cld = A.c_ld > 0 ? A.c_ld : ncol;
  const int nrows = nrows_of(E, A.rows_e);
  const int r0 = blockIdx.x * RT_ROWS;
  if (r0 >= nrows) return;
  int c0[2], c1[2];
  for (int o = 0; o < 2; ++o) {
    c0[o] = A.c_blockrows > 0 ? A.c0[o] * kS : A.c0[o];
    c1[o] = A.c_blockrows > 0 ? A.c1[o] * kS : A.c1[o];
  }
  __shared__ __attribute__((aligned(16))) unsigned short scb[3][NCT * 16][RB_PITCH];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int kl = lane >> 4;
  int rrow[RT_RT];
#pragma unroll
  for (int u = 0; u < RT_RT; ++u) rrow[u] = r0 + (w * RT_RT + u) * 16 + (lane & 15);
  const int nct = (ncol + 15) / 16;
  const double* Cm = E.small + soff(A.c_off, E);
  f4v acc[RT_RT][NCT];
#pragma unroll
  for (int u = 0; u < RT_RT; ++u)
#pragma unroll
    for (int t = 0; t < NCT; ++t) acc[u][t] = f4v{0.f, 0.f, 0.f, 0.f};
  const int nseg = A.nout > 1 ? 2 : 1;
  for (int sg = 0; sg < nseg; ++sg) {
    int lo, hi;
    if (A.nout > 1) {
      lo = sg == 0 ? c0[1] : c0[0];
      hi = sg == 0 ? c1[1] : c0[1];
    } else {
      lo = c0[0];
      hi = c1[0];
    }
    // S values of the next step (columns cb + 8 kl + i, rows rrow[u]) are loaded
    // while the current step is multiplied
    // block bases resolved once (a per-column lookup of the block table puts a
    // dependent pointer load before every column load); branch-free global loads from
    // clamped valid addresses, out-of-range values zeroed
    const float* sb0 = reinterpret_cast<const float*>(E.blk[A.S.blk[0]]);
    const long long d1 = A.S.nb > 1 ? reinterpret_cast<const float*>(E.blk[A.S.blk[1]]) - sb0 : 0;
    const long long d2 = A.S.nb > 2 ? reinterpret_cast<const float*>(E.blk[A.S.blk[2]]) - sb0 : 0;
    const long long ldS = E.ld;
    auto scol = [&](int c) -> const float* {
      const bool b1 = c >= kS, b2 = c >= 2 * kS;
      const long long off = (b2 ? d2 : (b1 ? d1 : 0LL)) + (long long)(c - (b2 ? 2 * kS : (b1 ? kS : 0))) * ldS;
      return sb0 + off;
    };
    float sv[RT_RT][8], sn[RT_RT][8];
    auto load_s = [&](int cb, float (&dst)[RT_RT][8]) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int c = cb + 8 * kl + i;
        const bool cin = c < hi;
        const float* col = scol(cin ? c : lo);
#pragma unroll
        for (int u = 0; u < RT_RT; ++u) {
          const bool ok = cin && rrow[u] < nrows;
          const float v = gload<float>(col + (rrow[u] < nrows ? rrow[u] : 0));
          dst[u][i] = ok ? v : 0.f;
        }
      }
    };
    // with six column tiles the C rows of the next step are prefetched into registers
    // too; with three they are read when staged (the registers would cost occupancy)
    constexpr bool kPrefC = NCT > 3;
    constexpr int CPT = (RB_K * NCT * 16 + RT_THREADS - 1) / RT_THREADS;
    double cn[kPrefC ? CPT : 1];
    auto load_c = [&](int cb) {
#pragma unroll
      for (int u = 0; u < CPT; ++u) {
        const int idx = threadIdx.x + u * RT_THREADS;
        const int j = idx % (NCT * 16), k = idx / (NCT * 16);
        const int c = cb + k;
        if constexpr (kPrefC) {
          const bool ok = idx < RB_K * NCT * 16 && c < hi && j < ncol;
          const double v = gload<double>(Cm + (ok ? (size_t)c * cld + j : 0));
          cn[u] = ok ? v : 0.0;
        }
      }
    };
    if (lo < hi) {
      load_s(lo, sn);
      if constexpr (kPrefC) load_c(lo);
    }
    for (int cb = lo; cb < hi; cb += RB_K) {
      __syncthreads();
      // C rows cb .. cb+31 as three BF16 planes, transposed (scb[piece][column j][row k])
#pragma unroll
      for (int u = 0; u < CPT; ++u) {
        const int idx = threadIdx.x + u * RT_THREADS;
        if (idx >= RB_K * NCT * 16) continue;
        const int j = idx % (NCT * 16), k = idx / (NCT * 16);
        double v;
        if constexpr (kPrefC) {
          v = cn[u];
        } else {
          const int c = cb + k;
          v = (c < hi && j < ncol) ? Cm[(size_t)c * cld + j] : 0.0;
        }
        const unsigned short h0 = bf16_bits_rn((float)v);
        const double v1 = v - (double)bf16_to_float(h0);
        const unsigned short h1 = bf16_bits_rn((float)v1);
        const unsigned short h2 = bf16_bits_rn((float)(v1 - (double)bf16_to_float(h1)));
        scb[0][j][k] = h0;
        scb[1][j][k] = h1;
        scb[2][j][k] = h2;
      }
#pragma unroll
      for (int u = 0; u < RT_RT; ++u)
#pragma unroll
        for (int i = 0; i < 8; ++i) sv[u][i] = sn[u][i];
      __syncthreads();
      if (cb + RB_K < hi) {
        load_s(cb + RB_K, sn);
        if constexpr (kPrefC) load_c(cb + RB_K);
      }
      bf16x8 b0[RT_RT], b1[RT_RT], b2[RT_RT];
#pragma unroll
      for (int u = 0; u < RT_RT; ++u) {
        us8v p0, p1, p2;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float x = sv[u][i];
          const unsigned short h0 = bf16_bits_rn(x);
          const float x1 = x - bf16_to_float(h0);
          const unsigned short h1 = bf16_bits_rn(x1);
          p0[i] = h0;
          p1[i] = h1;
          p2[i] = bf16_bits_rn(x1 - bf16_to_float(h1));
        }
        b0[u] = __builtin_bit_cast(bf16x8, p0);
        b1[u] = __builtin_bit_cast(bf16x8, p1);
        b2[u] = __builtin_bit_cast(bf16x8, p2);
      }
#pragma unroll
      for (int t = 0; t < NCT; ++t) {
        if (t >= nct) continue;
        const int j = t * 16 + (lane & 15);
        const bf16x8 a0 = *reinterpret_cast<const bf16x8*>(&scb[0][j][8 * kl]);
        const bf16x8 a1 = *reinterpret_cast<const bf16x8*>(&scb[1][j][8 * kl]);
        const bf16x8 a2 = *reinterpret_cast<const bf16x8*>(&scb[2][j][8 * kl]);
#pragma unroll
        for (int u = 0; u < RT_RT; ++u) {
          f4v s = acc[u][t];
          s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a2, b0[u], s, 0, 0, 0);
          s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, b1[u], s, 0, 0, 0);
          s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b2[u], s, 0, 0, 0);
          s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, b0[u], s, 0, 0, 0);
          s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b1[u], s, 0, 0, 0);
          acc[u][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b0[u], s, 0, 0, 0);
        }
      }
    }
    // store the output this segment completes: lane holds out[row rrow[u]][col 16 t + 4 kl + q]
    const int o = (A.nout > 1 && sg == 0) ? 1 : 0;
    float* out = reinterpret_cast<float*>(E.blk[A.out_blk[o]]);
#pragma unroll
    for (int t = 0; t < NCT; ++t) {
      if (t >= nct) continue;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = t * 16 + 4 * kl + q;
        if (j >= ncol) continue;
#pragma unroll
        for (int u = 0; u < RT_RT; ++u) {
          if (rrow[u] >= nrows) continue;
          float* p = out + (size_t)j * E.ld + rrow[u];
          const double prev = A.beta[o] != 0.0 ? A.beta[o] * (double)*p : 0.0;
          *p = (float)(prev + A.alpha * (double)acc[u][t][q]);
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// residual norms and preconditioner energies
// res_i = ||hx_i - theta_i x_i||,  ekin_i = max(theta_i - x_i^T V x_i, 0.05)
// ---------------------------------------------------------------------------
struct ResArgs {
  const ElemDev* elems;
  const int* active;
  int x_blk, hx_blk;
  int ncol;
  int kp;              // small storage order (kmax3 + 2)
};

// one workgroup of RES_THREADS per column; each thread keeps four rows in flight
constexpr int RES_THREADS = 1024;

template <typename T>
__global__ void __launch_bounds__(RES_THREADS) k_residual(ResArgs A) {
  const int e = blockIdx.y;
  const ElemDev& E = A.elems[e];
  const int i = blockIdx.x;
  const int ncol = kcode(A.ncol, E);
  if (i >= ncol) return;
  if (A.active && !A.active[e]) return;
  const int KP = E.kmax3 + 2;
  double* vec = E.small + SmallLayout::vec(KP);
  const double th = vec[VS_THETA * KP + i];
  const T* x = reinterpret_cast<const T*>(E.blk[A.x_blk]) + (size_t)i * E.ld;
  const T* hx = reinterpret_cast<const T*>(E.blk[A.hx_blk]) + (size_t)i * E.ld;
  double s1[4] = {0.0, 0.0, 0.0, 0.0}, s2[4] = {0.0, 0.0, 0.0, 0.0};
  for (int r0 = threadIdx.x; r0 < E.N; r0 += 4 * RES_THREADS) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = r0 + u * RES_THREADS;
      if (r < E.N) {
        const double xv = double(x[r]);
        const double rv = double(hx[r]) - th * xv;
        s1[u] += rv * rv;
        s2[u] += E.v64[r] * xv * xv;
      }
    }
  }
  __shared__ double sh[16];
  const double t1 = block_sum((s1[0] + s1[1]) + (s1[2] + s1[3]), sh);
  const double t2 = block_sum((s2[0] + s2[1]) + (s2[2] + s2[3]), sh);
  if (threadIdx.x == 0) {
    vec[VS_RES * KP + i] = sqrt(t1);
    vec[VS_EKIN * KP + i] = fmax(th - t2, 0.05);
  }
}

// per element: active = max_{i<J} res_i > tol ; count of active elements; the
// Rayleigh-Ritz breakdowns (status 2) since the last check are added to count[2]
// and their flags cleared
__global__ void k_check(const ElemDev* elems, int n_elem, int* active, double tol, int* count,
                        double* maxres, int* iter_count, int* status) {
  __shared__ double sh[16];
  if (threadIdx.x == 0) {
    int brk = 0;
    for (int e = 0; e < n_elem; ++e)
      if (status[e] != 0) {
        ++brk;
        status[e] = 0;
      }
    count[2] += brk;
  }
  __syncthreads();
  for (int e = 0; e < n_elem; ++e) {
    const ElemDev& E = elems[e];
    const int KP = E.kmax3 + 2;
    const double* res = E.small + SmallLayout::vec(KP) + VS_RES * KP;
    double m = 0.0;
    int bad = 0;
    for (int i = threadIdx.x; i < E.J; i += blockDim.x) {
      const double r = res[i];
      bad |= !(r == r);          // fmax drops NaN: flag it separately
      m = fmax(m, r);
    }
    m = block_max(m, sh);
    if (__syncthreads_or(bad)) m = __builtin_nan("");
    if (threadIdx.x == 0) {
      if (active[e] && !(m <= tol)) {
      } else {
        active[e] = 0;
      }
      if (!(m == m)) active[e] = -1;   // NaN
      maxres[e] = m;
      if (iter_count && active[e] > 0) ++iter_count[e];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    int c = 0, nan = 0;
    for (int e = 0; e < n_elem; ++e) {
      c += active[e] > 0;
      nan += active[e] < 0;
    }
    count[0] = c;
    count[1] = nan;
  }
}

// ---------------------------------------------------------------------------
// copies between caller buffers (packed) and blocks
// mode 0: packed <-> block (all N rows)      mode 1: block E_k rows -> packed
// mode 2: block E_k rows -> block rows 0..|E_k|-1
// ---------------------------------------------------------------------------
struct CopyArgs {
  const ElemDev* elems;
  int blk, blk2;
  void* ptr;                  // packed caller buffer (FP64 or FP32 as prec)
  const long long* off;       // per element offsets into ptr (elements), or nullptr
  long long off_mult;         // multiplier applied to off[e]
  int elem_only;              // >= 0: this element only, ptr offset 0
  int ncol;                   // column code
  int to_packed;              // 1: block -> ptr
  int mode;
  long long ld;               // mode 0: > 0 caller leading dimension (element blocks ld * ncol apart)
};

template <typename T>
__global__ void __launch_bounds__(256) k_copy(CopyArgs A) {
  const int e = A.elem_only >= 0 ? A.elem_only : blockIdx.z;
  const ElemDev& E = A.elems[e];
  const int ncol = kcode(A.ncol, E);
  const int j = blockIdx.y;
  if (j >= ncol) return;
  const int ne = E.en[0] * E.en[1] * E.en[2];
  const int nrows = A.mode == 0 ? E.N : ne;
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= nrows) return;
  int gr = r;
  if (A.mode != 0) {
    const int x = r % E.en[0], y = (r / E.en[0]) % E.en[1], z = r / (E.en[0] * E.en[1]);
    gr = (x + E.elo[0]) + E.nx * ((y + E.elo[1]) + E.ny * (z + E.elo[2]));
  }
  T* b = reinterpret_cast<T*>(E.blk[A.blk]) + (size_t)j * E.ld;
  if (A.mode == 2) {
    T* d = reinterpret_cast<T*>(E.blk[A.blk2]) + (size_t)j * E.ld;
    d[r] = b[gr];
    return;
  }
  long long base, cstride = nrows;
  if (A.ld > 0) {
    base = A.elem_only >= 0 ? 0 : (long long)e * A.ld * ncol;
    cstride = A.ld;
  } else {
    base = (A.elem_only >= 0 || !A.off) ? 0 : A.off[e] * A.off_mult;
  }
  T* p = reinterpret_cast<T*>(A.ptr) + base + (size_t)j * cstride + r;
  if (A.to_packed) *p = b[gr];
  else b[gr] = *p;
}

// packed FP64 source (x0) into a block of either precision
template <typename T>
__global__ void __launch_bounds__(256) k_copy_in64(const ElemDev* elems, int blk, const double* src,
                                                    const long long* off, int ncol_code) {
  const int e = blockIdx.z;
  const ElemDev& E = elems[e];
  const int ncol = kcode(ncol_code, E);
  const int j = blockIdx.y;
  if (j >= ncol) return;
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= E.N) return;
  reinterpret_cast<T*>(E.blk[blk])[(size_t)j * E.ld + r] = T(src[off[e] + (size_t)j * E.N + r]);
}

// convert a block between precisions (separate blocks)
__global__ void __launch_bounds__(256) k_convert(const ElemDev* elems, int src_blk, int src_prec,
                                                  int dst_blk, int dst_prec, int ncol_code) {
  const int e = blockIdx.z;
  const ElemDev& E = elems[e];
  const int ncol = kcode(ncol_code, E);
  const int j = blockIdx.y;
  if (j >= ncol) return;
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= E.N) return;
  const size_t o = (size_t)j * E.ld + r;
  double v = src_prec == DG_FP64 ? reinterpret_cast<const double*>(E.blk[src_blk])[o]
                                 : double(reinterpret_cast<const float*>(E.blk[src_blk])[o]);
  if (dst_prec == DG_FP64) reinterpret_cast<double*>(E.blk[dst_blk])[o] = v;
  else reinterpret_cast<float*>(E.blk[dst_blk])[o] = float(v);
}

// Mixed refinement, per active element and column j < K: the residual
// r_j = hx_j - theta_j x_j, formed in FP64 and stored in FP32 (its rounding is relative
// to r, not to hx), and x_j rounded to FP32.
__global__ void __launch_bounds__(256) k_mixed_split(const ElemDev* elems, const int* active, int x_blk,
                                                     int hx_blk, int r_blk, int x32_blk) {
  const int e = blockIdx.z;
  const ElemDev& E = elems[e];
  if (active && !active[e]) return;
  const int j = blockIdx.y;
  if (j >= E.K) return;
  const int KP = E.kmax3 + 2;
  const double th = E.small[SmallLayout::vec(KP) + VS_THETA * KP + j];
  const double* X = reinterpret_cast<const double*>(E.blk[x_blk]) + (size_t)j * E.ld;
  const double* HX = reinterpret_cast<const double*>(E.blk[hx_blk]) + (size_t)j * E.ld;
  float* R = reinterpret_cast<float*>(E.blk[r_blk]) + (size_t)j * E.ld;
  float* X32 = reinterpret_cast<float*>(E.blk[x32_blk]) + (size_t)j * E.ld;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int r = blockIdx.x * 1024 + u * 256 + threadIdx.x;
    if (r >= E.N) break;
    const double x = X[r];
    R[r] = (float)(HX[r] - th * x);
    X32[r] = (float)x;
  }
}

// Mixed refinement: the projected matrices of [X W P] (G: overlap, A: H) from the FP32
// Grams of S' = [W P X32] (Gs = S'^T S') and T' = [HW HP R] (As = S'^T T', upper blocks):
//   G_XX = I and A_XX = Theta (X holds Ritz vectors),
//   G_QX = Gs_QX and A_QX = Q^T R + G_QX Theta for Q = W, P,
//   G_QQ', A_QQ' = Gs, As,
// both symmetric.  A_QX - theta_j G_QX e_j = Q^T r_j holds whatever the rounding of
// G_QX, so the FP32 Grams perturb the correction only in second order.
__global__ void __launch_bounds__(256) k_mixed_fix(const ElemDev* elems, const int* active, int nb) {
  const int e = blockIdx.x;
  const ElemDev& E = elems[e];
  if (active && !active[e]) return;
  const int K = E.K, n = nb * K;
  const int KP = E.kmax3 + 2;
  const double* Gs = E.small + SmallLayout::V(KP);
  const double* As = E.small + SmallLayout::U(KP);
  double* G = E.small + SmallLayout::G(KP);
  double* Am = E.small + SmallLayout::A(KP);
  const double* th = E.small + SmallLayout::vec(KP) + VS_THETA * KP;
  for (int idx = threadIdx.x; idx < n * n; idx += blockDim.x) {
    const int i = idx / n, j = idx % n;
    const int bi = i / K, bj = j / K;
    // [X W P] index -> [W P X] index
    const int oi = (bi == 0 ? nb - 1 : bi - 1) * K + (i - bi * K);
    const int oj = (bj == 0 ? nb - 1 : bj - 1) * K + (j - bj * K);
    double g, a;
    if (bi == 0 && bj == 0) {
      g = i == j ? 1.0 : 0.0;
      a = i == j ? th[i] : 0.0;
    } else if (bi == 0 || bj == 0) {
      // one index in X: read the (Q row, X column) entries, computed directly in As
      const int q = bi == 0 ? oj : oi, x = bi == 0 ? oi : oj;
      const int xi = bi == 0 ? i : j;
      g = Gs[(size_t)q * n + x];
      a = As[(size_t)q * n + x] + g * th[xi];
    } else {
      g = Gs[(size_t)oi * n + oj];
      a = As[(size_t)oi * n + oj];
    }
    G[(size_t)i * n + j] = g;
    Am[(size_t)i * n + j] = a;
  }
}

// Seeded Gaussian start: value (row r, column j) of element g = e + elem_base is a
// Box-Muller normal from two SplitMix64 outputs of the counter (seed, g, j, r), so
// the block does not depend on how the batch is split into element groups.
__device__ __forceinline__ unsigned long long splitmix64(unsigned long long x) {
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}

template <typename T>
__global__ void __launch_bounds__(256) k_random_block(const ElemDev* elems, int blk, unsigned long long seed,
                                                       int elem_base) {
  const int e = blockIdx.z;
  const ElemDev& E = elems[e];
  const int j = blockIdx.y;
  if (j >= E.K) return;
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= E.N) return;
  const unsigned long long key =
      splitmix64(seed ^ splitmix64(((unsigned long long)(e + elem_base) << 32) | (unsigned)j)) ^ (unsigned long long)r;
  const unsigned long long h1 = splitmix64(2 * key), h2 = splitmix64(2 * key + 1);
  // u1 in (0, 1], u2 in [0, 1)
  const double u1 = ((double)(h1 >> 11) + 1.0) * (1.0 / 9007199254740992.0);
  const double u2 = (double)(h2 >> 11) * (1.0 / 9007199254740992.0);
  const double v = sqrt(-2.0 * log(u1)) * cospi(2.0 * u2);
  reinterpret_cast<T*>(E.blk[blk])[(size_t)j * E.ld + r] = T(v);
}

// J (all = 0) or J + g (all = 1) values per element from the small-vector slots
// into packed outputs
__global__ void k_extract(const ElemDev* elems, const long long* off, int slot0, double* out0,
                          int slot1, double* out1, int all) {
  const int e = blockIdx.x;
  const ElemDev& E = elems[e];
  const int KP = E.kmax3 + 2;
  const double* vec = E.small + SmallLayout::vec(KP);
  const int n = all ? E.K : E.J;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    if (out0) out0[off[e] + i] = vec[slot0 * KP + i];
    if (out1) out1[off[e] + i] = vec[slot1 * KP + i];
  }
}

// first |E_k| rows of a block -> packed |E_k| x J output
__global__ void __launch_bounds__(256) k_copy_rows(const ElemDev* elems, int blk, double* out,
                                                    const long long* off) {
  const int e = blockIdx.z;
  const ElemDev& E = elems[e];
  const int j = blockIdx.y;
  if (j >= E.J) return;
  const int ne = E.en[0] * E.en[1] * E.en[2];
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= ne) return;
  out[off[e] + (size_t)j * ne + r] = reinterpret_cast<const double*>(E.blk[blk])[(size_t)j * E.ld + r];
}

// Block roles move with each element: after a rotation the logical blocks of
// every active element are re-pointed (new[i] = old[perm[i]]); converged
// elements keep theirs.
struct Perm8 {
  int p[kMaxBlocks];
};

__global__ void k_permute_blocks(ElemDev* elems, int n_elem, const int* active, Perm8 perm) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n_elem) return;
  if (active && active[e] <= 0) return;
  void* old[kMaxBlocks];
  for (int i = 0; i < kMaxBlocks; ++i) old[i] = elems[e].blk[i];
  for (int i = 0; i < kMaxBlocks; ++i) elems[e].blk[i] = old[perm.p[i]];
}

int launch_permute(Ctx& c, const int* perm, const int* active) {
  Perm8 p;
  for (int i = 0; i < kMaxBlocks; ++i) p.p[i] = perm[i];
  hipLaunchKernelGGL(k_permute_blocks, dim3((c.n_elem + 63) / 64), dim3(64), 0, c.stream, c.elems_dev,
                     c.n_elem, active, p);
  DG_HIP(hipGetLastError());
  return DG_OK;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static void max_dims(Ctx& c, int code, int* maxk, int* maxN, int* maxE) {
  *maxk = *maxN = *maxE = 0;
  for (int e = 0; e < c.n_elem; ++e) {
    const int k = code > 0 ? code : (code == 0 ? c.K[e] : c.J[e]);
    *maxk = std::max(*maxk, k);
    *maxN = std::max(*maxN, c.N[e]);
    *maxE = std::max(*maxE, c.en[0][e] * c.en[1][e] * c.en[2][e]);
  }
}

static bool set_lds_limit(const void* fn, int bytes) {
  return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
}

// Gram instantiations: blocks per wave 1..6 x staging per thread (FP64 and FP32: 16-byte
// pieces of 64 columns a pass, 1, 2, 3, 4 or 6; BF16x3: values of 16 columns, 8 or 18).
template <int MB>
static void gram_attrs() {
  set_lds_limit((const void*)k_gram<MB, 1>, GP_LDS_LIMIT);
  set_lds_limit((const void*)k_gram<MB, 2>, GP_LDS_LIMIT);
  set_lds_limit((const void*)k_gram<MB, 3>, GP_LDS_LIMIT);
  set_lds_limit((const void*)k_gram<MB, 4>, GP_LDS_LIMIT);
  set_lds_limit((const void*)k_gram<MB, 6>, GP_LDS_LIMIT);
  set_lds_limit((const void*)k_gram_bf16<MB, 8>, 96000);
  set_lds_limit((const void*)k_gram_bf16<MB, 18>, 96000);
  set_lds_limit((const void*)k_gram32<MB, 1>, GP_LDS_LIMIT);
  set_lds_limit((const void*)k_gram32<MB, 2>, GP_LDS_LIMIT);
  set_lds_limit((const void*)k_gram32<MB, 3>, GP_LDS_LIMIT);
  set_lds_limit((const void*)k_gram32<MB, 4>, GP_LDS_LIMIT);
  set_lds_limit((const void*)k_gram32<MB, 6>, GP_LDS_LIMIT);
}

template <int MB>
static void launch_gram_mb(int prec, int pf, dim3 g, size_t lds, hipStream_t s, const GramArgs& ga, bool bf16) {
  if (prec != DG_FP64 && !bf16) {
    switch (pf) {
      case 1: hipLaunchKernelGGL((k_gram32<MB, 1>), g, dim3(GP_THREADS), lds, s, ga); break;
      case 2: hipLaunchKernelGGL((k_gram32<MB, 2>), g, dim3(GP_THREADS), lds, s, ga); break;
      case 3: hipLaunchKernelGGL((k_gram32<MB, 3>), g, dim3(GP_THREADS), lds, s, ga); break;
      case 4: hipLaunchKernelGGL((k_gram32<MB, 4>), g, dim3(GP_THREADS), lds, s, ga); break;
      default: hipLaunchKernelGGL((k_gram32<MB, 6>), g, dim3(GP_THREADS), lds, s, ga);
    }
    return;
  }
  if (prec == DG_FP64) {
    switch (pf) {
      case 1: hipLaunchKernelGGL((k_gram<MB, 1>), g, dim3(GP_THREADS), lds, s, ga); break;
      case 2: hipLaunchKernelGGL((k_gram<MB, 2>), g, dim3(GP_THREADS), lds, s, ga); break;
      case 3: hipLaunchKernelGGL((k_gram<MB, 3>), g, dim3(GP_THREADS), lds, s, ga); break;
      case 4: hipLaunchKernelGGL((k_gram<MB, 4>), g, dim3(GP_THREADS), lds, s, ga); break;
      default: hipLaunchKernelGGL((k_gram<MB, 6>), g, dim3(GP_THREADS), lds, s, ga);
    }
  } else {
    if (pf <= 8) hipLaunchKernelGGL((k_gram_bf16<MB, 8>), g, dim3(GP_THREADS), lds, s, ga);
    else hipLaunchKernelGGL((k_gram_bf16<MB, 18>), g, dim3(GP_THREADS), lds, s, ga);
  }
}

// dynamic-LDS limits of every kernel variant, set once before any launch (and so
// never from inside a stream capture)
void init_kernel_attributes() {
  static const bool done = [] {
    gram_attrs<1>();
    gram_attrs<2>();
    gram_attrs<3>();
    gram_attrs<4>();
    gram_attrs<5>();
    gram_attrs<6>();
    return true;
  }();
  (void)done;
}

// pair: also S^T S (to out_off_ss) from the same staging of [S | T]
// Tile side for a Gram launch: the tb that stages the fewest columns in total
// (over the tiles of every element shape in the launch) while each tile's blocks
// fit 8 waves x max_blocks and its staged columns max_cols.
struct GramPlan {
  int tb = 1, maxblk = 0, maxnc = 0, ntiles = 0;
};

// blocks per wave of a plan's largest tile: the instantiation to launch.  No element of the
// launch has more: the plan goes over every number of block rows there is, with the most
// block columns (fewer make no tile larger).
static int gram_blocks_per_wave(const GramPlan& pl) { return (pl.maxblk + 7) / 8; }

// dynamic LDS of a Gram launch: two panels (FP64, FP32), or three BF16 planes and the
// column pointers
static size_t gram_lds_bytes(const GramPlan& pl, bool fp64, bool bf16) {
  return fp64    ? (size_t)2 * GP_RP * pl.maxnc * sizeof(double)
         : !bf16 ? (size_t)2 * G3_RP * pl.maxnc * sizeof(float)
                 : (size_t)3 * pl.maxnc * GB_PITCH * 2 + (size_t)pl.maxnc * sizeof(void*);
}

static GramPlan plan_gram_tiles(const std::vector<int>& bis, int bj_max, int sym, int same, int pair,
                                int max_blocks, int max_cols) {
  int bi_max = 0;
  for (int b : bis) bi_max = std::max(bi_max, b);
  GramPlan best;
  long long best_staged = -1;
  for (int tb = std::max(bi_max, bj_max); tb >= 1; --tb) {
    GramPlan pl;
    pl.tb = tb;
    long long staged = 0;
    for (int bi : bis) {
      const int bj = sym ? bi : bj_max;
      const int nt = gram_ntiles(bi, bj, tb, sym);
      if (bi == bi_max) pl.ntiles = nt;
      for (int t = 0; t < nt; ++t) {
        const GramTile g = gram_tile(t, bi, bj, tb, sym, same, pair);
        pl.maxblk = std::max(pl.maxblk, g.nloc * (pair ? 2 : 1));
        pl.maxnc = std::max(pl.maxnc, g.ncA + g.ncB + g.ncC);
        if (bi == bi_max) staged += g.ncA + g.ncB + g.ncC;
      }
    }
    if (pl.maxblk > 8 * max_blocks || pl.maxnc > max_cols) continue;
    if (best_staged < 0 || staged < best_staged) {
      best = pl;
      best_staged = staged;
    }
  }
  return best;
}

static int gram_impl(Ctx& c, int prec, const ColSet& S, int kS, const ColSet& T, int kT,
                     long long out_off, const int* active, int rows_e, int sym, bool pair = false,
                     long long out_off_ss = 0) {
  int ks, kt, maxN, maxE;
  max_dims(c, kS, &ks, &maxN, &maxE);
  max_dims(c, kT, &kt, &maxN, &maxE);
  const int maxni = S.nb * ks, maxnj = T.nb * kt;
  const int rows = rows_e ? maxE : maxN;
  const bool same = S.nb == T.nb && kS == kT &&
                    std::equal(S.blk, S.blk + S.nb, T.blk);
  if (sym && maxni != maxnj) { set_error("symmetric Gram of a non-square shape"); return DG_ERR_ARG; }
  const long long part_sq = (long long)c.gram_part_ld * c.gram_part_ld;
  if (pair) {
    // both products from one staging of S (symmetric, T != S) when the partial area
    // holds both sets of partial sums; else two separate Grams
    const bool fits = sym && !same && c.gram_part_stride >= 2 * part_sq;
    if (!fits) {
      if (int st = gram_impl(c, prec, S, kS, S, kS, out_off_ss, active, rows_e, sym)) return st;
      return gram_impl(c, prec, S, kS, T, kT, out_off, active, rows_e, sym);
    }
  }
  // block-row counts of the element shapes in this launch
  std::vector<int> bis;
  for (int e = 0; e < c.n_elem; ++e) {
    const int ke = kS > 0 ? kS : (kS == 0 ? c.K[e] : c.J[e]);
    const int b = (S.nb * ke + 15) / 16;
    if (std::find(bis.begin(), bis.end(), b) == bis.end()) bis.push_back(b);
  }
  const int bj_max = (maxnj + 15) / 16;
  // FP64 and FP32 (FP32 matrix cores): at most 6 blocks per wave and 384 staged columns;
  // BF16x3 (DG_BF16=1): 6 blocks and 128 columns
  const bool bf16 = prec != DG_FP64 && c.bf16;
  const int cap_blocks = 6;
  const int cap_cols = prec == DG_FP64 ? GP_MAXCOL : (bf16 ? 128 : G3_MAXCOL);
  if (prec != DG_FP64 && !bf16)   // k_gram32 takes whole panels: every supported grid has some
    for (int e = 0; e < c.n_elem; ++e)
      if (rows_e || c.N[e] % G3_R != 0) {
        set_error("FP32 Gram of a number of rows that is no multiple of " + std::to_string(G3_R));
        return DG_ERR_SHAPE;
      }
  const GramPlan pl = plan_gram_tiles(bis, bj_max, sym, same ? 1 : 0, pair ? 1 : 0, cap_blocks, cap_cols);
  if (pl.maxblk == 0) {
    set_error("Gram: no tile fits the per-workgroup limits");
    return DG_ERR_SHAPE;
  }
  const int maxb = gram_blocks_per_wave(pl);   // at most cap_blocks
  // staged per thread: FP64 and FP32 a 16-byte piece of 64 columns per pass; BF16 a value of 16
  const int pf = bf16 ? (pl.maxnc + 15) / 16 : (pl.maxnc + 63) / 64;
  const int groups = pl.ntiles;
  // row-range split: row ranges of about 8192 rows of the largest element, and at least
  // 2048 workgroups over the launch (long single ranges leave the launch to a tail of
  // the largest elements), at least 256 rows each (the pair keeps two sets of partials);
  // with DG_TUNE=1 half or twice that where it is timed faster
  const int split_cap = std::max(1, std::min(pair ? (int)(c.gram_part_stride / (2 * part_sq)) : c.gram_max_split,
                                             rows / 256));
  int nsplit = std::max((rows + 8191) / 8192, (2048 + groups * c.n_elem - 1) / (groups * c.n_elem));
  nsplit = std::max(1, std::min(split_cap, nsplit));
  const long long key =
      ((((((long long)prec * 1024 + maxni) * 1024 + maxnj) * 2 + sym) * 2 + (same ? 1 : 0)) * 2 + rows_e) * 2 +
      (pair ? 1 : 0);
  auto tuned = c.gram_split_table.find(key);
  if (tuned != c.gram_split_table.end()) nsplit = tuned->second;
  GramArgs ga{c.elems_dev, active, S, T, kS, kT, nsplit, rows_e, sym, same ? 1 : 0, pl.tb, pl.ntiles,
              c.n_elem, c.gram_part, c.gram_part_stride, c.gram_part_ld, pair ? 1 : 0, 0};
  // algorithmic flops: 2 r n_i n_j per product, n (n + 1) r for a symmetric n x n result
  double flops = 0.0;
  for (int e = 0; e < c.n_elem; ++e) {
    if (active && !c.active_host.empty() && !c.active_host[e]) continue;
    const int ke = kS > 0 ? kS : (kS == 0 ? c.K[e] : c.J[e]);
    const int kt = kT > 0 ? kT : (kT == 0 ? c.K[e] : c.J[e]);
    const double r = rows_e ? (double)c.en[0][e] * c.en[1][e] * c.en[2][e] : (double)c.N[e];
    const double ni = S.nb * ke, nj = T.nb * kt;
    flops += (sym ? r * ni * (ni + 1.0) : 2.0 * r * ni * nj) * (pair ? 2.0 : 1.0);
  }
  const size_t lds = gram_lds_bytes(pl, prec == DG_FP64, bf16);
  auto launch = [&](int ns) -> int {
    ga.nsplit = ns;
    ga.part_pair = ns * part_sq;
    // 1D grid: tiles x row ranges (split, element), the row ranges padded to a multiple of 8
    const long long n_rr8 = ((long long)ns * c.n_elem + 7) / 8 * 8;
    dim3 g1((unsigned)(groups * n_rr8));
    switch (maxb) {
      case 1: launch_gram_mb<1>(prec, pf, g1, lds, c.stream, ga, bf16); break;
      case 2: launch_gram_mb<2>(prec, pf, g1, lds, c.stream, ga, bf16); break;
      case 3: launch_gram_mb<3>(prec, pf, g1, lds, c.stream, ga, bf16); break;
      case 4: launch_gram_mb<4>(prec, pf, g1, lds, c.stream, ga, bf16); break;
      case 5: launch_gram_mb<5>(prec, pf, g1, lds, c.stream, ga, bf16); break;
      case 6: launch_gram_mb<6>(prec, pf, g1, lds, c.stream, ga, bf16); break;
      default:
        set_error("Gram: unsupported block count");
        return DG_ERR_SHAPE;
    }
    return DG_OK;
  };
  if (tuned == c.gram_split_table.end() && c.autotune && !c.capturing) {
    // DG_TUNE=1: time the candidate splits on this launch's data, in turn in three rounds,
    // and keep the heuristic split unless another is at least 30 % faster in each of them.
    // Not by default: the split decides how the row sums are grouped, so a choice made by
    // timing changes the last bits from one context to the next (other element groups share
    // the GPU meanwhile; with 3 %, and with 10 % in each round, fresh contexts of twelve
    // uneven elements on three streams now and then chose differently), and over 71 shapes
    // of 24 batches no candidate beat the heuristic by 3 % without that noise.
    const int cand[3] = {nsplit, std::max(1, nsplit / 2), std::min(split_cap, nsplit * 2)};
    float best = 1e30f, worst_ratio[3] = {0.f, 0.f, 0.f}, ms_min[3] = {1e30f, 1e30f, 1e30f};
    int best_ns = nsplit;
    struct Events {   // destroyed on every return path
      hipEvent_t e[2] = {nullptr, nullptr};
      ~Events() {
        for (hipEvent_t x : e)
          if (x) (void)hipEventDestroy(x);
      }
    } evs;
    hipEvent_t* ev = evs.e;
    DG_HIP(hipEventCreate(&ev[0]));
    DG_HIP(hipEventCreate(&ev[1]));
    for (int round = 0; round < 3; ++round) {
      float base = 0.f;
      for (int ci = 0; ci < 3; ++ci) {
        if (ci > 0 && cand[ci] == nsplit) continue;
        DG_HIP(hipEventRecord(ev[0], c.stream));
        if (int st = launch(cand[ci])) return st;
        DG_HIP(hipEventRecord(ev[1], c.stream));
        DG_HIP(hipEventSynchronize(ev[1]));
        float ms = 0.f;
        DG_HIP(hipEventElapsedTime(&ms, ev[0], ev[1]));
        if (ci == 0) base = ms;
        ms_min[ci] = std::min(ms_min[ci], ms);
        worst_ratio[ci] = std::max(worst_ratio[ci], ms / std::max(base, 1e-6f));
      }
    }
    best = ms_min[0];
    for (int ci = 1; ci < 3; ++ci)
      if (cand[ci] != nsplit && worst_ratio[ci] < 0.7f && ms_min[ci] < best) {
        best = ms_min[ci];
        best_ns = cand[ci];
      }
    c.gram_split_table[key] = best_ns;
    nsplit = best_ns;
    if (c.log_level > 0)
      fprintf(stderr, "[dg] gram autotune %dx%d sym=%d prec=%d pair=%d tile=%d (%d tiles, %d blocks/wg): split %d "
              "(%.3f ms)\n", maxni, maxnj, sym, prec, pair ? 1 : 0, pl.tb, groups, pl.maxblk, best_ns, best);
  }
  TimedScope ts(c, TC_GRAM, flops);
  if (int st = launch(nsplit)) return st;
  GramReduceArgs ra{c.elems_dev, active, sym, S.nb, T.nb, kS, kT, nsplit, c.gram_part,
                    c.gram_part_stride, c.gram_part_ld, out_off, 0};
  dim3 g2((maxni * maxnj + 255) / 256, c.n_elem);
  hipLaunchKernelGGL(k_gram_reduce, g2, dim3(256), 0, c.stream, ra);
  if (pair) {
    GramReduceArgs rs{c.elems_dev, active, sym, S.nb, S.nb, kS, kS, nsplit, c.gram_part + nsplit * part_sq,
                      c.gram_part_stride, c.gram_part_ld, out_off_ss, 0};
    hipLaunchKernelGGL(k_gram_reduce, g2, dim3(256), 0, c.stream, rs);
  }
  DG_HIP(hipGetLastError());
  return DG_OK;
}

int launch_gram(Ctx& c, int prec, const ColSet& S, int kS, const ColSet& T, int kT,
                long long out_off, const int* active, int sym) {
  return gram_impl(c, prec, S, kS, T, kT, out_off, active, 0, sym);
}

int launch_gram_rows(Ctx& c, int prec, const ColSet& S, int kS, const ColSet& T, int kT,
                     long long out_off, int rows_e, int sym) {
  return gram_impl(c, prec, S, kS, T, kT, out_off, nullptr, rows_e, sym);
}

int launch_gram_pair(Ctx& c, int prec, const ColSet& S, int kS, const ColSet& T, int kT, long long out_off_st,
                     long long out_off_ss, const int* active) {
  return gram_impl(c, prec, S, kS, T, kT, out_off_st, active, 0, 1, true, out_off_ss);
}

int launch_rotate(Ctx& c, int prec, const RotArgs& a_in) {
  RotArgs a = a_in;
  a.elems = c.elems_dev;
  int k, maxN, maxE;
  max_dims(c, a.ncol, &k, &maxN, &maxE);
  const int rows = a.rows_e ? maxE : maxN;
  double flops = 0.0;
  for (int e = 0; e < c.n_elem; ++e) {
    if (a.active && !c.active_host.empty() && !c.active_host[e]) continue;
    const int ks = a.kS > 0 ? a.kS : (a.kS == 0 ? c.K[e] : c.J[e]);
    const int nc = a.ncol > 0 ? a.ncol : (a.ncol == 0 ? c.K[e] : c.J[e]);
    const double r = a.rows_e ? (double)c.en[0][e] * c.en[1][e] * c.en[2][e] : (double)c.N[e];
    for (int o = 0; o < a.nout; ++o) {
      const int span = a.c_blockrows > 0 ? (a.c1[o] - a.c0[o]) * ks : (a.c1[o] - a.c0[o]);
      flops += 2.0 * r * span * nc;
    }
  }
  TimedScope ts(c, TC_ROT, flops);
  // output column tiles: 3 (up to 48 columns) or 6 (up to 96); FP32 blocks on FP32 matrix
  // cores (BF16 matrix cores with DG_BF16=1)
  const bool k3 = k <= 48;
  const dim3 g((rows + RT_ROWS - 1) / RT_ROWS, c.n_elem);
  if (prec == DG_FP64) {
    const int rr = rt_rows(k3 ? 3 : 6);
    const dim3 g64((rows + rr - 1) / rr, c.n_elem);
    if (k3) hipLaunchKernelGGL((k_rotate<3>), g64, dim3(rt_threads(3)), 0, c.stream, a);
    else hipLaunchKernelGGL((k_rotate<6>), g64, dim3(rt_threads(6)), 0, c.stream, a);
  } else if (!c.bf16) {
    if (k3) hipLaunchKernelGGL((k_rotate32<3>), g, dim3(RT_THREADS), 0, c.stream, a);
    else hipLaunchKernelGGL((k_rotate32<6>), g, dim3(RT_THREADS), 0, c.stream, a);
  } else {
    if (k3) hipLaunchKernelGGL((k_rotate_bf16<3>), g, dim3(RT_THREADS), 0, c.stream, a);
    else hipLaunchKernelGGL((k_rotate_bf16<6>), g, dim3(RT_THREADS), 0, c.stream, a);
  }
  DG_HIP(hipGetLastError());
  return DG_OK;
}

int launch_residual(Ctx& c, int prec, int x_blk, int hx_blk, int ncol, const int* active) {
  int maxk, maxN, maxE;
  max_dims(c, ncol, &maxk, &maxN, &maxE);
  ResArgs a{c.elems_dev, active, x_blk, hx_blk, ncol, 0};
  dim3 g(maxk, c.n_elem);
  TimedScope ts(c, TC_OTHER);
  if (prec == DG_FP64) hipLaunchKernelGGL(k_residual<double>, g, dim3(RES_THREADS), 0, c.stream, a);
  else hipLaunchKernelGGL(k_residual<float>, g, dim3(RES_THREADS), 0, c.stream, a);
  DG_HIP(hipGetLastError());
  return DG_OK;
}

int launch_check(Ctx& c, int* active, double tol) {
  hipLaunchKernelGGL(k_check, dim3(1), dim3(256), 0, c.stream, c.elems_dev, c.n_elem, active, tol,
                     c.dev_count, c.dev_maxres, c.dev_iters, c.dev_status);
  DG_HIP(hipGetLastError());
  return DG_OK;
}

int launch_copy_ext(Ctx& c, int prec, int blk, const void* ptr, int elem, int ncol, int to_packed,
                    long long ld) {
  int maxk, maxN, maxE;
  max_dims(c, ncol, &maxk, &maxN, &maxE);
  CopyArgs a{c.elems_dev, blk, 0, const_cast<void*>(ptr), c.dev_off_grid, ncol, elem, ncol, to_packed, 0, ld};
  dim3 g((maxN + 255) / 256, maxk, elem >= 0 ? 1 : c.n_elem);
  if (prec == DG_FP64) hipLaunchKernelGGL(k_copy<double>, g, dim3(256), 0, c.stream, a);
  else hipLaunchKernelGGL(k_copy<float>, g, dim3(256), 0, c.stream, a);
  DG_HIP(hipGetLastError());
  return DG_OK;
}

int launch_copy_packed(Ctx& c, int prec, int blk, const double* ptr, const long long* off, int ncol,
                       int to_packed) {
  int maxk, maxN, maxE;
  max_dims(c, ncol, &maxk, &maxN, &maxE);
  dim3 g((maxN + 255) / 256, maxk, c.n_elem);
  if (!to_packed) {
    if (prec == DG_FP64) hipLaunchKernelGGL(k_copy_in64<double>, g, dim3(256), 0, c.stream, c.elems_dev, blk, ptr, off, ncol);
    else hipLaunchKernelGGL(k_copy_in64<float>, g, dim3(256), 0, c.stream, c.elems_dev, blk, ptr, off, ncol);
  } else {
    CopyArgs a{c.elems_dev, blk, 0, const_cast<double*>(ptr), off, 1, -1, ncol, 1, 0, 0};
    hipLaunchKernelGGL(k_copy<double>, g, dim3(256), 0, c.stream, a);
  }
  DG_HIP(hipGetLastError());
  return DG_OK;
}

int launch_gather_e(Ctx& c, int src_blk, int dst_blk) {
  int maxk, maxN, maxE;
  max_dims(c, -1, &maxk, &maxN, &maxE);
  CopyArgs a{c.elems_dev, src_blk, dst_blk, nullptr, nullptr, 0, -1, -1, 0, 2, 0};
  dim3 g((maxE + 255) / 256, maxk, c.n_elem);
  hipLaunchKernelGGL(k_copy<double>, g, dim3(256), 0, c.stream, a);
  DG_HIP(hipGetLastError());
  return DG_OK;
}

int launch_copy_rows_out(Ctx& c, int blk, double* out) {
  // blk holds |E_k| x J in its first rows: mode 0 semantics over |E_k| rows
  int maxk, maxN, maxE;
  max_dims(c, -1, &maxk, &maxN, &maxE);
  dim3 g((maxE + 255) / 256, maxk, c.n_elem);
  hipLaunchKernelGGL(k_copy_rows, g, dim3(256), 0, c.stream, c.elems_dev, blk, out, c.dev_off_alb);
  DG_HIP(hipGetLastError());
  return DG_OK;
}

int launch_random_block(Ctx& c, int prec, int blk, unsigned long long seed) {
  int maxk, maxN, maxE;
  max_dims(c, 0, &maxk, &maxN, &maxE);
  dim3 g((maxN + 255) / 256, maxk, c.n_elem);
  if (prec == DG_FP64)
    hipLaunchKernelGGL(k_random_block<double>, g, dim3(256), 0, c.stream, c.elems_dev, blk, seed, c.elem_base);
  else
    hipLaunchKernelGGL(k_random_block<float>, g, dim3(256), 0, c.stream, c.elems_dev, blk, seed, c.elem_base);
  DG_HIP(hipGetLastError());
  return DG_OK;
}

int launch_mixed_split(Ctx& c, int x_blk, int hx_blk, int r_blk, int x32_blk, const int* active) {
  int maxk, maxN, maxE;
  max_dims(c, 0, &maxk, &maxN, &maxE);
  dim3 g((maxN + 1023) / 1024, maxk, c.n_elem);
  TimedScope ts(c, TC_OTHER);
  hipLaunchKernelGGL(k_mixed_split, g, dim3(256), 0, c.stream, c.elems_dev, active, x_blk, hx_blk, r_blk, x32_blk);
  DG_HIP(hipGetLastError());
  return DG_OK;
}

int launch_mixed_fix(Ctx& c, int nb, const int* active) {
  TimedScope ts(c, TC_OTHER);
  hipLaunchKernelGGL(k_mixed_fix, dim3(c.n_elem), dim3(256), 0, c.stream, c.elems_dev, active, nb);
  DG_HIP(hipGetLastError());
  return DG_OK;
}

int launch_convert(Ctx& c, int src_blk, int src_prec, int dst_blk, int dst_prec, int ncol) {
  int maxk, maxN, maxE;
  max_dims(c, ncol, &maxk, &maxN, &maxE);
  dim3 g((maxN + 255) / 256, maxk, c.n_elem);
  hipLaunchKernelGGL(k_convert, g, dim3(256), 0, c.stream, c.elems_dev, src_blk, src_prec, dst_blk,
                     dst_prec, ncol);
  DG_HIP(hipGetLastError());
  return DG_OK;
}

int launch_extract_eig(Ctx& c, double* eig, double* resid) {
  hipLaunchKernelGGL(k_extract, dim3(c.n_elem), dim3(128), 0, c.stream, c.elems_dev, c.dev_off_eig,
                     (int)VS_THETA, eig, (int)VS_RES, resid, 0);
  DG_HIP(hipGetLastError());
  return DG_OK;
}

int launch_extract_kall(Ctx& c, double* theta, double* resid) {
  hipLaunchKernelGGL(k_extract, dim3(c.n_elem), dim3(128), 0, c.stream, c.elems_dev, c.dev_off_kall,
                     (int)VS_THETA, theta, (int)VS_RES, resid, 1);
  DG_HIP(hipGetLastError());
  return DG_OK;
}

int launch_extract_theta(Ctx& c, double* out) {
  hipLaunchKernelGGL(k_extract, dim3(c.n_elem), dim3(128), 0, c.stream, c.elems_dev, c.dev_off_eig,
                     (int)VS_THETA, out, (int)VS_THETA, (double*)nullptr, 0);
  DG_HIP(hipGetLastError());
  return DG_OK;
}

}  // namespace dg
