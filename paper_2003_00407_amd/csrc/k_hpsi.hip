// H*psi on gfx950: kinetic term by line FFTs, local potential, nonlocal projectors;
// and the Teter preconditioner by a 3D FFT built from the same line FFTs.
//
// Eq. (1): H = -1/2 Laplacian + V_eff + sum gamma |b><b|, plane waves on Q_k.
// The kinetic symbol |G|^2/2 = gx(kx) + gy(ky) + gz(kz) separates, so
//   T x = Tx x + Ty x + Tz x,  T_axis = F_axis^{-1} diag(g_axis) F_axis,
// exactly (up to rounding) the 3D FFT definition.  Two passes over HBM:
//   pass 1 (per z-plane, LDS):   y1 = Tx x + Ty x + V x
//   pass 2 (per z-column, regs): y  = y1 + Tz x
// then the projector term y += B diag(gamma) B^T x (overlap before, apply after).
//
// The Teter preconditioner (Eq. (3)) multiplies the full 3D spectrum by a
// non-separable K(|G|^2 / 2E); it uses three passes: 2D forward per plane,
// z forward * K * z inverse per column, 2D inverse per plane, in place in W.
//
// Real vectors are processed in pairs (columns 2p, 2p+1) packed as one complex
// line; an odd last column pairs with zero.
#include "dense_ops.h"
#include "fft_line.h"

#include <algorithm>
#include <type_traits>

namespace dg {

template <typename T>
__device__ __forceinline__ const T* vptr(const ElemDev& E);
template <>
__device__ __forceinline__ const double* vptr<double>(const ElemDev& E) { return E.v64; }
template <>
__device__ __forceinline__ const float* vptr<float>(const ElemDev& E) { return E.v32; }

__device__ __forceinline__ int signed_freq(int k, int n) { return (2 * k < n) ? k : k - n; }
// column-count code of the H*psi-family kernels for "the element's J" (<= 0 otherwise: K)
constexpr int kNcolsJ = -2;

// frequency of a first derivative: the Nyquist mode's odd derivative vanishes on the grid
__device__ __forceinline__ int deriv_freq(int k, int n) { return (2 * k == n) ? 0 : signed_freq(k, n); }

// 1/q from the hardware reciprocal (FP64: two Newton steps, a few ulps; FP32: one ulp)
__device__ __forceinline__ double fast_recip(double q) {
  double r = __builtin_amdgcn_rcp(q);
  double t = fma(-q, r, 1.0);
  r = fma(r, t, r);
  t = fma(-q, r, 1.0);
  return fma(r, t, r);
}
__device__ __forceinline__ float fast_recip(float q) { return __builtin_amdgcn_rcpf(q); }

// HPSI: y = (T_x + T_y + V) x; TFWD/TINV: Teter passes; DX/DY: y = d/dx x, d/dy x
enum PlaneMode { PM_HPSI = 0, PM_TFWD = 1, PM_TINV = 2, PM_DX = 3, PM_DY = 4 };

struct PlaneArgs {
  const ElemDev* elems;
  const int* elem_list;   // shape class members
  const int* active;      // per element flag (nullptr = all)
  int in_blk, out_blk, aux_blk;   // HPSI: x -> y ; TFWD: x=X, aux=HX, out=W ; TINV: out=W (in place)
  int ncols;              // columns per element (<= 0: E.K)
  const double* theta_base;  // TFWD: per-element theta at small + vec(VS_THETA)
  int k3;                 // small-layout K3 (for theta lookup)
  ExtBufs ext;            // caller buffers for block ids kExtX / kExtY
  int r_given = 0;        // TFWD: aux already holds r = HX - X theta (in_blk is not read)
};

// Columns 2p and 2p+1 of a block.  Where the second is absent, b repeats a: it is loaded
// without a branch, taken as zero and not stored.  Loads and stores go through the global
// address space: the pointers come from memory, and flat accesses also count as LDS
// accesses, so that LDS waits wait for them.
template <typename T>
struct PairCols {
  T* a;
  T* b;
  bool two;
  __device__ __forceinline__ cplx<T> load(size_t o) const {
    const T re = gload<T>(a + o), im = gload<T>(b + o);
    return {re, two ? im : T(0)};
  }
  // v[i] to at(i), i < N: one branch for the second column
  template <int N, typename F>
  __device__ __forceinline__ void store(const cplx<T> (&v)[N], F at) const {
    sfor<0, N>([&](auto i) { gstore(a + at(i), v[CV(i)].re); });
    if (two) sfor<0, N>([&](auto i) { gstore(b + at(i), v[CV(i)].im); });
  }
};

// First value and leading dimension of element e's columns in block blk, or in a
// caller buffer (blk = kExtX / kExtY)
template <typename T>
__device__ __forceinline__ T* block_base(const ElemDev& E, int e, int blk, const ExtBufs& X, long long& ld) {
  if (blk >= 0) {
    ld = E.ld;
    return reinterpret_cast<T*>(E.blk[blk]);
  }
  const long long l = blk == kExtX ? X.ldx : X.ldy;
  T* p = reinterpret_cast<T*>(blk == kExtX ? const_cast<void*>(X.x) : X.y);
  ld = l > 0 ? l : E.N;
  if (X.elem_only >= 0) return p;
  return p + (l > 0 ? (long long)e * l * X.nvec : X.off_grid[e] * X.nvec);
}

template <typename T>
__device__ __forceinline__ PairCols<T> pair_cols(const ElemDev& E, int e, int blk, int pair, int ncols,
                                                 const ExtBufs& X) {
  long long ld;
  T* base = block_base<T>(E, e, blk, X, ld);
  PairCols<T> pc;
  pc.a = base + (size_t)(2 * pair) * ld;
  pc.two = 2 * pair + 1 < ncols;
  pc.b = pc.two ? pc.a + ld : pc.a;
  return pc;
}

// ---------------------------------------------------------------------------
// plane pass: x-lines and y-lines of one z-plane, several planes per block
// ---------------------------------------------------------------------------
// Waves per SIMD asked of the compiler.  FP64 planes of 48 points take workgroups of six
// waves and 38 KB of LDS: at 100 VGPRs two share a CU, at 96 (five spilled) three: 681 us
// for 48 vectors on 16 elements of 48x48x64, 725 us.  The other sizes are below a step of
// the register file, or bound by LDS (64 points).
template <typename T, int NX, int MODE>
constexpr int plane_waves() {
  return sizeof(T) == 8 && NX == 48 && MODE == PM_HPSI ? 5 : 1;
}
template <typename T, int NX, int NY, int TL, int MODE>
__global__ void __launch_bounds__(512, (plane_waves<T, NX, MODE>())) k_plane(PlaneArgs A) {
  constexpr int NL = NX > NY ? NX : NY;
  constexpr int TPP = NL * TL;
  constexpr int PPW = (256 / TPP) > 0 ? 256 / TPP : 1;
  // LDS row pitch: with 8 lanes per line, NX + 2 (complex) makes the column reads of
  // a 16-lane group (2 lines x 8 lanes) fall in distinct banks
  constexpr int PITCH = NX + (TL == 8 ? 2 : 1);
  constexpr int MX = NX / TL, MY = NY / TL;
  using FX = LineFFT<T, NX, TL>;
  using FY = LineFFT<T, NY, TL>;
  __shared__ cplx<T> sm[PPW * NY * PITCH];

  const int e = A.elem_list[blockIdx.z];
  const ElemDev& E = A.elems[e];
  if (A.active && !A.active[e]) return;
  const int ncols = A.ncols > 0 ? A.ncols : (A.ncols == kNcolsJ ? E.J : E.K);
  const int pair = blockIdx.y;
  if (2 * pair >= ncols) return;
  const int slot = threadIdx.x / TPP;
  const int lt = threadIdx.x % TPP;
  const int line = lt / TL;
  const int t = lt % TL;
  const int z = blockIdx.x * PPW + slot;
  const bool zok = (slot < PPW) && (z < E.nz);
  constexpr int NXY = NX * NY;
  const size_t zoff = (size_t)z * NXY;
  cplx<T>* P = sm + (slot < PPW ? slot : 0) * NY * PITCH;

  // ---- load the plane (pair) into LDS: this thread's values are column lt % NX of the
  // rows lt / NX + TL i.  All loads go out before the first wait, and the stores at the
  // end without a branch each.  48 vectors on 16 elements of 48x48x64: 725 us, 757 us as a
  // loop with a wait per row and V read after the barrier (the first Teter pass 459 us,
  // 490 us; the last 296 us, 345 us).  The rest is the transforms: about 1400 vector
  // instructions and 120 LDS accesses a wave.
  constexpr int NI = NXY / TPP;
  static_assert(NX == NY && NXY % TPP == 0, "square planes, a whole number of rows per pass");
  const int lr = lt / NX, lc = lt % NX;
  auto at = [&](auto i) { return zoff + lt + TPP * CV(i); };
  const T* V = vptr<T>(E);
  T vv[MODE == PM_HPSI ? MY : 1];
  cplx<T> ld[NI];
  if constexpr (MODE == PM_HPSI || MODE == PM_TINV || MODE == PM_DX || MODE == PM_DY) {
    const int blk = (MODE == PM_TINV) ? A.out_blk : A.in_blk;
    const PairCols<T> in = pair_cols<T>(E, e, blk, pair, MODE == PM_TINV ? 2 * pair + 2 : ncols, A.ext);
    if (zok) {
      sfor<0, NI>([&](auto i) { ld[CV(i)] = in.load(at(i)); });
      if constexpr (MODE == PM_HPSI)
        sfor<0, MY>([&](auto i) { vv[CV(i)] = gload<T>(V + zoff + (t + TL * CV(i)) * NX + line); });
    }
  } else {  // PM_TFWD: r = HX - theta X
    const PairCols<T> xx = pair_cols<T>(E, e, A.in_blk, pair, ncols, A.ext);
    const PairCols<T> hx = pair_cols<T>(E, e, A.aux_blk, pair, ncols, A.ext);
    const int KP = E.kmax3 + 2;
    const double* th = E.small + SmallLayout::vec(KP) + VS_THETA * KP;
    const T ta = T(th[2 * pair]);
    const T tb = xx.two ? T(th[2 * pair + 1]) : T(0);
    if (zok) {
      sfor<0, NI>([&](auto i) { ld[CV(i)] = hx.load(at(i)); });
      if (!A.r_given) {
        cplx<T> x[NI];
        sfor<0, NI>([&](auto i) { x[CV(i)] = xx.load(at(i)); });
        sfor<0, NI>([&](auto i) {
          ld[CV(i)].re = ld[CV(i)].re - ta * x[CV(i)].re;
          ld[CV(i)].im = xx.two ? (ld[CV(i)].im - tb * x[CV(i)].im) : T(0);
        });
      }
    }
  }
  if (zok) sfor<0, NI>([&](auto i) { P[(lr + TL * CV(i)) * PITCH + lc] = ld[CV(i)]; });
  lds_barrier();

  if constexpr (MODE == PM_HPSI) {
    const T gys = T(E.ky / NY), gxs = T(E.kx / NX);
    cplx<T> acc[MY];
    // y-lines (line = x): Ty x + V x
    if (zok && line < NX) {
      cplx<T> v[MY];
      sfor<0, MY>([&](auto i) {
        const int y = t + TL * CV(i);
        v[CV(i)] = P[y * PITCH + line];
        acc[CV(i)] = {vv[CV(i)] * v[CV(i)].re, vv[CV(i)] * v[CV(i)].im};
      });
      FY::forward(v, t);
      sfor<0, MY>([&](auto i) {
        const int f = signed_freq(FY::freq(CV(i), t), NY);
        const T g = gys * T(f * f);
        v[CV(i)].re *= g;
        v[CV(i)].im *= g;
      });
      FY::inverse(v, t);
      sfor<0, MY>([&](auto i) { acc[CV(i)] = cadd(acc[CV(i)], v[CV(i)]); });
    }
    // x-lines (line = y): Tx x
    cplx<T> w[MX];
    const bool xl = zok && line < NY;
    if (xl) {
      sfor<0, MX>([&](auto i) { w[CV(i)] = P[line * PITCH + t + TL * CV(i)]; });
      FX::forward(w, t);
      sfor<0, MX>([&](auto i) {
        const int f = signed_freq(FX::freq(CV(i), t), NX);
        const T g = gxs * T(f * f);
        w[CV(i)].re *= g;
        w[CV(i)].im *= g;
      });
      FX::inverse(w, t);
    }
    lds_barrier();
    if (xl) sfor<0, MX>([&](auto i) { P[line * PITCH + t + TL * CV(i)] = w[CV(i)]; });
    lds_barrier();
    if (zok && line < NX) {
      const PairCols<T> out = pair_cols<T>(E, e, A.out_blk, pair, ncols, A.ext);
      sfor<0, MY>([&](auto i) { acc[CV(i)] = cadd(acc[CV(i)], P[(t + TL * CV(i)) * PITCH + line]); });
      out.store(acc, [&](auto i) { return zoff + (t + TL * CV(i)) * NX + line; });
    }
  } else if constexpr (MODE == PM_DX) {
    // d/dx along the rows: multiply the spectrum by i 2 pi f / L_x (normalised by 1/NX)
    const T g = T(sqrt(2.0 * E.kx) / NX);
    if (zok && line < NY) {
      cplx<T> w[MX];
      sfor<0, MX>([&](auto i) { w[CV(i)] = P[line * PITCH + t + TL * CV(i)]; });
      FX::forward(w, t);
      sfor<0, MX>([&](auto i) {
        const T m = g * T(deriv_freq(FX::freq(CV(i), t), NX));
        w[CV(i)] = {-m * w[CV(i)].im, m * w[CV(i)].re};
      });
      FX::inverse(w, t);
      const PairCols<T> out = pair_cols<T>(E, e, A.out_blk, pair, ncols, A.ext);
      out.store(w, [&](auto i) { return zoff + line * NX + t + TL * CV(i); });
    }
  } else if constexpr (MODE == PM_DY) {
    // d/dy along the columns
    const T g = T(sqrt(2.0 * E.ky) / NY);
    if (zok && line < NX) {
      cplx<T> v[MY];
      sfor<0, MY>([&](auto i) { v[CV(i)] = P[(t + TL * CV(i)) * PITCH + line]; });
      FY::forward(v, t);
      sfor<0, MY>([&](auto i) {
        const T m = g * T(deriv_freq(FY::freq(CV(i), t), NY));
        v[CV(i)] = {-m * v[CV(i)].im, m * v[CV(i)].re};
      });
      FY::inverse(v, t);
      const PairCols<T> out = pair_cols<T>(E, e, A.out_blk, pair, ncols, A.ext);
      out.store(v, [&](auto i) { return zoff + (t + TL * CV(i)) * NX + line; });
    }
  } else if constexpr (MODE == PM_TFWD) {
    // forward along x (rows), back to LDS at frequency positions, then along y
    cplx<T> w[MX];
    const bool xl = zok && line < NY;
    if (xl) {
      sfor<0, MX>([&](auto i) { w[CV(i)] = P[line * PITCH + t + TL * CV(i)]; });
      FX::forward(w, t);
    }
    lds_barrier();
    if (xl) sfor<0, MX>([&](auto i) { P[line * PITCH + FX::freq(CV(i), t)] = w[CV(i)]; });
    lds_barrier();
    if (zok && line < NX) {
      cplx<T> v[MY];
      sfor<0, MY>([&](auto i) { v[CV(i)] = P[(t + TL * CV(i)) * PITCH + line]; });
      FY::forward(v, t);
      const PairCols<T> out = pair_cols<T>(E, e, A.out_blk, pair, 2 * pair + 2, A.ext);
      out.store(v, [&](auto i) { return zoff + FY::freq(CV(i), t) * NX + line; });
    }
  } else {  // PM_TINV: inverse along y (columns), then x (rows); real pair out
    const bool yl = zok && line < NX;
    cplx<T> v[MY];
    if (yl) {
      // LDS holds [ky][kx]; register i of lane t takes frequency FY::freq(i, t)
      sfor<0, MY>([&](auto i) { v[CV(i)] = P[FY::freq(CV(i), t) * PITCH + line]; });
      FY::inverse(v, t);
    }
    lds_barrier();
    // after the inverse, register i of lane t is grid row y = t + TL * i
    if (yl) sfor<0, MY>([&](auto i) { P[(t + TL * CV(i)) * PITCH + line] = v[CV(i)]; });
    lds_barrier();
    if (zok && line < NY) {
      cplx<T> w[MX];
      sfor<0, MX>([&](auto i) { w[CV(i)] = P[line * PITCH + FX::freq(CV(i), t)]; });
      FX::inverse(w, t);
      const PairCols<T> out = pair_cols<T>(E, e, A.out_blk, pair, ncols, A.ext);
      out.store(w, [&](auto i) { return zoff + line * NX + t + TL * CV(i); });
    }
  }
}

// ---------------------------------------------------------------------------
// z-column pass
// ---------------------------------------------------------------------------
// STEP: HPSI, and the other terms of a filter step on its result
enum ZMode { ZM_HPSI = 0, ZM_TETER = 1, ZM_DZ = 2, ZM_STEP = 3 };

struct ZArgs {
  const ElemDev* elems;
  const int* elem_list;
  const int* active;
  int in_blk, out_blk;
  int ncols;
  int k3;
  ExtBufs ext;
  FilterStep f;
};

template <typename T, int NZ, int TL, int MODE>
__global__ void __launch_bounds__(256) k_zcol(ZArgs A) {
  constexpr int M = NZ / TL;
  using FZ = LineFFT<T, NZ, TL>;
  const int e = A.elem_list[blockIdx.z];
  const ElemDev& E = A.elems[e];
  if (A.active && !A.active[e]) return;
  const int ncols = A.ncols > 0 ? A.ncols : (A.ncols == kNcolsJ ? E.J : E.K);
  const int pair = blockIdx.y;
  if (2 * pair >= ncols) return;
  const int nxy = E.nx * E.ny;
  const int col = blockIdx.x * (256 / TL) + threadIdx.x / TL;
  const int t = threadIdx.x % TL;
  if (col >= nxy) return;  // whole lane groups leave together
  const cplx<T> wz = FZ::root(t);   // one root selection for both transforms

  // All loads of a kind go out together, and the stores after them (with out += v value by
  // value, each load waited for the store before it).  Bound by memory: 48 vectors on 16
  // elements of 48x48x64 take 655 us, 4.15 TB/s, either way; one element, 40 vectors: 36
  // us, 40 us before, and a filter step 45 us, 55 us.
  cplx<T> v[M];
  auto at = [&](auto i) { return (size_t)(t + TL * CV(i)) * nxy + col; };
  if constexpr (MODE == ZM_HPSI || MODE == ZM_STEP) {
    const PairCols<T> in = pair_cols<T>(E, e, A.in_blk, pair, ncols, A.ext);
    const PairCols<T> out = pair_cols<T>(E, e, A.out_blk, pair, ncols, A.ext);
    sfor<0, M>([&](auto i) { v[CV(i)] = in.load(at(i)); });
    FZ::forward(v, t, wz);
    const T gzs = T(E.kz / NZ);
    sfor<0, M>([&](auto i) {
      const int f = signed_freq(FZ::freq(CV(i), t), NZ);
      const T g = gzs * T(f * f);
      v[CV(i)].re *= g;
      v[CV(i)].im *= g;
    });
    FZ::inverse(v, t, wz);
    cplx<T> y[M];
    sfor<0, M>([&](auto i) { y[CV(i)] = out.load(at(i)); });
    if constexpr (MODE == ZM_HPSI) {
      sfor<0, M>([&](auto i) { v[CV(i)] = cadd(y[CV(i)], v[CV(i)]); });
    } else {
      // FP64: the three-term recurrence on the spot (x comes from the caches, it was read
      // above).  As a kernel of its own (k_filter_step) it read y, x and the third term and
      // wrote y again: 240 us of 1000 us a step for 48 vectors on six elements of 48x48x64
      const double* cf = A.f.coef + e * A.f.stride;
      const T al = cf[0], c = cf[1], be = A.f.prev_blk >= 0 ? cf[A.f.beta_at] : 0.0;
      cplx<T> x[M];
      sfor<0, M>([&](auto i) { x[CV(i)] = in.load(at(i)); });
      sfor<0, M>([&](auto i) {
        v[CV(i)].re = al * (y[CV(i)].re + v[CV(i)].re - c * x[CV(i)].re);
        v[CV(i)].im = al * (y[CV(i)].im + v[CV(i)].im - c * x[CV(i)].im);
      });
      if (A.f.prev_blk >= 0) {
        const PairCols<T> pv = pair_cols<T>(E, e, A.f.prev_blk, pair, ncols, A.ext);
        sfor<0, M>([&](auto i) { x[CV(i)] = pv.load(at(i)); });
        sfor<0, M>([&](auto i) {
          v[CV(i)].re -= be * x[CV(i)].re;
          v[CV(i)].im -= be * x[CV(i)].im;
        });
      }
    }
    out.store(v, at);
  } else if constexpr (MODE == ZM_DZ) {
    // d/dz along the columns of z
    const PairCols<T> in = pair_cols<T>(E, e, A.in_blk, pair, ncols, A.ext);
    sfor<0, M>([&](auto i) { v[CV(i)] = in.load(at(i)); });
    FZ::forward(v, t, wz);
    const T g = T(sqrt(2.0 * E.kz) / NZ);
    sfor<0, M>([&](auto i) {
      const T m = g * T(deriv_freq(FZ::freq(CV(i), t), NZ));
      v[CV(i)] = {-m * v[CV(i)].im, m * v[CV(i)].re};
    });
    FZ::inverse(v, t, wz);
    const PairCols<T> out = pair_cols<T>(E, e, A.out_blk, pair, ncols, A.ext);
    out.store(v, at);
  } else {
    // Teter: complex spectrum pair in W columns (2p: re, 2p+1: im), in place
    const PairCols<T> w = pair_cols<T>(E, e, A.out_blk, pair, 2 * pair + 2, A.ext);
    sfor<0, M>([&](auto i) { v[CV(i)] = w.load(at(i)); });
    FZ::forward(v, t, wz);
    const int KP = E.kmax3 + 2;
    const double* ek = E.small + SmallLayout::vec(KP) + VS_EKIN * KP;
    const double ea = ek[2 * pair];
    const double eb = (2 * pair + 1 < ncols) ? ek[2 * pair + 1] : ea;
    const T inv_e = T(2.0 / (ea + eb));
    const int kx = signed_freq(col % E.nx, E.nx);
    const int ky = signed_freq(col / E.nx, E.ny);
    const T gxy = T(E.kx * (double)(kx * kx) + E.ky * (double)(ky * ky));
    const T norm = T(1.0 / (double(E.nx) * E.ny * NZ));
    sfor<0, M>([&](auto i) {
      const int f = signed_freq(FZ::freq(CV(i), t), NZ);
      const T x = (gxy + T(E.kz) * T(f * f)) * inv_e;
      const T num = T(27) + x * (T(18) + x * (T(12) + T(8) * x));
      const T x2 = x * x;
      const T kf = norm * num * fast_recip(num + T(16) * x2 * x2);
      v[CV(i)].re *= kf;
      v[CV(i)].im *= kf;
    });
    FZ::inverse(v, t, wz);
    w.store(v, at);
  }
}

// ---------------------------------------------------------------------------
// nonlocal projectors: C = B^T X (per group of projectors sharing a support)
// ---------------------------------------------------------------------------
struct NlArgs {
  const ElemDev* elems;
  const int* active;
  int in_blk, out_blk;
  int ncols;
  int elem_only;   // >= 0: only this element (gridDim.z == 1)
  ExtBufs ext;
  FilterStep f;
};

// projector overlaps of element e: the element's own slice (nproj x kmax3), or the
// caller-independent scratch (nproj x nvec) of the no-allocation H*psi
__device__ __forceinline__ double* nlc_base(const ElemDev& E, int e, const ExtBufs& X, int& ld) {
  if (X.nlc) {
    ld = X.nvec;
    return X.nlc + (X.elem_only >= 0 ? 0 : X.nproj_off[e] * X.nvec);
  }
  ld = E.kmax3;
  return E.nlc;
}

constexpr int kNlCols = 8;
// NC: columns per workgroup; U: support points of a thread in flight (4 or 8 columns and
// 1 to 4 points measure the same within 3 %).
//
// Bound by latency (index, then x) and by the number of loads.  A workgroup has one
// group's four projectors; thread t sums the points t, t + 256, .. in that order, whatever
// NC.  48 vectors, 16 elements of 48x48x64 with 40 groups of 2000 points: 248 us, 270 us
// with one point in flight and a wave sum for each of the 32 values before; one element,
// 40 vectors: 20 us, 46 us.
template <typename T, int NC, int U>
__global__ void __launch_bounds__(256) k_nl_overlap(NlArgs A) {
  const int e = A.elem_only >= 0 ? A.elem_only : blockIdx.z;
  const ElemDev& E = A.elems[e];
  if (A.active && !A.active[e]) return;
  const int g = blockIdx.x;
  if (g >= E.ngrp) return;
  const int ncols = A.ncols > 0 ? A.ncols : (A.ncols == kNcolsJ ? E.J : E.K);
  const int c0 = blockIdx.y * NC;
  if (c0 >= ncols) return;
  const int s0 = E.grp_sptr[g], s1 = E.grp_sptr[g + 1];
  const int len = s1 - s0;
  const int p0 = E.grp_pbase[g], np = E.grp_pbase[g + 1] - p0;
  const long long vb = E.grp_vbase[g];
  long long ldx;
  const T* X = block_base<T>(E, e, A.in_blk, A.ext, ldx);
  int nld;
  double* nlc = nlc_base(E, e, A.ext, nld);
  const T* val = nullptr;
  if constexpr (sizeof(T) == 8) val = reinterpret_cast<const T*>(E.grp_val64);
  else val = reinterpret_cast<const T*>(E.grp_val32);
  // columns and projectors past the end repeat the last one and are not stored
  const T* xc[NC];
  const T* bq[4];
#pragma unroll
  for (int j = 0; j < NC; ++j) xc[j] = X + (size_t)min(c0 + j, ncols - 1) * ldx;
#pragma unroll
  for (int q = 0; q < 4; ++q) bq[q] = val + vb + (long long)min(q, np - 1) * len;
  const int* idx = E.grp_idx + s0;
  double acc[4 * NC];
#pragma unroll
  for (int i = 0; i < 4 * NC; ++i) acc[i] = 0.0;
  const int full = len / (256 * U) * (256 * U);   // points in whole steps of the workgroup
  int s = threadIdx.x;
  for (; s < full; s += 256 * U) {
    int r[U];
    T b[U][4], x[U][NC];
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = gload<int>(idx + s + 256 * u);
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int q = 0; q < 4; ++q) b[u][q] = gload<T>(bq[q] + s + 256 * u);
#pragma unroll
      for (int j = 0; j < NC; ++j) x[u][j] = gload<T>(xc[j] + r[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int j = 0; j < NC; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q * NC + j] += double(b[u][q]) * double(x[u][j]);
  }
  for (; s < len; s += 256) {
    const int r = gload<int>(idx + s);
    T b[4], x[NC];
#pragma unroll
    for (int q = 0; q < 4; ++q) b[q] = gload<T>(bq[q] + s);
#pragma unroll
    for (int j = 0; j < NC; ++j) x[j] = gload<T>(xc[j] + r);
#pragma unroll
    for (int j = 0; j < NC; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[q * NC + j] += double(b[q]) * double(x[j]);
  }
  // block reduction in a fixed order: rows of 16 lanes, then rows, then waves
  __shared__ double red[16][4 * NC];
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int h = 0; h < NC / 4; ++h) {
    double v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = acc[16 * h + i];
    red[threadIdx.x >> 4][16 * h + (lane & 15)] = row_sums16(v);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 4 * NC; i += blockDim.x) {
    double t = 0.0;
    for (int w = 0; w < 16; w += 4) t += (red[w][i] + red[w + 1][i]) + (red[w + 2][i] + red[w + 3][i]);
    const int q = i / NC, j = i % NC;
    if (q < np && c0 + j < ncols) gstore(nlc + (size_t)(p0 + q) * nld + c0 + j, t);
  }
}

// y[r, j] += sum_{p in row r} b_p(r) gamma_p C[p, j] over the active points (times the
// step's alpha after a filter step)
// NC: columns per thread.  Bound by latency: y and the entries of a point are loaded
// ahead of the sums.  LDS row pitch of the gamma C table: NC + 2, so that a row is read
// in 16-byte pairs.  48 vectors, 16 elements of 48x48x64, 43000 points with about eight
// entries each: 199 us, 374 us with y loaded last and one entry at a time before; one
// element, 40 vectors: 17 us, 29 us.
constexpr int kNlApplyPad = 2;
constexpr size_t nl_apply_lds(int nproj, int nc) { return (size_t)nproj * (nc + kNlApplyPad) * sizeof(double); }

template <typename T, int NC>
__global__ void __launch_bounds__(256) k_nl_apply(NlArgs A) {
  constexpr int kPitch = NC + kNlApplyPad, B = 4;   // B: entries in flight
  const int e = A.elem_only >= 0 ? A.elem_only : blockIdx.z;
  const ElemDev& E = A.elems[e];
  if (A.active && !A.active[e]) return;
  const int ncols = A.ncols > 0 ? A.ncols : (A.ncols == kNcolsJ ? E.J : E.K);
  const int c0 = blockIdx.y * NC;
  if (c0 >= ncols || E.nact == 0 || blockIdx.x * 256 >= E.nact) return;
  const int nc = min(NC, ncols - c0);
  extern __shared__ __align__(16) double gc[];   // nproj x kPitch: gamma_p C[p, c0 + j]
  // points past the end repeat the last one and are not stored
  const int a = blockIdx.x * 256 + threadIdx.x;
  const int ac = min(a, E.nact - 1);
  const int r = gload<int>(E.act_idx + ac);
  const int q0 = gload<int>(E.act_ptr + ac), q1 = gload<int>(E.act_ptr + ac + 1);
  long long ldy;
  T* Y = block_base<T>(E, e, A.out_blk, A.ext, ldy);
  T y[NC];
#pragma unroll
  for (int j = 0; j < NC; ++j) y[j] = gload<T>(Y + (size_t)(c0 + min(j, nc - 1)) * ldy + r);
  int nld;
  const double* nlc = nlc_base(E, e, A.ext, nld);
  for (int i = threadIdx.x; i < E.nproj * NC; i += 256) {
    const int p = i / NC, j = i % NC;
    gc[p * kPitch + j] = (j < nc) ? gload<double>(E.gamma + p) * gload<double>(nlc + (size_t)p * nld + c0 + j) : 0.0;
  }
  lds_barrier();
  double acc[NC];
#pragma unroll
  for (int j = 0; j < NC; ++j) acc[j] = 0.0;
  const T* ev = nullptr;
  if constexpr (sizeof(T) == 8) ev = reinterpret_cast<const T*>(E.ent_val64);
  else ev = reinterpret_cast<const T*>(E.ent_val32);
  auto add = [&](int p, double bv) {
    const double2* row = reinterpret_cast<const double2*>(gc + p * kPitch);
#pragma unroll
    for (int m = 0; m < NC / 2; ++m) {
      const double2 v = row[m];
      acc[2 * m] += bv * v.x;
      acc[2 * m + 1] += bv * v.y;
    }
  };
  int q = q0;
  for (; q + B <= q1; q += B) {
    int p[B];
    double bv[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      p[u] = gload<int>(E.ent_proj + q + u);
      bv[u] = double(gload<T>(ev + q + u));
    }
#pragma unroll
    for (int u = 0; u < B; ++u) add(p[u], bv[u]);
  }
  for (; q < q1; ++q) add(gload<int>(E.ent_proj + q), double(gload<T>(ev + q)));
  if (a >= E.nact) return;
  if (A.f.coef) {
    const double al = A.f.coef[e * A.f.stride];
#pragma unroll
    for (int j = 0; j < NC; ++j) acc[j] *= al;
  }
#pragma unroll
  for (int j = 0; j < NC; ++j)
    if (j < nc) gstore(Y + (size_t)(c0 + j) * ldy + r, T(y[j] + T(acc[j])));
}

// hy <- alpha (hy - c x) - beta prev on H x in FP32: H x is rounded to FP32, projector term
// included, before the step.  The fused pass would not keep that at the points that have
// projector entries (their term comes after it)
__global__ void __launch_bounds__(256) k_filter_step(const ElemDev* elems, const int* active, int x_blk, int hy_blk,
                                                     int cols, FilterStep f) {
  const int e = blockIdx.z;
  const ElemDev& E = elems[e];
  if (active && !active[e]) return;
  const int j = blockIdx.y;
  if (j >= (cols > 0 ? cols : E.K)) return;
  const double* cf = f.coef + e * f.stride;
  const double al = cf[0], c = cf[1], be = f.prev_blk >= 0 ? cf[f.beta_at] : 0.0;
  const float* x = reinterpret_cast<const float*>(E.blk[x_blk]) + (size_t)j * E.ld;
  float* hy = reinterpret_cast<float*>(E.blk[hy_blk]) + (size_t)j * E.ld;
  const float* pv = f.prev_blk >= 0 ? reinterpret_cast<const float*>(E.blk[f.prev_blk]) + (size_t)j * E.ld : nullptr;
  for (int r = blockIdx.x * 256 + threadIdx.x; r < E.N; r += gridDim.x * 256) {
    double v = al * (double(hy[r]) - c * double(x[r]));
    if (pv) v -= be * double(pv[r]);
    hy[r] = float(v);
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <typename T, int NXY, int TL, int MODE>
static void plane_launch(const PlaneArgs& a, int nz, int npairs, int nel, hipStream_t s) {
  constexpr int TPP = NXY * TL;
  constexpr int PPW = (256 / TPP) > 0 ? 256 / TPP : 1;
  dim3 grid((nz + PPW - 1) / PPW, npairs, nel);
  hipLaunchKernelGGL((k_plane<T, NXY, NXY, TL, MODE>), grid, dim3(PPW * TPP), 0, s, a);
}

template <typename T, int NZ, int TL, int MODE>
static void z_launch(const ZArgs& a, int nxy, int npairs, int nel, hipStream_t s) {
  dim3 grid((nxy + (256 / TL) - 1) / (256 / TL), npairs, nel);
  hipLaunchKernelGGL((k_zcol<T, NZ, TL, MODE>), grid, dim3(256), 0, s, a);
}

// lanes per FFT line: lines of 32..64 points on 8 lanes (M = 4..8 values per
// lane), shorter lines on 4; the same for FP32 and FP64 (fewer values per lane keep
// the register count, and so the occupancy, of the long-line kernels up)
template <typename T, int N>
constexpr int lanes_per_line() {
  return N >= 32 ? 8 : 4;
}

template <typename T, int MODE>
static bool dispatch_plane(int nxy, const PlaneArgs& a, int nz, int npairs, int nel, hipStream_t s) {
  switch (nxy) {
    case 8: plane_launch<T, 8, lanes_per_line<T, 8>(), MODE>(a, nz, npairs, nel, s); return true;
    case 12: plane_launch<T, 12, lanes_per_line<T, 12>(), MODE>(a, nz, npairs, nel, s); return true;
    case 16: plane_launch<T, 16, lanes_per_line<T, 16>(), MODE>(a, nz, npairs, nel, s); return true;
    case 24: plane_launch<T, 24, lanes_per_line<T, 24>(), MODE>(a, nz, npairs, nel, s); return true;
    case 32: plane_launch<T, 32, lanes_per_line<T, 32>(), MODE>(a, nz, npairs, nel, s); return true;
    case 48: plane_launch<T, 48, lanes_per_line<T, 48>(), MODE>(a, nz, npairs, nel, s); return true;
    case 64: plane_launch<T, 64, lanes_per_line<T, 64>(), MODE>(a, nz, npairs, nel, s); return true;
    default: return false;
  }
}

template <typename T, int MODE>
static bool dispatch_z(int nz, const ZArgs& a, int nxy, int npairs, int nel, hipStream_t s) {
  switch (nz) {
    case 8: z_launch<T, 8, lanes_per_line<T, 8>(), MODE>(a, nxy, npairs, nel, s); return true;
    case 12: z_launch<T, 12, lanes_per_line<T, 12>(), MODE>(a, nxy, npairs, nel, s); return true;
    case 16: z_launch<T, 16, lanes_per_line<T, 16>(), MODE>(a, nxy, npairs, nel, s); return true;
    case 24: z_launch<T, 24, lanes_per_line<T, 24>(), MODE>(a, nxy, npairs, nel, s); return true;
    case 32: z_launch<T, 32, lanes_per_line<T, 32>(), MODE>(a, nxy, npairs, nel, s); return true;
    case 48: z_launch<T, 48, lanes_per_line<T, 48>(), MODE>(a, nxy, npairs, nel, s); return true;
    case 64: z_launch<T, 64, lanes_per_line<T, 64>(), MODE>(a, nxy, npairs, nel, s); return true;
    default: return false;
  }
}

// algorithmic bytes of the H*psi passes for the elements a launch covers
struct HpsiWork {
  double plane = 0, zcol = 0, nl = 0;
};

static HpsiWork hpsi_work(Ctx& c, int elem, int ncols, size_t sz, const std::vector<int>& members,
                          const int* active_host, bool third = false) {
  HpsiWork w;
  for (int e : members) {
    if (elem >= 0 && e != elem) continue;
    if (active_host && !active_host[e]) continue;
    const double N = c.N[e], k = ncols > 0 ? ncols : c.K[e];
    w.plane += (2.0 * k + 1.0) * N * sz;          // read x, write y1, read V
    w.zcol += (third ? 4.0 : 3.0) * k * N * sz;   // read x, read y1 (and a step's third term), write y
    const double nnz = c.nnz[e], nact = c.elems_host[e].nact;
    w.nl += nnz * (sz + 4) + 3.0 * nact * k * sz;  // projectors; x read, y read+write at active points
  }
  return w;
}

template <typename T>
static int hpsi_typed(Ctx& c, int elem, int ncols, int in_blk, int out_blk, const int* active,
                      const ExtBufs& ext = ExtBufs(), const FilterStep& f = FilterStep()) {
  hipStream_t s = c.stream;
  const int* act_host = (active && !c.active_host.empty()) ? c.active_host.data() : nullptr;
  const int* iota = c.iota_dev;
  if (c.timing && !c.capturing) {
    // algorithmic bytes of the state applications: read psi, write H psi, V and the
    // projectors (nnz values + int32 indices) amortised over the J wanted states
    const double sz = sizeof(T);
    for (int e = 0; e < c.n_elem; ++e) {
      if ((elem >= 0 && e != elem) || (act_host && !act_host[e])) continue;
      const double N = c.N[e], k = ncols > 0 ? ncols : c.K[e], J = c.J[e];
      c.tacc.hpsi_alg += k * (2.0 * N * sz + N * sz / J + c.nnz[e] * (sz + 4.0) / J);
    }
  }
  // projector overlaps first (reads x only)
  {
    NlArgs na{c.elems_dev, active, in_blk, out_blk, ncols, elem, ext};
    int ng = 0, np = 0, kk = 0;
    for (int e = 0; e < c.n_elem; ++e) {
      if (elem >= 0 && e != elem) continue;
      ng = std::max(ng, c.elems_host[e].ngrp);
      np = std::max(np, c.elems_host[e].nproj);
      kk = std::max(kk, ncols > 0 ? ncols : c.K[e]);
    }
    if (ng > 0) {
      std::vector<int> all(c.n_elem);
      for (int e = 0; e < c.n_elem; ++e) all[e] = e;
      TimedScope ts(c, TC_NL, hpsi_work(c, elem, ncols, sizeof(T), all, act_host).nl);
      const int nel = elem >= 0 ? 1 : c.n_elem;
      hipLaunchKernelGGL((k_nl_overlap<T, kNlCols, 2>), dim3(ng, (kk + kNlCols - 1) / kNlCols, nel), dim3(256), 0, s, na);
    }
    c.nl_pending_np = np;
    c.nl_pending_kk = kk;
  }
  for (const ShapeClass& sc : c.classes) {
    const int* list = sc.elem_list_dev;
    int nel = sc.nelem;
    int maxk = 0;
    if (elem >= 0) {
      bool member = false;
      for (int x : sc.elem_list_host) member |= (x == elem);
      if (!member) continue;
      list = iota + elem;
      nel = 1;
      maxk = ncols > 0 ? ncols : c.K[elem];
    } else {
      maxk = ncols > 0 ? ncols : sc.max_k;
    }
    const int npairs = (maxk + 1) / 2;
    PlaneArgs pa{c.elems_dev, list, active, in_blk, out_blk, -1, ncols, nullptr, 0, ext};
    const HpsiWork hw = hpsi_work(c, elem, ncols, sizeof(T), sc.elem_list_host, act_host, f.prev_blk >= 0);
    {
      TimedScope ts(c, TC_PLANE, hw.plane);
      if (!dispatch_plane<T, PM_HPSI>(sc.nx, pa, sc.nz, npairs, nel, s)) {
        set_error("unsupported grid");
        return DG_ERR_SHAPE;
      }
    }
    ZArgs za{c.elems_dev, list, active, in_blk, out_blk, ncols, 0, ext, f};
    {
      TimedScope ts(c, TC_ZCOL, hw.zcol);
      bool ok;
      if constexpr (sizeof(T) == 8)
        ok = f.coef ? dispatch_z<T, ZM_STEP>(sc.nz, za, sc.nx * sc.ny, npairs, nel, s)
                    : dispatch_z<T, ZM_HPSI>(sc.nz, za, sc.nx * sc.ny, npairs, nel, s);
      else
        ok = dispatch_z<T, ZM_HPSI>(sc.nz, za, sc.nx * sc.ny, npairs, nel, s);
      if (!ok) {
        set_error("unsupported grid");
        return DG_ERR_SHAPE;
      }
    }
  }
  if (c.nl_pending_np > 0) {
    NlArgs na{c.elems_dev, active, in_blk, out_blk, ncols, elem, ext, f};
    int nact = 0;
    for (int e = 0; e < c.n_elem; ++e)
      if (elem < 0 || e == elem) nact = std::max(nact, c.elems_host[e].nact);
    TimedScope ts(c, TC_NL);
    const int nel = elem >= 0 ? 1 : c.n_elem;
    // 16 columns, and 8 where the table of the most projectors (480) exceeds 64 KB of LDS
    auto apply = [&](auto nc) {
      constexpr int NC = decltype(nc)::value;
      hipLaunchKernelGGL((k_nl_apply<T, NC>), dim3((nact + 255) / 256, (c.nl_pending_kk + NC - 1) / NC, nel), dim3(256),
                         nl_apply_lds(c.nl_pending_np, NC), s, na);
    };
    if (nl_apply_lds(c.nl_pending_np, 16) <= 65536) apply(std::integral_constant<int, 16>());
    else apply(std::integral_constant<int, 8>());
  }
  DG_HIP(hipGetLastError());
  return DG_OK;
}

int launch_hpsi(Ctx& c, int elem, int ncols, int prec, int in_blk, int out_blk, const int* active) {
  if (c.dg_op.active) return launch_dg_bsr(c, in_blk, out_blk, ncols, active);
  return prec == DG_FP64 ? hpsi_typed<double>(c, elem, ncols, in_blk, out_blk, active)
                         : hpsi_typed<float>(c, elem, ncols, in_blk, out_blk, active);
}

int launch_hpsi_step(Ctx& c, int ncols, int prec, int in_blk, int out_blk, const int* active, const FilterStep& f) {
  if (c.dg_op.active) return launch_dg_bsr(c, in_blk, out_blk, ncols, active, f);
  if (prec == DG_FP64) return hpsi_typed<double>(c, -1, ncols, in_blk, out_blk, active, ExtBufs(), f);
  if (int st = hpsi_typed<float>(c, -1, ncols, in_blk, out_blk, active)) return st;
  int n = 0, k = std::max(ncols, 0);
  for (int e = 0; e < c.n_elem; ++e) {
    n = std::max(n, c.N[e]);
    if (ncols <= 0) k = std::max(k, c.K[e]);
  }
  TimedScope ts(c, TC_OTHER);
  hipLaunchKernelGGL(k_filter_step, dim3(std::min(64, (n + 255) / 256), k, c.n_elem), dim3(256), 0, c.stream,
                     c.elems_dev, active, in_blk, out_blk, ncols, f);
  DG_HIP(hipGetLastError());
  return DG_OK;
}

int launch_hpsi_ext(Ctx& c, int elem, int ncols, int prec, const ExtBufs& ext) {
  return prec == DG_FP64 ? hpsi_typed<double>(c, elem, ncols, kExtX, kExtY, nullptr, ext)
                         : hpsi_typed<float>(c, elem, ncols, kExtX, kExtY, nullptr, ext);
}

// W <- Teter(HX - X theta), three passes, for every element in place in W (r_given:
// hx_blk already holds the residual)
template <typename T>
static int teter_typed(Ctx& c, int x_blk, int hx_blk, int w_blk, int k3, const int* active, bool r_given) {
  hipStream_t s = c.stream;
  double tw = 0.0;
  for (int e = 0; e < c.n_elem; ++e)
    if (c.active_host.empty() || c.active_host[e]) tw += 3.0 * c.K[e] * (double)c.N[e] * sizeof(T);
  TimedScope ts(c, TC_TETER, tw);   // read X, HX, write W
  for (const ShapeClass& sc : c.classes) {
    const int npairs = (sc.max_k + 1) / 2;
    PlaneArgs pa{c.elems_dev, sc.elem_list_dev, active, r_given ? hx_blk : x_blk, w_blk, hx_blk, -1, nullptr, k3};
    pa.r_given = r_given ? 1 : 0;
    if (!dispatch_plane<T, PM_TFWD>(sc.nx, pa, sc.nz, npairs, sc.nelem, s)) return DG_ERR_SHAPE;
    ZArgs za{c.elems_dev, sc.elem_list_dev, active, w_blk, w_blk, -1, k3};
    if (!dispatch_z<T, ZM_TETER>(sc.nz, za, sc.nx * sc.ny, npairs, sc.nelem, s)) return DG_ERR_SHAPE;
    PlaneArgs pc{c.elems_dev, sc.elem_list_dev, active, w_blk, w_blk, -1, -1, nullptr, k3};
    if (!dispatch_plane<T, PM_TINV>(sc.nx, pc, sc.nz, npairs, sc.nelem, s)) return DG_ERR_SHAPE;
  }
  DG_HIP(hipGetLastError());
  return DG_OK;
}

int launch_teter(Ctx& c, int prec, int x_blk, int hx_blk, int w_blk, int k3, const int* active, bool r_given) {
  return prec == DG_FP64 ? teter_typed<double>(c, x_blk, hx_blk, w_blk, k3, active, r_given)
                         : teter_typed<float>(c, x_blk, hx_blk, w_blk, k3, active, r_given);
}

// d/dx, d/dy, d/dz of the first J_k columns of block in_blk into out blocks (FP64,
// every element)
int launch_gradient(Ctx& c, int in_blk, const int out_blk[3]) {
  hipStream_t s = c.stream;
  const int ncols = kNcolsJ;
  for (const ShapeClass& sc : c.classes) {
    int maxk = 0;
    for (int e : sc.elem_list_host) maxk = std::max(maxk, c.J[e]);
    const int npairs = (maxk + 1) / 2;
    PlaneArgs px{c.elems_dev, sc.elem_list_dev, nullptr, in_blk, out_blk[0], -1, ncols, nullptr, 0};
    if (!dispatch_plane<double, PM_DX>(sc.nx, px, sc.nz, npairs, sc.nelem, s)) return DG_ERR_SHAPE;
    PlaneArgs py{c.elems_dev, sc.elem_list_dev, nullptr, in_blk, out_blk[1], -1, ncols, nullptr, 0};
    if (!dispatch_plane<double, PM_DY>(sc.nx, py, sc.nz, npairs, sc.nelem, s)) return DG_ERR_SHAPE;
    ZArgs zz{c.elems_dev, sc.elem_list_dev, nullptr, in_blk, out_blk[2], ncols, 0};
    if (!dispatch_z<double, ZM_DZ>(sc.nz, zz, sc.nx * sc.ny, npairs, sc.nelem, s)) return DG_ERR_SHAPE;
  }
  DG_HIP(hipGetLastError());
  return DG_OK;
}

bool grid_supported(int nx, int ny, int nz) {
  auto ok = [](int n) { return n == 8 || n == 12 || n == 16 || n == 24 || n == 32 || n == 48 || n == 64; };
  return nx == ny && ok(nx) && ok(nz);
}

}  // namespace dg
