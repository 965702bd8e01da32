// Host check of the Gram launch plans in k_dense.hip, built for the CPU only (no kernel is
// launched): the kernel that a plan instantiates has room for the blocks per wave and the
// staged columns of every tile of every element of the launch (a wave with more blocks
// than its instantiation would form no products), the dynamic LDS of the two panels is
// within the limit that the kernels are registered with, and every grid that elements can
// have fills whole 32-row panels of the FP32 kernel.
#include "../../paper_2003_00407_amd/csrc/k_dense.hip"

#include <cstdio>
#include <random>

namespace dg {
// the launchers' error sink and timing scope live in other translation units
void set_error(const std::string&) {}
TimedScope::TimedScope(Ctx& ctx, int k, double w) : c(ctx), cls(k), work(w) {}
TimedScope::~TimedScope() {}
}  // namespace dg

// one launch: K_e of every element, nbS and nbT blocks of columns per operand
static int check_launch(const std::vector<int>& K, int nbS, int nbT, int sym, int same, int pair, bool fp64) {
  std::vector<int> bis;
  int bj_max = 0;
  for (int k : K) {
    bis.push_back((nbS * k + 15) / 16);
    bj_max = std::max(bj_max, (nbT * k + 15) / 16);
  }
  const dg::GramPlan pl = dg::plan_gram_tiles(bis, bj_max, sym, same, pair, 6, fp64 ? dg::GP_MAXCOL : dg::G3_MAXCOL);
  const int maxb = dg::gram_blocks_per_wave(pl), pf = (pl.maxnc + 63) / 64;
  const int staged = pf == 5 ? 6 * 64 : pf * 64;   // instantiations: 1, 2, 3, 4 and 6 pieces
  if (maxb < 1 || maxb > 6 || pf < 1 || pf > 6 || dg::gram_lds_bytes(pl, fp64, false) > (size_t)dg::GP_LDS_LIMIT) {
    printf("plan without a kernel: maxb=%d pf=%d maxnc=%d\n", maxb, pf, pl.maxnc);
    return 1;
  }
  for (int k : K) {
    const int bi = (nbS * k + 15) / 16, bj = (nbT * k + 15) / 16;
    const int nt = dg::gram_ntiles(bi, bj, pl.tb, sym);
    if (nt > pl.ntiles) {
      printf("element with %d tiles, launch with %d\n", nt, pl.ntiles);
      return 1;
    }
    for (int t = 0; t < nt; ++t) {
      const dg::GramTile g = dg::gram_tile(t, bi, bj, pl.tb, sym, same, pair);
      const int cs = ((pair ? 2 : 1) * g.nloc + 7) >> 3, nc = g.ncA + g.ncB + g.ncC;
      if (cs < 1 || cs > maxb || nc > pl.maxnc || nc > staged) {
        printf("tile outside its kernel: K=%d bi=%d bj=%d tb=%d cs=%d of %d, %d of %d columns\n", k, bi, bj, pl.tb, cs,
               maxb, nc, pl.maxnc);
        return 1;
      }
    }
  }
  return 0;
}

int main() {
  std::mt19937 rng(9);
  int launches = 0;
  for (int n = 0; n < 600; ++n) {
    std::vector<int> K;   // 1 .. 88 columns per block, batches of one to twelve elements
    const int count = n < 88 ? 1 : 1 + (int)(rng() % 12);
    for (int e = 0; e < count; ++e) K.push_back(n < 88 ? n + 1 : 1 + (int)(rng() % 88));
    for (int nb = 1; nb <= 3; ++nb)
      for (int fp64 = 0; fp64 <= 1; ++fp64) {
        // S^T S, [S^T S, S^T T] at once, S^T T symmetric and general
        const int modes[4][3] = {{1, 1, 0}, {1, 0, 1}, {1, 0, 0}, {0, 0, 0}};
        for (const auto& m : modes) {
          if (int r = check_launch(K, nb, nb, m[0], m[1], m[2], fp64 != 0)) return r;
          ++launches;
        }
      }
  }
  const int lines[7] = {8, 12, 16, 24, 32, 48, 64};
  for (int nx : lines)
    for (int nz : lines)
      if (nx * nx * nz % dg::G3_R != 0) {
        printf("grid %d x %d x %d leaves a partial panel\n", nx, nx, nz);
        return 1;
      }
  printf("plans: %d launches, every tile within its kernel\n", launches);
  return 0;
}
