// Transfer weights of the P2 multigrid on the structured grid: the table of the restriction (host
// export and tests), and the check of the weights that the kernels compile in (afcell.h).
#include <cstdlib>
#include <cstring>

#include "kernels.h"
#include "lattice.h"

namespace fsi {

// ---------------------------------------------------------------- P2 restriction weights
// Host: the restriction weights do not depend on the level (nested uniform refinement),
// so they are read off at interior coarse nodes of a 16 x 16 fine grid.
void p2_restrict_tables(P2RestrTable &t) {
  std::memset(&t, 0, sizeof(t));
  const int nf = 16;
  for (int cls = 0; cls < 4; ++cls) {
    const int Ic = 4 + (cls & 1), Jc = 4 + (cls >> 1);
    int cnt = 0;
    for (int dJ = -4; dJ <= 4; ++dJ)
      for (int dI = -4; dI <= 4; ++dI) {
        int ic[6], jc[6];
        double w[6];
        const int m = p2_prolong_weights(2 * Ic + dI, 2 * Jc + dJ, nf, ic, jc, w);
        for (int q = 0; q < m; ++q)
          if (ic[q] == Ic && jc[q] == Jc) {
            FSI_REQUIRE(cnt < kRestrMax, FSI_E_ARG, "restriction table overflow");
            t.off[cls][cnt][0] = dI;
            t.off[cls][cnt][1] = dJ;
            t.w[cls][cnt] = w[q];
            ++cnt;
          }
      }
    t.count[cls] = cnt;
  }
  // the compiled transfer weights (afcell.h) against the interpolation they stand for
  for (int B = 0; B < 4; ++B)
    for (int A = 0; A < 4; ++A) {
      int ic[6], jc[6];
      double w[6], v[9] = {};
      const int m = p2_prolong_weights(4 + A, 4 + B, nf, ic, jc, w);
      for (int q = 0; q < m; ++q) v[3 * (jc[q] - 2) + ic[q] - 2] = w[q];
      for (int q = 0; q < 9; ++q)
        FSI_REQUIRE(v[q] == prolong_weight(A, B, q % 3, q / 3), FSI_E_ARG,
                    "the compiled prolongation weights differ from the interpolation");
    }
  for (int cls = 0; cls < 4; ++cls) {
    double sum = 0.0;
    for (int k = 0; k < t.count[cls]; ++k) {
      const int *o = t.off[cls][k];
      sum += t.w[cls][k];
      FSI_REQUIRE(std::abs(o[0]) <= 3 && std::abs(o[1]) <= 3 &&
                      t.w[cls][k] == restrict_weight(cls & 1, cls >> 1, o[0], o[1]),
                  FSI_E_ARG, "the compiled restriction weights differ from the transposed interpolation");
    }
    for (int dJ = -3; dJ <= 3; ++dJ)
      for (int dI = -3; dI <= 3; ++dI) sum -= restrict_weight(cls & 1, cls >> 1, dI, dJ);
    FSI_REQUIRE(sum == 0.0, FSI_E_ARG, "a compiled restriction weight has no entry in the table");
  }
}

}  // namespace fsi
