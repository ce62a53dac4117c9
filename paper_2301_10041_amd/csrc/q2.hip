// Class stencils of the paper's element pair (Q2 velocity, discontinuous P1 pressure) and the
// coefficients of the cell form that its velocity V-cycle uses.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "ctx.h"
#include "q2.h"
#include "q2cell.h"

namespace fsi {

// Class stencils of the Q2 A_f: the row of an interior node of each class summed over its cells
// as k_asm_q2q2 sums them (node (2 + a, 2 + b) of class a + 2 b has every cell inside for n >= 2).
void q2_tables(int n, double nu, double rdt, Q2Table &t) {
  FSI_REQUIRE(n >= 2, FSI_E_ARG, "Q2 class stencils need n >= 2");
  std::vector<double> E;
  q2_element_table(n, nu, E);
  std::memset(&t, 0, sizeof(t));
  for (int cls = 0; cls < 4; ++cls) {
    const int I = 2 + (cls & 1), J = 2 + (cls >> 1);
    const int i0 = std::max(0, (I - 1) >> 1), i1 = std::min(n - 1, I >> 1);
    const int j0 = std::max(0, (J - 1) >> 1), j1 = std::min(n - 1, J >> 1);
    int cnt = 0;
    for (int J2 = 2 * j0; J2 <= 2 * j1 + 2; ++J2)
      for (int I2 = 2 * i0; I2 <= 2 * i1 + 2; ++I2) {
        double m = 0.0, kk[4] = {0.0, 0.0, 0.0, 0.0};
        for (int cj = j0; cj <= j1; ++cj) {
          const int b = J - 2 * cj, b2 = J2 - 2 * cj;
          if (b2 < 0 || b2 > 2) continue;
          for (int ci = i0; ci <= i1; ++ci) {
            const int a = I - 2 * ci, a2 = I2 - 2 * ci;
            if (a2 < 0 || a2 > 2) continue;
            const int li = a + 3 * b, lj = a2 + 3 * b2;
            m += E[QE_M + 9 * li + lj];
            for (int q = 0; q < 4; ++q) kk[q] += E[QE_K + (q * 9 + li) * 9 + lj];
          }
        }
        FSI_REQUIRE(cnt < kQ2Max, FSI_E_ARG, "Q2 stencil too wide");
        const double v[4] = {rdt * m + kk[0], kk[1], kk[2], rdt * m + kk[3]};
        t.off[cls][cnt][0] = I2 - I;
        t.off[cls][cnt][1] = J2 - J;
        for (int q = 0; q < 4; ++q) t.coef[cls][cnt][q] = v[q];
        ++cnt;
      }
    t.count[cls] = cnt;
  }
}

static Q2Coef<double> q2_closed_form(int n, double nu, double rdt) {
  const double h = 1.0 / n;
  Q2Coef<double> c;
  c.a = nu / 90.0;
  c.b = nu / 180.0;
  c.g = rdt * h * h / 900.0;
  c.k = nu / 72.0;
  c.dv = 1.0 / (112 * (c.a + c.b) + 64 * c.g);
  c.d1 = 1.0 / (128 * c.a + 224 * c.b + 128 * c.g);
  c.d2 = 1.0 / (224 * c.a + 128 * c.b + 128 * c.g);
  c.dc = 1.0 / (256 * (c.a + c.b) + 256 * c.g);
  return c;
}

// Every entry of the class stencils, summed from the element matrices, has to be the one that
// cell_products takes for it: the parts of nu and of rho/dt each at a unit value (A_f is linear in them),
// so that a caller's parameters decide nothing here.
static void check_q2_closed_form(int n) {
  static const double M[2][5] = {{-1, 2, 8, 2, -1}, {0, 2, 16, 2, 0}}, K[2][5] = {{1, -8, 14, -8, 1}, {0, -8, 16, -8, 0}},
                      G[2][5] = {{-1, 4, 0, -4, 1}, {0, 4, 0, -4, 0}};
  for (int part = 0; part < 2; ++part) {
    const double nu = part == 0 ? 1.0 : 0.0, rdt = 1.0 - nu;
    const Q2Coef<double> c = q2_closed_form(n, nu, rdt);
    Q2Table t;
    q2_tables(n, nu, rdt, t);
    const double tol = 1e-13 * 256 * (c.a + c.b + c.g);
    for (int cls = 0; cls < 4; ++cls)
      for (int e = 0; e < t.count[cls]; ++e) {
        const int u = cls & 1, v = cls >> 1, i = t.off[cls][e][0] + 2, j = t.off[cls][e][1] + 2;
        const double km = K[u][i] * M[v][j], mk = M[u][i] * K[v][j], mm = M[u][i] * M[v][j], gg = G[u][i] * G[v][j];
        const double want[4] = {c.a * km + c.b * mk + c.g * mm, -c.k * gg, -c.k * gg, c.b * km + c.a * mk + c.g * mm};
        for (int k = 0; k < 4; ++k)
          FSI_REQUIRE(std::abs(t.coef[cls][e][k] - want[k]) <= tol, FSI_E_STATE,
                      "an entry of the Q2 A_f differs from its closed form");
        if (i == 2 && j == 2) {
          const double d[2] = {cls == 0 ? c.dv : cls == 1 ? c.d1 : cls == 2 ? c.d2 : c.dc,
                               cls == 0 ? c.dv : cls == 1 ? c.d2 : cls == 2 ? c.d1 : c.dc};
          FSI_REQUIRE(std::abs(d[0] * want[0] - 1.0) <= 1e-12 && std::abs(d[1] * want[3] - 1.0) <= 1e-12, FSI_E_STATE,
                      "an inverse diagonal of the Q2 A_f differs from its closed form");
        }
      }
  }
}

void q2_coefs(int n, double nu, double rdt, Q2Coef<double> &c, Q2Coef<float> &f) {
  check_q2_closed_form(n);
  c = q2_closed_form(n, nu, rdt);
  const double *p = &c.a;
  float *q = &f.a;
  static_assert(sizeof(Q2Coef<double>) == 8 * sizeof(double) && sizeof(Q2Coef<float>) == 8 * sizeof(float),
                "coefficients only");
  for (int i = 0; i < 8; ++i) q[i] = (float)p[i];
}

}  // namespace fsi
