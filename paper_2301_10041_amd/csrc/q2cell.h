// A_f of the paper's pair (Q2 on squares) cell by cell, as afcell.h has it for the triangle pair.
//
// With the 1D Q2 matrices of a uniform grid, M (mass), K (stiffness) and G (int phi_i' phi_j), the
// interior rows of A_f are tensor products (x factor first):
//   xx: (rho/dt) M x M + nu (K x M + 1/2 M x K),   xy = yx: 1/2 nu G x G^T (up to sign: -, with G x G),
//   yy: the two factors of xx exchanged.
// Rows of 1D vertices (offsets -2 .. 2): M (-1, 2, 8, 2, -1), K (1, -8, 14, -8, 1), G (-1, 4, 0, -4, 1);
// of midpoints (-1 .. 1): M (2, 16, 2), K (-8, 16, -8), G (4, 0, -4); units h / 30, 1 / (3 h), 1 / 6.
// So the four rows of a cell (vertex, (1, 0), (0, 1), (1, 1)) take their 25-node window lattice row by
// lattice row: the 1D sums along x first, then their share of the sums along y; five coefficients
// in all, where the 2 x 2 blocks of the class stencils are 256.
#pragma once

#include "afcell.h"

namespace fsi {

template <typename T>
struct Q2Coef {
  T a, b, g, k;          // nu / 90, nu / 180, (rho/dt) h^2 / 900, nu / 72
  T dv, d1, d2, dc;      // 1 / diagonal: vertex; edge along and across its direction; centre
};

// the biquadratic of a coarse cell: weight of its node (a, b) at its fine node (A, B)
__host__ __device__ constexpr double q2_line(int A, int a) {   // 1D, at A / 4
  const double t = 0.25 * A;
  return a == 0 ? 2.0 * (t - 0.5) * (t - 1.0) : a == 1 ? 4.0 * t * (1.0 - t) : 2.0 * t * (t - 0.5);
}
__host__ __device__ constexpr double q2_prolong_weight(int A, int B, int a, int b) {
  return q2_line(A, a) * q2_line(B, b);
}

template <typename T, int PL, int HW>
__device__ __forceinline__ void cell_products(const V2<T> *p, const Q2Coef<T> &c, V2<T> (&x)[4], V2<T> (&s)[4]) {
  auto W = [&](int dI, int dJ) -> V2<T> { return p[(dI & 1) * PL + dJ * HW + (dI >> 1)]; };
  auto row = [&](auto r_tag) {
    constexpr int R = decltype(r_tag)::value;   // lattice row -2 .. 2
    const V2<T> l2 = W(-2, R), l1 = W(-1, R), o = W(0, R), r1 = W(1, R), r2 = W(2, R);
    if constexpr (R == 0) {
      x[0] = o;
      x[1] = r1;
    }
    if constexpr (R == 1) {
      x[2] = o;
      x[3] = r1;
    }
    // 1D sums along x at the vertex column (col 0) and at the midpoint column (col 1)
    auto col = [&](auto col_tag) {
      constexpr int C = decltype(col_tag)::value;
      auto mk = [&](T vl2, T vl1, T vo, T vr1, T vr2, T &m, T &k, T &g) {
        if constexpr (C == 0) {
          const T e1 = vl1 + vr1, e2 = vl2 + vr2;
          m = fma(T(8), vo, fma(T(2), e1, -e2));
          k = fma(T(14), vo, fma(T(-8), e1, e2));
          g = fma(T(4), vl1 - vr1, vr2 - vl2);
        } else {
          const T e = vo + vr2;
          m = fma(T(16), vr1, T(2) * e);
          k = fma(T(16), vr1, T(-8) * e);
          g = T(4) * (vo - vr2);
        }
      };
      T mx, kx, gx, my, ky, gy;
      mk(l2.x, l1.x, o.x, r1.x, r2.x, mx, kx, gx);
      mk(l2.y, l1.y, o.y, r1.y, r2.y, my, ky, gy);
      // along y: mass of p, stiffness of q, and g of the other component's g
      const T px = fma(c.a, kx, c.g * mx), qx = c.b * mx, py = fma(c.b, ky, c.g * my), qy = c.a * my;
      gx *= -c.k;
      gy *= -c.k;
      if constexpr (R == -2) s[C] = V2<T>{(qx - px) - gy, (qy - py) - gx};
      if constexpr (R == 2) s[C] = V2<T>{s[C].x + ((qx - px) + gy), s[C].y + ((qy - py) + gx)};
      if constexpr (R == -1 || R == 1) {
        constexpr T G = R == 1 ? T(-4) : T(4);
        s[C].x = fma(T(2), px, fma(T(-8), qx, fma(G, gy, s[C].x)));
        s[C].y = fma(T(2), py, fma(T(-8), qy, fma(G, gx, s[C].y)));
      }
      if constexpr (R == 0) {
        s[C].x = fma(T(8), px, fma(T(14), qx, s[C].x));
        s[C].y = fma(T(8), py, fma(T(14), qy, s[C].y));
        s[2 + C] = V2<T>{(T)fma(T(2), px, fma(T(-8), qx, T(4) * gy)), (T)fma(T(2), py, fma(T(-8), qy, T(4) * gx))};
      }
      if constexpr (R == 1) {
        s[2 + C].x = fma(T(16), px + qx, s[2 + C].x);
        s[2 + C].y = fma(T(16), py + qy, s[2 + C].y);
      }
      if constexpr (R == 2) {
        s[2 + C].x = fma(T(2), px, fma(T(-8), qx, fma(T(-4), gy, s[2 + C].x)));
        s[2 + C].y = fma(T(2), py, fma(T(-8), qy, fma(T(-4), gx, s[2 + C].y)));
      }
    };
    col(std::integral_constant<int, 0>{});
    col(std::integral_constant<int, 1>{});
    __builtin_amdgcn_sched_barrier(0);   // row by row: the window is never live as a whole
  };
  row(std::integral_constant<int, -2>{});
  row(std::integral_constant<int, -1>{});
  row(std::integral_constant<int, 0>{});
  row(std::integral_constant<int, 1>{});
  row(std::integral_constant<int, 2>{});
#pragma unroll
  for (int q = 0; q < 4; ++q) asm volatile("" : "+v"(s[q].x), "+v"(s[q].y));   // the sums stay in this order
}

// z = D^{-1} r at node q of a cell (the diagonal blocks are diagonal)
template <typename T>
__device__ __forceinline__ V2<T> cell_dinv(const Q2Coef<T> &c, int q, V2<T> r) {
  const T dx = q == 0 ? c.dv : q == 1 ? c.d1 : q == 2 ? c.d2 : c.dc;
  const T dy = q == 0 ? c.dv : q == 1 ? c.d2 : q == 2 ? c.d1 : c.dc;
  return V2<T>{dx * r.x, dy * r.y};
}

template <typename T>
struct TransferOf<Q2Coef<T>> {
  static constexpr double at(int A, int B, int a, int b) { return q2_prolong_weight(A, B, a, b); }
};

// Host: the coefficients on an n x n grid, checked against the class stencils (q2.hip)
void q2_coefs(int n, double nu, double rdt, Q2Coef<double> &c64, Q2Coef<float> &c32);

}  // namespace fsi
