// A_f = (rho/dt) M_f + K_f on the uniform triangulated grid, cell by cell.
//
// The rows of A_f at the four nodes of a cell (i, j), the vertex (2i, 2j), the edge nodes
// (2i + 1, 2j) and (2i, 2j + 1) and the diagonal node (2i + 1, 2j + 1), together read the 19
// nodes that the vertex row alone reads, so one thread per cell reads 19 node values for four
// rows (a thread per node reads 19 + 9 + 9 + 9).  Opposite neighbours carry the same
// coefficient, so every pair is added before it is multiplied, and all the coefficients are
// multiples of nu (K_f) and of (rho/dt) h^2 (M_f): 14 values in all, which the kernels hold in
// scalar registers for their whole life instead of loading about 150 of them in every pass.
#pragma once

#include "common.h"

namespace fsi {

template <typename T>
struct alignas(2 * sizeof(T)) V2 {   // both velocity components of a node
  T x, y;
};
template <typename T>
struct NodePair {   // two neighbouring nodes of one component in device memory (aligned to T)
  T a, b;
};

// The distinct entries of A_f and of the inverses of its diagonal blocks.  With M = (rho/dt)
// h^2 / 720:
//   cv, ce     diagonal entries of vertex and edge rows (3 nu + 72 M, 4 nu + 128 M)
//   k2 .. k32  nu / 24 times 2, 8, 12, 16, 32
//   v2p, v2n   vertex to vertex along and across the component (8 nu / 24 - 4 M, 4 nu / 24 - 4 M)
//   e1p, e1n   edge to edge along and across the component (-32 nu / 24 + 32 M, -16 nu / 24 + 32 M)
//   m4, m8, m32  -4 M, -8 M, 32 M
//   dvd, dvo, ded, deo  the inverse 2x2 diagonal blocks of vertex and edge rows (diagonal, off)
template <typename T>
struct AfCoef {
  T cv, ce, k2, k8, k12, k16, k32, v2p, v2n, e1p, e1n, m4, m8, m32;
  T dvd, dvo, ded, deo;
};

// rows of A_f times x at the four nodes of the cell whose vertex is *p, in a staged array of two
// planes of even and odd lattice columns (plane stride PL, row stride HW): x (the four values
// themselves) and s (the products), in the order vertex, (1, 0), (0, 1), (1, 1).  PART 1: only the
// vertex and (1, 0) (all 19 nodes); PART 2: only (0, 1) and (1, 1) (12 nodes); the other entries of
// x and s are left alone.  DIV: also *div = 6 / h times the row of B at the cell's P1 vertex times x
// (B_q = int q div u: its entries are 0, +-h/6 and +-h/3, none of them at vertices).
enum { CELL_ALL = 0, CELL_ROW0 = 1, CELL_ROW1 = 2 };
template <typename T, int PL, int HW, int PART = CELL_ALL, bool DIV = false>
__device__ __forceinline__ void cell_products(const V2<T> *p, const AfCoef<T> &c, V2<T> (&x)[4], V2<T> (&s)[4],
                                              T *div = nullptr) {
  static_assert(!DIV || PART == CELL_ALL, "the B row needs all the edge nodes");
  constexpr bool R0 = PART != CELL_ROW1, R1 = PART != CELL_ROW0;
  auto W = [&](int dI, int dJ) -> V2<T> { return p[(dI & 1) * PL + dJ * HW + (dI >> 1)]; };
  auto add = [](V2<T> a, V2<T> b) -> V2<T> { return V2<T>{a.x + b.x, a.y + b.y}; };
  // The window comes in four groups, each read one group ahead of its use, and the vertex row's
  // pairs are formed as their members arrive: about 100 registers are live in FP64.  Left to
  // itself the compiler reads all 19 nodes first and spills beside b and d (128 registers at four
  // waves per SIMD).
  auto hold = [] { __builtin_amdgcn_sched_barrier(0); };
  const V2<T> o = W(0, 0), e = W(1, 0), f = W(0, 1), g = W(1, 1);
  const V2<T> n22 = W(2, 2), n20 = W(2, 0), n02 = W(0, 2), n12 = W(1, 2), n21 = W(2, 1);
  V2<T> l0m2, l0m1, l1m1;
  if constexpr (R0) {
    l0m2 = W(0, -2);
    l0m1 = W(0, -1);
    l1m1 = W(1, -1);
  }
  hold();
  if constexpr (R1) {   // (1, 1): neighbours inside the cell
    const V2<T> p10 = add(f, n21), p01 = add(e, n12), q = add(n20, n02), d = add(o, n22);
    const T cx = p10.x + p01.x - d.x, cy = p10.y + p01.y - d.y;
    x[2] = f;
    x[3] = g;
    s[3].x = fma(c.k8, cy, fma(-c.k16, g.y, fma(c.m8, q.x, fma(c.e1n, p01.x, fma(c.e1p, p10.x, c.ce * g.x)))));
    s[3].y = fma(c.k8, cx, fma(-c.k16, g.x, fma(c.m8, q.y, fma(c.e1p, p01.y, fma(c.e1n, p10.y, c.ce * g.y)))));
  }
  const V2<T> lm20 = W(-2, 0), lm10 = W(-1, 0), lm11 = W(-1, 1);
  hold();
  V2<T> v1, v2, six;
  if constexpr (DIV)
    *div = 2 * (e.x - lm10.x + f.y - l0m1.y) + (l0m1.x - f.x) + (lm10.y - e.y) + (l1m1.x - lm11.x) + (lm11.y - l1m1.y) +
           (g.x + g.y) + n21.x + n12.y;
  if constexpr (R0) {   // (1, 0)
    const V2<T> p10 = add(o, n20), p01 = add(l1m1, g), p11 = add(l0m1, n21), p12 = add(l0m2, n22);
    const T cx = p10.x + p01.x - p11.x, cy = p10.y + p01.y - p11.y;
    x[0] = o;
    x[1] = e;
    s[1].x = fma(c.k8, cy, fma(-c.k16, e.y, fma(c.m8, p12.x, fma(c.m32, p11.x, fma(c.e1n, p01.x, fma(-c.k32, p10.x, c.ce * e.x))))));
    s[1].y = fma(c.k8, cx, fma(-c.k16, e.x, fma(c.m8, p12.y, fma(c.m32, p11.y, fma(c.e1p, p01.y, fma(-c.k16, p10.y, c.ce * e.y))))));
    v1 = add(l0m1, f);
    v2 = add(l0m2, n02);
    six = add(add(n12, n21), l1m1);
  }
  V2<T> lm1m1, lm2m2, lm1m2, lm2m1;
  if constexpr (R0) {
    lm1m1 = W(-1, -1);
    lm2m2 = W(-2, -2);
    lm1m2 = W(-1, -2);
    lm2m1 = W(-2, -1);
  }
  hold();
  if constexpr (R1) {   // (0, 1)
    const V2<T> p10 = add(lm11, g), p01 = add(o, n02), p11 = add(lm10, n12), p21 = add(lm20, n22);
    const T cx = p10.x + p01.x - p11.x, cy = p10.y + p01.y - p11.y;
    s[2].x = fma(c.k8, cy, fma(-c.k16, f.y, fma(c.m8, p21.x, fma(c.m32, p11.x, fma(-c.k16, p01.x, fma(c.e1p, p10.x, c.ce * f.x))))));
    s[2].y = fma(c.k8, cx, fma(-c.k16, f.x, fma(c.m8, p21.y, fma(c.m32, p11.y, fma(-c.k32, p01.y, fma(c.e1n, p10.y, c.ce * f.y))))));
  }
  if constexpr (DIV) *div -= (lm1m1.x + lm1m1.y) + lm2m1.x + lm1m2.y;
  if constexpr (R0) {   // (0, 0)
    const V2<T> h1 = add(lm10, e), h2 = add(lm20, n20), d1 = add(lm1m1, g), d2 = add(lm2m2, n22);
    six = add(six, add(add(lm1m2, lm2m1), lm11));
    const T ax = h1.x + v1.x - d1.x, ay = h1.y + v1.y - d1.y, bx = h2.x + v2.x - d2.x, by = h2.y + v2.y - d2.y;
    s[0].x = fma(c.k8, ay, fma(-c.k2, by, fma(-c.k12, o.y, fma(c.m4, d2.x, fma(c.m8, six.x, fma(c.v2n, v2.x,
             fma(c.v2p, h2.x, fma(-c.k16, v1.x, fma(-c.k32, h1.x, c.cv * o.x)))))))));
    s[0].y = fma(c.k8, ax, fma(-c.k2, bx, fma(-c.k12, o.x, fma(c.m4, d2.y, fma(c.m8, six.y, fma(c.v2p, v2.y,
             fma(c.v2n, h2.y, fma(-c.k32, v1.y, fma(-c.k16, h1.y, c.cv * o.y)))))))));
  }
  // the sums stay here: a caller that selects by node would have them moved into its branches,
  // out of the order above
#pragma unroll
  for (int q = R0 ? 0 : 2; q < (R1 ? 4 : 2); ++q) asm volatile("" : "+v"(s[q].x), "+v"(s[q].y));
}

// z = D^{-1} r at node q of a cell (0: vertex, else an edge node)
template <typename T>
__device__ __forceinline__ V2<T> cell_dinv(const AfCoef<T> &c, int q, V2<T> r) {
  const T d = q == 0 ? c.dvd : c.ded, o = q == 0 ? c.dvo : c.deo;
  return V2<T>{fma(o, r.y, d * r.x), fma(d, r.y, o * r.x)};
}

// The coefficients as values of their own in scalar registers: used straight from the kernel
// arguments they may be loaded again in every pass, a scalar-cache round trip each time
template <typename T>
__device__ __forceinline__ AfCoef<T> pinned_coefs(const AfCoef<T> &c) {
  AfCoef<T> r = c;
  T *const v[18] = {&r.cv,  &r.ce,  &r.k2, &r.k8, &r.k12, &r.k16, &r.k32, &r.v2p, &r.v2n,
                    &r.e1p, &r.e1n, &r.m4, &r.m8, &r.m32, &r.dvd, &r.dvo, &r.ded, &r.deo};
#pragma unroll
  for (int i = 0; i < 18; ++i) asm volatile("" : "+s"(*v[i]));
  return r;
}

// Which of the cell's four nodes are interior: not on the Dirichlet boundary and in the lattice
struct CellIn {
  bool q[4];
};
__device__ __forceinline__ CellIn cell_inside(int i, int j, int n) {
  const bool vx = i > 0 && i < n, vy = j > 0 && j < n, ex = i >= 0 && i < n, ey = j >= 0 && j < n;
  return CellIn{{vx && vy, ex && vy, vx && ey, ex && ey}};
}

// Interpolation weight of the coarse P2 node (a, b) (0 .. 2 from the coarse cell's corner) at
// the fine node (A, B) (0 .. 3): the P2 basis of the cell's lower-right (A >= B) or upper-left
// triangle at (A / 4, B / 4)
__host__ __device__ constexpr double prolong_weight(int A, int B, int a, int b) {
  const double xi = 0.25 * A, eta = 0.25 * B;
  const bool lo = A >= B;
  const double l0 = lo ? 1 - xi : 1 - eta, l1 = lo ? xi - eta : xi, l2 = lo ? eta : eta - xi;
  // vertices 0, 1, 2 of the triangle: (0, 0), (2, 0) or (2, 2), (2, 2) or (0, 2)
  if (a == 0 && b == 0) return l0 * (2 * l0 - 1);
  if (lo) {
    if (a == 2 && b == 0) return l1 * (2 * l1 - 1);
    if (a == 2 && b == 2) return l2 * (2 * l2 - 1);
    if (a == 1 && b == 0) return 4 * l0 * l1;
    if (a == 2 && b == 1) return 4 * l1 * l2;
    if (a == 1 && b == 1) return 4 * l2 * l0;
  } else {
    if (a == 2 && b == 2) return l1 * (2 * l1 - 1);
    if (a == 0 && b == 2) return l2 * (2 * l2 - 1);
    if (a == 1 && b == 1) return 4 * l0 * l1;
    if (a == 1 && b == 2) return 4 * l1 * l2;
    if (a == 0 && b == 1) return 4 * l2 * l0;
  }
  return 0.0;
}

// The interpolation weights that belong to a level's coefficients: here the triangle pair's
template <typename C>
struct TransferOf {
  static constexpr double at(int A, int B, int a, int b) { return prolong_weight(A, B, a, b); }
};

// the coarse quadratic at fine node (A, B) of a coarse cell from its nine nodes c[3 b + a]
template <typename C, int A, int B, typename T>
__device__ __forceinline__ V2<T> prolong_node(const V2<T> (&c)[9]) {
  V2<T> s{T(0), T(0)};
  auto term = [&](auto q_tag) {
    constexpr int Q = decltype(q_tag)::value;
    constexpr double w = TransferOf<C>::at(A, B, Q % 3, Q / 3);
    if constexpr (w != 0.0) {
      s.x = fma(T(w), c[Q].x, s.x);
      s.y = fma(T(w), c[Q].y, s.y);
    }
  };
  term(std::integral_constant<int, 0>{});
  term(std::integral_constant<int, 1>{});
  term(std::integral_constant<int, 2>{});
  term(std::integral_constant<int, 3>{});
  term(std::integral_constant<int, 4>{});
  term(std::integral_constant<int, 5>{});
  term(std::integral_constant<int, 6>{});
  term(std::integral_constant<int, 7>{});
  term(std::integral_constant<int, 8>{});
  return s;
}

// Weight of the fine node at offset (dI, dJ) of (2 Ic, 2 Jc) in the restriction R = P^T at a
// coarse node of class (pa, pb) = (Ic mod 2, Jc mod 2): the coarse basis function there, from
// the coarse cell holding the fine node
template <typename Tr>
__host__ __device__ constexpr double restrict_weight_of(int pa, int pb, int dI, int dJ) {
  // fine position relative to the coarse cell corner of (Ic - pa, Jc - pb): 2 pa + dI
  const int X = 2 * pa + dI + 8, Y = 2 * pb + dJ + 8;   // 8: two cells over, keeps them positive
  const int ci = X / 4 - 2, cj = Y / 4 - 2;
  const int a = pa - 2 * ci, b = pb - 2 * cj;           // the coarse node in that cell
  return a < 0 || a > 2 || b < 0 || b > 2 ? 0.0 : Tr::at(X % 4, Y % 4, a, b);
}
__host__ __device__ constexpr double restrict_weight(int pa, int pb, int dI, int dJ) {
  return restrict_weight_of<TransferOf<void>>(pa, pb, dI, dJ);
}

// Host: the coefficients on an n x n grid (nu the viscosity, rdt = rho / dt), checked against
// the stencil table summed from the element matrices (assemble.hip)
void af_coefs(int n, double nu, double rdt, AfCoef<double> &c64, AfCoef<float> &c32);

}  // namespace fsi
