// Coefficient tables of the matrix-free A_f products (see stencil.hip).
#pragma once

#include "afcell.h"
#include "common.h"

namespace fsi {

constexpr int kStencilMax = 25;   // a P2 node couples with at most 19 nodes (5 x 5 window)

// Node classes: bit 0 = I odd, bit 1 = J odd (0 vertex, 1 horizontal edge, 2 vertical
// edge, 3 diagonal edge).  coef[c][k] is the 2x2 block (xx, xy, yx, yy) of A_f coupling a
// node of class c with the node at lattice offset off[c][k]; dinv[c] is the inverse of the
// diagonal block.
struct StencilTable {
  int count[4];
  int off[4][kStencilMax][2];
  double coef[4][kStencilMax][4];
  double dinv[4][4];
};

// Neighbour counts of the classes on the triangulated grid (vertex, h-edge, v-edge, diagonal).
constexpr int kStencilCount[4] = {19, 9, 9, 9};

// The neighbour offsets (dI, dJ) of each class, in the order of the tables (dJ, then dI,
// ascending).  They follow from the triangulation alone; the table builder checks them.
struct StencilOffsets {
  int d[4][kStencilMax][2];
};
__host__ __device__ constexpr StencilOffsets stencil_offsets() {
  return StencilOffsets{{
      {{-2, -2}, {-1, -2}, {0, -2}, {-2, -1}, {-1, -1}, {0, -1}, {1, -1}, {-2, 0}, {-1, 0}, {0, 0},
       {1, 0}, {2, 0}, {-1, 1}, {0, 1}, {1, 1}, {2, 1}, {0, 2}, {1, 2}, {2, 2}},
      {{-1, -2}, {-1, -1}, {0, -1}, {-1, 0}, {0, 0}, {1, 0}, {0, 1}, {1, 1}, {1, 2}},
      {{-2, -1}, {-1, -1}, {0, -1}, {-1, 0}, {0, 0}, {1, 0}, {0, 1}, {1, 1}, {2, 1}},
      {{-1, -1}, {0, -1}, {1, -1}, {-1, 0}, {0, 0}, {1, 0}, {-1, 1}, {0, 1}, {1, 1}},
  }};
}

// Entries whose cross-component couplings (xy, yx) vanish for every viscosity and time step:
// the symmetric-gradient form couples the components only through mixed derivatives, which
// integrate to zero for these neighbour pairs on the triangulated grid (the table builder
// checks that both values are exactly 0).
struct CrossZero {
  bool z[4][kStencilMax];
};
__host__ __device__ constexpr CrossZero cross_zero() {
  CrossZero c{};
  c.z[0][1] = c.z[0][3] = c.z[0][15] = c.z[0][17] = true;   // vertex: (-1,-2), (-2,-1), (2,1), (1,2)
  c.z[1][0] = c.z[1][8] = true;                              // horizontal edge: (-1,-2), (1,2)
  c.z[2][0] = c.z[2][8] = true;                              // vertical edge: (-2,-1), (2,1)
  return c;
}

// Divergence blocks on the structured grid.  B^T row of an interior P2 node of class c:
// the P1 vertices of the triangles around it (offsets from P1 node (I >> 1, J >> 1)) with
// the pair (B_x, B_y)(k, node).  B row of a P1 node (i, j): the P2 nodes of the triangles
// around it (lattice offsets from (2i, 2j)).  Rows of Dirichlet P2 nodes of B^T and the
// matching columns of B are zero; so are row 0 of B and column 0 of B^T (pinned pressure).
// Every triangle holding an interior P2 node lies in the domain, so one B row serves every
// P1 node, boundary ones included, once the Dirichlet values of x_u are read as zero.
constexpr int kBtMax = 7;
constexpr int kBMax = 19;
constexpr int kBtCount[4] = {7, 4, 4, 4};
// Entry order of both tables: by dJ, then dI (the builder sorts and checks).  B^T offsets
// are P1 lattice offsets from (I >> 1, J >> 1); B offsets are P2 lattice offsets from
// (2i, 2j), the pattern of the vertex class of A_f.
struct DivOffsets {
  int bt[4][kBtMax][2];
};
__host__ __device__ constexpr DivOffsets div_offsets() {
  return DivOffsets{{
      {{-1, -1}, {0, -1}, {-1, 0}, {0, 0}, {1, 0}, {0, 1}, {1, 1}},
      {{0, -1}, {0, 0}, {1, 0}, {1, 1}},
      {{-1, 0}, {0, 0}, {0, 1}, {1, 1}},
      {{0, 0}, {1, 0}, {0, 1}, {1, 1}},
  }};
}
struct DivTable {
  int bt_count[4];
  int bt_off[4][kBtMax][2];
  double bt_coef[4][kBtMax][2];
  int b_count;
  int b_off[kBMax][2];
  double b_coef[kBMax][2];
};

// Launchers run K independent systems (lane = blockIdx.y) over per-lane views (LP); the
// vector views of one launch share one lane stride.  K = 1: one system.

// Fluid rows of the operator on [u_x | u_y | p]:
//   y_u = A_f x_u - B^T x_p (+ C_f^T x_lam, a launch of its own, when cft_rp is given; lam_x at xl, lam_y
//   at xl + Ns)
//   y_p = -B x_u, and y_p[0] = x_p[0] (pinned node)
void a11_rows(int n, const AfCoef<double> &cf, const double *x, double *y, const int *cft_rp, const int *cft_col,
              const double *cft_val, const double *xl, int64_t Ns, hipStream_t s);

// b = [rdt M_f u | 0] on [u_x | u_y | p] (Dirichlet rows 0, Dirichlet values of u left out)
void mass_rows(int n, double rdt, const double *u, double *b, hipStream_t s);

// The three-term update of the inner MINRES, taken by pre3 while it stages its right-hand side:
// q = y1 - alfa s r2 on [u_x | u_y | p], alfa the sum of nparts parts (of stride lp per lane; stored to
// *alfa), or with nparts = 0 the value of *alfa.  y1, r2 and q have one lane stride, alfa and s another.
struct MsFold {
  LP<const double> y1, r2;
  LP<double> q;
  const double *part = nullptr;
  int nparts = 0;
  int64_t lp = 0;
  double *alfa = nullptr;
  const double *s = nullptr;
  int64_t ls = 0;
};

// Chebyshev smoothing of a velocity level, three steps per launch (C: AfCoef<T> for the triangle pair,
// Q2Coef<T> for the paper's):
// pre3 : x = s D^{-1} b, then the steps (c1a, c2a), (c1b, c2b); writes x.  With fold, b is the velocity
//        part of q; q (all three parts) is written, and for T = float also the copy b.
//        With bc (where pre3_restricts(n, K)) also bc = R (b - A_f x), as resid_restrict.
// post3: from x + P xc (xc the coarse correction of lattice n / 2) a step with c1 = 0 (c2a) and
//        the steps (c1b, c2b), (c1c, c2c); writes y (stored as TY: double or T; x is not
//        written).  With dot, tile t of lane k stores the sum over its nodes of b . y (FP64, y as
//        stored) at dot.at(k)[t] (post3_dot_count(n) tiles); with b64 the sums take that FP64
//        right-hand side in place of b (the FP32 cycle of the mixed form).
template <typename T, typename C>
void pre3(int n, const C &cf, LP<T> b, LP<T> x, T s, T c1a, T c2a, T c1b, T c2b, hipStream_t st, int K,
          const MsFold *fold = nullptr, LP<T> bc = LP<T>());
bool pre3_restricts(int n, int K);
template <typename T, typename TY, typename C>
void post3(int n, const C &cf, LP<const T> x, LP<const T> b, LP<TY> y, T c2a, T c1b, T c2b, T c1c, T c2c,
           hipStream_t st, int K, LP<const T> xc, LP<double> dot = LP<double>(),
           LP<const double> b64 = LP<const double>());
int post3_dot_count(int n);

// The A11 rows inside the inner MINRES, per lane: v = s y, then s (A11 y) + c r1 written over r1, with s
// and c of the lane's state, and one partial sum of their product per tile in part
// (a11_tile_count(n); r1 used only when c != 0).  v goes to the state's slot (clamped to [0, B - 1]) of the
// Lanczos block: vh + slot vs + lane r1.s.  nb > 0: the state is first taken one step further, from
// st with the nb parts of beta^2 at bpart to out (other memory than st), recorded in hist and told.
struct MinresState;
struct MsA11 {
  const MinresState *st = nullptr;
  MinresState *out = nullptr;
  LP<const double> bpart;
  int nb = 0;
  double *hist = nullptr;
  double *vh = nullptr;
  int64_t vs = 0;
  int B = 0;
  LP<double> part;
  unsigned long long *word = nullptr, seq = 0;
};
template <typename C>
void a11_minres(int n, const C &cf, LP<const double> y, LP<double> r1, const MsA11 &m, hipStream_t s,
                int K = 1);
int a11_tile_count(int n);

// Host: the tables of A_f on an n x n grid from the element matrices (assemble.hip).
void stencil_tables(int n, double nu, double rdt, StencilTable &t);
void div_tables(int n, DivTable &t);
void check_div_closed_form(int n);   // the entries of B and B^T that the kernels are compiled with

}  // namespace fsi
