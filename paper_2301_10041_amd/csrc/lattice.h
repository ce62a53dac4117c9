// Matrix-free pieces of the two multigrid hierarchies on the structured grid: the launches of the
// pressure parts and of the velocity cycle's coarse end, and host tables of the P1 operators and of the P2
// restriction (exported to tests; the kernels hold these numbers in closed form).
#pragma once

#include "common.h"
#include "stencil.h"

namespace fsi {

// P1 lattice (n + 1)^2 with the diagonal of each cell from (i, j) to (i + 1, j + 1): a node
// couples with itself and the six nodes at these offsets.
constexpr int kP1Nbr = 7;
// offsets: self, (-1,0), (+1,0), (0,-1), (0,+1), (-1,-1), (+1,+1)

// Node classes by position: ci = 0 (i = 0), 1 (interior), 2 (i = n); the same for j;
// class = 3 cj + ci.  coef[c][k] couples a node of class c with the node at offset k
// (zero where that node is outside the lattice).  With the pin the row of node 0 is the
// identity and its column is zero (the pressure level is fixed at node 0).
struct P1Table {
  double coef[9][kP1Nbr];
  double dinv[9];
};

// P2 restriction R = P^T: for each class of coarse node (bit 0 = Ic odd, bit 1 = Jc odd),
// the fine nodes (offsets from the fine node 2 Ic, 2 Jc) whose interpolated value uses the
// coarse node, with the coarse basis function's value there as weight.
constexpr int kRestrMax = 81;
struct P2RestrTable {
  int count[4];
  int off[4][kRestrMax][2];
  double w[4][kRestrMax];
};

// Lattice offsets (units h/2 from the cell's lower-left node) of the six P2 nodes of
// triangle t of a cell: T0 = (v00, v10, v11), T1 = (v00, v11, v01); vertices a, b, c
// then edge midpoints ab, bc, ca.
__host__ __device__ inline void p2_node_offset(int t, int b, int &dI, int &dJ) {
  const int vx[2][3] = {{0, 2, 2}, {0, 2, 0}};
  const int vy[2][3] = {{0, 0, 2}, {0, 2, 2}};
  if (b < 3) {
    dI = vx[t][b];
    dJ = vy[t][b];
  } else {
    const int p = b - 3, q = (p + 1) % 3;
    dI = (vx[t][p] + vx[t][q]) / 2;
    dJ = (vy[t][p] + vy[t][q]) / 2;
  }
}

// Coarse P2 interpolation at fine lattice node (I, J) of an nf grid (coarse grid nf / 2,
// nested): the coarse triangle holding the node, its barycentric coordinates (multiples of
// 1/4) and the non-zero values of the six coarse basis functions there.  Writes the coarse
// lattice coordinates and weights of up to 6 nodes; boundary nodes are not excluded.
__host__ __device__ inline int p2_prolong_weights(int I, int J, int nf, int *Ic, int *Jc, double *w) {
  const int nc = nf / 2;
  int ci = I / 4, cj = J / 4;
  if (ci > nc - 1) ci = nc - 1;
  if (cj > nc - 1) cj = nc - 1;
  const double xi = (I - 4 * ci) * 0.25, eta = (J - 4 * cj) * 0.25;
  int t;
  double l0, l1, l2;
  if (xi >= eta) {
    t = 0; l0 = 1.0 - xi; l1 = xi - eta; l2 = eta;
  } else {
    t = 1; l0 = 1.0 - eta; l1 = xi; l2 = eta - xi;
  }
  const double phi[6] = {l0 * (2 * l0 - 1), l1 * (2 * l1 - 1), l2 * (2 * l2 - 1),
                         4 * l0 * l1,       4 * l1 * l2,       4 * l2 * l0};
  int cnt = 0;
  for (int b = 0; b < 6; ++b) {
    if (phi[b] == 0.0) continue;
    int dI, dJ;
    p2_node_offset(t, b, dI, dJ);
    Ic[cnt] = 2 * ci + dI;
    Jc[cnt] = 2 * cj + dJ;
    w[cnt] = phi[b];
    ++cnt;
  }
  return cnt;
}

// Host table builders (which: kTableMp = pressure mass, kTableLp = pressure Laplacian)
constexpr int kTableMp = 216, kTableLp = 225;   // offsets of the P1 blocks in the element tables
void p1_tables(int n, int which, int pin, P1Table &t);   // assemble.hip
void p2_restrict_tables(P2RestrTable &t);                // lattice.hip

// Launchers (stream-ordered, no synchronisation) over K independent systems (lane =
// blockIdx.y; each vector is a per-lane view, K = 1 for one system).

// The pressure part of the A11 preconditioner (pressure.hip).  L_p V-cycle with two Chebyshev steps
// before and after the coarse correction; s, c1, c2: the coefficients of p1_cheb_coefs.
// Descent of a level of n cells (even): x = the steps from zero for right-hand side b (of type TB,
// rounded to T; b[0] read as 0), bc = R (b - L_p x).  Lane strides lb, lx, lc.
template <typename T, typename TB>
struct P1DownArgs {
  int n;
  const TB *b;
  T *x, *bc;
  T s, c1, c2;
  int64_t lb, lx, lc;
};
template <typename T, typename TB>
void p1_down(const P1DownArgs<T, TB> &a, hipStream_t s, int K);
// Ascent: y = the steps from x + P xc (P1_Y); on the finest level z = nu M_p^{-1} b + rdt y with the
// pinned entry z[0] = b[0] rounded through T, the mass solve from zero (scale ms[0], steps m1, m2; mdinv
// = 12 / h^2, munit = h^2 / 12), and per tile the part of sum b z at
// part, if given (P1_Z; p1_up_tiles(n) parts per lane); the same with y read from xc (P1_ZW).  Lane
// strides: lb for b, lx for x and y, lc for xc, lz for z, lp for part.
enum { P1_Y = 0, P1_Z = 1, P1_ZW = 2 };
template <typename T, typename TB>
struct P1UpArgs {
  int n;
  const TB *b;
  const T *x, *xc;
  T *y;
  T c1[2], c2[2];
  double *z;
  T ms[1], m1[2], m2[2], mdinv, munit, nu, rdt;
  double *part;
  int64_t lb, lx, lc, lz, lp;
};
template <typename T, typename TB, int OUT>
void p1_up(const P1UpArgs<T, TB> &a, hipStream_t s, int K);
int p1_up_tiles(int n);
// The coarse end in one launch per system: levels lv[0..nlev) (n <= kPTailMaxN cells, each the next
// one's fine level) and the coarsest level's dense inverse cinv (m x m).  LDS (offsets in T): level
// l's two buffers at lv[l].off ((n + 3)^2 each), its right-hand side at lv[l].offb (l > 0), the
// second buffer of the mass solve at offw (OUT), all zeroed up to offz; the coarsest b and x at
// offc (m each), its inverse at offm when it fits (else -1: read from device memory); lds = the
// total.  Result: x, or with OUT (lv[0] the finest level) z and one part of sum r z as p1_up's.
constexpr int kPTailMax = 6, kPTailMaxN = 64, kPTailPer = 5, kPTailDenseMax = 6 * 64;
template <typename T>
struct PTailLevel {
  int n, off, offb;
  T c1[2], c2[2];
};
template <typename T, typename TB>
struct PTailArgs {
  int nlev;
  PTailLevel<T> lv[kPTailMax];
  int offc, offm, offw, offz, m, lds;
  const T *cinv;
  const TB *b;
  T *x;
  double *z;
  T ms, m1[2], m2[2], mdinv, munit, nu, rdt;
  double *part;
  int64_t lb, lx, lz, lp;
};
template <typename T, typename TB, bool OUT>
void p1_tail(const PTailArgs<T, TB> &a, hipStream_t s, int K);
int p1_tail_lds_limit();

// The paper's pair (qpressure.hip): descent and ascent of a level of its pressure cycle (n even).  down:
// x = s D^{-1} b and the step (c1, c2), bc = P^T (b - L x).  up: x + P xc, a step with c1 = 0 (s) and the step
// (c1, c2) into y, or with z the output z = nu mpinv b + rdt of that (z[0] = b[0] rounded through T).
template <typename T, typename TB>
struct QpDownArgs {
  int n;
  const TB *b;
  T *x, *bc;
  T s, c1, c2;
};
template <typename T, typename TB>
void qp_down(const QpDownArgs<T, TB> &a, hipStream_t s);
template <typename T, typename TB>
struct QpUpArgs {
  int n;
  const TB *b;
  const T *x, *xc;
  T *y;
  TB *z;
  const T *mpinv;
  T s, c1, c2, nu, rdt;
  double *part;   // with z: per block (qp_up_tiles(n)) the part of sum b z, or null
};
template <typename T, typename TB>
void qp_up(const QpUpArgs<T, TB> &a, hipStream_t s);
int qp_up_tiles(int n);

// The coarse end of a velocity V-cycle in one launch per system (mgtail.hip): levels
// lv[0..nlev) (n <= kTailMaxN cells, each the next one's fine level) and the coarsest
// level's dense inverse cinv (m x m, symmetric).  LDS: two buffers of kTailLevelV2 nodes per
// level, the right-hand sides (two nodes per thread and level), the coarsest b and x (m each)
// and, at byte offp, the partial sums of the dense solve in FP64; lds = the total in bytes.  b and x
// in device memory: the first level's right-hand side and result (lane stride lb).
constexpr int kTailMax = 3, kTailSteps = 3, kTailMaxN = 16, kTailDenseMax = 6 * 64;
constexpr int kTailDenseReg = 54;   // entries of the dense inverse that a thread keeps in registers
constexpr int kTailLevelV2 = 2 * (2 * kTailMaxN + 5) * (kTailMaxN + 3);
// Largest LDS block of the tail launch on the current device (queried once, at most 160 KiB).
int tail_lds_limit();
template <typename T>
struct TailLevel {
  int n;
  AfCoef<T> cf;
  T s;                                     // 1 / theta: the first step of both smoothings
  T c1[kTailSteps - 1], c2[kTailSteps - 1];   // the later Chebyshev steps
};
template <typename T>
struct TailArgs {
  int nlev;
  TailLevel<T> lv[kTailMax];
  int offp, m, lds;
  const T *cinv;
  const T *b;
  T *x;
  int64_t lb;
};
template <typename T>
void mg_tail(const TailArgs<T> &a, hipStream_t s, int K = 1);
// bc = R (b - A_f x) in one launch (stencil.hip): the residual lives only in LDS
template <typename T, typename C>
void resid_restrict(int nf, const C &cf, LP<const T> x, LP<const T> b, LP<T> bc, hipStream_t s, int K = 1);

}  // namespace fsi
