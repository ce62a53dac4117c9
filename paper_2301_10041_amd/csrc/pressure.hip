// The pressure part of the A11 preconditioner on the structured grid: the Cahouet-Chabard form
// z = nu M_p^{-1} r + (rho/dt) L_p^{-1} r (Sec. 4), with L_p^{-1} one V-cycle of the pinned P1
// Laplacian and M_p^{-1} three Chebyshev-Jacobi steps.
//
// On this triangulation a P1 node is joined by L_p to its four axis neighbours only, with weight 1,
// or 1/2 along the boundary (the diagonal edge's weight is the cotangent of a right angle, 0), and
// its diagonal entry is the sum of its weights; by M_p, in units of h^2 / 12, to all six neighbours
// with weight 1 (1/2 along the boundary), and the diagonal entry is again their sum.  So no table
// is read: a value outside the grid is kept as 0 and the weights follow from the position.  The
// pinned node 0 holds 0 in every vector of the L_p cycle (its right-hand side is 0 and its row
// the identity), which also takes out its column.
//
// Three launches serve all levels:
//   k_p1_down  right-hand side -> two smoothing steps from zero, residual, restriction
//   k_p1_tail  the levels of at most 64 x 64 cells and the dense coarsest solve, one block
//              (from the finest level on: the mass solve and the output too)
//   k_p1_up    coarse correction, two smoothing steps; on the finest level the mass solve and the
//              output z with the parts of r . z
// The part runs beside the velocity cycle and is a chain of small dependent launches: bound by
// latency below 256^2 and by the launches themselves.  As one launch per step and transfer, with
// tables of coefficients read per node, it took 14 launches and 150 us per application at 256^2
// (FP32) and 24 launches at 1024^2; now 5 (33 us) and 9.  The coarse end alone: 44 -> 16 us from
// 64^2 (FP32), and 28 us plus 19 for the copies, the mass solve and the output -> 12 us with all of
// it at 32^2 (FP64).
#include <cmath>

#include "ctx.h"
#include "kernels.h"
#include "lattice.h"

namespace fsi {

namespace {

// Edge weights at grid position (i, j) of an n x n grid: along x on row j, along y on column i
struct P1Weights {
  bool in;          // the node exists
  bool pin;         // the pinned node
  bool wx, wy;      // half weight along x / y (the node lies on a horizontal / vertical wall)
  int i, j, n;
};
__device__ __forceinline__ P1Weights p1_weights(int i, int j, int n) {
  return P1Weights{i >= 0 && j >= 0 && i <= n && j <= n, i == 0 && j == 0, j == 0 || j == n, i == 0 || i == n, i, j, n};
}
// diagonal of L_p (4 inside, 2 on a wall, 1 in a corner) and its inverse
template <typename T>
__device__ __forceinline__ T lp_diag(const P1Weights &w) {
  return T(w.wx && w.wy ? 1 : w.wx || w.wy ? 2 : 4);
}
template <typename T>
__device__ __forceinline__ T lp_dinv(const P1Weights &w) {
  return w.wx && w.wy ? T(1) : w.wx || w.wy ? T(0.5) : T(0.25);
}
// (L_p x) at a node from its own value and its four axis neighbours (0 outside the grid)
template <typename T>
__device__ __forceinline__ T lp_apply(const P1Weights &w, T c, T l, T r, T d, T u) {
  const T hx = l + r, vy = d + u;
  return lp_diag<T>(w) * c - (w.wx ? T(0.5) * hx : hx) - (w.wy ? T(0.5) * vy : vy);
}
// The diagonal of M_p in units of h^2 / 12: the number of triangles around the node
__device__ __forceinline__ int mp_count(const P1Weights &w) {
  if (w.wx && w.wy) return (w.i == 0) == (w.j == 0) ? 2 : 1;   // the diagonal runs through two corners
  return w.wx || w.wy ? 3 : 6;
}
template <typename T>
__device__ __forceinline__ T mp_inv(const P1Weights &w) {   // 1 / mp_count
  const int c = mp_count(w);
  return c == 6 ? T(1.0 / 6.0) : c == 3 ? T(1.0 / 3.0) : c == 2 ? T(0.5) : T(1);
}
// (M_p x) in units of h^2 / 12; a, b: the diagonal neighbours (-1, -1) and (1, 1)
template <typename T>
__device__ __forceinline__ T mp_apply(const P1Weights &w, T c, T l, T r, T d, T u, T a, T b) {
  const T hx = l + r, vy = d + u;
  return T(mp_count(w)) * c + (w.wx ? T(0.5) * hx : hx) + (w.wy ? T(0.5) * vy : vy) + (a + b);
}

// Regions of the launches: 8 waves, wave w owns RPT consecutive rows of 64 columns (lane = column)
constexpr int kP1Waves = 8, kP1S = kWave + 2;   // row stride in LDS (a column of zeros on each side)

// linear interpolation at fine node (i, j) from the coarse lattice (side Lc)
template <typename T>
__device__ __forceinline__ T p1_interp(const T *xc, int Lc, int i, int j) {
  const int64_t k = (int64_t)(j >> 1) * Lc + (i >> 1);
  const T v = xc[k];
  if (!(i & 1) && !(j & 1)) return v;
  return T(0.5) * v + T(0.5) * xc[k + ((j & 1) ? Lc : 0) + (i & 1)];
}

}  // namespace

// ---------------------------------------------------------------- descent
// x = two Chebyshev steps from zero for L_p x = b, bc = R (b - L_p x): tile of 29 x CR coarse nodes
// (58 x 2 CR fine ones), b and the first step on the tile with a halo of 3, the second step 2, the
// residual 1.
constexpr int kDownC = (kWave - 5) / 2;
template <typename T, typename TB, int RPT>
__global__ void __launch_bounds__(kWave *kP1Waves) k_p1_down(P1DownArgs<T, TB> a, int tiles_x) {
  constexpr int RH = kP1Waves * RPT, CR = (RH - 5) / 2;
  __shared__ T XA[(RH + 2) * kP1S], XB[(RH + 2) * kP1S];
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave, ln = blockIdx.y, n = a.n, L = n + 1, Lc = n / 2 + 1;
  const TB *b = a.b + ln * a.lb;
  const int C0 = (blockIdx.x % tiles_x) * kDownC, R0 = (blockIdx.x / tiles_x) * CR;
  const int i = 2 * C0 - 3 + lane, jb = 2 * R0 - 3 + w * RPT;   // the thread's column and first row
  T bv[RPT], dv[RPT], xv[RPT];
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const P1Weights wt = p1_weights(i, jb + q, n);
    bv[q] = wt.in && !wt.pin ? (T)b[(int64_t)(jb + q) * L + i] : T(0);
  }
  T *const pa = XA + (w * RPT + 1) * kP1S + lane + 1, *const pb = XB + (w * RPT + 1) * kP1S + lane + 1;
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    dv[q] = a.s * (lp_dinv<T>(p1_weights(i, jb + q, n)) * bv[q]);
    pa[q * kP1S] = dv[q];
  }
  __syncthreads();
  // The rows just above and below the region and the columns beside it are never written; what is
  // computed from them lies outside the halo that the next pass needs.
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const P1Weights wt = p1_weights(i, jb + q, n);
    const T *p = pa + q * kP1S;
    const T s = lp_apply<T>(wt, p[0], p[-1], p[1], p[-kP1S], p[kP1S]);
    xv[q] = wt.in && !wt.pin ? dv[q] + (a.c1 * dv[q] + a.c2 * (lp_dinv<T>(wt) * (bv[q] - s))) : T(0);
    pb[q * kP1S] = xv[q];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const P1Weights wt = p1_weights(i, jb + q, n);
    const T *p = pb + q * kP1S;
    const T s = lp_apply<T>(wt, p[0], p[-1], p[1], p[-kP1S], p[kP1S]);
    pa[q * kP1S] = wt.in && !wt.pin ? bv[q] - s : T(0);
    const int rr = w * RPT + q;   // the tile's nodes
    if (wt.in && lane >= 3 && lane < 3 + 2 * kDownC && rr >= 3 && rr < 3 + 2 * CR)
      a.x[ln * a.lx + (int64_t)(jb + q) * L + i] = xv[q];
  }
  __syncthreads();
  // a coarse node collects the fine node on it and, with weight 1/2, the six edge midpoints around
  // it; lanes 0-28 and 32-60 of a wave take two coarse rows
  static_assert(CR <= 2 * kP1Waves && kDownC <= 32, "one pass over the coarse nodes");
  const int k = lane & 31, kr = 2 * w + (lane >> 5), Ic = C0 + k, Jc = R0 + kr;
  if (k < kDownC && kr < CR && Ic < Lc && Jc < Lc) {
    const T *p = XA + (2 * kr + 4) * kP1S + 2 * k + 4;
    const T edges = p[-1] + p[1] + p[-kP1S] + p[kP1S] + p[kP1S + 1] + p[-kP1S - 1];
    a.bc[ln * a.lc + (int64_t)Jc * Lc + Ic] = Ic == 0 && Jc == 0 ? T(0) : p[0] + T(0.5) * edges;
  }
}

// ---------------------------------------------------------------- ascent and output
// y = two Chebyshev steps from x + P xc (OUT = P1_Y), or z = nu M_p^{-1} r + (rho/dt) y with the
// mass solve's three steps from zero, the pinned entry r[0] and the tile's part of sum r z
// (OUT = P1_Z; P1_ZW: y is read from xc instead, the whole L_p cycle having run elsewhere).  Tile of
// 60 x (RH - 4) nodes; the values they start from with a halo of 2, the first step 1.
template <typename T, typename TB, int RPT, int OUT>
__global__ void __launch_bounds__(kWave *kP1Waves) k_p1_up(P1UpArgs<T, TB> a, int tiles_x) {
  constexpr int RH = kP1Waves * RPT, TR = RH - 4, TC = kWave - 4, NE = (RH + 2) * kP1S;
  constexpr bool UP = OUT != P1_ZW, MASS = OUT != P1_Y;
  __shared__ T XA[UP ? NE : 1], XB[UP ? NE : 1], MA[MASS ? NE : 1], MB[MASS ? NE : 1];
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave, ln = blockIdx.y, n = a.n, L = n + 1, Lc = n / 2 + 1;
  const TB *b = a.b + ln * a.lb;
  const int i = (blockIdx.x % tiles_x) * TC - 2 + lane, jb = (blockIdx.x / tiles_x) * TR - 2 + w * RPT;
  const int o = (w * RPT + 1) * kP1S + lane + 1;
  T bv[RPT], dv[RPT], xv[RPT], md[RPT], mv[RPT];
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const P1Weights wt = p1_weights(i, jb + q, n);
    const int64_t r = (int64_t)(jb + q) * L + i;
    bv[q] = wt.in && !wt.pin ? (T)b[r] : T(0);
    if constexpr (UP) {
      xv[q] = wt.in && !wt.pin ? a.x[ln * a.lx + r] + p1_interp(a.xc + ln * a.lc, Lc, i, jb + q) : T(0);
      XA[o + q * kP1S] = xv[q];
    }
    if constexpr (MASS) {
      mv[q] = md[q] = wt.in ? a.ms[0] * (a.mdinv * mp_inv<T>(wt) * bv[q]) : T(0);
      MA[o + q * kP1S] = mv[q];
    }
  }
  __syncthreads();
  auto step = [&](const T *X, const T *M, T c1, T c2, T m1, T m2, bool first) {
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
      const P1Weights wt = p1_weights(i, jb + q, n);
      if constexpr (UP) {
        const T *p = X + o + q * kP1S;
        const T s = lp_apply<T>(wt, p[0], p[-1], p[1], p[-kP1S], p[kP1S]);
        const T z = lp_dinv<T>(wt) * (bv[q] - s);
        dv[q] = first ? c2 * z : c1 * dv[q] + c2 * z;
        xv[q] = wt.in && !wt.pin ? xv[q] + dv[q] : T(0);
      }
      if constexpr (MASS) {
        const T *p = M + o + q * kP1S;
        const T s = mp_apply<T>(wt, p[0], p[-1], p[1], p[-kP1S], p[kP1S], p[-kP1S - 1], p[kP1S + 1]);
        md[q] = m1 * md[q] + m2 * (a.mdinv * mp_inv<T>(wt) * (bv[q] - a.munit * s));
        mv[q] = wt.in ? mv[q] + md[q] : T(0);
      }
    }
  };
  step(XA, MA, T(0), a.c2[0], a.m1[0], a.m2[0], true);
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    if constexpr (UP) XB[o + q * kP1S] = xv[q];
    if constexpr (MASS) MB[o + q * kP1S] = mv[q];
  }
  __syncthreads();
  step(XB, MB, a.c1[1], a.c2[1], a.m1[1], a.m2[1], false);
  double acc = 0.0;
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const int rr = w * RPT + q, j = jb + q;
    if (lane < 2 || lane >= 2 + TC || rr < 2 || rr >= 2 + TR || i > n || j > n) continue;
    const int64_t r = (int64_t)j * L + i;
    if constexpr (OUT == P1_Y) {
      a.y[ln * a.lx + r] = xv[q];
    } else {
      T y;
      if constexpr (UP) y = xv[q];
      else y = a.xc[ln * a.lc + r];
      const double rv = b[r], v = r == 0 ? (T)rv : (a.nu * mv[q] + a.rdt * y);
      a.z[ln * a.lz + r] = v;
      acc += rv * v;
    }
  }
  if constexpr (MASS) {
    if (a.part) {   // uniform; the tile's sum in a fixed order
      __shared__ double red[kP1Waves];
      const double t = wave_sum(acc);
      if (lane == 0) red[w] = t;
      __syncthreads();
      if (threadIdx.x == 0) {
        double s = 0.0;
        for (int k = 0; k < kP1Waves; ++k) s += red[k];
        a.part[ln * a.lp + blockIdx.x] = s;
      }
    }
  }
}

// ---------------------------------------------------------------- coarse end
// One 1024-thread block per system runs the levels of at most kPTailMaxN cells with every vector in
// LDS.  A level's iterate lies in two buffers with a border of zeros, row stride n + 3; node
// k of a level (row-major) belongs to thread k mod 1024 in every pass, which keeps its right-hand
// side and direction in registers, so a pass is four LDS reads per node and one barrier.  With OUT
// the first level is the finest: the block reads r, adds the mass solve and writes z with the sum of
// r z.
constexpr int kPTailThreads = 1024;
template <typename T, typename TB, bool OUT>
__global__ void __launch_bounds__(kPTailThreads) k_p1_tail(PTailArgs<T, TB> a) {
  extern __shared__ unsigned char ptail_smem[];
  T *const sm = reinterpret_cast<T *>(ptail_smem);
  const int tid = threadIdx.x, ln = blockIdx.y;
  const TB *bg = a.b + ln * a.lb;
  constexpr int PER = kPTailPer;
  // the node's row and column: k / L with k < 2^13 and L <= 65, exact in float
  auto coords = [&](int k, int L, int &i, int &j) {
    j = (int)(((float)k + 0.5f) * (1.0f / (float)L));
    i = k - j * L;
  };
  T b[PER], d[PER], bf[PER];
  {
    const int L = a.lv[0].n + 1, N = L * L;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int k = tid + kPTailThreads * q;
      b[q] = k < N && k > 0 ? (T)bg[k] : T(0);
      bf[q] = b[q];   // kept for the ascent and the mass solve
    }
  }
  for (int k = tid; k < a.offz; k += kPTailThreads) sm[k] = T(0);
  for (int k = tid; k < a.m * a.m && a.offm >= 0; k += kPTailThreads) sm[a.offm + k] = a.cinv[k];
  __syncthreads();
  // one step on a level from buffer X (into Y): ZERO c1 for the first step from x
  auto step = [&](int n, const T *X, T *Y, T c1, T c2, bool first) {
    const int L = n + 1, N = L * L, S = n + 3;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int k = tid + kPTailThreads * q;
      if (k >= N) break;
      int i, j;
      coords(k, L, i, j);
      const P1Weights wt = p1_weights(i, j, n);
      const T *p = X + (j + 1) * S + i + 1;
      const T s = lp_apply<T>(wt, p[0], p[-1], p[1], p[-S], p[S]);
      const T z = lp_dinv<T>(wt) * (b[q] - s);
      d[q] = first ? c2 * z : c1 * d[q] + c2 * z;
      Y[(j + 1) * S + i + 1] = k > 0 ? p[0] + d[q] : T(0);
    }
    __syncthreads();
  };
  // descent; b holds the level's right-hand side
  for (int l = 0; l < a.nlev; ++l) {
    const int n = a.lv[l].n, L = n + 1, N = L * L, S = n + 3;
    T *X = sm + a.lv[l].off, *Y = X + S * S;
    const T s0 = a.lv[l].c2[0];
#pragma unroll
    for (int q = 0; q < PER; ++q) {   // first step from zero
      const int k = tid + kPTailThreads * q;
      if (k >= N) break;
      int i, j;
      coords(k, L, i, j);
      d[q] = s0 * (lp_dinv<T>(p1_weights(i, j, n)) * b[q]);
      X[(j + 1) * S + i + 1] = d[q];
      if (l > 0) sm[a.lv[l].offb + k] = b[q];
    }
    __syncthreads();
    step(n, X, Y, a.lv[l].c1[1], a.lv[l].c2[1], false);
#pragma unroll
    for (int q = 0; q < PER; ++q) {   // the residual over the first buffer
      const int k = tid + kPTailThreads * q;
      if (k >= N) break;
      int i, j;
      coords(k, L, i, j);
      const T *p = Y + (j + 1) * S + i + 1;
      const T s = lp_apply<T>(p1_weights(i, j, n), p[0], p[-1], p[1], p[-S], p[S]);
      X[(j + 1) * S + i + 1] = k > 0 ? b[q] - s : T(0);
    }
    __syncthreads();
    const int Lc = n / 2 + 1, Nc = Lc * Lc;
    const bool coarsest = l + 1 == a.nlev;
#pragma unroll
    for (int q = 0; q < 2; ++q) {   // restriction: the thread's nodes of the next level
      const int k = tid + kPTailThreads * q;
      if (k >= Nc) break;
      int i, j;
      coords(k, Lc, i, j);
      const T *p = X + (2 * j + 1) * S + 2 * i + 1;
      const T edges = p[-1] + p[1] + p[-S] + p[S] + p[S + 1] + p[-S - 1];
      b[q] = k > 0 ? p[0] + T(0.5) * edges : T(0);
      if (coarsest) sm[a.offc + k] = b[q];
    }
  }
  __syncthreads();
  {   // coarsest level: x = C^{-1} b, 16 lanes per row, sums in double
    const T *bc = sm + a.offc;
    T *xc = sm + a.offc + a.m;
    const T *cm = a.offm >= 0 ? sm + a.offm : a.cinv;
    const int g = tid >> 4, t = tid & 15;
    for (int r = g; r < a.m; r += kPTailThreads / 16) {
      double s = 0.0;
      for (int k = t; k < a.m; k += 16) s += (double)cm[(int64_t)r * a.m + k] * (double)bc[k];
      s = group_sum<16>(s);
      if (t == 0) xc[r] = (T)s;
    }
  }
  __syncthreads();
  // ascent
  for (int l = a.nlev - 1; l >= 0; --l) {
    const int n = a.lv[l].n, L = n + 1, N = L * L, S = n + 3, Lc = n / 2 + 1;
    T *X = sm + a.lv[l].off, *Y = X + S * S;
    const bool coarsest = l + 1 == a.nlev;
    // the coarse iterate: row-major on the coarsest level, else in the second buffer
    const int Sc = coarsest ? Lc : Lc + 2;
    const T *xc = coarsest ? sm + a.offc + a.m : sm + a.lv[l + 1].off + Sc * Sc + Sc + 1;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int k = tid + kPTailThreads * q;
      if (k >= N) break;
      int i, j;
      coords(k, L, i, j);
      b[q] = l > 0 ? sm[a.lv[l].offb + k] : bf[q];
      if (k > 0) Y[(j + 1) * S + i + 1] += p1_interp(xc, Sc, i, j);
    }
    __syncthreads();
    step(n, Y, X, T(0), a.lv[l].c2[0], true);
    step(n, X, Y, a.lv[l].c1[1], a.lv[l].c2[1], false);
  }
  const int n = a.lv[0].n, L = n + 1, N = L * L, S = n + 3;
  T *const X = sm + a.lv[0].off;
  const T *const Y = X + S * S;
  if constexpr (!OUT) {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int k = tid + kPTailThreads * q;
      if (k >= N) break;
      int i, j;
      coords(k, L, i, j);
      a.x[ln * a.lx + k] = Y[(j + 1) * S + i + 1];
    }
  } else {
    // the mass solve in two buffers of its own (the first takes the residual's place)
    T *const M0 = X, *const M1 = sm + a.offw;
    T y[PER], mv[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int k = tid + kPTailThreads * q;
      if (k >= N) break;
      int i, j;
      coords(k, L, i, j);
      y[q] = Y[(j + 1) * S + i + 1];
      mv[q] = d[q] = a.ms * (a.mdinv * mp_inv<T>(p1_weights(i, j, n)) * bf[q]);
      M0[(j + 1) * S + i + 1] = mv[q];
    }
    __syncthreads();
    auto mstep = [&](const T *M, T m1, T m2) {
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        const int k = tid + kPTailThreads * q;
        if (k >= N) break;
        int i, j;
        coords(k, L, i, j);
        const P1Weights wt = p1_weights(i, j, n);
        const T *p = M + (j + 1) * S + i + 1;
        const T s = mp_apply<T>(wt, p[0], p[-1], p[1], p[-S], p[S], p[-S - 1], p[S + 1]);
        d[q] = m1 * d[q] + m2 * (a.mdinv * mp_inv<T>(wt) * (bf[q] - a.munit * s));
        mv[q] += d[q];
      }
    };
    mstep(M0, a.m1[0], a.m2[0]);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int k = tid + kPTailThreads * q;
      if (k >= N) break;
      int i, j;
      coords(k, L, i, j);
      M1[(j + 1) * S + i + 1] = mv[q];
    }
    __syncthreads();
    mstep(M1, a.m1[1], a.m2[1]);
    double acc = 0.0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int k = tid + kPTailThreads * q;
      if (k >= N) break;
      const double rv = bg[k], v = k == 0 ? (T)rv : (a.nu * mv[q] + a.rdt * y[q]);
      a.z[ln * a.lz + k] = v;
      acc += rv * v;
    }
    if (a.part) {
      __shared__ double red[kPTailThreads / kWave];
      const double t = wave_sum(acc);
      if (tid % kWave == 0) red[tid / kWave] = t;
      __syncthreads();
      if (tid == 0) {
        double s = 0.0;
        for (int k = 0; k < kPTailThreads / kWave; ++k) s += red[k];
        a.part[ln * a.lp] = s;
      }
    }
  }
}

// ---------------------------------------------------------------- launches
// Rows per thread of the tiled launches: 4 from kP1WideN cells on (less of the halo recomputed), 2
// below, where the tiles of 4 would leave most of the chip idle
constexpr int kP1WideN = 512;

template <int RPT>
static int p1_up_tiles_r(int n, int &tx) {
  tx = (n + kWave - 4) / (kWave - 4);
  constexpr int TR = kP1Waves * RPT - 4;
  return tx * ((n + TR) / TR);
}
int p1_up_tiles(int n) {
  int tx;
  return n >= kP1WideN ? p1_up_tiles_r<4>(n, tx) : p1_up_tiles_r<2>(n, tx);
}

template <typename T, typename TB>
void p1_down(const P1DownArgs<T, TB> &a, hipStream_t s, int K) {
  FSI_REQUIRE(a.n % 2 == 0 && a.n >= 4 && K >= 1 && K <= 65535, FSI_E_ARG, "pressure level out of range");
  auto go = [&](auto r_tag) {
    constexpr int RPT = decltype(r_tag)::value, CR = (kP1Waves * RPT - 5) / 2;
    const int tx = (a.n / 2 + kDownC) / kDownC, ty = (a.n / 2 + CR) / CR;
    hipLaunchKernelGGL((k_p1_down<T, TB, RPT>), dim3((unsigned)(tx * ty), (unsigned)K), dim3(kWave * kP1Waves), 0, s,
                       a, tx);
  };
  if (a.n >= kP1WideN) go(std::integral_constant<int, 4>{});
  else go(std::integral_constant<int, 2>{});
  FSI_CHECK_LAUNCH();
}

template <typename T, typename TB, int OUT>
void p1_up(const P1UpArgs<T, TB> &a, hipStream_t s, int K) {
  FSI_REQUIRE((OUT == P1_ZW || (a.n % 2 == 0 && a.n >= 4)) && K >= 1 && K <= 65535, FSI_E_ARG,
              "pressure level out of range");
  auto go = [&](auto r_tag) {
    constexpr int RPT = decltype(r_tag)::value;
    int tx;
    const int tiles = p1_up_tiles_r<RPT>(a.n, tx);
    hipLaunchKernelGGL((k_p1_up<T, TB, RPT, OUT>), dim3((unsigned)tiles, (unsigned)K), dim3(kWave * kP1Waves), 0, s,
                       a, tx);
  };
  if (a.n >= kP1WideN) go(std::integral_constant<int, 4>{});
  else go(std::integral_constant<int, 2>{});
  FSI_CHECK_LAUNCH();
}

// LDS grant of the tail launches (device limit, at most 160 KiB), set once
int p1_tail_lds_limit() {
  static int limit = [] {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
      v = 65536;
    v = v < 65536 ? v : v > 163840 ? 163840 : v;
    if (v > 65536) {
      const void *ks[] = {(const void *)k_p1_tail<double, double, false>,
                          (const void *)k_p1_tail<float, float, false>,
                          (const void *)k_p1_tail<double, double, true>,
                          (const void *)k_p1_tail<float, double, true>};
      for (const void *k : ks)
        if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, v) != hipSuccess) {
          (void)hipGetLastError();
          v = 65536;
          break;
        }
    }
    return v;
  }();
  return limit;
}

template <typename T, typename TB, bool OUT>
void p1_tail(const PTailArgs<T, TB> &a, hipStream_t s, int K) {
  FSI_REQUIRE(a.nlev >= 1 && a.nlev <= kPTailMax, FSI_E_ARG, "pressure tail shape out of range");
  FSI_REQUIRE(a.lv[0].n <= kPTailMaxN && (a.lv[0].n + 1) * (a.lv[0].n + 1) <= kPTailPer * kPTailThreads, FSI_E_ARG,
              "pressure tail level too fine");
  for (int l = 0; l < a.nlev; ++l) {
    FSI_REQUIRE(a.lv[l].n % 2 == 0, FSI_E_ARG, "pressure tail level without a coarser one");
    FSI_REQUIRE(l + 1 == a.nlev || a.lv[l + 1].n * 2 == a.lv[l].n, FSI_E_ARG, "pressure tail levels not nested");
  }
  FSI_REQUIRE(a.m == (a.lv[a.nlev - 1].n / 2 + 1) * (a.lv[a.nlev - 1].n / 2 + 1) && a.m <= kPTailDenseMax, FSI_E_ARG,
              "pressure tail coarsest level out of range");
  FSI_REQUIRE(K >= 1 && K <= 65535 && (K == 1 || a.lb > 0), FSI_E_ARG, "lane count out of range");
  FSI_REQUIRE(a.lds * (int)sizeof(T) <= p1_tail_lds_limit(), FSI_E_ARG, "pressure tail exceeds the LDS of a block");
  hipLaunchKernelGGL((k_p1_tail<T, TB, OUT>), dim3(1, (unsigned)K), dim3(kPTailThreads), a.lds * (int)sizeof(T), s,
                     a);
  FSI_CHECK_LAUNCH();
}

#define FSI_P1_INST(T)                                                                \
  template void p1_up<T, double, P1_Z>(const P1UpArgs<T, double> &, hipStream_t, int);  \
  template void p1_up<T, double, P1_ZW>(const P1UpArgs<T, double> &, hipStream_t, int); \
  template void p1_up<T, T, P1_Y>(const P1UpArgs<T, T> &, hipStream_t, int);            \
  template void p1_tail<T, double, true>(const PTailArgs<T, double> &, hipStream_t, int); \
  template void p1_tail<T, T, false>(const PTailArgs<T, T> &, hipStream_t, int);        \
  template void p1_down<T, double>(const P1DownArgs<T, double> &, hipStream_t, int);
FSI_P1_INST(double)
FSI_P1_INST(float)
#undef FSI_P1_INST
template void p1_down<float, float>(const P1DownArgs<float, float> &, hipStream_t, int);

}  // namespace fsi
