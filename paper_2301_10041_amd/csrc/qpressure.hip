// The pressure V-cycle of the paper's pair, L = B D^{-1} B^T on the discontinuous P1 pressure (three
// unknowns per cell: 1, (x - x_c) / h, (y - y_c) / h; D the lumped velocity mass), cell by cell.
//
// L couples a cell with the eight around it, but it is cheaper through the velocity nodes: w = D^{-1}
// B^T p at a cell's four nodes from the cells that share them, then B w over the nine nodes of a
// cell.  B is a tensor product of the 1D numbers
//   G0 = int phi' (-1, 0, 1), G1 = int phi' (x - 1/2) (1, -2, 1) / 3, S0 = int phi (1, 4, 1) / 6,
//   S1 = int phi (x - 1/2) (-1, 0, 1) / 12        (over a unit cell, for its three nodes)
// times h, and D is h^2 / 9 times 1, 2, 2, 4 at vertices, edge nodes and centres, so L has no h.
// Dirichlet nodes hold w = 0, which is all that the boundary changes; the pinned unknown (the constant
// of cell 0) is held at 0 and its row is left out.
//
// A block of 8 waves owns 8 x 64 cells, one per thread; a product is valid one cell further in, and
// both launches take two: the descent (first step from zero, second step, residual, restriction) and
// the ascent (coarse correction, two steps, at the finest level also the output) keep 4 x 60.  Both
// are bound by the latency of their passes: at 128^2 4.6 and 5.4 us, where the assembled form took seven
// launches per level of 2.6 to 6.7 us (the chain 130 -> 33 us, now behind the velocity cycle).
#include "ctx.h"
#include "kernels.h"
#include "lattice.h"

namespace fsi {

namespace {

constexpr int kQpW = 8, kQpT = kWave * kQpW;          // waves, threads
constexpr int kQpC = kWave - 4, kQpR = kQpW - 4;      // output cells of a block
static_assert(kQpC % 2 == 0 && kQpR % 2 == 0, "whole coarse cells");

template <typename T>
struct V3 {
  T c, x, y;   // constant, slopes
};

template <typename T>
struct QpLds {
  T p[3][kQpT];
  V2<T> w[4][kQpT];   // w at the cell's vertex, (1, 0), (0, 1), (1, 1)
};

// L p for the thread's cell (i, j) of an n x n grid; valid where the cell and its neighbours belong to
// the block's region.  Cells outside the grid pass p = 0.
template <typename T>
__device__ __forceinline__ V3<T> qp_product(QpLds<T> &s, V3<T> p, int i, int j, int n) {
  const int t = threadIdx.x, lane = t % kWave, row = t / kWave;
  __syncthreads();   // the w of the product before have been read
  s.p[0][t] = p.c;
  s.p[1][t] = p.x;
  s.p[2][t] = p.y;
  __syncthreads();
  const int tl = lane > 0 ? t - 1 : t, td = row > 0 ? t - kWave : t, tld = lane > 0 ? td - 1 : td;
  const V3<T> l{s.p[0][tl], s.p[1][tl], s.p[2][tl]}, d{s.p[0][td], s.p[1][td], s.p[2][td]};
  const V3<T> e{s.p[0][tld], s.p[1][tld], s.p[2][tld]};
  const T k6 = T(1.0 / 6.0), k18 = T(1.0 / 18.0), k12 = T(1.0 / 12.0), k9 = T(1.0 / 9.0);
  const bool ex = i >= 0 && i < n, ey = j >= 0 && j < n, vx = i > 0 && i < n, vy = j > 0 && j < n;
  const V2<T> o{T(0), T(0)};
  // 9 (vertex), 9/2 (edges), 9/4 (centre) times B^T p
  s.w[0][t] = vx && vy ? V2<T>{T(9) * (k6 * ((l.c + e.c) - (p.c + d.c)) + k18 * ((p.x + l.x) + (d.x + e.x)) +
                                       k12 * ((p.y - l.y) + (e.y - d.y))),
                               T(9) * (k6 * ((d.c + e.c) - (p.c + l.c)) + k12 * ((p.x - l.x) + (e.x - d.x)) +
                                       k18 * ((p.y + l.y) + (d.y + e.y)))}
                       : o;
  s.w[1][t] = ex && vy ? V2<T>{T(-4.5) * k9 * (p.x + d.x), T(3) * (d.c - p.c) + (p.y + d.y)} : o;
  s.w[2][t] = vx && ey ? V2<T>{T(3) * (l.c - p.c) + (p.x + l.x), T(-4.5) * k9 * (p.y + l.y)} : o;
  s.w[3][t] = ex && ey ? V2<T>{-p.x, -p.y} : o;
  __syncthreads();
  const int tr = lane < kWave - 1 ? t + 1 : t, tu = row < kQpW - 1 ? t + kWave : t, tru = lane < kWave - 1 ? tu + 1 : tu;
  const V2<T> v00 = s.w[0][t], v20 = s.w[0][tr], v02 = s.w[0][tu], v22 = s.w[0][tru];
  const V2<T> b = s.w[1][t], u = s.w[1][tu], lf = s.w[2][t], r = s.w[2][tr], c = s.w[3][t];
  const T k23 = T(2.0 / 3.0), k29 = T(2.0 / 9.0);
  V3<T> y;
  y.c = k6 * ((v20.x + v22.x) - (v00.x + v02.x) + (v02.y + v22.y) - (v00.y + v20.y)) +
        k23 * ((r.x - lf.x) + (u.y - b.y));
  y.x = k18 * ((v00.x + v20.x) + (v02.x + v22.x)) + k12 * ((v00.y - v20.y) + (v22.y - v02.y)) - k9 * (b.x + u.x) +
        k29 * (lf.x + r.x) - T(4) * k9 * c.x;
  y.y = k18 * ((v00.y + v20.y) + (v02.y + v22.y)) + k12 * ((v00.x - v20.x) + (v22.x - v02.x)) - k9 * (lf.y + r.y) +
        k29 * (b.y + u.y) - T(4) * k9 * c.y;
  return y;
}

// 1 / the diagonal of L at cell (i, j): its interior vertices, horizontal and vertical edges and centre
template <typename T>
__device__ __forceinline__ V3<T> qp_dinv(int i, int j, int n) {
  const double h = (j > 0) + (j < n - 1), v = (i > 0) + (i < n - 1), nv = h * v;
  return V3<T>{(T)(1.0 / (0.5 * nv + 2.0 * (h + v))), (T)(1.0 / (13.0 / 144.0 * nv + h / 18.0 + (2.0 * v + 4.0) / 9.0)),
               (T)(1.0 / (13.0 / 144.0 * nv + v / 18.0 + (2.0 * h + 4.0) / 9.0))};
}

template <typename T, typename TS>
__device__ __forceinline__ V3<T> qp_load(const TS *v, int64_t cell, bool in) {
  if (!in) return V3<T>{T(0), T(0), T(0)};
  const TS *q = v + 3 * cell;
  return V3<T>{cell == 0 ? T(0) : (T)q[0], (T)q[1], (T)q[2]};   // the pinned unknown reads as 0
}
template <typename T>
__device__ __forceinline__ V3<T> qp_step(const V3<T> &z, T c1, const V3<T> &d, T c2, const V3<T> &b, const V3<T> &s) {
  return V3<T>{fma(c2, z.c * (b.c - s.c), c1 * d.c), fma(c2, z.x * (b.x - s.x), c1 * d.x),
               fma(c2, z.y * (b.y - s.y), c1 * d.y)};
}
template <typename T>
__device__ __forceinline__ V3<T> qp_add(const V3<T> &a, const V3<T> &b) {
  return V3<T>{a.c + b.c, a.x + b.x, a.y + b.y};
}

// the block's region and the thread's cell
struct QpCell {
  int i, j, n;
  bool in, out;   // in the grid; one of the block's output cells
  int64_t cell;
  __device__ QpCell(int n_, int tiles_x) : n(n_) {
    const int lane = threadIdx.x % kWave, row = threadIdx.x / kWave;
    i = (int)(blockIdx.x % tiles_x) * kQpC - 2 + lane;
    j = (int)(blockIdx.x / tiles_x) * kQpR - 2 + row;
    in = i >= 0 && j >= 0 && i < n && j < n;
    out = in && lane >= 2 && lane < 2 + kQpC && row >= 2 && row < 2 + kQpR;
    cell = (int64_t)j * n + i;
  }
};

template <typename T, typename TB>
__global__ void __launch_bounds__(kQpT) k_qp_down(QpDownArgs<T, TB> a, int tiles_x) {
  __shared__ QpLds<T> s;
  const QpCell q(a.n, tiles_x);
  const V3<T> b = qp_load<T>(a.b, q.cell, q.in), z = qp_dinv<T>(q.i, q.j, q.n);
  V3<T> x{a.s * z.c * b.c, a.s * z.x * b.x, a.s * z.y * b.y};   // b = 0 outside the grid
  auto pinned = [&](V3<T> v) -> V3<T> {
    if (!q.in) return V3<T>{T(0), T(0), T(0)};
    if (q.cell == 0) v.c = T(0);
    return v;
  };
  x = pinned(x);
  V3<T> y = qp_product(s, x, q.i, q.j, q.n);
  x = pinned(qp_add(x, qp_step(z, a.c1, x, a.c2, b, y)));
  if (q.out) {
    T *xg = a.x + 3 * q.cell;
    xg[0] = x.c;
    xg[1] = x.x;
    xg[2] = x.y;
  }
  y = qp_product(s, x, q.i, q.j, q.n);
  const V3<T> r = pinned(V3<T>{b.c - y.c, b.x - y.x, b.y - y.y});
  // the four children of a coarse cell: constants, and slopes about its centre
  __syncthreads();
  s.p[0][threadIdx.x] = r.c;
  s.p[1][threadIdx.x] = r.x;
  s.p[2][threadIdx.x] = r.y;
  __syncthreads();
  if (!q.out || (q.i & 1) || (q.j & 1)) return;
  const int t = threadIdx.x, t1 = t + 1, t2 = t + kWave, t3 = t2 + 1;
  const T *c = s.p[0], *gx = s.p[1], *gy = s.p[2];
  const int64_t cc = (int64_t)(q.j >> 1) * (q.n / 2) + (q.i >> 1);
  T *bc = a.bc + 3 * cc;
  bc[0] = cc == 0 ? T(0) : (c[t] + c[t1]) + (c[t2] + c[t3]);
  bc[1] = T(0.25) * ((c[t1] - c[t]) + (c[t3] - c[t2])) + T(0.5) * ((gx[t] + gx[t1]) + (gx[t2] + gx[t3]));
  bc[2] = T(0.25) * ((c[t2] - c[t]) + (c[t3] - c[t1])) + T(0.5) * ((gy[t] + gy[t1]) + (gy[t2] + gy[t3]));
}

template <typename T, typename TB, bool OUT>
__global__ void __launch_bounds__(kQpT) k_qp_up(QpUpArgs<T, TB> a, int tiles_x) {
  __shared__ QpLds<T> s;
  const QpCell q(a.n, tiles_x);
  const V3<T> b = qp_load<T>(a.b, q.cell, q.in), z = qp_dinv<T>(q.i, q.j, q.n);
  auto pinned = [&](V3<T> v) -> V3<T> {
    if (!q.in) return V3<T>{T(0), T(0), T(0)};
    if (q.cell == 0) v.c = T(0);
    return v;
  };
  V3<T> x = qp_load<T>(a.x, q.cell, q.in);
  {   // + P xc
    const V3<T> c = qp_load<T>(a.xc, (int64_t)(q.j >> 1) * (q.n / 2) + (q.i >> 1), q.in);
    const T sx = (q.i & 1) ? T(0.25) : T(-0.25), sy = (q.j & 1) ? T(0.25) : T(-0.25);
    x = pinned(V3<T>{x.c + (c.c + (sx * c.x + sy * c.y)), x.x + T(0.5) * c.x, x.y + T(0.5) * c.y});
  }
  V3<T> y = qp_product(s, x, q.i, q.j, q.n);
  V3<T> d = pinned(qp_step(z, T(0), V3<T>{T(0), T(0), T(0)}, a.s, b, y));
  x = qp_add(x, d);
  y = qp_product(s, x, q.i, q.j, q.n);
  x = pinned(qp_add(x, qp_step(z, a.c1, d, a.c2, b, y)));
  double acc = 0.0;   // OUT: the thread's part of b . z
  if (q.out) {
  if constexpr (OUT) {   // z = nu M_p^{-1} r + (rho/dt) x, the pinned unknown r rounded through T
    const T *m = a.mpinv + 3 * q.cell;
    const TB *r = a.b + 3 * q.cell;
    TB *zg = a.z + 3 * q.cell;
    const TB v[3] = {(TB)(q.cell == 0 ? (T)r[0] : a.nu * m[0] * (T)r[0] + a.rdt * x.c),
                     (TB)(a.nu * m[1] * (T)r[1] + a.rdt * x.x), (TB)(a.nu * m[2] * (T)r[2] + a.rdt * x.y)};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      zg[k] = v[k];
      acc = fma((double)r[k], (double)v[k], acc);
    }
  } else {
    T *yg = a.y + 3 * q.cell;
    yg[0] = x.c;
    yg[1] = x.x;
    yg[2] = x.y;
  }
  }
  if constexpr (OUT) {
    if (a.part) {   // uniform; the block's sum in a fixed order
      __shared__ double red[kQpW];
      acc = wave_sum(acc);
      if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = acc;
      __syncthreads();
      if (threadIdx.x == 0) {
        double t = 0.0;
#pragma unroll
        for (int k = 0; k < kQpW; ++k) t += red[k];
        a.part[blockIdx.x] = t;
      }
    }
  }
}

int qp_tiles(int n, int &tx) {
  FSI_REQUIRE(n >= 2 && n % 2 == 0, FSI_E_ARG, "the pressure levels above the coarsest have even grids");
  tx = (n + kQpC - 1) / kQpC;
  return tx * ((n + kQpR - 1) / kQpR);
}

}  // namespace

int qp_up_tiles(int n) {
  int tx;
  return qp_tiles(n, tx);
}

template <typename T, typename TB>
void qp_down(const QpDownArgs<T, TB> &a, hipStream_t s) {
  int tx;
  const int tiles = qp_tiles(a.n, tx);
  hipLaunchKernelGGL((k_qp_down<T, TB>), dim3((unsigned)tiles), dim3(kQpT), 0, s, a, tx);
  FSI_CHECK_LAUNCH();
}
template <typename T, typename TB>
void qp_up(const QpUpArgs<T, TB> &a, hipStream_t s) {
  int tx;
  const int tiles = qp_tiles(a.n, tx);
  if (a.z) hipLaunchKernelGGL((k_qp_up<T, TB, true>), dim3((unsigned)tiles), dim3(kQpT), 0, s, a, tx);
  else hipLaunchKernelGGL((k_qp_up<T, TB, false>), dim3((unsigned)tiles), dim3(kQpT), 0, s, a, tx);
  FSI_CHECK_LAUNCH();
}
template void qp_down<double, double>(const QpDownArgs<double, double> &, hipStream_t);
template void qp_down<float, double>(const QpDownArgs<float, double> &, hipStream_t);
template void qp_down<float, float>(const QpDownArgs<float, float> &, hipStream_t);
template void qp_up<double, double>(const QpUpArgs<double, double> &, hipStream_t);
template void qp_up<float, double>(const QpUpArgs<float, double> &, hipStream_t);
template void qp_up<float, float>(const QpUpArgs<float, float> &, hipStream_t);

}  // namespace fsi
