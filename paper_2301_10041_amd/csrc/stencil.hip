// Matrix-free products with A_f on the structured P2 lattice (multigrid smoothing and
// residuals).  Every interior row of A_f = (rho/dt) M_f + K_f is one of four stencils,
// fixed by the parities of the node's lattice coordinates (vertex, horizontal edge,
// vertical edge, diagonal edge); rows of boundary nodes are the identity and columns of
// boundary nodes are zero (the Dirichlet condition imposed by value).  The coefficients are
// closed forms (AfCoef), checked on the host against the sums over the element matrices that the
// assembled A_f holds; products read no matrix and no indices.
#include <initializer_list>
#include <type_traits>
#include <utility>

#include "afcell.h"
#include "ctx.h"
#include "kernels.h"
#include "lattice.h"
#include "minres.h"
#include "q2cell.h"
#include "stencil.h"

namespace fsi {

// Workgroups are dispatched to the 8 XCDs round-robin (block b to XCD b % 8); each XCD
// gets a contiguous band of tiles in row-major order, so the halo rows a tile shares with
// the tile below are still in that XCD's L2.
constexpr int kXcd = 8;

// One lane stride for the vectors of a launch (null views take any)
static int64_t common_stride(std::initializer_list<std::pair<const void *, int64_t>> v, int K) {
  int64_t s = -1;
  for (const auto &e : v) {
    if (!e.first) continue;
    if (s < 0) s = e.second;
    FSI_REQUIRE(K == 1 || e.second == s, FSI_E_ARG, "lane views of one launch need one stride");
  }
  return s < 0 ? 0 : s;
}

// ---------------------------------------------------------------- smoothing, cell by cell
// The Chebyshev steps of a velocity level and its residual with one thread per cell
// (cell_products, afcell.h).  A block owns a region of 8 rows of 64, 32 or 16 cells (16 x 16 with the
// restriction in the first launch): a thread is the same cell, row w and column lane of the region, in
// every pass, so its right-hand side, directions and values stay in its registers from one step to the
// next.  x is staged in LDS as two planes of
// even and odd lattice columns, [parity][row][column / 2], with both components of a node side
// by side, so that the lanes of a wave read consecutive 16-byte (FP32: 8-byte) words; each step
// writes its values over the ones before it between two barriers.  Dirichlet and out-of-lattice
// nodes are staged as 0 (zero columns); Dirichlet rows are the identity, stepped pointwise from
// device memory.
//
// On coarse levels a launch is bound by the latency of its dependent passes, on fine ones by
// memory (pre3 with the MINRES update: 294 MB at 1024^2, 3.5 TB/s of the 4.3 that a copy reaches) and,
// in post3, by the FP64 issue of the steps it recomputes on the halo.  Against one thread per node with
// the coefficients loaded through the scalar cache in every pass (kernel times in a step in us, FP64):
//   1024^2, finest level  pre-smoothing 79.7 -> 37.6 (84 with the update, launches of 75 before),
//                         residual and restriction 51.2 -> 36.0, post-smoothing 139 -> 92.7
//   512^2 level           28.5 -> 15.4, 18.4 -> 11.8, 41.5 -> 25.0
//   32^2, finest level    8.6 and 7.9 -> 8.0 in one launch with the update, 12.0 -> 6.2
constexpr int kCellRows = 8;                          // cell rows of a region
constexpr int kCellH = 2 * kCellRows + 3;             // its staged rows: a halo of one cell
// the names of a kernel on regions of LW cells per row
#define FSI_CELL_REGION(LW) FSI_CELL_REGION_R(LW, kCellRows)
#define FSI_CELL_REGION_R(LW, R)                                                                               \
  constexpr int kThreads = (LW) * (R), kWaves = kThreads / kWave;       /* one thread per cell */              \
  constexpr int kCellHW = (LW) + 2, kCellPL = (2 * (R) + 3) * kCellHW;  /* plane width and stride, with halo */ \
  const int lane = threadIdx.x % (LW), w = region_row<LW>();            /* the thread's cell */                \
  (void)kWaves, (void)kCellPL, (void)lane, (void)w
template <int LW>
__device__ __forceinline__ int region_row() {
  static_assert(LW == kWave || 2 * LW == kWave || 4 * LW == kWave, "whole rows per wave");
  return LW == kWave ? __builtin_amdgcn_readfirstlane(threadIdx.x / kWave) : threadIdx.x / LW;
}
constexpr int kPreTileR = kCellRows - 2, kPostTileR = kCellRows - 4;
template <int LW> constexpr int kPreTile = LW - 2;     // tile widths in cells (restriction: coarse cells)
template <int LW> constexpr int kPostTile = LW - 4;
template <int LW> constexpr int kRRTile = (LW - 3) / 2;

// Regions are 64 cells wide, narrower on grids whose launches leave most of the chip idle: a block's waves
// queue for the LDS and the FP64 units of one CU, and twice the blocks of half as many waves queue
// less.  Kernel times at 64 / 32 / 16 cells in us:
//   smoothing      32^2 (FP64, in MINRES) 8.5 and 7.5 / 7.1 and 6.5 / 6.2 and 6.0; 64^2 level 6.1 and 8.2
//                  / 5.8 and 6.2 / 5.1 and 5.9; 256^2 (FP32) 9.3 and 10.5 / 8.6 and 9.4, 512^2 in FP64 23
//                  and 27 at 64, where the halo's recomputation begins to count
//   restriction    4.8 / 4.2 / 4.5 on 32^2 cells (where it is a launch of its own, by pre3_restricts, a
//                  level has 65^2 cells or more)
//   A11 rows       32^2 8.0 / 7.8 / 8.9 (two waves sum beta^2), 256^2 10.2 / 11.4
template <typename F>
static void smooth_width(int n, F f) {   // post-smoothing
  if (n <= 64) f(std::integral_constant<int, kWave / 4>{});
  else if (n <= 256) f(std::integral_constant<int, kWave / 2>{});
  else f(std::integral_constant<int, kWave>{});
}
template <typename F>
static void rows_width(int n, F f) {   // restriction and A11
  if (n <= 128) f(std::integral_constant<int, kWave / 2>{});
  else f(std::integral_constant<int, kWave>{});
}

// device-memory nodes (2 i, J), (2 i + 1, J) of one component of a vector
template <typename T>
__device__ __forceinline__ NodePair<T> ld_pair(const T *v, int64_t r) {
  return *reinterpret_cast<const NodePair<T> *>(v + r);
}

// The four nodes of cell (i, j) of a vector (component stride N, lattice side L = 2n + 1) in the
// order of cell_products; zero outside the lattice
template <typename T>
__device__ __forceinline__ void load_cell(const T *v, int64_t N, int L, int n, int i, int j, V2<T> (&q)[4]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) q[k] = V2<T>{T(0), T(0)};
  if (i < 0 || j < 0 || i > n || j > n) return;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (h == 1 && j == n) continue;
    const int64_t r = (int64_t)(2 * j + h) * L + 2 * i;
    if (i < n) {
      const NodePair<T> a = ld_pair(v, r), b = ld_pair(v, N + r);
      q[2 * h] = V2<T>{a.a, b.a};
      q[2 * h + 1] = V2<T>{a.b, b.b};
    } else {
      q[2 * h] = V2<T>{v[r], v[N + r]};
    }
  }
}

// v = q at the four nodes of cell (i, j), those in the lattice
template <typename T, typename TY>
__device__ __forceinline__ void store_cell(TY *v, int64_t N, int L, int n, int i, int j, const V2<T> (&q)[4]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (h == 1 && j == n) continue;
    const int64_t r = (int64_t)(2 * j + h) * L + 2 * i;
    if (i < n) {
      *reinterpret_cast<NodePair<TY> *>(v + r) = NodePair<TY>{(TY)q[2 * h].x, (TY)q[2 * h + 1].x};
      *reinterpret_cast<NodePair<TY> *>(v + N + r) = NodePair<TY>{(TY)q[2 * h].y, (TY)q[2 * h + 1].y};
    } else {
      v[r] = (TY)q[2 * h].x;
      v[N + r] = (TY)q[2 * h].y;
    }
  }
}

// the thread's four values at its place in the staged planes (vertex at row r, column h)
template <typename T, int PL, int HW>
__device__ __forceinline__ void put_cell(V2<T> *X, int r, int h, const V2<T> (&q)[4]) {
  V2<T> *p = X + r * HW + h;
  p[0] = q[0];
  p[PL] = q[1];
  p[HW] = q[2];
  p[PL + HW] = q[3];
}

// x (a pair of nodes of each staged row, interior nodes only) of the region whose first cell is
// (i0, j0), with the halo of one cell; f maps a node's value before it is stored (row parity,
// column parity, value)
template <typename T, int ROWS, int LW, int NT = LW *kCellRows, typename F>
__device__ __forceinline__ void stage_pairs(V2<T> *X, const T *v, int64_t N, int L, int n, int i0, int j0, F f) {
  constexpr int HW = LW + 2, NE = ROWS * HW, IT = (NE + NT - 1) / NT, PL = NE;
  NodePair<T> a[IT], b[IT];
#pragma unroll
  for (int q = 0; q < IT; ++q) {
    const int e = threadIdx.x + NT * q, lr = e / HW, i = i0 - 1 + e % HW, J = 2 * (j0 - 1) + lr;
    a[q] = b[q] = NodePair<T>{T(0), T(0)};
    if (e < NE && i >= 0 && i < n && J > 0 && J < 2 * n) {
      const int64_t r = (int64_t)J * L + 2 * i;
      a[q] = ld_pair(v, r);
      b[q] = ld_pair(v, N + r);
      if (i == 0) a[q].a = b[q].a = T(0);
    }
  }
#pragma unroll
  for (int q = 0; q < IT; ++q) {
    const int e = threadIdx.x + NT * q, lr = e / HW;
    if (e < NE) {
      X[e] = f(lr & 1, 0, V2<T>{a[q].a, b[q].a});
      X[PL + e] = f(lr & 1, 1, V2<T>{a[q].b, b[q].b});
    }
  }
}

// The restriction sums of the CW x CR coarse cells from (C0, R0) on: R is the place of the first one's fine
// vertex in the staged residual (column-parity planes of stride PL, rows of HW).
template <typename T, typename C, int HW, int PL, int CW, int CR, int WAVES>
__device__ __forceinline__ void restrict_cells(const V2<T> *R, int n, int C0, int R0, T *bcg) {
  const int Lc = n + 1;
  const int64_t Nc = (int64_t)Lc * Lc;
  // coarse classes (vertex, (1, 0), (0, 1), (1, 1)) of the CW x CR coarse cells, 64 cells a pass
  constexpr int NC = CW * CR, PASS = (NC + kWave - 1) / kWave;
  for (int u = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave); u < 4 * PASS; u += WAVES) {
    const int c = (u >> 2) * kWave + threadIdx.x % kWave;
    if (c >= NC) continue;
    const int ck = c % CW, cr = c / CW;
    auto gather = [&](auto pa_tag, auto pb_tag) {
      constexpr int PA = decltype(pa_tag)::value, PB = decltype(pb_tag)::value;
      const int Ic = 2 * (C0 + ck) + PA, Jc = 2 * (R0 + cr) + PB;
      if (Ic >= Lc || Jc >= Lc) return;
      V2<T> sum{T(0), T(0)};
      if (Ic > 0 && Jc > 0 && Ic < n && Jc < n) {
        // fine node (2 Ic + dI, 2 Jc + dJ) relative to the tile's first node
        const V2<T> *r = R + 4 * cr * HW + 2 * ck;
        auto row = [&](auto dj_tag) {
          constexpr int DJ = decltype(dj_tag)::value;
          auto term = [&](auto di_tag) {
            constexpr int DI = decltype(di_tag)::value;
            constexpr double wt = restrict_weight_of<TransferOf<C>>(PA, PB, DI, DJ);
            if constexpr (wt != 0.0) {
              constexpr int u0 = 2 * PA + DI, v0 = 2 * PB + DJ;
              const V2<T> v = r[(u0 & 1) * PL + v0 * HW + (u0 >> 1)];
              sum.x = fma(T(wt), v.x, sum.x);
              sum.y = fma(T(wt), v.y, sum.y);
            }
          };
          term(std::integral_constant<int, -3>{});
          term(std::integral_constant<int, -2>{});
          term(std::integral_constant<int, -1>{});
          term(std::integral_constant<int, 0>{});
          term(std::integral_constant<int, 1>{});
          term(std::integral_constant<int, 2>{});
          term(std::integral_constant<int, 3>{});
        };
        row(std::integral_constant<int, -3>{});
        row(std::integral_constant<int, -2>{});
        row(std::integral_constant<int, -1>{});
        row(std::integral_constant<int, 0>{});
        row(std::integral_constant<int, 1>{});
        row(std::integral_constant<int, 2>{});
        row(std::integral_constant<int, 3>{});
      }
      const int64_t k = (int64_t)Jc * Lc + Ic;
      bcg[k] = sum.x;
      bcg[Nc + k] = sum.y;
    };
    using std::integral_constant;
    switch (u & 3) {
      case 0: gather(integral_constant<int, 0>{}, integral_constant<int, 0>{}); break;
      case 1: gather(integral_constant<int, 1>{}, integral_constant<int, 0>{}); break;
      case 2: gather(integral_constant<int, 0>{}, integral_constant<int, 1>{}); break;
      default: gather(integral_constant<int, 1>{}, integral_constant<int, 1>{}); break;
    }
  }
}

template <typename T, typename C>
struct PreArgs {
  int n;
  C cf;
  T *b;                      // read, or written with the update (FP32 only)
  T *y;
  T s, c1a, c2a, c1b, c2b;   // the first step's scale, the two stencil steps
  int64_t lb, ly;            // lane strides of b and y (lane = blockIdx.y)
  MsFold f;                  // MS
  int64_t np;                // its pressure entries
  T *bc;                     // RR: the coarse right-hand side
  int64_t lc;                // its lane stride
};

// The pre-smoothing of a degree-3 smoother: x = d = s D^{-1} b, then two steps; reads b, writes x
// (4 w per node).  The first stencil step runs on 8 x 64 cells, the second on the inner 6 x 62,
// which are the block's tile.
//
// MS: in MINRES b is made here, q = y1 - alfa s r2, from the parts of alfa that the A11 launch
// left: every block sums them (in the same order) while its loads of y1 and r2 are in flight, and
// blocks past the tiles update the pressure part.  Two launches and one pass over three vectors
// less per inner step, without the restriction: 9 us against 6.2 + 2.6 + 1.9 and two gaps at 32^2, 84
// against 37 + 38 + 4 and two gaps at 1024^2 (FP64); 72 at 1024^2 with FP32 arithmetic, where the FP32
// copy of q is written here too.
//
// RR: the residual and its restriction too, in regions of 16 x 16 cells: x2 is right on the inner 14 x 14,
// the residual on 12 x 12, which gives 4 x 4 coarse cells, so 8 x 8 of the region's cells are the tile's.
// Four times the tile's work against a launch, its gap and two passes over memory less: small levels are
// bound by launches.  The values are those of k_pre3 and k_resid_restrict bit for bit.
constexpr int kPrePres = 2048;   // pressure entries per block
constexpr int kPreRRRows = 16, kPreRRc = (16 + 2 - 6 - 3) / 2;   // region rows; coarse cells per tile and side
template <typename T, typename C, int LW, bool MS, bool RR>
__global__ void __launch_bounds__(LW *(RR ? kPreRRRows : kCellRows), RR ? 1 : LW / 16)
    k_pre3(PreArgs<T, C> a, int tiles_x, int tiles, int band) {
  constexpr int kRows = RR ? kPreRRRows : kCellRows;
  static_assert(!RR || LW == kPreRRRows, "square regions");
  FSI_CELL_REGION_R(LW, kRows);
  // the first cell of the tile in the region, and its cells (a region's outermost cells are halo)
  constexpr int kOff = RR ? 4 : 1, kPreW = RR ? 2 * kPreRRc : kPreTile<LW>, kPreR = RR ? 2 * kPreRRc : kPreTileR;
  using TS = typename std::conditional<MS, double, T>::type;   // staged first
  __shared__ V2<TS> XS[2 * kCellPL];
  V2<T> *const X = reinterpret_cast<V2<T> *>(XS);
  const bool pres = MS && (int)blockIdx.x >= band * kXcd;
  const int t = (blockIdx.x % kXcd) * band + blockIdx.x / kXcd;
  if (!pres && t >= tiles) return;
  T *bg = a.b + (int64_t)blockIdx.y * a.lb;
  T *yg = a.y + (int64_t)blockIdx.y * a.ly;
  const int n = a.n, L = 2 * n + 1;
  const int64_t N = (int64_t)L * L;
  const int i0 = (t % tiles_x) * kPreW - kOff, j0 = (t / tiles_x) * kPreR - kOff;   // first cell of the region
  const int i = i0 + lane, j = j0 + w;
  const C &cf = a.cf;
  auto first = [&](int pj, int pi, V2<T> v) -> V2<T> {
    const V2<T> z = cell_dinv(cf, pi + 2 * pj, v);
    return V2<T>{a.s * z.x, a.s * z.y};
  };
  V2<T> b[4];
  if constexpr (MS) {
    const int64_t lane_v = (int64_t)blockIdx.y * a.f.q.s;
    const double *y1 = a.f.y1.p + lane_v, *r2 = a.f.r2.p + lane_v;
    double *q = a.f.q.p + lane_v;
    // the staged nodes (as in stage_pairs), in flight over the sum of alfa
    constexpr int NT = kThreads, NE = kCellPL, IT = (NE + NT - 1) / NT;
    NodePair<double> ya[IT], yb[IT], ra[IT], rb[IT];
    if (!pres) {
#pragma unroll
      for (int k = 0; k < IT; ++k) {
        const int e = threadIdx.x + NT * k, lr = e / kCellHW, ci = i0 - 1 + e % kCellHW, J = 2 * (j0 - 1) + lr;
        ya[k] = yb[k] = ra[k] = rb[k] = NodePair<double>{0.0, 0.0};
        if (e < NE && ci >= 0 && ci < n && J > 0 && J < 2 * n) {
          const int64_t r = (int64_t)J * L + 2 * ci;
          ya[k] = ld_pair(y1, r);
          yb[k] = ld_pair(y1, N + r);
          ra[k] = ld_pair(r2, r);
          rb[k] = ld_pair(r2, N + r);
          if (ci == 0) ya[k].a = yb[k].a = ra[k].a = rb[k].a = 0.0;
        }
      }
    }
    __shared__ double red[kWaves];
    double *alfa = a.f.alfa + (int64_t)blockIdx.y * a.f.ls;
    double al = 0.0;
    if (a.f.nparts > 0) {
      const double *part = a.f.part + (int64_t)blockIdx.y * a.f.lp;
      for (int k = threadIdx.x; k < a.f.nparts; k += NT) al += part[k];
      al = wave_sum(al);
      if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = al;
      __syncthreads();
      al = 0.0;
#pragma unroll
      for (int k = 0; k < kWaves; ++k) al += red[k];
      if (blockIdx.x == 0 && threadIdx.x == 0) *alfa = al;
    } else {
      al = *alfa;
    }
    al *= -a.f.s[(int64_t)blockIdx.y * a.f.ls];
    auto upd = [&](double y, double r) -> double { return al != 0.0 ? fma(al, r, y) : y; };
    if (pres) {
      const int64_t p0 = (int64_t)((int)blockIdx.x - band * kXcd) * kPrePres + threadIdx.x;
#pragma unroll
      for (int k = 0; k < kPrePres / NT; ++k) {
        const int64_t e = p0 + NT * k;
        if (e < a.np) q[2 * N + e] = upd(y1[2 * N + e], r2[2 * N + e]);
      }
      return;
    }
    // q through LDS: a thread's own cell is read there, not once more from device memory
    V2<double> qa[IT], qb[IT], by[4];
#pragma unroll
    for (int k = 0; k < IT; ++k) {
      const int e = threadIdx.x + NT * k;
      qa[k] = V2<double>{upd(ya[k].a, ra[k].a), upd(yb[k].a, rb[k].a)};
      qb[k] = V2<double>{upd(ya[k].b, ra[k].b), upd(yb[k].b, rb[k].b)};
      if (e < NE) {
        XS[e] = qa[k];
        XS[kCellPL + e] = qb[k];
      }
    }
    __syncthreads();
    {
      const V2<TS> *p = XS + (2 * w + 2) * kCellHW + lane + 1;
      by[0] = p[0];
      by[1] = p[kCellPL];
      by[2] = p[kCellHW];
      by[3] = p[kCellPL + kCellHW];
    }
    if (i == 0 || j == 0 || i >= n || j >= n) {   // Dirichlet nodes, staged as 0 (none outside the lattice)
      V2<double> y4[4], r4[4];
      load_cell(y1, N, L, n, i, j, y4);
      load_cell(r2, N, L, n, i, j, r4);
#pragma unroll
      for (int k = 0; k < 4; ++k) by[k] = V2<double>{upd(y4[k].x, r4[k].x), upd(y4[k].y, r4[k].y)};
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) b[k] = V2<T>{(T)by[k].x, (T)by[k].y};
    __syncthreads();
#pragma unroll
    for (int k = 0; k < IT; ++k) {
      const int e = threadIdx.x + NT * k, lr = e / kCellHW;
      if (e < NE) {
        X[e] = first(lr & 1, 0, V2<T>{(T)qa[k].x, (T)qa[k].y});
        X[kCellPL + e] = first(lr & 1, 1, V2<T>{(T)qb[k].x, (T)qb[k].y});
      }
    }
    if (w >= kOff && w < kOff + kPreR && j <= n && lane >= kOff && lane < kOff + kPreW && i <= n) {
      store_cell<double, double>(q, N, L, n, i, j, by);
      if constexpr (!std::is_same<T, double>::value) store_cell<T, T>(bg, N, L, n, i, j, b);
    }
  } else {
    load_cell((const T *)bg, N, L, n, i, j, b);
    stage_pairs<T, 2 * kRows + 3, LW, kThreads>(X, (const T *)bg, N, L, n, i0, j0, first);
  }
  const CellIn in = cell_inside(i, j, n);
  const int row = 2 * w + 2, h = lane + 1;
  const V2<T> *p = X + row * kCellHW + h;
  V2<T> x[4], s[4], d[4];
  __syncthreads();
  cell_products<T, kCellPL, kCellHW>(p, cf, x, s);
#pragma unroll
  for (int q = 0; q < 4; ++q) {   // the direction of the first step is x itself
    const V2<T> z = cell_dinv(cf, q, V2<T>{b[q].x - s[q].x, b[q].y - s[q].y});
    d[q] = V2<T>{fma(a.c2a, z.x, a.c1a * x[q].x), fma(a.c2a, z.y, a.c1a * x[q].y)};
    x[q] = in.q[q] ? V2<T>{x[q].x + d[q].x, x[q].y + d[q].y} : V2<T>{T(0), T(0)};
  }
  __syncthreads();
  put_cell<T, kCellPL, kCellHW>(X, row, h, x);
  __syncthreads();
  const bool mine = w >= kOff && w < kOff + kPreR && j <= n && lane >= kOff && lane < kOff + kPreW && i <= n;
  if (!RR && (w < 1 || w > kPreR || j > n)) return;
  cell_products<T, kCellPL, kCellHW>(p, cf, x, s);
  if (!RR && !mine) return;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (in.q[q]) {
      const V2<T> z = cell_dinv(cf, q, V2<T>{b[q].x - s[q].x, b[q].y - s[q].y});
      x[q].x += fma(a.c2b, z.x, a.c1b * d[q].x);
      x[q].y += fma(a.c2b, z.y, a.c1b * d[q].y);
    } else {   // Dirichlet row: the identity, stepped pointwise
      auto steps = [&](T bv) -> T {
        const T x0 = a.s * bv, e = a.c1a * x0 + a.c2a * (bv - x0), x1 = x0 + e;
        return x1 + (a.c1b * e + a.c2b * (bv - x1));
      };
      x[q] = V2<T>{steps(b[q].x), steps(b[q].y)};
    }
  }
  if (!RR || mine) store_cell<T, T>(yg, N, L, n, i, j, x);
  if constexpr (RR) {
    // x is right on the region without its outermost cells, r on one cell less at each side
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = in.q[q] ? x[q] : V2<T>{T(0), T(0)};
    __syncthreads();
    put_cell<T, kCellPL, kCellHW>(X, row, h, x);
    __syncthreads();
    cell_products<T, kCellPL, kCellHW>(p, cf, x, s);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      b[q] = in.q[q] ? V2<T>{b[q].x - s[q].x, b[q].y - s[q].y} : V2<T>{T(0), T(0)};
    __syncthreads();   // every wave has read x: r goes over it
    put_cell<T, kCellPL, kCellHW>(X, row, h, b);
    __syncthreads();
    const int C0 = (t % tiles_x) * kPreRRc, R0 = (t / tiles_x) * kPreRRc;
    restrict_cells<T, C, kCellHW, kCellPL, kPreRRc, kPreRRc, kWaves>(
        X + (2 * kOff + 2) * kCellHW + kOff + 1, n, C0, R0, a.bc + (int64_t)blockIdx.y * a.lc);
  }
}

// The coarse correction and the whole post-smoothing of a degree-3 smoother: x + P xc staged,
// then a step with c1 = 0 and two more; reads x, b and xc, writes y (stored as TY: the mixed
// form writes FP32 results into an FP64 vector), and with DOT the tile's sum of b . y.  The first
// step runs on 8 x 64 cells, the second on the inner 6 x 62, the third on 4 x 60, the tile.
// x is staged by coarse cells (4 x 4 fine nodes; one thread takes two of its rows), so that the
// interpolation weights are compile-time constants and no coarse value goes through LDS.

template <typename T, typename TY, typename C>
struct PostArgs {
  int n;
  C cf;
  const T *x, *b;
  TY *y;
  T c2a, c1b, c2b, c1c, c2c;
  int64_t lx, lb, ly;  // lane strides of x, b, y (lane = blockIdx.y)
  const T *xc;         // coarse correction (lattice n / 2, two components)
  int64_t lc;          // its lane stride
  double *dot;         // per-tile sums of b . y (FP64), or null
  int64_t ldot;        // their lane stride
  const double *b64;   // with dot: the FP64 right-hand side the sums use instead of b, or null
  int64_t lb64;        // its lane stride
};

template <typename T, typename TY, typename C, int LW, bool DOT>
__global__ void __launch_bounds__(LW *kCellRows, LW / 16) k_post3(PostArgs<T, TY, C> a, int tiles_x, int tiles, int band) {
  FSI_CELL_REGION(LW);
  constexpr int kPostW = kPostTile<LW>, kPostR = kPostTileR;
  static_assert(kPostW % 2 == 0 && kPostR % 2 == 0, "tile origins on coarse cell corners");
  __shared__ V2<T> X[2 * kCellPL];
  const int t = (blockIdx.x % kXcd) * band + blockIdx.x / kXcd;
  if (t >= tiles) return;
  const T *xg = a.x + (int64_t)blockIdx.y * a.lx, *bg = a.b + (int64_t)blockIdx.y * a.lb;
  const T *xcg = a.xc + (int64_t)blockIdx.y * a.lc;
  TY *yg = a.y + (int64_t)blockIdx.y * a.ly;
  const int n = a.n, L = 2 * n + 1;
  const int64_t N = (int64_t)L * L;
  const int i0 = (t % tiles_x) * kPostW - 2, j0 = (t / tiles_x) * kPostR - 2;   // first cell of the region
  const int i = i0 + lane, j = j0 + w;
  const C &cf = a.cf;
  {   // stage x + P xc: coarse cell (ci, cj), its fine rows 0, 1 (first four waves) or 2, 3
    constexpr int CX = (kCellHW + 2) / 2, CY = (kCellH + 4) / 4 + 1;
    static_assert(CX * CY <= kThreads / 2, "two threads per coarse cell");
    const int c = threadIdx.x % (kThreads / 2), half = w / (kCellRows / 2);
    const int kx = c % CX, ky = c / CX;
    const int ci = i0 / 2 - 1 + kx, cj = j0 / 2 - 1 + ky;   // i0 and j0 are even
    const int nc = n / 2, Lc = n + 1;
    const int64_t Nc = (int64_t)Lc * Lc;
    V2<T> v[2][4], k9[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) k9[q] = V2<T>{T(0), T(0)};
#pragma unroll
    for (int B = 0; B < 2; ++B)
#pragma unroll
      for (int A = 0; A < 4; ++A) v[B][A] = V2<T>{T(0), T(0)};
    const bool live = ky < CY && ci >= 0 && cj >= 0 && ci < nc && cj < nc;
    if (live) {
#pragma unroll
      for (int B = 0; B < 2; ++B) {
        const int64_t r = (int64_t)(4 * cj + 2 * half + B) * L + 4 * ci;
#pragma unroll
        for (int A = 0; A < 4; A += 2) {
          const NodePair<T> px = ld_pair(xg, r + A), py = ld_pair(xg, N + r + A);
          v[B][A] = V2<T>{px.a, py.a};
          v[B][A + 1] = V2<T>{px.b, py.b};
        }
      }
#pragma unroll
      for (int bq = 0; bq < 3; ++bq) {
        const int64_t r = (int64_t)(2 * cj + bq) * Lc + 2 * ci;
        const NodePair<T> px = ld_pair(xcg, r), py = ld_pair(xcg, Nc + r);
        k9[3 * bq] = V2<T>{px.a, py.a};
        k9[3 * bq + 1] = V2<T>{px.b, py.b};
        k9[3 * bq + 2] = V2<T>{xcg[r + 2], xcg[Nc + r + 2]};
      }
      // Dirichlet coarse nodes are read as 0
#pragma unroll
      for (int q = 0; q < 9; ++q) {
        const int Ic = 2 * ci + q % 3, Jc = 2 * cj + q / 3;
        if (Ic == 0 || Jc == 0 || Ic == n || Jc == n) k9[q] = V2<T>{T(0), T(0)};
      }
      auto addp = [&](auto h_tag) {
        constexpr int H = decltype(h_tag)::value;
        auto node = [&](auto a_tag, auto b_tag) {
          constexpr int A = decltype(a_tag)::value, B = decltype(b_tag)::value;
          const V2<T> p = prolong_node<C, A, 2 * H + B, T>(k9);
          v[B][A].x += p.x;
          v[B][A].y += p.y;
        };
        using std::integral_constant;
        node(integral_constant<int, 0>{}, integral_constant<int, 0>{});
        node(integral_constant<int, 1>{}, integral_constant<int, 0>{});
        node(integral_constant<int, 2>{}, integral_constant<int, 0>{});
        node(integral_constant<int, 3>{}, integral_constant<int, 0>{});
        node(integral_constant<int, 0>{}, integral_constant<int, 1>{});
        node(integral_constant<int, 1>{}, integral_constant<int, 1>{});
        node(integral_constant<int, 2>{}, integral_constant<int, 1>{});
        node(integral_constant<int, 3>{}, integral_constant<int, 1>{});
      };
      if (half) addp(std::integral_constant<int, 1>{});
      else addp(std::integral_constant<int, 0>{});
    }
#pragma unroll
    for (int B = 0; B < 2; ++B) {
      const int lr = 4 * ky - 2 + 2 * half + B;          // staged row: lattice row - 2 (j0 - 1)
      const bool wall = cj == 0 && half == 0 && B == 0;  // lattice row 0: Dirichlet
      if (ky < CY && lr >= 0 && lr < kCellH) {
#pragma unroll
        for (int A = 0; A < 4; ++A) {
          const int h = 2 * kx - 1 + A / 2;
          if (h >= 0 && h < kCellHW)
            X[(A & 1) * kCellPL + lr * kCellHW + h] = (wall || (A == 0 && ci == 0)) ? V2<T>{T(0), T(0)} : v[B][A];
        }
      }
    }
  }
  // b after the staging, whose registers it takes over: its latency runs behind the barrier
  V2<T> b[4];
  load_cell(bg, N, L, n, i, j, b);
  const CellIn in = cell_inside(i, j, n);
  const int row = 2 * w + 2, h = lane + 1;
  const V2<T> *p = X + row * kCellHW + h;
  V2<T> x[4], s[4], d[4];
  __syncthreads();
  cell_products<T, kCellPL, kCellHW>(p, cf, x, s);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const V2<T> z = cell_dinv(cf, q, V2<T>{b[q].x - s[q].x, b[q].y - s[q].y});
    d[q] = V2<T>{a.c2a * z.x, a.c2a * z.y};
    x[q] = in.q[q] ? V2<T>{x[q].x + d[q].x, x[q].y + d[q].y} : V2<T>{T(0), T(0)};
  }
  __syncthreads();
  put_cell<T, kCellPL, kCellHW>(X, row, h, x);
  __syncthreads();
  const bool in2 = w >= 1 && w <= kCellRows - 2;
  if (in2) {
    cell_products<T, kCellPL, kCellHW>(p, cf, x, s);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const V2<T> z = cell_dinv(cf, q, V2<T>{b[q].x - s[q].x, b[q].y - s[q].y});
      d[q] = V2<T>{fma(a.c2b, z.x, a.c1b * d[q].x), fma(a.c2b, z.y, a.c1b * d[q].y)};
      x[q] = in.q[q] ? V2<T>{x[q].x + d[q].x, x[q].y + d[q].y} : V2<T>{T(0), T(0)};
    }
  }
  __syncthreads();
  if (in2 && lane >= 1 && lane <= LW - 2) put_cell<T, kCellPL, kCellHW>(X, row, h, x);
  __syncthreads();
  double by = 0.0;   // the thread's part of b . y
  if (w >= 2 && w < 2 + kPostR && j <= n) {
    cell_products<T, kCellPL, kCellHW>(p, cf, x, s);
    if (lane >= 2 && lane < 2 + kPostW && i <= n) {
      V2<T> xb[4];
      if (i == 0 || j == 0 || i == n || j == n) load_cell(xg, N, L, n, i, j, xb);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (in.q[q]) {
          const V2<T> z = cell_dinv(cf, q, V2<T>{b[q].x - s[q].x, b[q].y - s[q].y});
          x[q].x += fma(a.c2c, z.x, a.c1c * d[q].x);
          x[q].y += fma(a.c2c, z.y, a.c1c * d[q].y);
        } else {   // Dirichlet row: the identity, stepped pointwise
          auto steps = [&](T bv, T x0) -> T {
            const T f = a.c2a * (bv - x0), x1 = x0 + f, e = a.c1b * f + a.c2b * (bv - x1), x2 = x1 + e;
            return x2 + (a.c1c * e + a.c2c * (bv - x2));
          };
          x[q] = V2<T>{steps(b[q].x, xb[q].x), steps(b[q].y, xb[q].y)};
        }
      }
      store_cell<T, TY>(yg, N, L, n, i, j, x);
      if constexpr (DOT) {
        V2<double> r[4];
        if (!std::is_same<T, double>::value && a.b64) {   // the FP64 right-hand side
          load_cell(a.b64 + (int64_t)blockIdx.y * a.lb64, N, L, n, i, j, r);
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) r[q] = V2<double>{(double)b[q].x, (double)b[q].y};
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)   // r = 0 outside the lattice
          if ((i < n || !(q & 1)) && (j < n || q < 2))
            by += r[q].x * (double)(TY)x[q].x + r[q].y * (double)(TY)x[q].y;
      }
    }
  }
  if constexpr (DOT) {   // the tile's sum in a fixed order: lanes by shuffles, then waves
    __shared__ double red[kWaves];
    by = wave_sum(by);
    if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = by;
    __syncthreads();
    if (threadIdx.x == 0) {
      double s0 = 0.0;
#pragma unroll
      for (int k = 0; k < kWaves; ++k) s0 += red[k];
      a.dot[(int64_t)blockIdx.y * a.ldot + t] = s0;
    }
  }
}

int post3_dot_count(int n) {
  int c = 0;
  smooth_width(n, [&](auto lw) {
    constexpr int W = kPostTile<decltype(lw)::value>;
    c = ((n + W) / W) * ((n + kPostTileR) / kPostTileR);
  });
  return c;
}

// tiles of W x R cells over the n + 1 cell columns and rows that hold nodes
static int cell_tiles(int n, int W, int R, int &tx) {
  tx = (n + W) / W;
  return tx * ((n + R) / R);
}

static void cell_launch_checks(int n, int K) {
  FSI_REQUIRE((int64_t)(2 * n + 1) * (2 * n + 1) < INT32_MAX, FSI_E_ARG, "grid too large for 32-bit stencil indices");
  FSI_REQUIRE(K >= 1 && K <= 65535, FSI_E_ARG, "lane count out of range");
}

// RR up to 256^2 cells in all lanes together, where its recomputation still fits beside the idle part of
// the chip.  Whole steps with / without it: 32^2 12.6 / 13.9 ms, 96^2 (block-diagonal) 62.7 / 69.0, 256^2
// mixed 33.3 / 36.2, 8 x 64^2 mixed 23.9 / 26.1; on the line 4 x 128^2 25.0 / 24.7 in FP64 and 21.7 / 22.4
// mixed; beyond it 2 x 256^2 47.7 / 46.6, 5 x 192^2 63.6 / 61.3, 512^2 32.8 / 31.2.  Up to 64^2 with any
// number of lanes, where the two are alike (17 x 64^2 30.1-31.2 / 31.3 ms, 32 x 64^2 46.0-47.9 / 47.0, mixed
// 40.1-41.5 / 41.7) and one form is enough.  A system's sums do not depend on the choice: both forms have
// blocks of 256 threads up to 256^2.
bool pre3_restricts(int n, int K) {
  return n % 2 == 0 && n >= 4 && (n <= 64 || (n <= 256 && (int64_t)K * n * n <= 256 * 256));
}

// Several systems at once: the triangle pair only.  A single one takes the launch with the restriction on
// every level of up to 256^2 cells, so the paper's pair never reaches the other forms of those sizes.
template <typename C>
constexpr bool kBatched = std::is_same<C, AfCoef<double>>::value || std::is_same<C, AfCoef<float>>::value;

template <typename T, typename C>
void pre3(int n, const C &cf, LP<T> b, LP<T> x, T s, T c1a, T c2a, T c1b, T c2b, hipStream_t st, int K,
          const MsFold *fold, LP<T> bc) {
  cell_launch_checks(n, K);
  FSI_REQUIRE(!bc.p || (pre3_restricts(n, K) && (K == 1 || bc.s > 0)), FSI_E_ARG, "no restriction in this launch");
  FSI_REQUIRE(K == 1 || (x.s > 0 && (b.s > 0 || !b.p)), FSI_E_ARG, "lane views need a stride");
  PreArgs<T, C> a{n, cf, b.p, x.p, s, c1a, c2a, c1b, c2b, b.s, x.s, MsFold(), 0, bc.p, bc.s};
  if (fold) {
    a.f = *fold;
    a.np = std::is_same<C, AfCoef<T>>::value ? (int64_t)(n + 1) * (n + 1) : 3 * (int64_t)n * n;
    a.f.q.s = common_stride({{a.f.y1.p, a.f.y1.s}, {a.f.r2.p, a.f.r2.s}, {a.f.q.p, a.f.q.s}}, K);
    FSI_REQUIRE(a.f.q.p != a.f.y1.p && a.f.q.p != a.f.r2.p, FSI_E_ARG, "the update reads its neighbours' operands");
  }
  const unsigned gp = fold ? (unsigned)((a.np + kPrePres - 1) / kPrePres) : 0u;
  if (bc.p) {
    constexpr int LW = kPreRRRows;
    int tx;
    const int tiles = cell_tiles(n / 2, kPreRRc, kPreRRc, tx), band = (tiles + kXcd - 1) / kXcd;
    const dim3 grid((unsigned)(band * kXcd) + gp, (unsigned)K), block(LW * kPreRRRows);
    if (fold) hipLaunchKernelGGL((k_pre3<T, C, LW, true, true>), grid, block, 0, st, a, tx, tiles, band);
    else hipLaunchKernelGGL((k_pre3<T, C, LW, false, true>), grid, block, 0, st, a, tx, tiles, band);
    FSI_CHECK_LAUNCH();
    return;
  }
  auto go = [&](auto lw) {
    constexpr int LW = decltype(lw)::value;
    int tx;
    const int tiles = cell_tiles(n, kPreTile<LW>, kPreTileR, tx), band = (tiles + kXcd - 1) / kXcd;
    const dim3 grid((unsigned)(band * kXcd) + gp, (unsigned)K), block(LW * kCellRows);
    if (fold) hipLaunchKernelGGL((k_pre3<T, C, LW, true, false>), grid, block, 0, st, a, tx, tiles, band);
    else hipLaunchKernelGGL((k_pre3<T, C, LW, false, false>), grid, block, 0, st, a, tx, tiles, band);
  };
  if constexpr (kBatched<C>) {
    if (n <= 256) {
      go(std::integral_constant<int, kWave / 2>{});
      FSI_CHECK_LAUNCH();
      return;
    }
  }
  go(std::integral_constant<int, kWave>{});
  FSI_CHECK_LAUNCH();
}
#define FSI_PRE3_INST(T, C) \
  template void pre3<T, C>(int, const C &, LP<T>, LP<T>, T, T, T, T, T, hipStream_t, int, const MsFold *, LP<T>);
FSI_PRE3_INST(double, AfCoef<double>)
FSI_PRE3_INST(float, AfCoef<float>)
FSI_PRE3_INST(double, Q2Coef<double>)
FSI_PRE3_INST(float, Q2Coef<float>)
#undef FSI_PRE3_INST

template <typename T, typename TY, typename C>
void post3(int n, const C &cf, LP<const T> x, LP<const T> b, LP<TY> y, T c2a, T c1b, T c2b, T c1c, T c2c,
           hipStream_t st, int K, LP<const T> xc, LP<double> dot, LP<const double> b64) {
  cell_launch_checks(n, K);
  FSI_REQUIRE(xc.p && n % 2 == 0 && n >= 4, FSI_E_ARG, "a coarse correction needs an even fluid grid");
  FSI_REQUIRE(K == 1 || xc.s > 0, FSI_E_ARG, "lane views of the coarse correction need a stride");
  FSI_REQUIRE(K == 1 || (x.s > 0 && b.s > 0 && y.s > 0), FSI_E_ARG, "lane views need a stride");
  FSI_REQUIRE(!dot.p || K == 1 || dot.s >= post3_dot_count(n), FSI_E_ARG, "lane stride of the tile sums too small");
  FSI_REQUIRE(!b64.p || (dot.p && (K == 1 || b64.s > 0) && !std::is_same<T, double>::value), FSI_E_ARG,
              "an FP64 right-hand side only for the sums of the FP32 form");
  PostArgs<T, TY, C> a{n, cf, x.p, b.p, y.p, c2a, c1b, c2b, c1c, c2c, x.s, b.s, y.s, xc.p, xc.s, dot.p, dot.s, b64.p, b64.s};
  smooth_width(n, [&](auto lw) {
    constexpr int LW = decltype(lw)::value;
    int tx;
    const int tiles = cell_tiles(n, kPostTile<LW>, kPostTileR, tx), band = (tiles + kXcd - 1) / kXcd;
    const dim3 grid((unsigned)(band * kXcd), (unsigned)K), block(LW * kCellRows);
    if (dot.p) hipLaunchKernelGGL((k_post3<T, TY, C, LW, true>), grid, block, 0, st, a, tx, tiles, band);
    else hipLaunchKernelGGL((k_post3<T, TY, C, LW, false>), grid, block, 0, st, a, tx, tiles, band);
  });
  FSI_CHECK_LAUNCH();
}
#define FSI_POST3_INST(T, TY, C)                                                                                 \
  template void post3<T, TY, C>(int, const C &, LP<const T>, LP<const T>, LP<TY>, T, T, T, T, T, hipStream_t, int, \
                                LP<const T>, LP<double>, LP<const double>);
FSI_POST3_INST(double, double, AfCoef<double>)
FSI_POST3_INST(float, float, AfCoef<float>)
FSI_POST3_INST(float, double, AfCoef<float>)
FSI_POST3_INST(double, double, Q2Coef<double>)
FSI_POST3_INST(float, float, Q2Coef<float>)
FSI_POST3_INST(float, double, Q2Coef<float>)
#undef FSI_POST3_INST

// ---------------------------------------------------------------- residual and restriction
// bc = R (b - A_f x) = P^T r for the multigrid descent (Sec. 4): the residual of the fine cells
// under a coarse tile is computed as in the smoothing launches and kept in LDS for the
// restriction sums, so r never goes to HBM (reads x and b, writes bc).  A coarse node gathers the
// interior fine nodes within 3 of its place, so C coarse cells need the residual of 2 C + 3 fine
// cells: a block takes Q rows of fine cells per row of its region, 30 coarse columns (14 where it is 32
// cells wide) and (8 Q - 3) / 2 coarse rows.  Q = 2 recomputes less (15 rows for 6 coarse rows, against 7 for 2) and is taken where
// that leaves the chip enough blocks; Q = 1 shortens the two dependent passes of a block.
// The restriction runs by coarse classes, one per wave pass, with compile-time weights.

template <typename T, typename C>
struct ResidRestrArgs {
  int n;
  C cf;
  const T *x, *b;
  T *bc;
  int64_t lx, lb, lc;   // lane strides of x, b and bc
};

template <typename T, typename C, int LW, int Q>
__global__ void __launch_bounds__(LW *kCellRows, LW / 16)
    k_resid_restrict(ResidRestrArgs<T, C> a, int tiles_x, int tiles, int band) {
  FSI_CELL_REGION(LW);
  constexpr int kRRc = kRRTile<LW>;
  constexpr int ROWS = 2 * kCellRows * Q + 3, PL = ROWS * kCellHW;
  constexpr int CR = (kCellRows * Q - 3) / 2;                      // coarse rows
  constexpr int RH = 2 * kCellRows * Q, RPL = RH * LW;          // residual planes
  static_assert(RPL <= PL, "the residual fits over the staged x");
  __shared__ V2<T> X[2 * PL];
  const int t = (blockIdx.x % kXcd) * band + blockIdx.x / kXcd;
  if (t >= tiles) return;
  const T *xg = a.x + (int64_t)blockIdx.y * a.lx, *bg = a.b + (int64_t)blockIdx.y * a.lb;
  T *bcg = a.bc + (int64_t)blockIdx.y * a.lc;
  const int n = a.n, L = 2 * n + 1;
  const int64_t N = (int64_t)L * L;
  const int C0 = (t % tiles_x) * kRRc, R0 = (t / tiles_x) * CR;     // first coarse cell of the tile
  const int i0 = 2 * C0 - 2, j0 = 2 * R0 - 2;                       // first fine cell of the region
  const int i = i0 + lane;
  const C &cf = a.cf;
  V2<T> b[Q][4];
  stage_pairs<T, ROWS, LW>(X, xg, N, L, n, i0, j0, [](int, int, V2<T> v) -> V2<T> { return v; });
  load_cell(bg, N, L, n, i, j0 + w * Q, b[0]);   // after the staging, whose registers it takes over
  __syncthreads();
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int j = j0 + w * Q + q;
    if (q > 0) load_cell(bg, N, L, n, i, j, b[q]);
    const CellIn in = cell_inside(i, j, n);
    V2<T> x[4], s[4];
    cell_products<T, PL, kCellHW>(X + (2 * (w * Q + q) + 2) * kCellHW + lane + 1, cf, x, s);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      b[q][k] = in.q[k] ? V2<T>{b[q][k].x - s[k].x, b[q][k].y - s[k].y} : V2<T>{T(0), T(0)};
  }
  __syncthreads();   // every wave has read x: r goes over it
  V2<T> *const R = X;
#pragma unroll
  for (int q = 0; q < Q; ++q) put_cell<T, RPL, LW>(R, 2 * (w * Q + q), lane, b[q]);
  __syncthreads();
  restrict_cells<T, C, LW, RPL, kRRc, CR, kWaves>(R + 4 * LW + 2, n, C0, R0, bcg);
}

constexpr int kRestrictWideN = 256;   // cells per side from which a block takes two rows per wave

template <typename T, typename C>
void resid_restrict(int nf, const C &cf, LP<const T> x, LP<const T> b, LP<T> bc, hipStream_t s, int K) {
  cell_launch_checks(nf, K);
  FSI_REQUIRE(nf % 2 == 0 && nf >= 4, FSI_E_ARG, "restriction needs an even fluid grid");
  FSI_REQUIRE(K == 1 || (x.s > 0 && b.s > 0 && bc.s > 0), FSI_E_ARG, "lane views need a stride");
  ResidRestrArgs<T, C> a{nf, cf, x.p, b.p, bc.p, x.s, b.s, bc.s};
  auto go = [&](auto lw, auto q_tag) {
    constexpr int LW = decltype(lw)::value, Q = decltype(q_tag)::value;
    int tx;
    const int tiles = cell_tiles(nf / 2, kRRTile<LW>, (kCellRows * Q - 3) / 2, tx), band = (tiles + kXcd - 1) / kXcd;
    hipLaunchKernelGGL((k_resid_restrict<T, C, LW, Q>), dim3((unsigned)(band * kXcd), (unsigned)K), dim3(LW * kCellRows),
                       0, s, a, tx, tiles, band);
  };
  if constexpr (kBatched<C>) {
    if (nf < kRestrictWideN) {
      rows_width(nf, [&](auto lw) { go(lw, std::integral_constant<int, 1>{}); });
      FSI_CHECK_LAUNCH();
      return;
    }
  }
  go(std::integral_constant<int, kWave>{}, std::integral_constant<int, 2>{});
  FSI_CHECK_LAUNCH();
}
#define FSI_RR_INST(T, C) \
  template void resid_restrict<T, C>(int, const C &, LP<const T>, LP<const T>, LP<T>, hipStream_t, int);
FSI_RR_INST(double, AfCoef<double>)
FSI_RR_INST(float, AfCoef<float>)
FSI_RR_INST(double, Q2Coef<double>)
FSI_RR_INST(float, Q2Coef<float>)
#undef FSI_RR_INST

// ---------------------------------------------------------------- A11 rows
// y = A11 x on [u_x | u_y | p] with one thread per cell: the cell's four velocity rows
// (cell_products and, from a staged pressure tile, the B^T rows of its three edge nodes; vertices
// have none) and the pressure row of its P1 vertex, whose 19 velocity nodes are the window the
// thread reads anyway.  No row is computed twice: a block of 8 waves owns 8 x 64 cells.
//
// Bound by memory where the vectors leave the caches: the form in MINRES reads x and r1 and writes
// y and v, 302 MB at 1024^2 in 59 us, more than a copy from device memory reaches, since part of them is
// still in the last-level cache.  One thread per node with the coefficients of its class read through the
// scalar cache took 84 us, and 8.0 at 32^2 against 6.2 (7.9 with the step before it at the head).
template <typename C>
struct A11Args {
  int n;
  C cf;
  double g;             // h / 6, the unit of the entries of B (Q2 pair: h)
  const double *x;
  double *y;            // in MINRES: r1, overwritten
  int64_t lv;           // lane stride of x, y and v (lane = blockIdx.y)
  MsA11 m;              // in MINRES
};

// the operator's rows; a step's head; the head with the step before it
enum { A11_ROWS = 0, A11_MS = 1, A11_MS_STEP = 2 };
// waves per SIMD: the paper's pair spills within the registers of four (14 us a launch at 128^2 against 10.5)
template <typename C>
constexpr int kA11Waves = std::is_same<C, AfCoef<double>>::value ? 4 : 2;
template <int MODE, typename C, int LW>
__global__ void __launch_bounds__(LW *kCellRows, (kA11Waves<C> * LW / kWave > 1 ? kA11Waves<C> * LW / kWave : 1)) k_a11(A11Args<C> a, int tiles_x, int tiles, int band) {
  FSI_CELL_REGION(LW);
  constexpr bool MS = MODE != A11_ROWS, STEP = MODE == A11_MS_STEP;
  // the paper's pair: three pressure unknowns per cell (qpressure.hip has their tensor numbers), MINRES only
  constexpr bool Q2 = !std::is_same<C, AfCoef<double>>::value;
  static_assert(MS || !Q2, "the operator's rows of the paper's pair are assembled");
  constexpr int NP = Q2 ? 3 : 1;
  __shared__ V2<double> X[2 * kCellPL];
  // P1 rows j0 - 1 .. j0 + 8 (Q2 pair: cells, three planes); the pinned entry read as 0
  constexpr int XPN = (kCellRows + 2) * kCellHW;
  __shared__ double XP[NP * XPN];
  const int t = (blockIdx.x % kXcd) * band + blockIdx.x / kXcd;
  if (t >= tiles) return;
  const double *xg = a.x + (int64_t)blockIdx.y * a.lv;
  double *yg = a.y + (int64_t)blockIdx.y * a.lv;
  const int n = a.n, L = 2 * n + 1;
  const int64_t N = (int64_t)L * L, o2 = 2 * N;
  const int i0 = (t % tiles_x) * LW, j0 = (t / tiles_x) * kCellRows;
  const int i = i0 + lane, j = j0 + w;
  const bool node = i <= n && j <= n;                    // the cell's vertex is in the lattice
  const int np1 = Q2 ? n : n + 1;                        // pressure places per row: cells, or vertices
  const bool pres = i < np1 && j < np1;
  const int64_t q0 = NP * ((int64_t)j * np1 + i);
  // the step first: beta^2, and s, c and the slot as ms_step forms them, kept in LDS for the end (in
  // registers they would be live over the products, which take all there are)
  __shared__ double msc[3];   // s, c, beta^2
  if constexpr (STEP) {
    __shared__ double bred[1024 / kWave];
    const double beta2 = ms_beta2<kThreads>(a.m.bpart.p + (int64_t)blockIdx.y * a.m.bpart.s, a.m.nb, bred);
    if (threadIdx.x == 0) {
      const MinresState &q = a.m.st[blockIdx.y];
      double sc = q.s, cc = q.c_r1;
      if (q.done == 0.0) {
        const double beta = sqrt(beta2 > 0.0 ? beta2 : 0.0);
        sc = beta > 0.0 ? 1.0 / beta : 0.0;
        cc = beta > 0.0 ? -beta / q.beta : 0.0;
      }
      msc[0] = sc;
      msc[1] = cc;
      msc[2] = beta2;
    }
  }
  {   // the pressure tile
    constexpr int NT = kThreads, IT = (XPN + NT - 1) / NT;
    double v[IT][NP];
#pragma unroll
    for (int k = 0; k < IT; ++k) {
      const int e = threadIdx.x + NT * k, pi = i0 - 1 + e % kCellHW, pj = j0 - 1 + e / kCellHW;
      const bool in = e < XPN && pi >= 0 && pj >= 0 && pi < np1 && pj < np1;
      const int64_t q = NP * ((int64_t)pj * np1 + pi);
#pragma unroll
      for (int u = 0; u < NP; ++u) v[k][u] = in && q + u != 0 ? xg[o2 + q + u] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < IT; ++k)
#pragma unroll
      for (int u = 0; u < NP; ++u)
        if (threadIdx.x + NT * k < XPN) XP[u * XPN + threadIdx.x + NT * k] = v[k][u];
  }
  stage_pairs<double, kCellH, LW>(X, xg, N, L, n, i0, j0, [](int, int, V2<double> v) -> V2<double> { return v; });
  V2<double> r1[4];
  double r1p[NP] = {};
  auto load_r1 = [&] {
    load_cell((const double *)yg, N, L, n, i, j, r1);
#pragma unroll
    for (int u = 0; u < NP; ++u)
      if (pres) r1p[u] = yg[o2 + q0 + u];
  };
  if constexpr (MS) load_r1();   // after the staging, whose registers it takes over
  __syncthreads();
  V2<double> x[4], s[4];
  double xp[NP], sp[NP];
  const V2<double> *XV = X + (2 * w + 2) * kCellHW + lane + 1;
  const double *P = XP + (w + 1) * kCellHW + lane + 1;
  if constexpr (Q2) {
    cell_products<double, kCellPL, kCellHW>(XV, a.cf, x, s);
    const double k6 = a.g / 6.0, k18 = a.g / 18.0, k12 = a.g / 12.0, k9 = a.g / 9.0, k23 = a.g * (2.0 / 3.0),
                 k29 = a.g * (2.0 / 9.0), k49 = a.g * (4.0 / 9.0);
    {   // - B^T x_p from the cells that share the node: here, left, below, below left
      const double *Px = P + XPN, *Py = Px + XPN;
      constexpr int D = kCellHW;
      s[0].x -= k6 * ((P[-1] + P[-D - 1]) - (P[0] + P[-D])) + k18 * ((Px[0] + Px[-1]) + (Px[-D] + Px[-D - 1])) +
                k12 * ((Py[0] - Py[-1]) + (Py[-D - 1] - Py[-D]));
      s[0].y -= k6 * ((P[-D] + P[-D - 1]) - (P[0] + P[-1])) + k12 * ((Px[0] - Px[-1]) + (Px[-D - 1] - Px[-D])) +
                k18 * ((Py[0] + Py[-1]) + (Py[-D] + Py[-D - 1]));
      s[1].x += k9 * (Px[0] + Px[-D]);
      s[1].y -= k23 * (P[-D] - P[0]) + k29 * (Py[0] + Py[-D]);
      s[2].x -= k23 * (P[-1] - P[0]) + k29 * (Px[0] + Px[-1]);
      s[2].y += k9 * (Py[0] + Py[-1]);
      s[3].x += k49 * Px[0];
      s[3].y += k49 * Py[0];
      xp[0] = P[0];
      xp[1] = Px[0];
      xp[2] = Py[0];
    }
    {   // - B x_u over the cell's nine nodes
      auto W = [&](int dI, int dJ) -> V2<double> { return XV[(dI & 1) * kCellPL + dJ * kCellHW + (dI >> 1)]; };
      const V2<double> v00 = W(0, 0), v20 = W(2, 0), v02 = W(0, 2), v22 = W(2, 2), bo = W(1, 0), up = W(1, 2),
                       lf = W(0, 1), rt = W(2, 1), ce = W(1, 1);
      sp[0] = -(k6 * (((v20.x + v22.x) - (v00.x + v02.x)) + ((v02.y + v22.y) - (v00.y + v20.y))) +
                k23 * ((rt.x - lf.x) + (up.y - bo.y)));
      sp[1] = -(k18 * ((v00.x + v20.x) + (v02.x + v22.x)) + k12 * ((v00.y - v20.y) + (v22.y - v02.y)) -
                k9 * (bo.x + up.x) + k29 * (lf.x + rt.x) - k49 * ce.x);
      sp[2] = -(k18 * ((v00.y + v20.y) + (v02.y + v22.y)) + k12 * ((v00.x - v20.x) + (v22.x - v02.x)) -
                k9 * (lf.y + rt.y) + k29 * (bo.y + up.y) - k49 * ce.y);
    }
  } else {
    double div;
    cell_products<double, kCellPL, kCellHW, CELL_ALL, true>(XV, a.cf, x, s, &div);
    // - B^T x_p at the edge nodes
    const double p00 = P[0], p10 = P[1], p01 = P[kCellHW], p11 = P[kCellHW + 1], pm = P[-1], p0m = P[-kCellHW];
    const double d1 = p10 - p00, d2 = p01 - p00, d3 = p11 - p01, d4 = p11 - p10;
    s[1].x = fma(2.0 * a.g, d1, s[1].x);
    s[1].y = fma(a.g, (p00 - p0m) + d4, s[1].y);
    s[2].x = fma(a.g, (p00 - pm) + d3, s[2].x);
    s[2].y = fma(2.0 * a.g, d2, s[2].y);
    s[3].x = fma(a.g, d1 + d3, s[3].x);
    s[3].y = fma(a.g, d2 + d4, s[3].y);
    xp[0] = p00;
    sp[0] = -a.g * div;
  }
  const CellIn in = cell_inside(i, j, n);
  if (i == 0 || j == 0 || i >= n || j >= n) {   // Dirichlet rows: the identity; zero outside the lattice
    V2<double> xb[4];
    load_cell(xg, N, L, n, i, j, xb);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (!in.q[q]) x[q] = s[q] = xb[q];
  }
  if (q0 == 0) xp[0] = sp[0] = xg[o2];   // the pinned entry
  if constexpr (MS) {
    const MinresState &q = a.m.st[blockIdx.y];
    const double sc = STEP ? msc[0] : q.s, cc = STEP ? msc[1] : q.c_r1;
    int sl = (int)q.slot + (STEP ? 1 : 0);
    sl = sl < 0 ? 0 : sl >= a.m.B ? a.m.B - 1 : sl;
    double *vg = a.m.vh + (int64_t)sl * a.m.vs + (int64_t)blockIdx.y * a.lv;
    double acc = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      s[q] = V2<double>{sc * s[q].x, sc * s[q].y};
      if (cc != 0.0) s[q] = V2<double>{fma(cc, r1[q].x, s[q].x), fma(cc, r1[q].y, s[q].y)};
      x[q] = V2<double>{sc * x[q].x, sc * x[q].y};
      acc = fma(x[q].y, s[q].y, fma(x[q].x, s[q].x, acc));
    }
    if (node) {
      store_cell<double, double>(yg, N, L, n, i, j, s);
      store_cell<double, double>(vg, N, L, n, i, j, x);
#pragma unroll
      for (int u = 0; u < NP; ++u) {
        if (!pres) continue;
        sp[u] *= sc;
        if (cc != 0.0) sp[u] = fma(cc, r1p[u], sp[u]);
        xp[u] *= sc;
        yg[o2 + q0 + u] = sp[u];
        vg[o2 + q0 + u] = xp[u];
        acc = fma(xp[u], sp[u], acc);
      }
    } else {
      acc = 0.0;
    }
    __shared__ double red[kWaves];   // the tile's part of v . y in a fixed order
    acc = wave_sum(acc);
    if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
      double b = 0.0;
#pragma unroll
      for (int k = 0; k < kWaves; ++k) b += red[k];
      a.m.part.p[(int64_t)blockIdx.y * a.m.part.s + t] = b;
      if constexpr (STEP) {
        if (blockIdx.x == 0) {
          MinresState o = a.m.st[blockIdx.y];
          o.beta2 = msc[2];
          ms_step(&o, a.m.hist + (int64_t)blockIdx.y * kMsRec * a.m.B, a.m.B);
          a.m.out[blockIdx.y] = o;
          ms_tell(a.m.word ? a.m.word + blockIdx.y : nullptr, a.m.seq, o);
        }
      }
    }
  } else {
    if (node) {
      store_cell<double, double>(yg, N, L, n, i, j, s);
      yg[o2 + q0] = sp[0];
    }
  }
}

// b_u = (rho/dt) M_f u with Dirichlet rows 0 and Dirichlet columns left out, b_p = 0: the velocity and
// pressure part of the step's right-hand side, cell by cell.  The entries of M_f are h^2 / 720 times
// 72, -4, -8 (vertex rows) and 128, 32, -8 (edge rows).  Bound by memory: 143 MB at 1024^2;
// 32 us, against 283 for the assembled M_f (4 lanes per CSR row; 12 bytes per entry).
struct MassArgs {
  int n;
  double m;   // (rho/dt) h^2 / 720
  const double *u;
  double *b;
};

__global__ void __launch_bounds__(kWave *kCellRows) k_mass(MassArgs a, int tiles_x, int tiles, int band) {
  FSI_CELL_REGION(kWave);
  __shared__ V2<double> X[2 * kCellPL];
  const int t = (blockIdx.x % kXcd) * band + blockIdx.x / kXcd;
  if (t >= tiles) return;
  const int n = a.n, L = 2 * n + 1;
  const int64_t N = (int64_t)L * L;
  const int i0 = (t % tiles_x) * kWave, j0 = (t / tiles_x) * kCellRows;
  const int i = i0 + lane, j = j0 + w;
  stage_pairs<double, kCellH, kWave>(X, a.u, N, L, n, i0, j0, [](int, int, V2<double> v) -> V2<double> { return v; });
  __syncthreads();
  if (i > n || j > n) return;
  const V2<double> *p = X + (2 * w + 2) * kCellHW + lane + 1;
  auto W = [&](int dI, int dJ) -> V2<double> { return p[(dI & 1) * kCellPL + dJ * kCellHW + (dI >> 1)]; };
  auto sum = [](auto... v) -> V2<double> { return V2<double>{(v.x + ...), (v.y + ...)}; };
  const V2<double> o = W(0, 0), e = W(1, 0), f = W(0, 1), g = W(1, 1);
  const V2<double> n22 = W(2, 2), n20 = W(2, 0), n02 = W(0, 2), n12 = W(1, 2), n21 = W(2, 1);
  const V2<double> l1m1 = W(1, -1), lm11 = W(-1, 1);
  V2<double> far[4], edge[4];   // vertex neighbours (edge rows: vertices), edge neighbours
  far[0] = sum(W(-2, 0), n20, W(0, -2), n02, W(-2, -2), n22);
  edge[0] = sum(n12, n21, l1m1, lm11, W(-1, -2), W(-2, -1));
  far[1] = sum(W(0, -2), n22);
  edge[1] = sum(l1m1, g, W(0, -1), n21);
  far[2] = sum(W(-2, 0), n22);
  edge[2] = sum(lm11, g, W(-1, 0), n12);
  far[3] = sum(n20, n02);
  edge[3] = sum(f, n21, e, n12);
  const V2<double> own[4] = {o, e, f, g};
  const CellIn in = cell_inside(i, j, n);
  V2<double> s[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double cd = q ? 128 * a.m : 72 * a.m, ce = q ? 32 * a.m : -8 * a.m, cf = q ? -8 * a.m : -4 * a.m;
    s[q] = in.q[q] ? V2<double>{fma(cf, far[q].x, fma(ce, edge[q].x, cd * own[q].x)),
                                fma(cf, far[q].y, fma(ce, edge[q].y, cd * own[q].y))}
                   : V2<double>{0.0, 0.0};
  }
  store_cell<double, double>(a.b, N, L, n, i, j, s);
  a.b[2 * N + (int64_t)j * (n + 1) + i] = 0.0;
}

void mass_rows(int n, double rdt, const double *u, double *b, hipStream_t s) {
  cell_launch_checks(n, 1);
  int tx;
  const int tiles = cell_tiles(n, kWave, kCellRows, tx), band = (tiles + kXcd - 1) / kXcd;
  hipLaunchKernelGGL(k_mass, dim3((unsigned)(band * kXcd)), dim3(kWave * kCellRows), 0, s,
                     MassArgs{n, rdt / (720.0 * n * n), u, b}, tx, tiles, band);
  FSI_CHECK_LAUNCH();
}

template <int MODE, int LW, typename C>
static void launch_a11(A11Args<C> a, hipStream_t s, int K) {
  cell_launch_checks(a.n, K);
  int tx;
  const int tiles = cell_tiles(a.n, LW, kCellRows, tx), band = (tiles + kXcd - 1) / kXcd;
  a.g = std::is_same<C, AfCoef<double>>::value ? 1.0 / (6.0 * a.n) : 1.0 / a.n;
  hipLaunchKernelGGL((k_a11<MODE, C, LW>), dim3((unsigned)(band * kXcd), (unsigned)K), dim3(LW * kCellRows), 0, s, a, tx,
                     tiles, band);
  FSI_CHECK_LAUNCH();
}

// y_u += C_f^T x_lam: one lane per row, which sums its entries in their order, every product fused into
// the sum.  The entries of the 64 rows of a wavefront come kCftSlice per row and round, a row's by
// neighbouring lanes, with the x_lam that they meet, through LDS, one round ahead; rows without entries
// (most of them) end after their pointers.
//
// Bound by the latency of a round where the solid is fine (rows of 40 to 1,000 entries), by the memory
// path of the scattered x_lam beyond 256^2.  As a part of the A11 launch, a wavefront summing two lattice
// rows of cells from segments of 256 entries, it left all lanes but one idle on long rows.  Whole operator in us,
// [one thread per node inside the row kernel] / [segments in the A11 launch] / now, at r = 0.2: 32^2 with
// rows of 7.8 entries 16.5 / 15.7 / 15.9, of 141 137 / 428 / 70; 128^2, 9.3 17.9 / 20.8 / 17.2, 124 203 / 713 / 84; 256^2,
// 9.4 24.1 / 31.8 / 19.6; 512^2, 9.5 61 / 55 / 44; 1024^2, 6.3 151 / 112 / 106, 18.6 624 / 288 / 298.
// Slices of 8 (twice the LDS): 141 at 1024^2, 165 against 228 at 512^2 with 45 entries.
struct CftArgs {
  int64_t N;   // rows
  const int *rp, *col;
  const double *val, *lx, *ly;
  double *y;   // two components
};
constexpr int kCftThreads = 256, kCftSlice = 4;

__global__ void __launch_bounds__(kCftThreads) k_cft_rows(CftArgs a) {
  constexpr int S = kCftSlice, G = kWave / S, ROW = kWave + 8;   // 8: the writes of a slice over all banks
  __shared__ V2<double> xs[kCftThreads / kWave][S * ROW];
  __shared__ double vs[kCftThreads / kWave][S * ROW];
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
  const int64_t r = (int64_t)blockIdx.x * kCftThreads + threadIdx.x;
  int k = a.rp[min(r, a.N)];
  const int k1 = a.rp[min(r + 1, a.N)];
  if (!__ballot(k < k1)) return;   // no barrier follows: a wavefront is on its own
  const bool any = k < k1;
  double sx = 0.0, sy = 0.0;
  if (any) {
    sx = a.y[r];
    sy = a.y[a.N + r];
  }
  // slice entry u of this lane: entry lane % S of the row of lane u G + lane / S
  double v[S];
  int c[S];
  auto fetch = [&](int pos) {
#pragma unroll
    for (int u = 0; u < S; ++u) {
      const int o = u * G + lane / S, p = __shfl(pos, o) + lane % S;
      const bool in = p < __shfl(k1, o);
      v[u] = in ? a.val[p] : 0.0;
      c[u] = in ? a.col[p] : -1;
    }
  };
  auto fence = [] {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  fetch(k);
  for (; __ballot(k < k1); k += S) {
    V2<double> x[S];
#pragma unroll
    for (int u = 0; u < S; ++u)
      if (c[u] >= 0) x[u] = V2<double>{a.lx[c[u]], a.ly[c[u]]};
#pragma unroll
    for (int u = 0; u < S; ++u)
      if (c[u] >= 0) {
        const int q = lane % S * ROW + u * G + lane / S;
        xs[w][q] = x[u];
        vs[w][q] = v[u];
      }
    fetch(k + S);
    fence();
#pragma unroll
    for (int t = 0; t < S; ++t)
      if (k + t < k1) {
        const V2<double> g = xs[w][t * ROW + lane];
        const double cv = vs[w][t * ROW + lane];
        sx = fma(cv, g.x, sx);
        sy = fma(cv, g.y, sy);
      }
    fence();
  }
  if (any) {
    a.y[r] = sx;
    a.y[a.N + r] = sy;
  }
}

void a11_rows(int n, const AfCoef<double> &cf, const double *x, double *y, const int *cft_rp, const int *cft_col,
              const double *cft_val, const double *xl, int64_t Ns, hipStream_t s) {
  A11Args<AfCoef<double>> a{};
  a.n = n;
  a.cf = cf;
  a.x = x;
  a.y = y;
  launch_a11<A11_ROWS, kWave>(a, s, 1);
  if (!cft_rp) return;
  const int64_t N = (int64_t)(2 * n + 1) * (2 * n + 1);
  hipLaunchKernelGGL(k_cft_rows, dim3((unsigned)((N + kCftThreads - 1) / kCftThreads)), dim3(kCftThreads), 0, s,
                     CftArgs{N, cft_rp, cft_col, cft_val, xl, xl + Ns, y});
  FSI_CHECK_LAUNCH();
}

template <typename C>
void a11_minres(int n, const C &cf, LP<const double> y, LP<double> r1, const MsA11 &m, hipStream_t s,
                int K) {
  FSI_REQUIRE(m.st && m.B >= 1 && m.part.p && (m.nb == 0 || (m.out && m.out != m.st)), FSI_E_ARG,
              "the A11 launch of an inner step needs its state, slots and parts");
  A11Args<C> a{};
  a.n = n;
  a.cf = cf;
  a.x = y.p;
  a.y = r1.p;
  a.lv = common_stride({{y.p, y.s}, {r1.p, r1.s}}, K);
  a.m = m;
  rows_width(n, [&](auto lw) {
    constexpr int LW = decltype(lw)::value;
    if (m.nb > 0) launch_a11<A11_MS_STEP, LW>(a, s, K);
    else launch_a11<A11_MS, LW>(a, s, K);
  });
}

template void a11_minres<AfCoef<double>>(int, const AfCoef<double> &, LP<const double>, LP<double>, const MsA11 &,
                                         hipStream_t, int);
template void a11_minres<Q2Coef<double>>(int, const Q2Coef<double> &, LP<const double>, LP<double>, const MsA11 &,
                                         hipStream_t, int);

int a11_tile_count(int n) {
  int c = 0, tx;
  rows_width(n, [&](auto lw) { c = cell_tiles(n, decltype(lw)::value, kCellRows, tx); });
  return c;
}

}  // namespace fsi
