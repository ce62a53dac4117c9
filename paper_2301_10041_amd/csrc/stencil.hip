// Matrix-free products with A_f on the structured P2 lattice (multigrid smoothing and
// residuals).  Every interior row of A_f = (rho/dt) M_f + K_f is one of four stencils,
// fixed by the parities of the node's lattice coordinates (vertex, horizontal edge,
// vertical edge, diagonal edge); rows of boundary nodes are the identity and columns of
// boundary nodes are zero (the Dirichlet condition imposed by value).  The coefficients
// come from the same element matrices as the assembled A_f (host tables per level), so the
// stencil product equals the CSR product up to the order of the sums.
//
// Bytes per node in the Chebyshev step: x, b, d read, d and y written (5 two-component
// vectors); no matrix and no indices.
#include <initializer_list>
#include <type_traits>
#include <utility>

#include "afcell.h"
#include "ctx.h"
#include "kernels.h"
#include "lattice.h"
#include "stencil.h"

namespace fsi {

template <typename T>
struct StencilArgs {
  int n;
  const StencilTable<T> *tab;   // device
  const T *x, *b;
  T *d, *y;
  int L2;                      // nodes per component (2n+1)^2
  T c1, c2;
  // SP_A11 only: fluid rows on [u_x | u_y | p] (x and y hold all three; see
  // stencil_fluid_rows), optional C_f^T x_lam on the velocity rows
  const DivTable<T> *dv;
  const int *cft_rp, *cft_col;
  const T *cft_val, *xlx, *xly;
  // SP_A11 inside MINRES (ms_s set): with device scalars s = *ms_s, c = *ms_c, write
  // v = s x and y = s (A11 x) + c r1 over r1 (ms_r1y; r1 read only where c != 0), and the
  // block's part of v . y to ms_part[tile]
  const double *ms_s, *ms_c;
  T *ms_v, *ms_r1y;
  double *ms_part;
  // lane strides (blockIdx.y = lane): vectors, MINRES scalars, per-tile parts.  The C_f^T
  // term (cft_*, xlx, xly) is one system's and is not shifted.
  int64_t lv, ls, lp;
  // in MINRES: ms_v is the base of the Lanczos block; v goes to slot *ms_slot (a device
  // scalar of the lane's state, clamped to [0, ms_nslot - 1]) at stride ms_vs
  const double *ms_slot;
  int64_t ms_vs;
  int ms_nslot;
};

// Views of lane blockIdx.y (null pointers stay null).
template <typename P>
__device__ __forceinline__ void lane_shift(P *&p, int64_t stride) {
  if (p) p += (int64_t)blockIdx.y * stride;
}
template <typename T>
__device__ __forceinline__ StencilArgs<T> lane_args(const StencilArgs<T> &a0) {
  StencilArgs<T> a = a0;
  lane_shift(a.x, a.lv);
  lane_shift(a.b, a.lv);
  lane_shift(a.d, a.lv);
  lane_shift(a.y, a.lv);
  lane_shift(a.ms_v, a.lv);
  lane_shift(a.ms_r1y, a.lv);
  lane_shift(a.ms_s, a.ls);
  lane_shift(a.ms_c, a.ls);
  lane_shift(a.ms_part, a.lp);
  lane_shift(a.ms_slot, a.ls);
  if (a.ms_slot) {
    int sl = (int)*a.ms_slot;
    sl = sl < 0 ? 0 : sl >= a.ms_nslot ? a.ms_nslot - 1 : sl;
    a.ms_v += (int64_t)sl * a.ms_vs;
  }
  return a;
}

// Tiled kernel.  A block owns kTileR lattice rows x kTileC nodes.  Phase 1 stages x with a
// halo of two nodes into LDS (stride-1, coalesced), storing 0 for boundary nodes and for
// nodes outside the lattice, so that interior rows need no column test.  Phase 2: wave w
// computes row w of the tile, first the even-I nodes then the odd-I nodes, so the node
// class (and the coefficient addresses) are uniform over the wave.  Phase 3 reads the
// products back in row-major order and does the mode's epilogue with coalesced global
// accesses.  Boundary rows are the identity.
constexpr int kTW = kTileC + 4;                 // tile width with halo
constexpr int kTH = kTileR + 4;

template <typename T, int CLS>
__device__ __forceinline__ void tile_row_products(const StencilTable<T> &tb, const T *X0, const T *X1,
                                                  int base, T &s0, T &s1) {
  constexpr StencilOffsets so = stencil_offsets();
  constexpr CrossZero cz = cross_zero();
  s0 = 0;
  s1 = 0;
#pragma unroll
  for (int k = 0; k < kStencilCount[CLS]; ++k) {
    const int o = base + so.d[CLS][k][1] * kTW + so.d[CLS][k][0];
    const T y0 = X0[o], y1 = X1[o];
    if (cz.z[CLS][k]) {   // xy = yx = 0 (fma with a zero coefficient adds nothing)
      s0 = fma(tb.coef[CLS][k][0], y0, s0);
      s1 = fma(tb.coef[CLS][k][3], y1, s1);
    } else {
      s0 = fma(tb.coef[CLS][k][1], y1, fma(tb.coef[CLS][k][0], y0, s0));
      s1 = fma(tb.coef[CLS][k][3], y1, fma(tb.coef[CLS][k][2], y0, s1));
    }
  }
}

// B^T x_p of a class-CLS node from the staged pressure tile (row width kPW), base = the
// tile position of P1 node (I >> 1, J >> 1)
constexpr int kPW = kTileC / 2 + 2, kPH = kTileR / 2 + 2;   // P1 tile with a halo of one
template <typename T, int CLS>
__device__ __forceinline__ void tile_bt_products(const DivTable<T> &dv, const T *XP, int base, T &s0, T &s1) {
  constexpr DivOffsets so = div_offsets();
#pragma unroll
  for (int k = 0; k < kBtCount[CLS]; ++k) {
    const T pv = XP[base + so.bt[CLS][k][1] * kPW + so.bt[CLS][k][0]];
    s0 = fma(-dv.bt_coef[CLS][k][0], pv, s0);
    s1 = fma(-dv.bt_coef[CLS][k][1], pv, s1);
  }
}

// Workgroups are dispatched to the 8 XCDs round-robin (block b to XCD b % 8); each XCD
// gets a contiguous band of tiles in row-major order, so the halo rows a tile shares with
// the tile below are still in that XCD's L2.
constexpr int kXcd = 8;

template <typename T, int MODE>
__global__ void __launch_bounds__(256) k_stencil(StencilArgs<T> a0, int tiles_x, int tiles, int band) {
  __shared__ T X[2][kTH * kTW];
  __shared__ T S[2][kTileR * kTileC];
  __shared__ T XP[MODE == SP_A11 ? kPH * kPW : 1];   // SP_A11: x_p tile (column 0 read as 0)
  const int t = (blockIdx.x % kXcd) * band + blockIdx.x / kXcd;
  if (t >= tiles) return;
  const StencilArgs<T> a = lane_args(a0);
  const int n2 = 2 * a.n, L = n2 + 1;
  const int I0 = (t % tiles_x) * kTileC, J0 = (t / tiles_x) * kTileR;
  const int tid = threadIdx.x;
  const StencilTable<T> &tb = *a.tab;
  double ms_acc = 0.0;   // SP_A11 in MINRES: this thread's part of v . y
  // epilogue operands of this thread's nodes (row-major, coalesced), loaded first; x only at
  // Dirichlet nodes (the staged tile holds 0 there), the interior x comes from the tile
  constexpr int EIT = kTileR * kTileC / 256;
  T ex[EIT][2], eb[EIT][2], ed[EIT][2];
#pragma unroll
  for (int q = 0; q < EIT; ++q) {
    const int e = tid + 256 * q, I = I0 + e % kTileC, J = J0 + e / kTileC;
    ex[q][0] = ex[q][1] = eb[q][0] = eb[q][1] = ed[q][0] = ed[q][1] = 0;
    if (I <= n2 && J <= n2) {
      const int r = J * L + I;
      if (I == 0 || J == 0 || I == n2 || J == n2) {
        ex[q][0] = a.x[r];
        ex[q][1] = a.x[a.L2 + r];
      }
      if constexpr (MODE == SP_RESID || MODE == SP_CHEB) {
        eb[q][0] = a.b[r];
        eb[q][1] = a.b[a.L2 + r];
      }
      if constexpr (MODE == SP_CHEB) {
        ed[q][0] = a.d[r];
        ed[q][1] = a.d[a.L2 + r];
      }
      if constexpr (MODE == SP_A11) {   // in MINRES: r1 (ed holds it)
        if (a.ms_s) {
          ed[q][0] = a.ms_r1y[r];
          ed[q][1] = a.ms_r1y[a.L2 + r];
        }
      }
    }
  }
  // SP_A11: the pressure tile (P1 rows J0/2 - 1 .. J0/2 + 2, columns I0/2 - 1 .. I0/2 + 64)
  // and, for the pressure rows of the tile (threads 0..127), x_p and r1 at the own node
  T pp_x = 0, pp_r1 = 0;
  if constexpr (MODE == SP_A11) {
    const int64_t o2 = 2 * (int64_t)a.L2;
    for (int e = tid; e < kPH * kPW; e += 256) {
      const int pi = (I0 >> 1) - 1 + e % kPW, pj = (J0 >> 1) - 1 + e / kPW;
      T pv = 0;
      if (pi >= 0 && pj >= 0 && pi <= a.n && pj <= a.n) {
        const int64_t q = (int64_t)pj * (a.n + 1) + pi;
        if (q != 0) pv = a.x[o2 + q];
      }
      XP[e] = pv;
    }
    if (tid < 2 * kWave) {
      const int pi = (I0 >> 1) + tid % kWave, pj = (J0 >> 1) + tid / kWave;
      if (pi <= a.n && pj <= a.n) {
        const int64_t q = (int64_t)pj * (a.n + 1) + pi;
        pp_x = a.x[o2 + q];
        if (a.ms_s) pp_r1 = a.ms_r1y[o2 + q];
      }
    }
  }
  // phase 1: x tile with halo (all loads issued before the LDS stores)
  constexpr int NE = kTH * kTW, IT = (NE + 255) / 256;
  T v[IT][2];
#pragma unroll
  for (int q = 0; q < IT; ++q) {
    const int e = tid + 256 * q, tr = e / kTW, tc = e % kTW;
    const int I = I0 - 2 + tc, J = J0 - 2 + tr;
    v[q][0] = 0;
    v[q][1] = 0;
    if (e < NE && I > 0 && J > 0 && I < n2 && J < n2) {
      const int r = J * L + I;
      v[q][0] = a.x[r];
      v[q][1] = a.x[a.L2 + r];
    }
  }
#pragma unroll
  for (int q = 0; q < IT; ++q) {
    const int e = tid + 256 * q;
    if (e < NE) {
      X[0][e] = v[q][0];
      X[1][e] = v[q][1];
    }
  }
  __syncthreads();
  // phase 2: products of the interior rows, one tile row per wave
  {
    const int w = tid / kWave, lane = tid % kWave;
    const int J = J0 + w;
    if (J > 0 && J < n2) {
#pragma unroll
      for (int par = 0; par < 2; ++par) {
        const int i = 2 * lane + par;
        const int I = I0 + i;
        T s0 = 0, s1 = 0;
        const int base = (w + 2) * kTW + (i + 2);
        if (I > 0 && I < n2) {
          // SP_A11: - B^T x_p from the pressure tile; P1 node (I >> 1, J >> 1) sits at
          // tile row (w >> 1) + 1, column lane + 1 (I0 and J0 are even)
          const int pbase = ((w >> 1) + 1) * kPW + lane + 1;
          if (J & 1) {
            if (par) {
              tile_row_products<T, 3>(tb, X[0], X[1], base, s0, s1);
              if constexpr (MODE == SP_A11) tile_bt_products<T, 3>(*a.dv, XP, pbase, s0, s1);
            } else {
              tile_row_products<T, 2>(tb, X[0], X[1], base, s0, s1);
              if constexpr (MODE == SP_A11) tile_bt_products<T, 2>(*a.dv, XP, pbase, s0, s1);
            }
          } else {
            if (par) {
              tile_row_products<T, 1>(tb, X[0], X[1], base, s0, s1);
              if constexpr (MODE == SP_A11) tile_bt_products<T, 1>(*a.dv, XP, pbase, s0, s1);
            } else {
              tile_row_products<T, 0>(tb, X[0], X[1], base, s0, s1);
              if constexpr (MODE == SP_A11) tile_bt_products<T, 0>(*a.dv, XP, pbase, s0, s1);
            }
          }
        }
        S[0][w * kTileC + i] = s0;
        S[1][w * kTileC + i] = s1;
      }
    }
  }
  __syncthreads();
  // phase 3: epilogue, row-major and coalesced
#pragma unroll
  for (int q = 0; q < EIT; ++q) {
    const int e = tid + 256 * q;
    const int j = e / kTileC, i = e % kTileC;
    const int I = I0 + i, J = J0 + j;
    if (I > n2 || J > n2) continue;
    const int r = J * L + I;
    const bool bnd = I == 0 || J == 0 || I == n2 || J == n2;
    const int xo = (j + 2) * kTW + (i + 2);   // the node in the staged tile
    const T x0 = bnd ? ex[q][0] : X[0][xo], x1 = bnd ? ex[q][1] : X[1][xo];
    const T s0 = bnd ? x0 : S[0][e], s1 = bnd ? x1 : S[1][e];
    if constexpr (MODE == SP_APPLY) {
      a.y[r] = s0;
      a.y[a.L2 + r] = s1;
    } else if constexpr (MODE == SP_A11) {
      T t0 = s0, t1 = s1;   // A_f x_u - B^T x_p (identity on Dirichlet rows)
      if (a.cft_rp) {
        for (int k = a.cft_rp[r]; k < a.cft_rp[r + 1]; ++k) {
          const T cv = a.cft_val[k];
          const int j = a.cft_col[k];
          t0 += cv * a.xlx[j];
          t1 += cv * a.xly[j];
        }
      }
      if (a.ms_s) {
        const T sc = (T)*a.ms_s, cc = (T)*a.ms_c;
        T y0 = sc * t0, y1 = sc * t1;
        if (cc != T(0)) {
          y0 += cc * ed[q][0];
          y1 += cc * ed[q][1];
        }
        const T v0 = sc * x0, v1 = sc * x1;
        a.ms_r1y[r] = y0;
        a.ms_r1y[a.L2 + r] = y1;
        a.ms_v[r] = v0;
        a.ms_v[a.L2 + r] = v1;
        ms_acc += (double)v0 * (double)y0 + (double)v1 * (double)y1;
      } else {
        a.y[r] = t0;
        a.y[a.L2 + r] = t1;
      }
    } else if constexpr (MODE == SP_RESID) {
      a.y[r] = eb[q][0] - s0;
      a.y[a.L2 + r] = eb[q][1] - s1;
    } else {
      const T r0 = eb[q][0] - s0, r1 = eb[q][1] - s1;
      T z0 = r0, z1 = r1;
      if (!bnd) {   // class-wise D^{-1}: scalar loads, picked per node
        const int cls = (I & 1) | ((J & 1) << 1);
        T di[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
          di[k] = cls == 0 ? tb.dinv[0][k] : cls == 1 ? tb.dinv[1][k] : cls == 2 ? tb.dinv[2][k] : tb.dinv[3][k];
        z0 = di[0] * r0 + di[1] * r1;
        z1 = di[2] * r0 + di[3] * r1;
      }
      const T d0 = a.c1 * ed[q][0] + a.c2 * z0, d1 = a.c1 * ed[q][1] + a.c2 * z1;
      a.d[r] = d0;
      a.d[a.L2 + r] = d1;
      a.y[r] = x0 + d0;
      a.y[a.L2 + r] = x1 + d1;
    }
  }
  if constexpr (MODE == SP_A11) {
    // phase 4: pressure rows of the P1 nodes at even lattice positions of the tile
    // (2 rows x 64 nodes), -B x_u from the staged x tile (Dirichlet values read as zero)
    if (tid < 2 * kWave) {
      const int pr = tid / kWave, pc = tid % kWave;
      const int pi = (I0 >> 1) + pc, pj = (J0 >> 1) + pr;
      if (pi <= a.n && pj <= a.n) {
        const DivTable<T> &dv = *a.dv;
        constexpr StencilOffsets so = stencil_offsets();   // B rows: the vertex pattern
        const int base = (2 * pr + 2) * kTW + (2 * pc + 2);
        T sp = 0;
#pragma unroll
        for (int k = 0; k < kBMax; ++k) {
          const int o = base + so.d[0][k][1] * kTW + so.d[0][k][0];
          sp = fma(dv.b_coef[k][1], X[1][o], fma(dv.b_coef[k][0], X[0][o], sp));
        }
        const int64_t q = (int64_t)pj * (a.n + 1) + pi;
        const int64_t o2 = 2 * (int64_t)a.L2;
        const T val = q == 0 ? pp_x : -sp;
        if (a.ms_s) {
          const T sc = (T)*a.ms_s, cc = (T)*a.ms_c;
          T yv = sc * val;
          if (cc != T(0)) yv += cc * pp_r1;
          const T vv = sc * pp_x;
          a.ms_r1y[o2 + q] = yv;
          a.ms_v[o2 + q] = vv;
          ms_acc += (double)vv * (double)yv;
        } else {
          a.y[o2 + q] = val;
        }
      }
    }
    if (a.ms_s) {   // the block's part of v . y (fixed order: deterministic)
      __shared__ double red[256 / kWave];
      const double wsum = wave_sum(ms_acc);
      if (tid % kWave == 0) red[tid / kWave] = wsum;
      __syncthreads();
      if (tid == 0) {
        double b = 0.0;
        for (int k = 0; k < 256 / kWave; ++k) b += red[k];
        a.ms_part[t] = b;
      }
    }
  }
}

template <typename T, int MODE>
static void launch_tiles(int n, const StencilArgs<T> &a, hipStream_t s, int K) {
  const int L = 2 * n + 1;
  const int tx = (L + kTileC - 1) / kTileC, ty = (L + kTileR - 1) / kTileR;
  const int tiles = tx * ty, band = (tiles + kXcd - 1) / kXcd;
  FSI_REQUIRE(K >= 1 && K <= 65535, FSI_E_ARG, "lane count out of range");
  hipLaunchKernelGGL((k_stencil<T, MODE>), dim3((unsigned)(band * kXcd), (unsigned)K), dim3(256), 0, s, a, tx,
                     tiles, band);
  FSI_CHECK_LAUNCH();
}

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

template <typename T, int MODE>
void stencil_launch(int n, const StencilTable<T> *tab, LP<const T> x, LP<const T> b, LP<T> d, LP<T> y, T c1,
                    T c2, hipStream_t s, int K) {
  FSI_REQUIRE((int64_t)(2 * n + 1) * (2 * n + 1) < INT32_MAX, FSI_E_ARG, "grid too large for 32-bit stencil indices");
  static_assert(kTileR * kWave == 256 && 2 * kWave == kTileC, "one tile row per wave, two nodes per lane");
  const int64_t lv = common_stride({{x.p, x.s}, {b.p, b.s}, {d.p, d.s}, {y.p, y.s}}, K);
  StencilArgs<T> a{n, tab, x.p, b.p, d.p, y.p, (2 * n + 1) * (2 * n + 1), c1, c2, nullptr, nullptr, nullptr,
                   nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, lv, 0, 0};
  launch_tiles<T, MODE>(n, a, s, K);
}

template <typename T>
void stencil_fluid_rows(int n, const StencilTable<T> *tab, const DivTable<T> *dv, const T *x, T *y,
                        const int *cft_rp, const int *cft_col, const T *cft_val, const T *xl, int64_t Ns,
                        hipStream_t s) {
  FSI_REQUIRE((int64_t)(2 * n + 1) * (2 * n + 1) < INT32_MAX, FSI_E_ARG, "grid too large for 32-bit stencil indices");
  static_assert(kTileC % 2 == 0 && kTileR % 2 == 0 && kTileC / 2 == kWave && kTileR / 2 * kWave <= 256,
                "a tile holds 2 x 64 P1 nodes, one per thread of the first two waves");
  const int L = 2 * n + 1, L2 = L * L;
  StencilArgs<T> a{n, tab, x, nullptr, nullptr, y, L2, T(0), T(0), dv, cft_rp, cft_col, cft_val, xl,
                   xl ? xl + Ns : nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, 0, 0, 0};
  launch_tiles<T, SP_A11>(n, a, s, 1);
}

int stencil_a11_minres(int n, const StencilTable<double> *tab, const DivTable<double> *dv, LP<const double> x,
                       LP<double> v, LP<double> r1y, LP<const double> s_dev, LP<const double> c_dev,
                       LP<const double> slot_dev, int64_t vs, int nslot, LP<double> part, hipStream_t s, int K) {
  FSI_REQUIRE((int64_t)(2 * n + 1) * (2 * n + 1) < INT32_MAX, FSI_E_ARG, "grid too large for 32-bit stencil indices");
  FSI_REQUIRE(slot_dev.p && nslot >= 1, FSI_E_ARG, "the Lanczos block needs a slot index and at least one slot");
  const int L = 2 * n + 1, L2 = L * L;
  const int64_t lv = common_stride({{x.p, x.s}, {v.p, v.s}, {r1y.p, r1y.s}}, K);
  const int64_t ls = common_stride({{s_dev.p, s_dev.s}, {c_dev.p, c_dev.s}, {slot_dev.p, slot_dev.s}}, K);
  StencilArgs<double> a{n, tab, x.p, nullptr, nullptr, nullptr, L2, 0.0, 0.0, dv, nullptr, nullptr, nullptr, nullptr,
                        nullptr, s_dev.p, c_dev.p, v.p, r1y.p, part.p, lv, ls, part.s, slot_dev.p, vs, nslot};
  launch_tiles<double, SP_A11>(n, a, s, K);
  const int tx = (L + kTileC - 1) / kTileC, ty = (L + kTileR - 1) / kTileR;
  return tx * ty;
}

int stencil_tile_count(int n) {
  const int L = 2 * n + 1;
  return ((L + kTileC - 1) / kTileC) * ((L + kTileR - 1) / kTileR);
}
template void stencil_fluid_rows<double>(int, const StencilTable<double> *, const DivTable<double> *,
                                         const double *, double *, const int *, const int *, const double *,
                                         const double *, int64_t, hipStream_t);
template void stencil_fluid_rows<float>(int, const StencilTable<float> *, const DivTable<float> *, const float *,
                                        float *, const int *, const int *, const float *, const float *, int64_t,
                                        hipStream_t);

// ---------------------------------------------------------------- smoothing, cell by cell
// The Chebyshev steps of a velocity level and its residual with one thread per cell
// (cell_products, afcell.h).  A block of 8 waves owns 8 rows of 64 cells: wave w is cell row w of
// the region, lane l cell column l, in every pass, so a thread's right-hand side, directions and
// values stay in its registers from one step to the next.  x is staged in LDS as two planes of
// even and odd lattice columns, [parity][row][column / 2], with both components of a node side
// by side, so that the lanes of a wave read consecutive 16-byte (FP32: 8-byte) words; each step
// writes its values over the ones before it between two barriers.  Dirichlet and out-of-lattice
// nodes are staged as 0 (zero columns); Dirichlet rows are the identity, stepped pointwise from
// device memory.
//
// On coarse levels a launch is bound by the latency of its dependent passes, on fine ones by
// memory (pre3: 134 MB at 1024^2, 3.6 TB/s of the 4.3 that a copy reaches) and, in post3, by the
// FP64 issue of the steps it recomputes on the halo.  Against one thread per node with the
// coefficients loaded through the scalar cache in every pass (kernel times in a step, FP64):
//   1024^2  pre-smoothing 79.7 -> 37.6 us, residual and restriction 51.2 -> 32.7, post-smoothing
//           139 -> 118 (beside the pressure part on the other stream)
//   512^2   28.5 -> 15.2, 18.4 -> 11.5, 41.5 -> 24.4
//   32^2    8.6 -> 6.2, 7.9 -> 4.8, 12.0 -> 8.1
constexpr int kCellWaves = 8;
constexpr int kCellHW = kWave + 2;                    // plane width: a halo of one cell
constexpr int kCellH = 2 * kCellWaves + 3;            // staged rows of 8 cell rows
constexpr int kCellPL = kCellH * kCellHW;             // plane stride

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
template <typename T, int ROWS, typename F>
__device__ __forceinline__ void stage_pairs(V2<T> *X, const T *v, int64_t N, int L, int n, int i0, int j0, F f) {
  constexpr int NT = kWave * kCellWaves, NE = ROWS * kCellHW, IT = (NE + NT - 1) / NT, PL = ROWS * kCellHW;
  NodePair<T> a[IT], b[IT];
#pragma unroll
  for (int q = 0; q < IT; ++q) {
    const int e = threadIdx.x + NT * q, lr = e / kCellHW, i = i0 - 1 + e % kCellHW, J = 2 * (j0 - 1) + lr;
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
    const int e = threadIdx.x + NT * q, lr = e / kCellHW;
    if (e < NE) {
      X[e] = f(lr & 1, 0, V2<T>{a[q].a, b[q].a});
      X[PL + e] = f(lr & 1, 1, V2<T>{a[q].b, b[q].b});
    }
  }
}

template <typename T>
struct PreArgs {
  int n;
  AfCoef<T> cf;
  const T *b;
  T *y;
  T s, c1a, c2a, c1b, c2b;   // the first step's scale, the two stencil steps
  int64_t lv;                // lane stride of b and y (lane = blockIdx.y)
};

// The pre-smoothing of a degree-3 smoother: x = d = s D^{-1} b, then two steps; reads b, writes x
// (4 w per node).  The first stencil step runs on 8 x 64 cells, the second on the inner 6 x 62,
// which are the block's tile.
constexpr int kPreW = kWave - 2, kPreR = kCellWaves - 2;
template <typename T>
__global__ void __launch_bounds__(kWave *kCellWaves, 4) k_pre3(PreArgs<T> a, int tiles_x, int tiles, int band) {
  __shared__ V2<T> X[2 * kCellPL];
  const int t = (blockIdx.x % kXcd) * band + blockIdx.x / kXcd;
  if (t >= tiles) return;
  const T *bg = a.b + (int64_t)blockIdx.y * a.lv;
  T *yg = a.y + (int64_t)blockIdx.y * a.lv;
  const int n = a.n, L = 2 * n + 1;
  const int64_t N = (int64_t)L * L;
  const int i0 = (t % tiles_x) * kPreW - 1, j0 = (t / tiles_x) * kPreR - 1;   // first cell of the region
  const int lane = threadIdx.x % kWave, w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int i = i0 + lane, j = j0 + w;
  const AfCoef<T> &cf = a.cf;
  V2<T> b[4];
  load_cell(bg, N, L, n, i, j, b);
  stage_pairs<T, kCellH>(X, bg, N, L, n, i0, j0, [&](int pj, int pi, V2<T> v) -> V2<T> {
    const V2<T> z = cell_dinv(cf, pi | pj, v);
    return V2<T>{a.s * z.x, a.s * z.y};
  });
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
  if (w < 1 || w > kPreR || j > n) return;
  cell_products<T, kCellPL, kCellHW>(p, cf, x, s);
  if (lane < 1 || lane > kPreW || i > n) return;
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
  store_cell<T, T>(yg, N, L, n, i, j, x);
}

// The coarse correction and the whole post-smoothing of a degree-3 smoother: x + P xc staged,
// then a step with c1 = 0 and two more; reads x, b and xc, writes y (stored as TY: the mixed
// form writes FP32 results into an FP64 vector), and with DOT the tile's sum of b . y.  The first
// step runs on 8 x 64 cells, the second on the inner 6 x 62, the third on 4 x 60, the tile.
// x is staged by coarse cells (4 x 4 fine nodes; one thread takes two of its rows), so that the
// interpolation weights are compile-time constants and no coarse value goes through LDS.
constexpr int kPostW = kWave - 4, kPostR = kCellWaves - 4;
static_assert(kPostW % 2 == 0 && kPostR % 2 == 0, "tile origins on coarse cell corners");

template <typename T, typename TY>
struct PostArgs {
  int n;
  AfCoef<T> cf;
  const T *x, *b;
  TY *y;
  T c2a, c1b, c2b, c1c, c2c;
  int64_t lv;          // lane stride of x, b, y (lane = blockIdx.y)
  const T *xc;         // coarse correction (lattice n / 2, two components)
  int64_t lc;          // its lane stride
  double *dot;         // per-tile sums of b . y (FP64), or null
  int64_t ldot;        // their lane stride
  const double *b64;   // with dot: the FP64 right-hand side the sums use instead of b, or null
  int64_t lb64;        // its lane stride
};

template <typename T, typename TY, bool DOT>
__global__ void __launch_bounds__(kWave *kCellWaves, 4) k_post3(PostArgs<T, TY> a, int tiles_x, int tiles, int band) {
  __shared__ V2<T> X[2 * kCellPL];
  const int t = (blockIdx.x % kXcd) * band + blockIdx.x / kXcd;
  if (t >= tiles) return;
  const T *xg = a.x + (int64_t)blockIdx.y * a.lv, *bg = a.b + (int64_t)blockIdx.y * a.lv;
  const T *xcg = a.xc + (int64_t)blockIdx.y * a.lc;
  TY *yg = a.y + (int64_t)blockIdx.y * a.lv;
  const int n = a.n, L = 2 * n + 1;
  const int64_t N = (int64_t)L * L;
  const int i0 = (t % tiles_x) * kPostW - 2, j0 = (t / tiles_x) * kPostR - 2;   // first cell of the region
  const int lane = threadIdx.x % kWave, w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int i = i0 + lane, j = j0 + w;
  const AfCoef<T> &cf = a.cf;
  {   // stage x + P xc: coarse cell (ci, cj), its fine rows 0, 1 (first four waves) or 2, 3
    constexpr int CX = (kCellHW + 2) / 2, CY = (kCellH + 4) / 4 + 1;
    static_assert(CX * CY <= kWave * kCellWaves / 2, "two threads per coarse cell");
    const int c = threadIdx.x % (kWave * kCellWaves / 2), half = w / (kCellWaves / 2);
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
          const V2<T> p = prolong_node<A, 2 * H + B, T>(k9);
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
  const bool in2 = w >= 1 && w <= kCellWaves - 2;
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
  if (in2 && lane >= 1 && lane <= kWave - 2) put_cell<T, kCellPL, kCellHW>(X, row, h, x);
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
    __shared__ double red[kPostR];
    by = wave_sum(by);
    if (lane == 0 && w >= 2 && w < 2 + kPostR) red[w - 2] = by;
    __syncthreads();
    if (threadIdx.x == 0) {
      double s0 = 0.0;
#pragma unroll
      for (int k = 0; k < kPostR; ++k) s0 += red[k];
      a.dot[(int64_t)blockIdx.y * a.ldot + t] = s0;
    }
  }
}

int post3_dot_count(int n) { return ((n + kPostW) / kPostW) * ((n + kPostR) / kPostR); }

// tiles of W x R cells over the n + 1 cell columns and rows that hold nodes
static int cell_tiles(int n, int W, int R, int &tx) {
  tx = (n + W) / W;
  return tx * ((n + R) / R);
}

static void cell_launch_checks(int n, int K) {
  FSI_REQUIRE((int64_t)(2 * n + 1) * (2 * n + 1) < INT32_MAX, FSI_E_ARG, "grid too large for 32-bit stencil indices");
  FSI_REQUIRE(K >= 1 && K <= 65535, FSI_E_ARG, "lane count out of range");
}

template <typename T>
void pre3(int n, const AfCoef<T> &cf, LP<const T> b, LP<T> x, T s, T c1a, T c2a, T c1b, T c2b, hipStream_t st, int K) {
  cell_launch_checks(n, K);
  int tx;
  const int tiles = cell_tiles(n, kPreW, kPreR, tx), band = (tiles + kXcd - 1) / kXcd;
  const int64_t lv = common_stride({{b.p, b.s}, {x.p, x.s}}, K);
  PreArgs<T> a{n, cf, b.p, x.p, s, c1a, c2a, c1b, c2b, lv};
  hipLaunchKernelGGL(k_pre3<T>, dim3((unsigned)(band * kXcd), (unsigned)K), dim3(kWave * kCellWaves), 0, st, a, tx,
                     tiles, band);
  FSI_CHECK_LAUNCH();
}
template void pre3<double>(int, const AfCoef<double> &, LP<const double>, LP<double>, double, double, double, double,
                           double, hipStream_t, int);
template void pre3<float>(int, const AfCoef<float> &, LP<const float>, LP<float>, float, float, float, float, float,
                          hipStream_t, int);

template <typename T, typename TY>
void post3(int n, const AfCoef<T> &cf, LP<const T> x, LP<const T> b, LP<TY> y, T c2a, T c1b, T c2b, T c1c, T c2c,
           hipStream_t st, int K, LP<const T> xc, LP<double> dot, LP<const double> b64) {
  cell_launch_checks(n, K);
  FSI_REQUIRE(xc.p && n % 2 == 0 && n >= 4, FSI_E_ARG, "a coarse correction needs an even fluid grid");
  FSI_REQUIRE(K == 1 || xc.s > 0, FSI_E_ARG, "lane views of the coarse correction need a stride");
  int tx;
  const int tiles = cell_tiles(n, kPostW, kPostR, tx), band = (tiles + kXcd - 1) / kXcd;
  const int64_t lv = common_stride({{x.p, x.s}, {b.p, b.s}, {y.p, y.s}}, K);
  FSI_REQUIRE(!dot.p || K == 1 || dot.s >= tiles, FSI_E_ARG, "lane stride of the tile sums too small");
  FSI_REQUIRE(!b64.p || (dot.p && (K == 1 || b64.s > 0) && !std::is_same<T, double>::value), FSI_E_ARG,
              "an FP64 right-hand side only for the sums of the FP32 form");
  PostArgs<T, TY> a{n, cf, x.p, b.p, y.p, c2a, c1b, c2b, c1c, c2c, lv, xc.p, xc.s, dot.p, dot.s, b64.p, b64.s};
  const dim3 grid((unsigned)(band * kXcd), (unsigned)K), block(kWave * kCellWaves);
  if (dot.p) hipLaunchKernelGGL((k_post3<T, TY, true>), grid, block, 0, st, a, tx, tiles, band);
  else hipLaunchKernelGGL((k_post3<T, TY, false>), grid, block, 0, st, a, tx, tiles, band);
  FSI_CHECK_LAUNCH();
}
#define FSI_POST3_INST(T, TY)                                                                                    \
  template void post3<T, TY>(int, const AfCoef<T> &, LP<const T>, LP<const T>, LP<TY>, T, T, T, T, T, hipStream_t, \
                             int, LP<const T>, LP<double>, LP<const double>);
FSI_POST3_INST(double, double)
FSI_POST3_INST(float, float)
FSI_POST3_INST(float, double)
#undef FSI_POST3_INST

// ---------------------------------------------------------------- residual and restriction
// bc = R (b - A_f x) = P^T r for the multigrid descent (Sec. 4): the residual of the fine cells
// under a coarse tile is computed as in the smoothing launches and kept in LDS for the
// restriction sums, so r never goes to HBM (reads x and b, writes bc).  A coarse node gathers the
// interior fine nodes within 3 of its place, so C coarse cells need the residual of 2 C + 3 fine
// cells: a block takes Q rows of fine cells per wave, 30 coarse columns and (8 Q - 3) / 2 coarse
// rows.  Q = 2 recomputes less (15 rows for 6 coarse rows, against 7 for 2) and is taken where
// that leaves the chip enough blocks; Q = 1 shortens the two dependent passes of a block.
// The restriction runs by coarse classes, one per wave pass, with compile-time weights.
constexpr int kRRc = (kWave - 3) / 2;

template <typename T>
struct ResidRestrArgs {
  int n;
  AfCoef<T> cf;
  const T *x, *b;
  T *bc;
  int64_t lv, lc;   // lane strides of the fine (x, b) and coarse (bc) vectors
};

template <typename T, int Q>
__global__ void __launch_bounds__(kWave *kCellWaves, 4)
    k_resid_restrict(ResidRestrArgs<T> a, int tiles_x, int tiles, int band) {
  constexpr int ROWS = 2 * kCellWaves * Q + 3, PL = ROWS * kCellHW;
  constexpr int CR = (kCellWaves * Q - 3) / 2;                      // coarse rows
  constexpr int RH = 2 * kCellWaves * Q, RPL = RH * kWave;          // residual planes
  static_assert(RPL <= PL, "the residual fits over the staged x");
  __shared__ V2<T> X[2 * PL];
  const int t = (blockIdx.x % kXcd) * band + blockIdx.x / kXcd;
  if (t >= tiles) return;
  const T *xg = a.x + (int64_t)blockIdx.y * a.lv, *bg = a.b + (int64_t)blockIdx.y * a.lv;
  T *bcg = a.bc + (int64_t)blockIdx.y * a.lc;
  const int n = a.n, L = 2 * n + 1, Lc = n + 1;
  const int64_t N = (int64_t)L * L, Nc = (int64_t)Lc * Lc;
  const int C0 = (t % tiles_x) * kRRc, R0 = (t / tiles_x) * CR;     // first coarse cell of the tile
  const int i0 = 2 * C0 - 2, j0 = 2 * R0 - 2;                       // first fine cell of the region
  const int lane = threadIdx.x % kWave, w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int i = i0 + lane;
  const AfCoef<T> &cf = a.cf;
  V2<T> b[Q][4];
  stage_pairs<T, ROWS>(X, xg, N, L, n, i0, j0, [](int, int, V2<T> v) -> V2<T> { return v; });
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
  for (int q = 0; q < Q; ++q) put_cell<T, RPL, kWave>(R, 2 * (w * Q + q), lane, b[q]);
  __syncthreads();
  // coarse classes (vertex, (1, 0), (0, 1), (1, 1)) of the kRRc x CR coarse cells, 64 cells a pass
  constexpr int NC = kRRc * CR, PASS = (NC + kWave - 1) / kWave;
  for (int u = w; u < 4 * PASS; u += kCellWaves) {
    const int c = (u >> 2) * kWave + lane;
    if (c >= NC) continue;
    const int ck = c % kRRc, cr = c / kRRc;
    auto gather = [&](auto pa_tag, auto pb_tag) {
      constexpr int PA = decltype(pa_tag)::value, PB = decltype(pb_tag)::value;
      const int Ic = 2 * (C0 + ck) + PA, Jc = 2 * (R0 + cr) + PB;
      if (Ic >= Lc || Jc >= Lc) return;
      V2<T> sum{T(0), T(0)};
      if (Ic > 0 && Jc > 0 && Ic < n && Jc < n) {
        // fine node (2 Ic + dI, 2 Jc + dJ) relative to the region's first node (2 i0, 2 j0)
        const V2<T> *r = R + (4 * cr + 4) * kWave + 2 * ck + 2;
        auto row = [&](auto dj_tag) {
          constexpr int DJ = decltype(dj_tag)::value;
          auto term = [&](auto di_tag) {
            constexpr int DI = decltype(di_tag)::value;
            constexpr double wt = restrict_weight(PA, PB, DI, DJ);
            if constexpr (wt != 0.0) {
              constexpr int u0 = 2 * PA + DI, v0 = 2 * PB + DJ;
              const V2<T> v = r[(u0 & 1) * RPL + v0 * kWave + (u0 >> 1)];
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

constexpr int kRestrictWideN = 256;   // cells per side from which a block takes two rows per wave

template <typename T>
void resid_restrict(int nf, const AfCoef<T> &cf, LP<const T> x, LP<const T> b, LP<T> bc, hipStream_t s, int K) {
  cell_launch_checks(nf, K);
  FSI_REQUIRE(nf % 2 == 0 && nf >= 4, FSI_E_ARG, "restriction needs an even fluid grid");
  FSI_REQUIRE(K == 1 || bc.s > 0, FSI_E_ARG, "lane views of the coarse vector need a stride");
  const int64_t lv = common_stride({{x.p, x.s}, {b.p, b.s}}, K);
  ResidRestrArgs<T> a{nf, cf, x.p, b.p, bc.p, lv, bc.s};
  auto go = [&](auto q_tag) {
    constexpr int Q = decltype(q_tag)::value;
    int tx;
    const int tiles = cell_tiles(nf / 2, kRRc, (kCellWaves * Q - 3) / 2, tx), band = (tiles + kXcd - 1) / kXcd;
    hipLaunchKernelGGL((k_resid_restrict<T, Q>), dim3((unsigned)(band * kXcd), (unsigned)K),
                       dim3(kWave * kCellWaves), 0, s, a, tx, tiles, band);
  };
  if (nf >= kRestrictWideN) go(std::integral_constant<int, 2>{});
  else go(std::integral_constant<int, 1>{});
  FSI_CHECK_LAUNCH();
}
template void resid_restrict<double>(int, const AfCoef<double> &, LP<const double>, LP<const double>, LP<double>,
                                     hipStream_t, int);
template void resid_restrict<float>(int, const AfCoef<float> &, LP<const float>, LP<const float>, LP<float>,
                                    hipStream_t, int);

#define FSI_STENCIL_INST(T, M)                                                                              \
  template void stencil_launch<T, M>(int, const StencilTable<T> *, LP<const T>, LP<const T>, LP<T>, LP<T>, T, T, \
                                     hipStream_t, int);
FSI_STENCIL_INST(double, SP_APPLY)
FSI_STENCIL_INST(double, SP_RESID)
FSI_STENCIL_INST(double, SP_CHEB)
FSI_STENCIL_INST(float, SP_APPLY)
FSI_STENCIL_INST(float, SP_RESID)
FSI_STENCIL_INST(float, SP_CHEB)
#undef FSI_STENCIL_INST

}  // namespace fsi
