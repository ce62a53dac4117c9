// The coarse end of the velocity V-cycle in one launch per system (Sec. 4 multigrid).  On
// levels of at most 16 x 16 cells every smoothing step, residual and transfer of the
// separate launches costs the latency of a whole kernel while the level holds a few
// thousand nodes; here one 512-thread block keeps the iterate of every remaining level in LDS
// and runs pre-smoothing, residual, restriction, the dense solve on the coarsest level,
// prolongation and post-smoothing with block barriers in between.  The steps are those of the
// per-level launches (the same Chebyshev coefficients, cell products and transfer weights).
//
// Threads: cell (i, j) of a level belongs to two threads, one for its nodes on the even lattice
// row (vertex and (1, 0): the first four waves) and one for those on the odd row, so that a wave's
// work is uniform and both halves of a cell run at once on two waves per SIMD.  A thread's
// right-hand side and direction stay in its registers over the steps of a level.  The iterate lies
// in LDS in two buffers, one step reading one and writing the other (one barrier per step), as
// even and odd column planes with both components of a node together and a halo of zeros; the
// residual takes the buffer that the iterate has left.  Dirichlet nodes hold 0 (a restricted
// right-hand side vanishes there), so only interior nodes are ever written.
//
// What bounds it is the latency of about 20 dependent passes.  The A_f entries come from the
// kernel arguments into scalar registers (AfCoef): read from LDS by every wave in every pass they
// took two thirds of a pass (6,800 of its cycles at 16^2; an LDS read of one uniform word costs
// as much as one of 64 words).  The dense inverse (162 x 162 words on 4^2) is fetched into
// registers at the start, behind the descent; read at its turn it took 9 of 43 us.  Now 20.6 us
// in FP64 and 17.0 in FP32 (43.6 and 41 in the form before); one thread per node, 1024 threads,
// measured 23.2 and 17.5 (registers spill in FP64, twice the waves per barrier).
#include <cmath>

#include "ctx.h"
#include "kernels.h"
#include "lattice.h"
#include "stencil.h"

namespace fsi {

namespace {

constexpr int kTailThreads = 512, kTailHalf = kTailThreads / 2;
// staged planes of a level: lattice columns -2 .. 2n + 2 as planes of n + 3, rows -2 .. 2n + 2
constexpr int kTailHW = kTailMaxN + 3, kTailPL = (2 * kTailMaxN + 5) * kTailHW;
static_assert(2 * kTailPL == kTailLevelV2, "LDS size of a level's buffer");
static_assert(kTailMaxN * kTailMaxN <= kTailHalf, "one thread per half cell");

// position of node (I, J) in a level's buffer
__device__ __forceinline__ int tail_at(int I, int J) { return (I & 1) * kTailPL + (J + 2) * kTailHW + (I >> 1) + 1; }

// restriction sum at coarse node (2 i + PA, 2 j + PB) from the fine residual r of a level
template <typename T, int PA, int PB>
__device__ __forceinline__ V2<T> tail_restrict(const V2<T> *r, int i, int j) {
  V2<T> sum{T(0), T(0)};
  const V2<T> *p = r + tail_at(4 * i, 4 * j);
  auto row = [&](auto dj_tag) {
    constexpr int DJ = decltype(dj_tag)::value;
    auto term = [&](auto di_tag) {
      constexpr int DI = decltype(di_tag)::value;
      constexpr double wt = restrict_weight(PA, PB, DI, DJ);
      if constexpr (wt != 0.0) {
        constexpr int U = 2 * PA + DI, V = 2 * PB + DJ;
        const V2<T> v = p[(U & 1) * kTailPL + V * kTailHW + (U >> 1)];
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
  return sum;
}

// coarse quadratic at fine node (A, B) (0 .. 3) of a coarse cell: the six P2 basis values of the
// triangle that holds it, in the order vertices 0, 1, 2, edges 01, 12, 20 (exact in float); c(a, b)
// reads the coarse node (a, b) (0 .. 2) of the cell
template <typename T, typename C>
__device__ __forceinline__ V2<T> tail_prolong(C c, int A, int B) {
  const bool lo = A >= B;
  const float xi = 0.25f * (float)A, eta = 0.25f * (float)B;
  const float l0 = lo ? 1.0f - xi : 1.0f - eta, l1 = lo ? xi - eta : xi, l2 = lo ? eta : eta - xi;
  const float phi[6] = {l0 * (2.0f * l0 - 1.0f), l1 * (2.0f * l1 - 1.0f), l2 * (2.0f * l2 - 1.0f),
                        4.0f * l0 * l1,         4.0f * l1 * l2,         4.0f * l2 * l0};
  const int di[6] = {0, 2, lo ? 2 : 0, 1, lo ? 2 : 1, lo ? 1 : 0};
  const int dj[6] = {0, lo ? 0 : 2, 2, lo ? 0 : 1, lo ? 1 : 2, 1};
  V2<T> s{T(0), T(0)};
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    const V2<T> v = c(di[q], dj[q]);
    s.x = fma((T)phi[q], v.x, s.x);
    s.y = fma((T)phi[q], v.y, s.y);
  }
  return s;
}

template <typename T>
__global__ void __launch_bounds__(kTailThreads, 2) k_mg_tail(TailArgs<T> a) {
  extern __shared__ unsigned char tail_smem[];
  V2<T> *const sv = reinterpret_cast<V2<T> *>(tail_smem);   // level l: buffers 2 l, 2 l + 1; then its b
  const int tid = threadIdx.x, half = __builtin_amdgcn_readfirstlane(tid / kTailHalf), cell = tid % kTailHalf;
  const T *bg = a.b + (int64_t)blockIdx.y * a.lb;
  T *xg = a.x + (int64_t)blockIdx.y * a.lb;
  // the dense inverse: P threads per row, kp consecutive columns each; the matrix is symmetric, so
  // thread (row, part) reads its entries down column `row` and the loads are coalesced
  const int m = a.m, P = kTailThreads / m, kp = (m + P - 1) / P, drow = tid % m, dpart = tid / m;
  const bool dlive = dpart < P;
  const bool pre = kp <= kTailDenseReg, even = kp == kTailDenseReg && P * kp == m;   // uniform
  T cr[kTailDenseReg];
  {
    const int c0 = (dlive ? dpart : 0) * kp;
    if (even) {   // no column to guard (a coarsest level of 4 x 4 cells: 162 = 3 x 54)
      const T *p = a.cinv + c0 * m + drow;
#pragma unroll
      for (int q = 0; q < kTailDenseReg; ++q) cr[q] = p[q * m];
    } else {
#pragma unroll
      for (int q = 0; q < kTailDenseReg; ++q)   // past the last column: any entry (it meets a zero of b)
        cr[q] = pre && q < kp ? a.cinv[(c0 + q < m ? c0 + q : 0) * m + drow] : T(0);
    }
  }
  auto buf = [&](int l, int k) -> V2<T> * { return sv + (2 * l + k) * kTailLevelV2; };
  V2<T> *const bs = sv + 2 * a.nlev * kTailLevelV2;         // right-hand sides: 2 per thread and level
  T *const db = reinterpret_cast<T *>(bs + 2 * kTailThreads * a.nlev), *const dx = db + m + kTailDenseReg;   // coarsest b (zeros after it) and x
  double *const dp = reinterpret_cast<double *>(tail_smem + a.offp);                         // partial sums
  // the first level's right-hand side (interior nodes), and the zeros of its last column and row
  V2<T> b[2] = {{T(0), T(0)}, {T(0), T(0)}};
  {
    const int n = a.lv[0].n, L = 2 * n + 1, NG = L * L, i = cell % n, j = cell / n;
    if (j < n) {
      const int r = (2 * j + half) * L + 2 * i;
      b[0] = V2<T>{bg[r], bg[NG + r]};
      b[1] = V2<T>{bg[r + 1], bg[NG + r + 1]};
    }
    for (int q = tid; q < L; q += kTailThreads) {
      xg[q * L + 2 * n] = xg[NG + q * L + 2 * n] = T(0);
      xg[2 * n * L + q] = xg[NG + 2 * n * L + q] = T(0);
    }
  }
  for (int q = tid; q < 2 * a.nlev * kTailLevelV2; q += kTailThreads) sv[q] = V2<T>{T(0), T(0)};
  for (int q = tid; q < m + kTailDenseReg; q += kTailThreads) db[q] = T(0);
  __syncthreads();
  // the thread's place on a level: its two nodes (2 i, J), (2 i + 1, J), J = 2 j + half
  struct Place {
    int i, j, at;
    bool in[2];
  };
  auto place = [&](int n) -> Place {
    const int i = cell % n, j = cell / n;
    const bool row = j < n && (half == 1 || j > 0);
    return Place{i, j, tail_at(2 * i, 2 * j), {row && i > 0, row}};
  };
  // products at the thread's nodes from buffer x (threads past the level's cells read cell 0)
  auto product = [&](const V2<T> *x, const Place &pl, const AfCoef<T> &cf, V2<T> (&xo)[2], V2<T> (&so)[2]) {
    const V2<T> *p = x + (pl.in[1] ? pl.at : tail_at(0, 0));
    V2<T> xx[4], ss[4];
    if (half) {
      cell_products<T, kTailPL, kTailHW, CELL_ROW1>(p, cf, xx, ss);
      xo[0] = xx[2];
      xo[1] = xx[3];
      so[0] = ss[2];
      so[1] = ss[3];
    } else {
      cell_products<T, kTailPL, kTailHW, CELL_ROW0>(p, cf, xx, ss);
      xo[0] = xx[0];
      xo[1] = xx[1];
      so[0] = ss[0];
      so[1] = ss[1];
    }
  };
  auto put = [&](V2<T> *x, const Place &pl, const V2<T> (&v)[2]) {
    V2<T> *p = x + pl.at + half * kTailHW;
    if (pl.in[0]) p[0] = v[0];
    if (pl.in[1]) p[kTailPL] = v[1];
  };
  V2<T> d[2];
  // one Chebyshev step on level l from buffer src: the new values of the thread's nodes
  auto cheb_step = [&](const AfCoef<T> &cf, const Place &pl, const V2<T> *src, T c1, T c2, V2<T> (&x)[2]) {
    V2<T> s[2];
    product(src, pl, cf, x, s);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const V2<T> z = cell_dinv(cf, 2 * half + q, V2<T>{b[q].x - s[q].x, b[q].y - s[q].y});
      d[q] = V2<T>{(T)fma(c2, z.x, c1 * d[q].x), (T)fma(c2, z.y, c1 * d[q].y)};
      x[q] = V2<T>{x[q].x + d[q].x, x[q].y + d[q].y};
    }
  };
  // descent: pre-smoothing, residual, restriction
#pragma unroll 1
  for (int l = 0; l < a.nlev; ++l) {
    const TailLevel<T> &lv = a.lv[l];
    const Place pl = place(lv.n);
    const AfCoef<T> cf = pinned_coefs(lv.cf);
    V2<T> x[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {   // first step from zero: x = d = s D^{-1} b
      bs[2 * (kTailThreads * l) + kTailThreads * q + tid] = b[q];
      const V2<T> z = cell_dinv(cf, 2 * half + q, b[q]);
      x[q] = d[q] = V2<T>{lv.s * z.x, lv.s * z.y};
    }
    int k = 0;
    put(buf(l, k), pl, x);
    __syncthreads();
#pragma unroll 1
    for (int j = 0; j + 1 < kTailSteps; ++j, k ^= 1) {
      cheb_step(cf, pl, buf(l, k), lv.c1[j], lv.c2[j], x);
      put(buf(l, k ^ 1), pl, x);
      __syncthreads();
    }
    {   // the residual into the other buffer
      V2<T> s[2];
      product(buf(l, k), pl, cf, x, s);
#pragma unroll
      for (int q = 0; q < 2; ++q) s[q] = V2<T>{b[q].x - s[q].x, b[q].y - s[q].y};
      put(buf(l, k ^ 1), pl, s);
    }
    __syncthreads();
    {   // restriction: the next level's right-hand side at the thread's nodes there
      const int nc = lv.n / 2;
      const Place pc = place(nc);
      const V2<T> *r = buf(l, k ^ 1);
      b[0] = b[1] = V2<T>{T(0), T(0)};
      if (half) {
        if (pc.in[0]) b[0] = tail_restrict<T, 0, 1>(r, pc.i, pc.j);
        if (pc.in[1]) b[1] = tail_restrict<T, 1, 1>(r, pc.i, pc.j);
      } else {
        if (pc.in[0]) b[0] = tail_restrict<T, 0, 0>(r, pc.i, pc.j);
        if (pc.in[1]) b[1] = tail_restrict<T, 1, 0>(r, pc.i, pc.j);
      }
      if (l + 1 == a.nlev) {   // the coarsest level, row-major as its dense inverse
        const int Lc = lv.n + 1, q = (2 * pc.j + half) * Lc + 2 * pc.i;
        if (pc.in[0]) {
          db[q] = b[0].x;
          db[Lc * Lc + q] = b[0].y;
        }
        if (pc.in[1]) {
          db[q + 1] = b[1].x;
          db[Lc * Lc + q + 1] = b[1].y;
        }
      }
    }
  }
  __syncthreads();
  // coarsest level: x = C^{-1} b, sums in double
  if (dlive) {
    double s0 = 0.0, s1 = 0.0;
    const int k0 = dpart * kp;
    // the loads' first use: without this the FP32 kernel converts to double as they arrive and so
    // waits for all of them at the start (31 us a launch instead of 17)
#pragma unroll
    for (int q = 0; q < kTailDenseReg; ++q) asm volatile("" : "+v"(cr[q]));
    if (even) {
#pragma unroll
      for (int q = 0; q < kTailDenseReg; ++q) (q & 1 ? s1 : s0) += (double)cr[q] * (double)db[k0 + q];
    } else if (pre) {
#pragma unroll
      for (int q = 0; q < kTailDenseReg; ++q)
        if (q < kp) (q & 1 ? s1 : s0) += (double)cr[q] * (double)db[k0 + q];
    } else {
      const int k1 = k0 + kp < m ? k0 + kp : m;
#pragma unroll 8
      for (int k = k0; k < k1; ++k) s0 += (double)a.cinv[(int64_t)k * m + drow] * (double)db[k];
    }
    dp[dpart * m + drow] = s0 + s1;
  }
  __syncthreads();
  if (tid < m) {
    double s = 0.0;
    for (int q = 0; q < P; ++q) s += dp[q * m + tid];
    dx[tid] = (T)s;
  }
  __syncthreads();
  // ascent: coarse correction, post-smoothing
  constexpr int kend = (kTailSteps - 1) & 1;   // buffer that the pre-smoothing left the iterate in
#pragma unroll 1
  for (int l = a.nlev - 1; l >= 0; --l) {
    const TailLevel<T> &lv = a.lv[l];
    const Place pl = place(lv.n);
    const AfCoef<T> cf = pinned_coefs(lv.cf);
    V2<T> x[2];
    b[0] = bs[2 * (kTailThreads * l) + tid];
    b[1] = bs[2 * (kTailThreads * l) + kTailThreads + tid];
    if (pl.in[1]) {
      const int Ib = 2 * (pl.i >> 1), Jb = 2 * (pl.j >> 1), A = 2 * (pl.i & 1), B = 2 * (pl.j & 1) + half;
      const V2<T> *p = buf(l, kend) + pl.at + half * kTailHW;
      x[0] = p[0];
      x[1] = p[kTailPL];
      auto add = [&](auto c) {
        const V2<T> p0 = tail_prolong<T>(c, A, B), p1 = tail_prolong<T>(c, A + 1, B);
        x[0] = V2<T>{x[0].x + p0.x, x[0].y + p0.y};
        x[1] = V2<T>{x[1].x + p1.x, x[1].y + p1.y};
      };
      if (l + 1 == a.nlev) {
        const int Lc = lv.n + 1;
        add([&](int ai, int bj) -> V2<T> {
          const int q = (Jb + bj) * Lc + Ib + ai;
          return V2<T>{dx[q], dx[Lc * Lc + q]};
        });
      } else {   // the next level's iterate: the buffer that its post-smoothing ended on
        const V2<T> *xc = buf(l + 1, kend ^ (kTailSteps & 1));
        add([&](int ai, int bj) -> V2<T> { return xc[tail_at(Ib + ai, Jb + bj)]; });
      }
    }
    put(buf(l, kend), pl, x);
    __syncthreads();
    int k = kend;
#pragma unroll 1
    for (int j = 0; j < kTailSteps; ++j, k ^= 1) {
      if (j == 0) d[0] = d[1] = V2<T>{T(0), T(0)};
      cheb_step(cf, pl, buf(l, k), j == 0 ? T(0) : lv.c1[j - 1], j == 0 ? lv.s : lv.c2[j - 1], x);
      if (l == 0 && j + 1 == kTailSteps) break;   // the result goes to device memory
      put(buf(l, k ^ 1), pl, x);
      __syncthreads();
    }
    if (l == 0 && pl.j < lv.n) {
      const int L = 2 * lv.n + 1, NG = L * L, r = (2 * pl.j + half) * L + 2 * pl.i;
      const V2<T> v0 = pl.in[0] ? x[0] : V2<T>{T(0), T(0)}, v1 = pl.in[1] ? x[1] : V2<T>{T(0), T(0)};
      xg[r] = v0.x;
      xg[r + 1] = v1.x;
      xg[NG + r] = v0.y;
      xg[NG + r + 1] = v1.y;
    }
  }
}

}  // namespace

int tail_lds_limit() {
  static int limit = [] {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
      v = 65536;
    v = v < 65536 ? v : v > 163840 ? 163840 : v;
    // dynamic LDS above 64 KiB is granted per kernel
    if (v > 65536 && (hipFuncSetAttribute((const void *)k_mg_tail<double>,
                                          hipFuncAttributeMaxDynamicSharedMemorySize, v) != hipSuccess ||
                      hipFuncSetAttribute((const void *)k_mg_tail<float>,
                                          hipFuncAttributeMaxDynamicSharedMemorySize, v) != hipSuccess)) {
      (void)hipGetLastError();
      v = 65536;
    }
    return v;
  }();
  return limit;
}

template <typename T>
void mg_tail(const TailArgs<T> &a, hipStream_t s, int K) {
  FSI_REQUIRE(a.nlev >= 1 && a.nlev <= kTailMax, FSI_E_ARG, "coarse tail shape out of range");
  FSI_REQUIRE(a.lv[0].n <= kTailMaxN, FSI_E_ARG, "coarse tail level too fine");
  for (int l = 0; l + 1 < a.nlev; ++l)
    FSI_REQUIRE(a.lv[l + 1].n * 2 == a.lv[l].n, FSI_E_ARG, "coarse tail levels not nested");
  FSI_REQUIRE(a.m == 2 * (a.lv[a.nlev - 1].n + 1) * (a.lv[a.nlev - 1].n + 1) && a.m <= kTailDenseMax, FSI_E_ARG,
              "coarse tail coarsest level out of range");
  FSI_REQUIRE(K >= 1 && K <= 65535 && (K == 1 || a.lb > 0), FSI_E_ARG, "lane count out of range");
  FSI_REQUIRE(a.lds <= tail_lds_limit(), FSI_E_ARG, "coarse tail exceeds the LDS of a block");
  hipLaunchKernelGGL(k_mg_tail<T>, dim3(1, (unsigned)K), dim3(kTailThreads), a.lds, s, a);
  FSI_CHECK_LAUNCH();
}
template void mg_tail<double>(const TailArgs<double> &, hipStream_t, int);
template void mg_tail<float>(const TailArgs<float> &, hipStream_t, int);

}  // namespace fsi
