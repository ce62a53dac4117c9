// Scalar state of the inner MINRES recurrence of one system and its step, shared by the launches that
// take it (solve.hip: on its own or behind the sum of beta^2; stencil.hip: at the head of the A11 launch).
#pragma once

#include "common.h"

namespace fsi {

struct MinresState {
  double alfa, beta2;                         // dot products of the iteration
  double beta, oldb, dbar, epsln, phibar, cs, sn, beta1, tol;
  double s, c_r1;                             // 1 / beta, -beta / oldb
  double e, d, ginv, phi;                     // direction update
  double it, done, apply;                     // iterations; converged; update valid
  double slot;                                // slot of this iteration's Lanczos vector
};
constexpr int kMsRec = 5;                     // recorded per iteration: e, d, 1/gamma, phi, applied
constexpr int kMsDoubles = sizeof(MinresState) / sizeof(double);

// After the two dot products of an iteration: Givens rotation and the next coefficients,
// recorded in slot st->slot of the lane's history (B slots of kMsRec; the host starts a new
// block before the slots run out, and a slot out of range records nothing).
__device__ inline void ms_step(MinresState *st, double *hist, int B) {
  const int sl = (int)st->slot;
  double *h = (sl >= 0 && sl < B) ? hist + kMsRec * sl : nullptr;
  st->slot += 1.0;
  if (st->done != 0.0) {
    st->apply = 0.0;
    if (h) h[4] = 0.0;
    return;
  }
  const double alfa = st->alfa, nb2 = st->beta2;
  const double oldb = st->beta;
  const double beta = sqrt(nb2 > 0.0 ? nb2 : 0.0);
  const double oldeps = st->epsln;
  // the fused products are written out: the step has the same bits in every launch that takes it
  const double delta = fma(st->cs, st->dbar, st->sn * alfa);
  const double gbar = fma(st->sn, st->dbar, -(st->cs * alfa));
  st->epsln = st->sn * beta;
  st->dbar = -st->cs * beta;
  double gamma = sqrt(fma(gbar, gbar, beta * beta));
  if (gamma < 1e-300) gamma = 1e-300;
  st->cs = gbar / gamma;
  st->sn = beta / gamma;
  st->phi = st->cs * st->phibar;
  st->phibar = st->sn * st->phibar;
  st->e = oldeps;
  st->d = delta;
  st->ginv = 1.0 / gamma;
  st->apply = 1.0;
  if (h) {
    h[0] = st->e;
    h[1] = st->d;
    h[2] = st->ginv;
    h[3] = st->phi;
    h[4] = 1.0;
  }
  st->it += 1.0;
  st->oldb = oldb;
  st->beta = beta;
  st->s = beta > 0.0 ? 1.0 / beta : 0.0;
  st->c_r1 = beta > 0.0 ? -beta / oldb : 0.0;
  if (!(st->phibar > st->tol * st->beta1) || beta == 0.0 || !(alfa == alfa)) st->done = 1.0;
}

// What the host polls: one word per system in pinned memory, the state's number and two flags in a
// single 8-byte store (so that no order between stores matters): bit 0 converged, bit 1 non-finite.
__device__ __forceinline__ void ms_tell(unsigned long long *word, unsigned long long seq, const MinresState &s) {
  if (!word) return;
  const bool bad = !(s.phibar == s.phibar && s.beta == s.beta);
  __hip_atomic_store(word, seq << 2 | (bad ? 2u : 0u) | (s.done != 0.0 ? 1u : 0u), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_SYSTEM);
}

// beta^2 = the velocity tile sums, then the pressure sums, in the order of a block of 1024 threads (the
// same wherever it is formed): virtual thread v adds the parts v, v + 1024, ..., then waves, then the
// 16 wave sums.  One block of NT threads; red: 16 doubles of LDS; every thread gets the sum.
template <int NT>
__device__ __forceinline__ double ms_beta2(const double *part, int n, double *red) {
  constexpr int V = 1024 / NT;
  double acc[V];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    acc[v] = 0.0;
    for (int i = threadIdx.x + NT * v; i < n; i += 1024) acc[v] += part[i];
    acc[v] = wave_sum(acc[v]);
    if (threadIdx.x % kWave == 0) red[v * (NT / kWave) + threadIdx.x / kWave] = acc[v];
  }
  __syncthreads();
  double b = 0.0;
#pragma unroll
  for (int k = 0; k < 1024 / kWave; ++k) b += red[k];
  return b;
}

}  // namespace fsi
