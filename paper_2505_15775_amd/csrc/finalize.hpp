// What the finalizers do with their totals, for the one-block kernels and for the
// kernels that run the finalizer of the one before in a block of their own.
#pragma once

#include <math.h>

#include "kernels.hpp"

namespace almbm {

// Objective totals of the DIAG family (one thread).  mode 0: API call, writes *f_out.
// mode 1: inner loop step 1 -- after max_inner steps stop (flag 2), else the
// stop test ||G|| ||R|| <= tol (1 + |<C,RR^T>|) (flag 1), else count the step.
__device__ __forceinline__ void finish_objgrad(const double* tot, DevScalars* sc, double sigma, int mode,
                                               double* f_out) {
  const double f = tot[P_C0] + tot[P_YBMA] + 0.5 * sigma * tot[P_EE];
  sc->f = f;
  if (!isfinite(f) || !isfinite(tot[P_GG])) sc->numeric_error = 1;
  if (f_out) *f_out = f;
  if (mode == 1) {
    const double lhs = sqrt(tot[P_GG]) * sqrt(tot[P_RR]);
    if (sc->iter >= sc->max_inner) {
      sc->flag = 2;
    } else if (lhs <= sc->tol * (1.0 + fabs(tot[P_C0])) || !isfinite(lhs)) {
      sc->flag = 1;
    } else {
      sc->iter += 1;
    }
  }
}

// Direction-dependent totals of the quartic (one thread).
__device__ __forceinline__ void finish_lsdir(const double* tot, DevScalars* sc, LbfgsState* S) {
  constexpr int K = 10;
  const int sl[K] = {P_GG, P_GP, P_YA1, P_YA2, P_EA1, P_EA2, P_A1A1, P_A1A2, P_A2A2, P_RG};
#pragma unroll
  for (int k = 0; k < K; ++k) sc->tot[sl[k]] = tot[sl[k]];
  S->ee = tot[P_GG];
}

// The stop flag as one thread reads it, for the kernels beside whose blocks a side
// block may be setting it: all waves of a block take the same way.
__device__ __forceinline__ bool block_stopped(const DevScalars* sc) {
  __shared__ int stop;
  if (threadIdx.x == 0) stop = sc->flag;
  __syncthreads();
  return stop != 0;
}

// The side block: true (and the work done) in the last block of a grid that has one.
__device__ __forceinline__ bool run_side_fin(const SideFin& f) {
  if (!f.part || blockIdx.x != gridDim.x - 1) return false;
  if (block_stopped(f.sc)) return true;
  __shared__ double tot[NUM_P];
  fin_rows<NUM_P, kBlock>(f.part, f.nb, tot);
  if (f.ls) {
    if (threadIdx.x == 0) finish_lsdir(tot, f.sc, f.ls);
  } else {
    if (threadIdx.x < NUM_P) f.sc->tot[threadIdx.x] = tot[threadIdx.x];
    if (threadIdx.x == 0) finish_objgrad(tot, f.sc, f.sigma, 1, nullptr);
  }
  return true;
}

}  // namespace almbm
