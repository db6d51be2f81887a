// Device-side scalars of the conjugate gradient kernels.
//
// One iteration is two launches.  The element kernel forms the direction as it gathers it,
// p = (z - zshift) + beta p_old with z = dinv r, applies the operator, and leaves the partial
// sums of p.Ap taken at the quadrature points (so they need no assembled vector); the update
// kernel assembles w = A p DoF by DoF, forms the same p again and writes p, x += alpha p,
// r -= alpha w with the partial sums of the new r.z and r.r.  Every block that needs a scalar
// sums the partials itself in a fixed order, on large problems what cg_fold_kernel and
// cg_finish_kernel have left of them (cg_plan.h).  The states alternate between two arrays, so
// that no block reads a value another block of the same launch writes: the element kernel
// reads the state the update left, adds beta (cg_next) and writes the other array; the
// update adds alpha (set_alpha).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"
#include "wave.h"

namespace sfem {

// A state in registers (copied field by field: a struct copy went through scratch memory).
__device__ __forceinline__ void copy_state(PcgScalars &to, const PcgScalars &from) {
  to.rho = from.rho;
  to.rr = from.rr;
  to.bb = from.bb;
  to.pw = from.pw;
  to.alpha = from.alpha;
  to.beta = from.beta;
  to.tol2 = from.tol2;
  to.active = from.active;
  to.status = from.status;
  to.iters = from.iters;
  to.pad = from.pad;
  to.zshift = from.zshift;
}

// CG step length from p.Ap (or the failure state).
__device__ __forceinline__ void set_alpha(PcgScalars &s, double pw) {
  s.pw = pw;
  s.alpha = 0.0;
  if (s.active) {
    if (!isfinite(pw)) {
      s.status = SFEM_E_NAN;
      s.active = 0;
    } else if (!(pw > 0.0)) {
      s.status = SFEM_E_BREAKDOWN;
      s.active = 0;
    } else {
      s.alpha = s.rho / pw;
    }
  }
}

// New direction coefficient from r.z and r.r, and the stopping test.
__device__ __forceinline__ void set_beta(PcgScalars &s, double rz, double rr) {
  s.beta = 0.0;
  if (s.active) {
    s.iters += 1;
    if (!isfinite(rz) || !isfinite(rr)) {
      s.status = SFEM_E_NAN;
      s.active = 0;
    } else {
      s.beta = rz / s.rho;
      s.rho = rz;
      s.rr = rr;
      if (rr <= s.tol2) s.active = 0;
    }
  }
}

// The state of the next iteration from the update's sums r.z, r.r, sum z and sum r over n
// unknowns; with nullspace the preconditioned residual is z - mean(z).
__device__ __forceinline__ void cg_next(PcgScalars &s, double rz, double rr, double sz, double sr,
                                        int nullspace, int64_t n) {
  const double zs = nullspace ? sz / (double)n : 0.0;
  if (s.active) s.zshift = zs;
  set_beta(s, rz - zs * sr, rr);
}

// The partials of K quantities (quantity k at p + k nblk, nblk <= kCgUpdateMax) that one thread of
// NW full waves sums: requested early (load), added and combined later (parts).  All loads are
// in flight together; a loop that waits for each costs microseconds at the head of every
// workgroup.
template <int NW, int K>
struct PartLoads {
  static_assert(4 * 64 * NW >= kCgUpdateMax, "partials beyond the loads would be dropped");
  double v[K][4];
  __device__ __forceinline__ void load(const double *__restrict__ p, int nblk) {
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = (int)threadIdx.x + j * NW * 64;
        v[k][j] = p[(int64_t)k * nblk + (i < nblk ? i : nblk - 1)];
      }
  }
  // sums of this wave into sh[k][wave]; a barrier has to follow (the last, partial wave of the
  // workgroup has no part in it)
  __device__ __forceinline__ void parts(double (&sh)[4][NW], int nblk) const {
    if (threadIdx.x >= NW * 64) return;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      double u = 0.0;
#pragma unroll
      for (int j = 0; j < 4; ++j) u += (int)threadIdx.x + j * NW * 64 < nblk ? v[k][j] : 0.0;
      u = wave_total(u);
      if ((threadIdx.x & 63) == 0) sh[k][threadIdx.x >> 6] = u;
    }
  }
};

// cg_next from the waves' parts of the update's sums (without nullspace only r.z and r.r).
template <int NW>
__device__ __forceinline__ void cg_next_from(PcgScalars &s, const double (&sh)[4][NW], int nullspace, int64_t n) {
  double u[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int w = 0; w < NW; ++w)
      if (k < 2 || nullspace) u[k] += sh[k][w];
  cg_next(s, u[0], u[1], u[2], u[3], nullspace, n);
}

// The direction at one entry; written with explicit fused operations so that every kernel
// that forms it gets the same bits.
__device__ __forceinline__ double cg_dir(double d, double r, double zs, double beta, double p) {
  return __builtin_fma(beta, p, __builtin_fma(d, r, -zs));
}
__device__ __forceinline__ float cg_dir(float d, float r, float zs, float beta, float p) {
  return __builtin_fmaf(beta, p, __builtin_fmaf(d, r, -zs));
}

}  // namespace sfem
