// Geometric factors of a trilinear hexahedron, formed where a kernel needs them.
//
// x(xi) = c0 + sum_d c_d xi_d + c12 xi_1 xi_2 + c13 xi_1 xi_3 + c23 xi_2 xi_3 + c123 xi_1 xi_2 xi_3,
// so along a line of fixed (xi_1, xi_2) the columns of J = dx/dxi are
//   J1 = P1 + xi_3 Q1,  J2 = P2 + xi_3 Q2,  J3 constant,
// and what the quadrature function needs is a short polynomial in xi_3 whose coefficients
// a thread that owns the line keeps in registers: one element is 21 doubles in memory
// instead of 6 or 9 factors per point.  Two forms:
//   LineGeom    the rows of adj(J) = |J| J^{-1}: r1 = J2 x J3, r2 = J3 x J1 (degree 1),
//               r3 = J1 x J2 (degree 2); w |J| J^{-1} J^{-T} = (w / |J|) adj adj^T is applied
//               as two products with adj;
//   LineMetric  the metric M = J^T J (degree at most 2) and adj adj^T = adj(M), 12 operations
//               per point.  adj(M) cancels where two columns of J are nearly parallel: its
//               entries lose 3e-16 / sin^2 of their angle (LineGeom: 1e-16 / sin).  It serves
//               the float32 operators, whose factors are rounded from it, on meshes without
//               such elements (kMetricLimit), and LineGeom those with.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rules.h"

namespace sfem {

// Stored per element, float64: c1, c2, c3, c12, c13, c23, c123 (3 components each), padded.
constexpr int kGeoStride = 24;

// Largest 1 / sin^2 of the angle between two columns of J (each of the element's largest length
// along its direction) at a quadrature point for which the float32 operators form their factors by
// LineMetric: 3e-10 of error at the limit, against 6e-8 of the rounding to float32.
constexpr double kMetricLimit = 1048576.0;

// Gauss rule with q points, indexed by the thread.
template <int Q>
__constant__ rules::GaussRule<Q> kGaussRule = rules::gauss<Q>();

__device__ __forceinline__ void cross3(const double (&u)[3], const double (&v)[3], double (&w)[3]) {
  w[0] = u[1] * v[2] - u[2] * v[1];
  w[1] = u[2] * v[0] - u[0] * v[2];
  w[2] = u[0] * v[1] - u[1] * v[0];
}
__device__ __forceinline__ double dot3(const double (&u)[3], const double (&v)[3]) {
  return u[0] * v[0] + u[1] * v[1] + u[2] * v[2];
}

// J1 = P1 + xi_3 Q1, J2 = P2 + xi_3 Q2 and J3 along the line (x1, x2) of an element with
// stored coefficients g.
__device__ __forceinline__ void line_columns(const double *g, double x1, double x2, double (&P1)[3],
                                             double (&Q1)[3], double (&P2)[3], double (&Q2)[3],
                                             double (&J3)[3]) {
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    P1[r] = g[r] + g[9 + r] * x2;
    Q1[r] = g[12 + r] + g[18 + r] * x2;
    P2[r] = g[3 + r] + g[9 + r] * x1;
    Q2[r] = g[15 + r] + g[18 + r] * x1;
    J3[r] = (g[6 + r] + g[12 + r] * x1) + Q2[r] * x2;
  }
}

// Coefficients of adj(J)'s rows and of |J| along a thread's xi_3 line.
struct LineGeom {
  double a1[3], b1[3], a2[3], b2[3], a3[3], b3[3], c3[3];
  double d0, d1, d2;

  __device__ __forceinline__ void init(const double *g, double x1, double x2) {
    double P1[3], Q1[3], P2[3], Q2[3], J3[3];
    line_columns(g, x1, x2, P1, Q1, P2, Q2, J3);
    double m[3];
    cross3(P2, J3, a1);
    cross3(Q2, J3, b1);
    cross3(J3, P1, a2);
    cross3(J3, Q1, b2);
    cross3(P1, P2, a3);
    d0 = dot3(J3, a3);
    cross3(P1, Q2, b3);
    cross3(Q1, P2, m);
#pragma unroll
    for (int r = 0; r < 3; ++r) b3[r] += m[r];
    d1 = dot3(J3, b3);
    cross3(Q1, Q2, c3);
    d2 = dot3(J3, c3);
  }
  // rows of adj(J) and |J| at xi_3 = x
  __device__ __forceinline__ void adj(double x, double (&r1)[3], double (&r2)[3], double (&r3)[3]) const {
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      r1[r] = a1[r] + x * b1[r];
      r2[r] = a2[r] + x * b2[r];
      r3[r] = (a3[r] + (x * x) * c3[r]) + x * b3[r];
    }
  }
  __device__ __forceinline__ double det(double x) const { return (d0 + (x * x) * d2) + x * d1; }
  // s adj adj^T at xi_3 = x as (11, 22, 33, 12, 13, 23), rounded to float32
  __device__ __forceinline__ void factors(double x, double s, float (&G)[6]) const {
    double r1[3], r2[3], r3[3];
    adj(x, r1, r2, r3);
    G[0] = (float)(s * dot3(r1, r1));
    G[1] = (float)(s * dot3(r2, r2));
    G[2] = (float)(s * dot3(r3, r3));
    G[3] = (float)(s * dot3(r1, r2));
    G[4] = (float)(s * dot3(r1, r3));
    G[5] = (float)(s * dot3(r2, r3));
  }
};

// Coefficients of the metric M = J^T J and of |J| along a thread's xi_3 line.
struct LineMetric {
  double m11[3], m22[3], m12[3], m13[2], m23[2], m33;
  double d0, d1, d2;

  __device__ __forceinline__ void init(const double *g, double x1, double x2) {
    double P1[3], Q1[3], P2[3], Q2[3], J3[3], u[3];
    line_columns(g, x1, x2, P1, Q1, P2, Q2, J3);
    m11[0] = dot3(P1, P1);
    m11[1] = 2.0 * dot3(P1, Q1);
    m11[2] = dot3(Q1, Q1);
    m22[0] = dot3(P2, P2);
    m22[1] = 2.0 * dot3(P2, Q2);
    m22[2] = dot3(Q2, Q2);
    m12[0] = dot3(P1, P2);
    m12[1] = dot3(P1, Q2) + dot3(Q1, P2);
    m12[2] = dot3(Q1, Q2);
    m13[0] = dot3(P1, J3);
    m13[1] = dot3(Q1, J3);
    m23[0] = dot3(P2, J3);
    m23[1] = dot3(Q2, J3);
    m33 = dot3(J3, J3);
    cross3(P2, J3, u);  // |J| = J1 . (J2 x J3)
    d0 = dot3(P1, u);
    d1 = dot3(Q1, u);
    cross3(Q2, J3, u);
    d1 += dot3(P1, u);
    d2 = dot3(Q1, u);
  }
  __device__ __forceinline__ double det(double x) const { return (d0 + (x * x) * d2) + x * d1; }

  // s adj(M) at xi_3 = x as (11, 22, 33, 12, 13, 23), rounded to float32
  __device__ __forceinline__ void factors(double x, double s, float (&G)[6]) const {
    const double a = (m11[0] + (x * x) * m11[2]) + x * m11[1];
    const double b = (m22[0] + (x * x) * m22[2]) + x * m22[1];
    const double c = (m12[0] + (x * x) * m12[2]) + x * m12[1];
    const double e = m13[0] + x * m13[1], f = m23[0] + x * m23[1];
    G[0] = (float)(s * (b * m33 - f * f));
    G[1] = (float)(s * (a * m33 - e * e));
    G[2] = (float)(s * (a * b - c * c));
    G[3] = (float)(s * (e * f - c * m33));
    G[4] = (float)(s * (c * f - e * b));
    G[5] = (float)(s * (c * e - a * f));
  }
};

// Component d (physical direction) of adj(J)'s three rows along a thread's xi_3 line, for
// kernels that take one physical direction after the other: 7 coefficients at a time.
// Sixty-four threads of a wave read the element's coefficients g from LDS.
struct LineAdjComp {
  double a1, b1, a2, b2, a3, b3, c3;

  __device__ __forceinline__ void init(const double *g, int d, double x1, double x2) {
    double P1[2], Q1[2], P2[2], Q2[2], J3[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {  // the two other components, in cyclic order
      const int r = d + 1 + k < 3 ? d + 1 + k : d - 2 + k;
      P1[k] = g[r] + g[9 + r] * x2;
      Q1[k] = g[12 + r] + g[18 + r] * x2;
      P2[k] = g[3 + r] + g[9 + r] * x1;
      Q2[k] = g[15 + r] + g[18 + r] * x1;
      J3[k] = (g[6 + r] + g[12 + r] * x1) + Q2[k] * x2;
    }
    auto cross = [](const double (&u)[2], const double (&v)[2]) { return u[0] * v[1] - u[1] * v[0]; };
    a1 = cross(P2, J3);
    b1 = cross(Q2, J3);
    a2 = cross(J3, P1);
    b2 = cross(J3, Q1);
    a3 = cross(P1, P2);
    b3 = cross(P1, Q2) + cross(Q1, P2);
    c3 = cross(Q1, Q2);
  }
  __device__ __forceinline__ void at(double x, double &r1, double &r2, double &r3) const {
    r1 = a1 + x * b1;
    r2 = a2 + x * b2;
    r3 = (a3 + (x * x) * c3) + x * b3;
  }
};

// 1 / d for the positive |J| of a valid element: the hardware estimate and Newton steps.
__device__ __forceinline__ double recip(double d) {
  double r = __builtin_amdgcn_rcp(d);
  r = __builtin_fma(r, __builtin_fma(-d, r, 1.0), r);
  return __builtin_fma(r, __builtin_fma(-d, r, 1.0), r);
}

}  // namespace sfem
