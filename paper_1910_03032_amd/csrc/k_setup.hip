// Setup kernels: the elements' trilinear coefficients, the check of |J|, physical
// quadrature-point coordinates, the coefficient w nu / |J| of the applies, the collocated
// mass, precision casts.
#include <hip/hip_runtime.h>

#include "geom.h"
#include "internal.h"
#include "flow.h"

namespace sfem {
namespace {

struct GaussArg {
  double x[SFEM_MAX_P + 2];
  double w[SFEM_MAX_P + 2];
};

// Trilinear map through the 8 vertices (vertex v = i + 2j + 4k at reference corner
// (2i-1, 2j-1, 2k-1)): position and Jacobian J[r][d] = dx_r / dxi_d.
__device__ inline void trilinear(const double *X, const double xi[3], double pos[3],
                                 double J[3][3]) {
  for (int r = 0; r < 3; ++r) {
    pos[r] = 0.0;
    for (int d = 0; d < 3; ++d) J[r][d] = 0.0;
  }
  for (int v = 0; v < 8; ++v) {
    double s[3], f[3];
    for (int d = 0; d < 3; ++d) {
      s[d] = ((v >> d) & 1) ? 1.0 : -1.0;
      f[d] = 0.5 * (1.0 + s[d] * xi[d]);
    }
    const double Nv = f[0] * f[1] * f[2];
    const double dN0 = 0.5 * s[0] * f[1] * f[2];
    const double dN1 = 0.5 * s[1] * f[0] * f[2];
    const double dN2 = 0.5 * s[2] * f[0] * f[1];
    for (int r = 0; r < 3; ++r) {
      const double Xr = X[v * 3 + r];
      pos[r] += Xr * Nv;
      J[r][0] += Xr * dN0;
      J[r][1] += Xr * dN1;
      J[r][2] += Xr * dN2;
    }
  }
}

// Rank of local node l among the surface nodes of an order-p element (same order as the
// host plan and the element kernels), -1 for an interior node.
__device__ inline int surface_rank_rt(int p, int l) {
  const int n = p + 1;
  const int i = l % n, j = (l / n) % n, k = l / (n * n);
  if (k == 0) return i + n * j;
  if (k == p) return n * n + i + n * j;
  const int base = 2 * n * n + (k - 1) * 4 * p;
  if (j == 0) return base + i;
  if (j == p) return base + n + i;
  if (i == 0 || i == p) return base + 2 * n + 2 * (j - 1) + (i == 0 ? 0 : 1);
  return -1;
}

// Collocated mass (Section 5.1): integrating the mass matrix with the GLL rule at the
// nodes themselves makes it diagonal; element node l contributes w_l |J(xi_l)| (tensor
// GLL weight times the Jacobian determinant at the node).  Written like an element
// output: sole DoFs directly into diag, shared nodes into their E-vector entry,
// essential DoFs not at all (the assembly sets them).
__global__ void colloc_mass_kernel(GaussArg g, int p, const double *__restrict__ xyz,
                                   const int32_t *__restrict__ map, const int32_t *__restrict__ pos,
                                   int compact, int64_t nelem, double *__restrict__ diag,
                                   double *__restrict__ Y) {
  const int n = p + 1, n3 = n * n * n;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= nelem * n3) return;
  const int64_t e = gid / n3;
  const int l = (int)(gid - e * n3);
  const int i = l % n, j = (l / n) % n, k = l / (n * n);
  const int32_t c = map[gid];
  if (c < 0) return;
  const double xi[3] = {g.x[i], g.x[j], g.x[k]};
  double x3[3], J[3][3];
  trilinear(xyz + e * 24, xi, x3, J);
  const double det = J[0][0] * (J[1][1] * J[2][2] - J[1][2] * J[2][1]) -
                     J[0][1] * (J[1][0] * J[2][2] - J[1][2] * J[2][0]) +
                     J[0][2] * (J[1][0] * J[2][1] - J[1][1] * J[2][0]);
  const double v = g.w[i] * g.w[j] * g.w[k] * det;
  if (c & kSoleBit) {
    diag[c & kDofMask] = v;
  } else {
    const int S = p == 1 ? 8 : 2 * n * n + (n - 2) * 4 * p;
    const int64_t q = compact ? e * S + surface_rank_rt(p, l) : gid;
    Y[pos ? pos[q] : q] = v;
  }
}

// |J| > 0 at the quadrature points (else, or not a number, bad[0] = 1), and no two columns of J
// nearly parallel there (else bad[1] = 1; kMetricLimit).
__global__ void check_det_kernel(GaussArg g, int q, const double *__restrict__ xyz, int64_t nei,
                                 int *__restrict__ bad) {
  const int64_t q3 = (int64_t)q * q * q;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= nei * q3) return;
  const int64_t e = gid / q3;
  const int qi = (int)(gid - e * q3);
  const int a = qi % q, b = (qi / q) % q, c = qi / (q * q);
  const double xi[3] = {g.x[a], g.x[b], g.x[c]};
  double pos[3], J[3][3];
  trilinear(xyz + e * 24, xi, pos, J);
  // |J| by the first column of the adjugate
  const double A00 = J[1][1] * J[2][2] - J[1][2] * J[2][1];
  const double A10 = J[1][2] * J[2][0] - J[1][0] * J[2][2];
  const double A20 = J[1][0] * J[2][1] - J[1][1] * J[2][0];
  const double det = J[0][0] * A00 + J[0][1] * A10 + J[0][2] * A20;
  if (!(det > 0.0)) bad[0] = 1;
  // squared lengths: the longest edge along each direction (halved, as the columns of J)
  const double *X = xyz + e * 24;
  double len[3] = {0.0, 0.0, 0.0};
  for (int d = 0; d < 3; ++d)
    for (int v = 0; v < 8; ++v) {
      if ((v >> d) & 1) continue;
      double s = 0.0;
      for (int r = 0; r < 3; ++r) {
        const double h = 0.5 * (X[(v + (1 << d)) * 3 + r] - X[v * 3 + r]);
        s += h * h;
      }
      len[d] = s > len[d] ? s : len[d];
    }
  for (int i = 0; i < 3; ++i) {
    const int j = i == 2 ? 0 : i + 1;
    const double u[3] = {J[0][i], J[1][i], J[2][i]}, v[3] = {J[0][j], J[1][j], J[2][j]};
    double c[3];
    cross3(u, v, c);
    if (len[i] * len[j] > kMetricLimit * dot3(c, c)) bad[1] = 1;
  }
}

__global__ void qpoint_coords_kernel(GaussArg g, int q, const double *__restrict__ xyz,
                                     int64_t nei, double *__restrict__ xq) {
  const int64_t q3 = (int64_t)q * q * q;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= nei * q3) return;
  const int64_t e = gid / q3;
  const int qi = (int)(gid - e * q3);
  const int a = qi % q, b = (qi / q) % q, c = qi / (q * q);
  const double xi[3] = {g.x[a], g.x[b], g.x[c]};
  double pos[3], J[3][3];
  trilinear(xyz + e * 24, xi, pos, J);
  const int64_t o = e * q3 + qi;
  const int64_t plane = nei * q3;
  xq[o] = pos[0];
  xq[plane + o] = pos[1];
  xq[2 * plane + o] = pos[2];
}

// Trilinear coefficients of the elements: sums of vertex differences, so that no digits are
// lost to the element's distance from the origin.
__global__ void geo_setup_kernel(const double *__restrict__ xyz, int64_t nei, double *__restrict__ geo) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= nei * 3) return;
  const int64_t e = gid / 3;
  const int r = (int)(gid - e * 3);
  const double *X = xyz + e * 24 + r;
  // differences along xi_1 of the edges (j, k), and along xi_2, xi_3 of the xi_1 = -1 face
  const double d00 = X[3] - X[0], d10 = X[9] - X[6], d01 = X[15] - X[12], d11 = X[21] - X[18];
  const double f0 = X[6] - X[0], f1 = X[9] - X[3], f2 = X[18] - X[12], f3 = X[21] - X[15];
  const double h0 = X[12] - X[0], h1 = X[15] - X[3], h2 = X[18] - X[6], h3 = X[21] - X[9];
  double *o = geo + e * kGeoStride + r;
  o[0] = 0.125 * ((d00 + d10) + (d01 + d11));
  o[3] = 0.125 * ((f0 + f1) + (f2 + f3));
  o[6] = 0.125 * ((h0 + h1) + (h2 + h3));
  o[9] = 0.125 * ((d10 - d00) + (d11 - d01));
  o[12] = 0.125 * ((d01 - d00) + (d11 - d10));
  o[15] = 0.125 * ((f2 - f0) + (f3 - f1));
  o[18] = 0.125 * ((d11 - d10) - (d01 - d00));
  o[21] = 0.0;
}

// cw[f][e][point] = w nu_f / |J|, the one coefficient the element kernel reads per point, and
// a copy of nu.
__global__ void fold_kernel(GaussArg g, int q, const double *__restrict__ geo,
                            const double *__restrict__ nu_user, int64_t nei, int nfield,
                            double *__restrict__ cw, double *__restrict__ nu64) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t q3 = (int64_t)q * q * q, per_field = nei * q3;
  if (gid >= per_field * nfield) return;
  const int64_t f = gid / per_field, r = gid - f * per_field, e = r / q3;
  const int qi = (int)(r - e * q3);
  const int a = qi % q, b = (qi / q) % q, c = qi / (q * q);
  LineGeom L;
  L.init(geo + e * kGeoStride, g.x[a], g.x[b]);
  const double nv = nu_user[gid];
  cw[gid] = g.w[a] * g.w[b] * g.w[c] * nv / L.det(g.x[c]);
  nu64[gid] = nv;
}

__global__ void cast_kernel(const double *__restrict__ src, float *__restrict__ dst, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    dst[i] = (float)src[i];
}

GaussArg gauss_arg(const double *rules_x, const double *rules_w, int q) {
  GaussArg g{};
  for (int i = 0; i < q; ++i) {
    g.x[i] = rules_x[i];
    g.w[i] = rules_w[i];
  }
  return g;
}

unsigned nblocks(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

hipError_t launch_check_det(int q, const double *gx, const double *gw, const double *xyz, int64_t nei,
                            int *bad, hipStream_t s) {
  const int64_t n = nei * (int64_t)q * q * q;
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(check_det_kernel, dim3(nblocks(n, 256)), dim3(256), 0, s, gauss_arg(gx, gw, q), q, xyz,
                     nei, bad);
  return hipGetLastError();
}

hipError_t launch_qpoint_coords(int q, const double *gx, const double *gw, const double *xyz,
                                int64_t nei, double *xq, hipStream_t s) {
  const int64_t n = nei * (int64_t)q * q * q;
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(qpoint_coords_kernel, dim3(nblocks(n, 256)), dim3(256), 0, s,
                     gauss_arg(gx, gw, q), q, xyz, nei, xq);
  return hipGetLastError();
}

hipError_t launch_geo_setup(const double *xyz, int64_t nei, double *geo, hipStream_t s) {
  if (nei == 0) return hipSuccess;
  hipLaunchKernelGGL(geo_setup_kernel, dim3(nblocks(nei * 3, 256)), dim3(256), 0, s, xyz, nei, geo);
  return hipGetLastError();
}

hipError_t launch_fold(int q, const double *gx, const double *gw, const double *geo, const double *nu_user,
                       int64_t nei, int nfield, double *cw, double *nu64, hipStream_t s) {
  const int64_t n = nei * (int64_t)q * q * q * nfield;
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(fold_kernel, dim3(nblocks(n, 256)), dim3(256), 0, s, gauss_arg(gx, gw, q), q, geo,
                     nu_user, nei, nfield, cw, nu64);
  return hipGetLastError();
}

hipError_t launch_colloc_mass(int p, const double *gll_x, const double *gll_w, const double *xyz,
                              const int32_t *map, const int32_t *pos, int compact, int64_t nelem,
                              double *diag, double *evec, hipStream_t s) {
  const int64_t n = nelem * (int64_t)(p + 1) * (p + 1) * (p + 1);
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(colloc_mass_kernel, dim3(nblocks(n, 256)), dim3(256), 0, s,
                     gauss_arg(gll_x, gll_w, p + 1), p, xyz, map, pos, compact, nelem, diag, evec);
  return hipGetLastError();
}

hipError_t launch_cast_f32(const double *src, float *dst, int64_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const int64_t nb = (n + 255) / 256;
  hipLaunchKernelGGL(cast_kernel, dim3((unsigned)(nb < 65536 ? nb : 65536)), dim3(256), 0, s, src,
                     dst, n);
  return hipGetLastError();
}

}  // namespace sfem
