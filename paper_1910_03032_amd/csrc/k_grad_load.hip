// Adjoint-gradient integrand and load vector, built from the same sum-factorized
// stages as the apply, with the geometric factors formed along each thread's xi_3 line
// (geom.h).
//
// Gradient: K depends on nu only through W = nu w|J| J^-1 J^-T (Section 3.1), so
// dJ/dnu_q = -lam^T (dA/dnu_q) u = -beta w|J| (J^-T grad_ref lam).(J^-T grad_ref u)
// = -beta (w / |J|) (adj^T grad_ref lam).(adj^T grad_ref u) at each quadrature point.  The
// result goes to the caller's element order.
//
// Load vector: b_i = sum_q w|J| f_q phi_i, i.e. the transposed stages with the
// mass weight only (B^T in each direction), assembled like the apply (the assembly
// kernel sets the essential entries to 0).
//
// Both were bound by the factors' bytes (6 and 1 of 8 per point); formed, the 25 x 26 x 24
// p = 4 gradient takes 35 instead of 58 us (17 x 18 x 16 p = 6: 31 of 73) and the load vector
// 23 instead of 34.
#include <hip/hip_runtime.h>

#include "apply_impl.h"

namespace sfem {
namespace {

// xi_3 lines of a field's three xi_1/xi_2-contracted forms, even-odd split.
template <int P>
struct Lines {
  eo::Split<P + 1, double> bb, gb, bg;
  __device__ __forceinline__ void read(const double *buf, int t) {
    double zbb[P + 1], zgb[P + 1], zbg[P + 1];
    load_z<P, double, true>(buf, t, zbb, zgb, zbg);
    bb = eo::split(zbb);
    gb = eo::split(zgb);
    bg = eo::split(zbg);
  }
  // reference gradient at slices c and q-1-c, and at the middle slice
  __device__ __forceinline__ void grad_pair(int c, double (&lo)[3], double (&hi)[3]) const {
    eo::out_pair<eo::Tab1<P, 0>>(bg, c, lo[0], hi[0]);
    eo::out_pair<eo::Tab1<P, 0>>(gb, c, lo[1], hi[1]);
    eo::out_pair<eo::Tab1<P, 1>>(bb, c, lo[2], hi[2]);
  }
  __device__ __forceinline__ void grad_mid(double (&m)[3]) const {
    m[0] = eo::out_mid<eo::Tab1<P, 0>>(bg);
    m[1] = eo::out_mid<eo::Tab1<P, 0>>(gb);
    m[2] = eo::out_mid<eo::Tab1<P, 1>>(bb);
  }
};

template <int P>
__global__ void __launch_bounds__(Dims<P>::THREADS, 2)
grad_kernel(const int32_t *__restrict__ map, const double *__restrict__ geo, double beta,
            int64_t nei, int nbatch, int64_t ndof, const double *__restrict__ u,
            const double *__restrict__ lam, double *__restrict__ g) {
  using D = Dims<P>;
  constexpr int Q = D::Q, Q2 = D::Q2, Q3 = D::Q3, TPE = D::TPE, E = D::E;
  constexpr rules::GaussRule<Q> gr = rules::gauss<Q>();
  __shared__ __align__(16) double smem[E * Lds<P>::BUF];
  __shared__ __align__(16) double sgeo[E * kGeoStride];
  const int le = threadIdx.x / TPE;
  const int t = threadIdx.x - le * TPE;
  const int64_t e0 = (int64_t)xcd_block() * E;
  const bool active = e0 + le < nei;
  const uint32_t rel = active ? le : 0;
  double *buf = smem + le * Lds<P>::BUF;
  Nodes<P> nd;
  nd.load_map(elem_tab<P>(map, nullptr, 1, e0), t, rel);
  load_geo<P>(sgeo + le * kGeoStride, geo, e0, rel, t);
  for (int m = 0; m < nbatch; ++m) {
    double uv[Nodes<P>::NL];  // both fields' nodal values in flight together
    nd.load_values(u + (int64_t)m * ndof, uv);
    Lines<P> a, b;
    gather_e<P, double>(buf, t, active, nd, lam + (int64_t)m * ndof);
    fwd_x<P, double, true>(buf, t);
    fwd_y<P, double, true>(buf, t);
    a.read(buf, t);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < Nodes<P>::NL; ++k)
      buf[Lds<P>::nodal(Nodes<P>::node(t, k))] = (active && nd.c[k] >= 0) ? uv[k] : 0.0;
    __syncthreads();
    fwd_x<P, double, true>(buf, t);
    fwd_y<P, double, true>(buf, t);
    b.read(buf, t);
    __syncthreads();  // buf is reused by the next member
    LineGeom L;
    L.init(sgeo + le * kGeoStride, kGaussRule<Q>.x[t % Q], kGaussRule<Q>.x[t / Q]);
    const double wab = kGaussRule<Q>.w[t % Q] * kGaussRule<Q>.w[t / Q];
    double *go = g + ((int64_t)m * nei + e0 + rel) * Q3 + t;
    auto point = [&](int c, const double (&x)[3], const double (&y)[3]) {
      double r1[3], r2[3], r3[3], s = 0.0;
      L.adj(gr.x[c], r1, r2, r3);
#pragma unroll
      for (int r = 0; r < 3; ++r)
        s += (r1[r] * x[0] + r2[r] * x[1] + r3[r] * x[2]) * (r1[r] * y[0] + r2[r] * y[1] + r3[r] * y[2]);
      if (active) go[c * Q2] = -beta * ((wab * gr.w[c]) * recip(L.det(gr.x[c]))) * s;
    };
#pragma unroll
    for (int c = 0; c < Q / 2; ++c) {
      double xl[3], xh[3], yl[3], yh[3];
      a.grad_pair(c, xl, xh);
      b.grad_pair(c, yl, yh);
      point(c, xl, yl);
      point(Q - 1 - c, xh, yh);
    }
    if constexpr (Q % 2 == 1) {
      double x[3], y[3];
      a.grad_mid(x);
      b.grad_mid(y);
      point(Q / 2, x, y);
    }
  }
}

template <int P, bool POS>
__global__ void __launch_bounds__(Dims<P>::THREADS)
load_kernel(const int32_t *__restrict__ map, const double *__restrict__ geo, int64_t nei,
            int nbatch, int64_t ndof, const double *__restrict__ f, double *__restrict__ b,
            double *__restrict__ Y, int64_t estride, const int32_t *__restrict__ pos, int compact) {
  using D = Dims<P>;
  using BT = eo::Tab1<P, 0>;
  constexpr int N = D::N, Q = D::Q, Q2 = D::Q2, Q3 = D::Q3, TPE = D::TPE, E = D::E;
  constexpr rules::GaussRule<Q> gr = rules::gauss<Q>();
  __shared__ __align__(16) double smem[E * Lds<P, false>::BUF];
  __shared__ __align__(16) double sgeo[E * kGeoStride];
  __shared__ int32_t smap_all[E * D::N3];
  const int le = threadIdx.x / TPE;
  const int t = threadIdx.x - le * TPE;
  const int64_t e0 = (int64_t)xcd_block() * E;
  const bool active = e0 + le < nei;
  const uint32_t rel = active ? le : 0;
  double *buf = smem + le * Lds<P, false>::BUF;
  int32_t *smap = smap_all + le * D::N3;
  double fv[Q];  // the next source's values at the line's points
  auto load_f = [&](int m) {
    const double *fe = f + ((int64_t)m * nei + e0 + rel) * Q3 + t;
#pragma unroll
    for (int c = 0; c < Q; ++c) fv[c] = fe[c * Q2];
  };
  {
    const ElemTab z = elem_tab<P>(map, pos, compact, e0);
    Nodes<P> nd;
    nd.load_map(z, t, rel);
    nd.load_rank(z, t);
    load_f(0);
    load_geo<P>(sgeo + le * kGeoStride, geo, e0, rel, t);
    nd.template load_dest<POS>(z, rel);
    nd.keep(smap, t);
  }
  __syncthreads();
  double wd[Q];  // w|J| along the line
  {
    LineGeom L;
    L.init(sgeo + le * kGeoStride, kGaussRule<Q>.x[t % Q], kGaussRule<Q>.x[t / Q]);
    const double wab = kGaussRule<Q>.w[t % Q] * kGaussRule<Q>.w[t / Q];
#pragma unroll
    for (int c = 0; c < Q; ++c) wd[c] = (wab * gr.w[c]) * L.det(gr.x[c]);
  }
  for (int m = 0; m < nbatch; ++m) {
    double p1[N];
#pragma unroll
    for (int c = 0; c < Q; ++c) fv[c] *= wd[c];
    eo::Acc<N, double> A;
    A.zero();
#pragma unroll
    for (int c = 0; c < Q / 2; ++c) A.template add_pair<BT>(c, fv[c], fv[Q - 1 - c]);
    if constexpr (Q % 2 == 1) A.template add_mid<BT>(fv[Q / 2]);
    A.finish(p1);
#pragma unroll
    for (int k = 0; k < N; ++k) buf[k * Lds<P, false>::SP + t] = p1[k];
    if (m + 1 < nbatch) load_f(m + 1);
    __syncthreads();
    bwd_y<P, double, false>(buf, t);
    bwd_x<P, double, false>(buf, t);
    emit_e<P, double, Lds<P, false>>(buf, t, active, smap, Y + (int64_t)m * estride,
                             b + (int64_t)m * ndof);
    __syncthreads();
  }
}

template <int P>
hipError_t launch_grad_p(const GradArgs &a, hipStream_t s) {
  using D = Dims<P>;
  if (a.nei <= 0 || a.nbatch <= 0) return hipSuccess;
  hipLaunchKernelGGL((grad_kernel<P>), dim3((unsigned)((a.nei + D::E - 1) / D::E)),
                     dim3(D::THREADS), 0, s, a.map, a.geo, a.beta, a.nei, a.nbatch,
                     a.ndof, a.u, a.lam, a.g);
  return hipGetLastError();
}

template <int P>
hipError_t launch_load_p(const LoadArgs &a, hipStream_t s) {
  using D = Dims<P>;
  const int64_t ne = a.nei;
  if (ne <= 0 || a.nbatch <= 0) return hipSuccess;
  constexpr bool POS = evec_dof_ordered(P);
  if ((a.pos != nullptr) != POS) return hipErrorInvalidValue;
  hipLaunchKernelGGL((load_kernel<P, POS>), dim3((unsigned)((ne + D::E - 1) / D::E)), dim3(D::THREADS),
                     0, s, a.map, a.geo, a.nei, a.nbatch, a.ndof, a.f, a.b, a.evec, a.estride,
                     a.pos, a.compact);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_grad(const GradArgs &a, hipStream_t s) {
#define SFEM_CALL(P) launch_grad_p<P>(a, s)
  SFEM_DISPATCH_P(a.p, SFEM_CALL)
#undef SFEM_CALL
}

hipError_t launch_load(const LoadArgs &a, hipStream_t s) {
#define SFEM_CALL(P) launch_load_p<P>(a, s)
  SFEM_DISPATCH_P(a.p, SFEM_CALL)
#undef SFEM_CALL
}

}  // namespace sfem
