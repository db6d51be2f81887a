// Exact diagonal of the assembled operator alpha M + beta K(nu), sum-factorized.
//
// With the factors m = w|J| and Gq = w|J| J^-1 J^-T (symmetric, 6 entries), formed from the
// element's trilinear map (geom.h), the diagonal entry of node (i, j, k) of an element is
//   alpha sum_abc m B2(a,i) B2(b,j) B2(c,k)
// + beta  sum_abc nu sum_{r,s} Gq_rs t_r t_s
// where t_1 = G(a,i) B(b,j) B(c,k), t_2 = B G B, t_3 = B B G (the rows of the tensor
// gradient of eq. tensorGradient evaluated on the node's own basis function).  Each
// of the 7 distinct (r, s) products factors per direction into a Hadamard product
// of 1D tables: B2 = B.B, G2 = G.G, BG = B.G, with the off-diagonal pairs doubled.
// Every term is then a three-stage contraction q^3 -> n^3; a thread owns a xi_3 line of the
// points, so a term's values and its xi_3 contraction stay in registers.  The element
// contributions are assembled like the apply's (sole DoFs directly, shared nodes via
// the E-vector and the assembly kernel, which sets the essential rows to 1).  Several elements
// share a workgroup as in the apply (one element per 64 threads left most lanes idle at low
// order): set_coeffs with this kernel at 31 x 32 x 30 p = 1 449 -> 112 us, 20 x 21 x 19 p = 5
// 869 -> 537 us.
#include <hip/hip_runtime.h>

#include "apply_impl.h"

namespace sfem {
namespace {

// Hadamard products of the compile-time 1D tables: 0: B.B, 1: G.G, 2: B.G
template <int P>
__device__ __forceinline__ constexpr double dtab(int which, int a, int i) {
  using TB = Tab<P, double>;
  return which == 0 ? TB::B(a, i) * TB::B(a, i)
                    : (which == 1 ? TB::G(a, i) * TB::G(a, i) : TB::B(a, i) * TB::G(a, i));
}

// (x, y, z) table of each term; term 0 = mass, 1..6 = G11, G22, G33, G12, G13, G23
__device__ constexpr int kTermTab[7][3] = {{0, 0, 0}, {1, 0, 0}, {0, 1, 0}, {0, 0, 1},
                                           {2, 2, 0}, {2, 0, 2}, {0, 2, 2}};

template <int P, bool POS>
__global__ void __launch_bounds__(Dims<P>::THREADS)
diag_kernel(const int32_t *__restrict__ map, const double *__restrict__ geo,
            const double *__restrict__ cw, double alpha, double beta, int64_t nelem,
            double *__restrict__ diag, double *__restrict__ Y, const int32_t *__restrict__ pos,
            int compact) {
  using D = Dims<P>;
  constexpr int N = D::N, Q = D::Q, N2 = D::N2, N3 = D::N3, Q2 = D::Q2, Q3 = D::Q3, TPE = D::TPE, E = D::E;
  constexpr rules::GaussRule<Q> gr = rules::gauss<Q>();
  __shared__ double s1_all[E * N * Q2];  // [k][b][a], at the end the nodal values [k][j][i]
  __shared__ double s2_all[E * N2 * Q];  // [k][j][a]
  __shared__ __align__(16) double sgeo[E * kGeoStride];
  __shared__ int32_t smap_all[E * N3];
  const int le = threadIdx.x / TPE;
  const int t = threadIdx.x - le * TPE;
  const int64_t e0 = (int64_t)xcd_block() * E;
  const bool active = e0 + le < nelem;
  const uint32_t rel = active ? le : 0;
  double *s1 = s1_all + le * N * Q2, *s2 = s2_all + le * N2 * Q, *sg = sgeo + le * kGeoStride;
  int32_t *smap = smap_all + le * N3;
  {
    const ElemTab z = elem_tab<P>(map, pos, compact, e0);
    Nodes<P> nd;
    nd.load_map(z, t, rel);
    nd.load_rank(z, t);
    load_geo<P>(sg, geo, e0, rel, t);
    nd.template load_dest<POS>(z, rel);
    nd.keep(smap, t);
  }
  __syncthreads();
  LineGeom L;
  L.init(sg, kGaussRule<Q>.x[t % Q], kGaussRule<Q>.x[t / Q]);
  const double wab = kGaussRule<Q>.w[t % Q] * kGaussRule<Q>.w[t / Q];
  const double *ce = cw ? cw + (e0 + rel) * Q3 + t : nullptr;
  double acc[N];
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = 0.0;

#pragma unroll
  for (int term = 0; term < 7; ++term) {
    const double coef = (term == 0) ? alpha : ((term <= 3) ? beta : 2.0 * beta);
    if (coef == 0.0) continue;  // uniform across the block
    const int tx = kTermTab[term][0], ty = kTermTab[term][1], tz = kTermTab[term][2];
    {  // the term at the line's points, contracted along c
      double r[N];
#pragma unroll
      for (int k = 0; k < N; ++k) r[k] = 0.0;
#pragma unroll
      for (int c = 0; c < Q; ++c) {
        const double w = wab * gr.w[c], det = L.det(gr.x[c]);
        double v;
        if (term == 0) {
          v = coef * (w * det);
        } else {
          double ad[3][3];
          L.adj(gr.x[c], ad[0], ad[1], ad[2]);
          const int i = term <= 3 ? term - 1 : (term == 6 ? 1 : 0), j = term <= 3 ? term - 1 : (term == 4 ? 1 : 2);
          v = coef * (ce ? ce[c * Q2] : w * recip(det)) *
              (ad[i][0] * ad[j][0] + ad[i][1] * ad[j][1] + ad[i][2] * ad[j][2]);
        }
#pragma unroll
        for (int k = 0; k < N; ++k) r[k] += dtab<P>(tz, c, k) * v;
      }
#pragma unroll
      for (int k = 0; k < N; ++k) s1[k * Q2 + t] = r[k];
    }
    __syncthreads();
    if (t < Q * N) {  // contract b: lines (a, k)
      const int a = t % Q, k = t / Q;
      double in[Q];
#pragma unroll
      for (int b = 0; b < Q; ++b) in[b] = s1[(k * Q + b) * Q + a];
#pragma unroll
      for (int j = 0; j < N; ++j) {
        double s = 0.0;
#pragma unroll
        for (int b = 0; b < Q; ++b) s += dtab<P>(ty, b, j) * in[b];
        s2[(k * N + j) * Q + a] = s;
      }
    }
    __syncthreads();
    if (t < N2) {  // contract a: lines (j, k)
      double in[Q];
#pragma unroll
      for (int a = 0; a < Q; ++a) in[a] = s2[t * Q + a];
#pragma unroll
      for (int i = 0; i < N; ++i) {
        double s = 0.0;
#pragma unroll
        for (int a = 0; a < Q; ++a) s += dtab<P>(tx, a, i) * in[a];
        acc[i] += s;
      }
    }
    // (the next term writes s1, whose last reads the barrier above has closed, and s2 only
    // after its own first barrier)
  }
  if (t < N2) {
#pragma unroll
    for (int i = 0; i < N; ++i) s1[t * N + i] = acc[i];
  }
  __syncthreads();
  emit_e<P, double>(s1, t, active, smap, Y, diag);
}

template <int P>
hipError_t launch_diag_p(const DiagArgs &a, hipStream_t s) {
  using D = Dims<P>;
  const int64_t ne = a.nelem;
  if (ne <= 0) return hipSuccess;
  constexpr bool POS = evec_dof_ordered(P);
  if ((a.pos != nullptr) != POS) return hipErrorInvalidValue;
  hipLaunchKernelGGL((diag_kernel<P, POS>), dim3((unsigned)((ne + D::E - 1) / D::E)), dim3(D::THREADS), 0,
                     s, a.map, a.geo, a.cw, a.alpha, a.beta, a.nelem, a.diag, a.evec, a.pos, a.compact);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_diag(const DiagArgs &a, hipStream_t s) {
#define SFEM_CALL(P) launch_diag_p<P>(a, s)
  SFEM_DISPATCH_P(a.p, SFEM_CALL)
#undef SFEM_CALL
}

}  // namespace sfem
