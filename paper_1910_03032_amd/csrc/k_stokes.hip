// Coupling blocks of the Taylor-Hood Stokes operator (Section 3, eq. gradient and
// eq. divergence): velocity in (Q_p)^3, pressure in Q_{p-1}, both nodal on the GLL
// points, on the same elements and the same q = p + 2 Gauss points.  With the
// coupling factor C = w |J| J^{-T} at each point (C_cd = w adj(J)_dc, formed from the
// element's trilinear map, geom.h), the physical
// gradient of a scalar f integrated against w|J| is C grad_ref f, so
//
//   (G p)_{l, c} = sum_Q phi_l(Q) (C_Q grad_ref p(Q))_c
//   (D u)_m      = sum_Q psi_m(Q) sum_c (C_Q grad_ref u_c(Q))_c
//
// Both are sum-factorized like the scalar operators (Section 3.1): the reference
// gradient by B/G contractions direction by direction, the test functions by the
// transposed B contractions.  One element per q^2 threads, the workgroups of the apply
// kernel (same LDS buffers, same thread-per-1D-line stages).  Outputs go through the
// same conflict-free assembly as the apply: values of DoFs owned by one element are
// written directly, those of shared DoFs to the E-vector of their space.
#include <hip/hip_runtime.h>

#include "apply_impl.h"
#include "flow.h"
#include "geom.h"

namespace sfem {
namespace {

// 1D tables of an order-PO space at the q points of order P (q = P + 2).
template <int PO, int Q>
struct Tab2 {
  static constexpr rules::Tables<PO, Q> c = rules::tables<PO, Q>();
  static constexpr double B(int a, int i) { return c.B[a][i]; }
  static constexpr double G(int a, int i) { return c.G[a][i]; }
};
// The same tables in the accessor form of the even-odd helpers (WHICH 0 = B, 1 = G): the
// GLL nodes of any order and the Gauss points are symmetric about 0, so B is
// centro-symmetric and G centro-antisymmetric for every (order, q) pair.
template <int PO, int Q, int WHICH>
struct TabEO {
  static constexpr int NO = Q, NI = PO + 1;
  static constexpr int S = WHICH == 0 ? 1 : -1;
  static constexpr double t(int a, int i) { return WHICH == 0 ? Tab2<PO, Q>::B(a, i) : Tab2<PO, Q>::G(a, i); }
  static constexpr double e(int a, int i) { return 0.5 * (t(a, i) + t(a, NI - 1 - i)); }
  static constexpr double o(int a, int i) { return 0.5 * (t(a, i) - t(a, NI - 1 - i)); }
};

// Where the stages keep a field of order PO in an element's buffer: [k][j][i] at NOD, then
// [k][j][a] (line stride LQ, plane SK, field XF), then [k][b][a] (plane SP, field YF).  Dense
// serves any (order, q); Padded the velocity, with the strides of Lds<P> and the nodal vector
// past the [k][j][a] fields, where the xi_1 stages need no barrier between reads and writes.
template <int PO, int Q>
struct Dense {
  static constexpr int NI = PO + 1, LQ = Q, SK = NI * Q, XF = NI * SK, SP = Q * Q, YF = NI * SP, NOD = 0;
};
template <int P>
struct Padded {
  static constexpr int LQ = Lds<P>::LQ, SK = Lds<P>::SK, XF = Lds<P>::XF, SP = Lds<P>::SP, YF = Lds<P>::YF,
                       NOD = Lds<P>::NOD;
  static_assert(Lds<P>::FULL >= NOD + (P + 1) * (P + 1) * (P + 1) && Lds<P>::FULL >= Dims<P>::BUF, "element buffer");
};
// (p = 8: the padded strides' addresses spill in the curl and coupling kernels, 11^3 curl 51.3 ->
// 52.7 us; p = 2, where a wave holds its elements: 42^3 curl 86 -> 78, Stokes 205 -> 188 us; p = 6
// 5 to 7 %, the others 0 to 3 %)
template <int P>
using VelLay = std::conditional_t<(P < 8), Padded<P>, Dense<P, P + 2>>;

// Forward reference gradient of a nodal field of order PO (NI = PO + 1 nodes per
// direction, in buf + NOD as [k][j][i]) for the q x q threads of an element: stages xi_1 and
// xi_2 through LDS (even-odd contractions); the xi_3 contraction is the caller's.
template <int PO, int Q, class L = Dense<PO, Q>>
__device__ __forceinline__ void fwd_grad_xy(double *buf, int t) {
  constexpr int NI = PO + 1;
  constexpr int N2 = NI * NI;
  using BT = TabEO<PO, Q, 0>;
  using GT = TabEO<PO, Q, 1>;
  {  // xi_1: [k][j][i] -> [k][j][a] (B and G)
    const bool w = t < N2;
    const int j = t % NI, k = t / NI;
    double ob[Q], og[Q];
    if (w) {
      double in[NI];
#pragma unroll
      for (int i = 0; i < NI; ++i) in[i] = buf[L::NOD + (k * NI + j) * NI + i];
      const auto sp = eo::split(in);
      eo::apply<BT>(sp, ob);
      eo::apply<GT>(sp, og);
    }
    if constexpr (L::NOD == 0) elem_sync<Q - 2>();
    if (w) {
#pragma unroll
      for (int a = 0; a < Q; ++a) {
        buf[k * L::SK + j * L::LQ + a] = ob[a];
        buf[L::XF + k * L::SK + j * L::LQ + a] = og[a];
      }
    }
    elem_sync<Q - 2>();
  }
  {  // xi_2: [k][j][a] -> [k][b][a]: B(Bx), G(Bx), B(Gx)
    const bool w = t < Q * NI;
    const int a = t % Q, k = t / Q;
    double obb[Q], ogb[Q], obg[Q];
    if (w) {
      double ib[NI], ig[NI];
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        ib[j] = buf[k * L::SK + j * L::LQ + a];
        ig[j] = buf[L::XF + k * L::SK + j * L::LQ + a];
      }
      const auto sb = eo::split(ib);
      eo::apply<BT>(sb, obb);
      eo::apply<GT>(sb, ogb);
      eo::apply<BT>(eo::split(ig), obg);
    }
    elem_sync<Q - 2>();
    if (w) {
#pragma unroll
      for (int b = 0; b < Q; ++b) {
        buf[k * L::SP + b * Q + a] = obb[b];
        buf[L::YF + k * L::SP + b * Q + a] = ogb[b];
        buf[2 * L::YF + k * L::SP + b * Q + a] = obg[b];
      }
    }
    elem_sync<Q - 2>();
  }
}

// Transposed mass-type contractions along xi_2 and xi_1 of NF fields given by their
// contracted xi_3 lines (r[f][k] of line (a, b)), down to nodal fields of order PO (NO = PO + 1
// nodes per direction), field f at buf + NOD + f * NO^3 ([k][j][i]); even-odd form.  Ends with
// a barrier and, with NOD = 0, starts with one (else a thread's lines replace lines of its own).
template <int PO, int Q>
__device__ __forceinline__ void mass_line(const double (&in)[Q], double (&out)[PO + 1]) {
  using BT = TabEO<PO, Q, 0>;
  eo::Acc<PO + 1, double> A;
  A.zero();
#pragma unroll
  for (int c = 0; c < Q / 2; ++c) A.template add_pair<BT>(c, in[c], in[Q - 1 - c]);
  if constexpr (Q % 2 == 1) A.template add_mid<BT>(in[Q / 2]);
  A.finish(out);
}
template <int PO, int Q, int NF, class L = Dense<PO, Q>>
__device__ __forceinline__ void bwd_mass_xy(double *buf, int t, const double (&p)[NF][PO + 1]) {
  constexpr int NO = PO + 1;
  constexpr int N3 = NO * NO * NO;
  static_assert(L::NOD == 0 || NF == 1, "one field past the [k][j][a] fields");
  if constexpr (L::NOD == 0) elem_sync<Q - 2>();
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int k = 0; k < NO; ++k) buf[f * L::YF + k * L::SP + t] = p[f][k];
  elem_sync<Q - 2>();
  {  // xi_2: [k][b][a] -> [k][j][a]
    const bool w = t < Q * NO;
    const int a = t % Q, k = t / Q;
    double r[NF][NO];
    if (w) {
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        double in[Q];
#pragma unroll
        for (int b = 0; b < Q; ++b) in[b] = buf[f * L::YF + k * L::SP + b * Q + a];
        mass_line<PO, Q>(in, r[f]);
      }
    }
    elem_sync<Q - 2>();
    if (w) {
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int j = 0; j < NO; ++j) buf[f * L::XF + k * L::SK + j * L::LQ + a] = r[f][j];
    }
    elem_sync<Q - 2>();
  }
  {  // xi_1: [k][j][a] -> [k][j][i]
    const bool w = t < NO * NO;
    const int j = t % NO, k = t / NO;
    double r[NF][NO];
    if (w) {
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        double in[Q];
#pragma unroll
        for (int a = 0; a < Q; ++a) in[a] = buf[f * L::XF + k * L::SK + j * L::LQ + a];
        mass_line<PO, Q>(in, r[f]);
      }
    }
    if constexpr (L::NOD == 0) elem_sync<Q - 2>();
    if (w) {
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int i = 0; i < NO; ++i) buf[L::NOD + f * N3 + (k * NO + j) * NO + i] = r[f][i];
    }
    elem_sync<Q - 2>();
  }
}

// The same from the fields at the q^3 points (each thread holds its xi_3 line v[f][c]).
template <int PO, int Q, int NF, class L = Dense<PO, Q>>
__device__ __forceinline__ void bwd_mass(double *buf, int t, const double (&v)[NF][Q]) {
  double r[NF][PO + 1];
#pragma unroll
  for (int f = 0; f < NF; ++f) mass_line<PO, Q>(v[f], r[f]);
  bwd_mass_xy<PO, Q, NF, L>(buf, t, r);
}

// Gather of a pressure-space element (order P - 1, no essential DoFs) into buf, for the q^2
// threads of the element (TPE = (P + 2)^2).
template <int P>
__device__ __forceinline__ void gather_pres(double *buf, int t, bool active, const int32_t *emap,
                                            const double *__restrict__ x) {
  constexpr int NP3 = P * P * P, TPE = (P + 2) * (P + 2);
  constexpr int NL = (NP3 + TPE - 1) / TPE;
  int32_t c[NL];
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    const int l0 = t + k * TPE;
    c[k] = emap[l0 < NP3 ? l0 : NP3 - 1];
  }
  double v[NL];
#pragma unroll
  for (int k = 0; k < NL; ++k) v[k] = x[c[k] & kDofMask];
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    const int l = t + k * TPE;
    if (l < NP3) buf[l] = active ? v[k] : 0.0;
  }
  __syncthreads();
}

// Output of a pressure-space element vector (element-ordered E-vector, surface ranks of
// order P - 1 when compact): sole DoFs -> y, shared nodes -> Y[e * epe + r].
template <int P>
__device__ __forceinline__ void emit_pres(const double *buf, int t, bool active,
                                          const int32_t *smap, int64_t e, bool compact,
                                          double *__restrict__ Y, double *__restrict__ y) {
  constexpr int NP3 = P * P * P, TPE = (P + 2) * (P + 2);
  constexpr int NL = (NP3 + TPE - 1) / TPE;
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    const int l0 = t + k * TPE;
    const int l = l0 < NP3 ? l0 : NP3 - 1;
    const int32_t c = smap[l];
    const double v = buf[l];
    const bool ok = active && l0 < NP3;
    const bool sole = (c & kSoleBit) != 0;
    const int64_t ye = compact ? e * surf_count<P - 1>() + kRankTable<P - 1>.r[l] : e * NP3 + l;
    double *dst = sole ? y + (c & kDofMask) : Y + ye;
    if (ok) *dst = v;
  }
}

template <int P>
struct SDims {
  using D = Dims<P>;
  static constexpr int N = P + 1, NP = P, Q = P + 2, Q2 = Q * Q, Q3 = Q * Q * Q;
  static constexpr int TPE = D::TPE, E = D::E, THREADS = D::THREADS;
  static_assert(D::BUF >= 3 * N * Q * Q && D::BUF >= 3 * Q * Q * NP && D::BUF >= 2 * Q * N * N,
                "element buffer");
  // minimum waves per SIMD the kernels below are compiled for
  static constexpr int OCC = 2;
  static constexpr int CONV_OCC = P <= 4 ? 4 : (P <= 6 ? 3 : 2);  // the most without spilling
};

// Output of a velocity element vector that adds into an apply's output: sole DoFs
// y[g] += v (each has exactly one writer), shared nodes -> their E-vector entry, essential
// -> nothing.  With the DoF-ordered E-vector (POS) the value is added into the entry the
// Helmholtz element kernel wrote, and one assembly sums both; with the element-ordered
// one (p >= 5) it is stored into an E-vector of its own, assembled into y afterwards
// (adding into the element-ordered entries measured 1-2 % slower than the second
// assembly).
template <int P, bool POS>
__device__ __forceinline__ void emit_add_vel(const double *buf, int t, bool active,
                                             const int32_t *smap, double *__restrict__ Y,
                                             double *__restrict__ y) {
  using D = Dims<P>;
  constexpr int NL = Per<P>::NL;
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    const int l = Nodes<P>::node(t, k);
    const int32_t c = smap[l];
    const double v = buf[l];
    if (!(active && t + k * D::TPE < D::N3 && c >= 0)) continue;
    if (c & kSoleBit) {
      y[c & kDofMask] += v;
    } else if constexpr (POS) {
      Y[c] += v;
    } else {
      Y[c] = v;
    }
  }
}

// Nodal values held in registers (Nodes::load_values) into buf[k][j][i], essential DoFs as 0
// unless ESS; no barrier.
template <int P, bool ESS>
__device__ __forceinline__ void put_nodal(double *buf, int t, bool active, const Nodes<P> &nd,
                                          const double (&v)[Nodes<P>::NL]) {
#pragma unroll
  for (int k = 0; k < Nodes<P>::NL; ++k)
    buf[Nodes<P>::node(t, k)] = (active && (ESS || nd.c[k] >= 0)) ? v[k] : 0.0;
}

// Even-odd xi_3 lines of the three fields fwd_grad_xy leaves for order PO.
template <int PO, int Q, class L = Dense<PO, Q>>
__device__ __forceinline__ void read_z3(const double *buf, int t, eo::Split<PO + 1, double> &bb,
                                        eo::Split<PO + 1, double> &gb, eo::Split<PO + 1, double> &bg) {
  constexpr int NI = PO + 1;
  double zb[NI], zg[NI], zx[NI];
#pragma unroll
  for (int k = 0; k < NI; ++k) {
    zb[k] = buf[k * L::SP + t];
    zg[k] = buf[L::YF + k * L::SP + t];
    zx[k] = buf[2 * L::YF + k * L::SP + t];
  }
  bb = eo::split(zb);
  gb = eo::split(zg);
  bg = eo::split(zx);
}

// Both coupling blocks in one pass over the elements: G p added into the three velocity
// components (the sole DoFs of yv directly, the shared nodes through the E-vector, members
// at stride vestride, as emit_add_vel describes) and -D P u into the pressure space
// (element-ordered E-vector Yp, sole DoFs of yp).  Component r needs the components
// C_rd = w adj(J)_dr of the three adjugate rows, formed along the thread's xi_3 line (the
// Stokes apply at 28 x 29 x 27 p = 3: 200 -> 152 us with the Helmholtz part's factors formed too).
template <int P, bool POS>
__global__ void __launch_bounds__(Dims<P>::THREADS, SDims<P>::OCC)
coupling_kernel(const int32_t *__restrict__ vmap, const int32_t *__restrict__ vpos, int vcompact,
                const int32_t *__restrict__ pmap, int pcompact, const double *__restrict__ geo,
                int64_t nelem, const double *__restrict__ u, const double *__restrict__ pres,
                int64_t nv, double *__restrict__ Yv, int64_t vestride, double *__restrict__ yv,
                double *__restrict__ Yp, double *__restrict__ yp) {
  using S = SDims<P>;
  constexpr int N = S::N, NP = S::NP, Q = S::Q, TPE = S::TPE, E = S::E;
  constexpr int N3 = N * N * N, NP3 = NP * NP * NP;
  constexpr rules::GaussRule<Q> gr = rules::gauss<Q>();
  __shared__ __align__(16) double smem[E * Lds<P>::FULL];
  __shared__ __align__(16) double sgeo[E * kGeoStride];
  __shared__ int32_t smap_all[E * N3];
  const int le = threadIdx.x / TPE;
  const int t0 = threadIdx.x - le * TPE;
  const int t = t0;
  const int64_t e0 = (int64_t)xcd_block() * E;
  const int64_t e = e0 + le;
  const bool active = e < nelem;
  const int64_t es = active ? e : e0;
  const uint32_t rel = (uint32_t)(es - e0);
  double *buf = smem + le * Lds<P>::FULL;
  const double *sg = sgeo + le * kGeoStride;
  int32_t *smap = smap_all + le * N3;
  const ElemTab z = elem_tab<P>(vmap, vpos, vcompact, e0);
  Nodes<P> nd;
  nd.load_map(z, t, rel);
  nd.load_rank(z, t);
  load_geo<P>(sgeo + le * kGeoStride, geo, e0, rel, t);
  // pressure element: the xi_3 lines of its reference gradient
  gather_pres<P>(buf, t, active, pmap + (int64_t)es * NP3, pres);
  nd.template load_dest<POS>(z, rel);
  double v[Nodes<P>::NL];  // the next component's nodal values
  nd.load_values(u, v);
  fwd_grad_xy<P - 1, Q>(buf, t);
  eo::Split<NP, double> pbb, pgb, pbg;  // xi_3 lines of the pressure, even-odd split
  read_z3<P - 1, Q>(buf, t, pbb, pgb, pbg);
  nd.keep(smap, t);  // the velocity nodes' destinations
  double s[1][Q];
#pragma unroll
  for (int c = 0; c < Q; ++c) s[0][c] = 0.0;
  const double x1 = kGaussRule<Q>.x[t % Q], x2 = kGaussRule<Q>.x[t / Q];
  const double wab = kGaussRule<Q>.w[t % Q] * kGaussRule<Q>.w[t / Q];
  // (one component at a time, not unrolled: fewer live registers)
#pragma unroll 1
  for (int r = 0; r < 3; ++r) {
    // indices derived from the thread are recomputed per component rather than kept live
    int t = t0;
    asm volatile("" : "+v"(t));
    elem_sync<P>();  // buf was read by the last component's output (or the pressure lines)
    // velocity component r (essential DoFs read as 0)
    put_nodal<P, false>(buf + VelLay<P>::NOD, t, active, nd, v);
    elem_sync<P>();
    if (r < 2) nd.load_values(u + (r + 1) * nv, v);
    fwd_grad_xy<P, Q, VelLay<P>>(buf, t);
    eo::Split<N, double> ubb, ugb, ubg;
    read_z3<P, Q, VelLay<P>>(buf, t, ubb, ugb, ubg);
    LineAdjComp L;
    L.init(sg, r, x1, x2);
    double n[1][Q];
    // row r of C times grad_ref p (G) and times grad_ref u_r (D) at slice c
    auto point = [&](int c, double ux, double uy, double uz, double px, double py, double pz) {
      double c0, c1, c2;
      L.at(gr.x[c], c0, c1, c2);
      const double w = wab * gr.w[c];
      n[0][c] = w * (c0 * px + c1 * py + c2 * pz);
      s[0][c] -= w * (c0 * ux + c1 * uy + c2 * uz);
    };
    using VB = TabEO<P, Q, 0>;
    using VG = TabEO<P, Q, 1>;
    using PB = TabEO<P - 1, Q, 0>;
    using PG = TabEO<P - 1, Q, 1>;
#pragma unroll
    for (int c = 0; c < Q / 2; ++c) {
      double uz0, uz1, uy0, uy1, ux0, ux1, pz0, pz1, py0, py1, px0, px1;
      eo::out_pair<VG>(ubb, c, uz0, uz1);
      eo::out_pair<VB>(ugb, c, uy0, uy1);
      eo::out_pair<VB>(ubg, c, ux0, ux1);
      eo::out_pair<PG>(pbb, c, pz0, pz1);
      eo::out_pair<PB>(pgb, c, py0, py1);
      eo::out_pair<PB>(pbg, c, px0, px1);
      point(c, ux0, uy0, uz0, px0, py0, pz0);
      point(Q - 1 - c, ux1, uy1, uz1, px1, py1, pz1);
    }
    if constexpr (Q % 2 == 1)
      point(Q / 2, eo::out_mid<VB>(ubg), eo::out_mid<VB>(ugb), eo::out_mid<VG>(ubb), eo::out_mid<PB>(pbg),
            eo::out_mid<PB>(pgb), eo::out_mid<PG>(pbb));
    // G p, component r: added into yv / the velocity E-vector
    bwd_mass<P, Q, 1, VelLay<P>>(buf, t, n);
    emit_add_vel<P, POS>(buf + VelLay<P>::NOD, t, active, smap, Yv + r * vestride, yv + r * nv);
  }
  // -D P u: one pressure field
  bwd_mass<P - 1, Q, 1>(buf, t, s);
  {
    constexpr int NL = (NP3 + TPE - 1) / TPE;
    const int32_t *em = pmap + (int64_t)es * NP3;
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const int l = t + k * TPE;
      if (l < NP3) smap[l] = em[l];
    }
    __syncthreads();
  }
  emit_pres<P>(buf, t, active, smap, es, pcompact != 0, Yp, yp);
}

// Interpolation of the three nodal fields in buf (field f at f n^3) to the points, stages
// xi_1 and xi_2 (B only): afterwards buf holds the fields [k][b][a] at f n q^2.
template <int P, int Q>
__device__ __forceinline__ void fwd_val3_xy(double *buf, int t) {
  constexpr int NI = P + 1, N2 = NI * NI, N3 = N2 * NI;
  using BT = TabEO<P, Q, 0>;
  {
    const bool w = t < N2;
    const int j = t % NI, k = t / NI;
    double ob[3][Q];
    if (w) {
#pragma unroll
      for (int f = 0; f < 3; ++f) {
        double in[NI];
#pragma unroll
        for (int i = 0; i < NI; ++i) in[i] = buf[f * N3 + (k * NI + j) * NI + i];
        eo::apply<BT>(eo::split(in), ob[f]);
      }
    }
    elem_sync<P>();
    if (w) {
#pragma unroll
      for (int f = 0; f < 3; ++f)
#pragma unroll
        for (int a = 0; a < Q; ++a) buf[f * N2 * Q + (k * NI + j) * Q + a] = ob[f][a];
    }
    elem_sync<P>();
  }
  {
    const bool w = t < Q * NI;
    const int a = t % Q, k = t / Q;
    double ob[3][Q];
    if (w) {
#pragma unroll
      for (int f = 0; f < 3; ++f) {
        double in[NI];
#pragma unroll
        for (int j = 0; j < NI; ++j) in[j] = buf[f * N2 * Q + (k * NI + j) * Q + a];
        eo::apply<BT>(eo::split(in), ob[f]);
      }
    }
    elem_sync<P>();
    if (w) {
#pragma unroll
      for (int f = 0; f < 3; ++f)
#pragma unroll
        for (int b = 0; b < Q; ++b) buf[f * NI * Q * Q + (k * Q + b) * Q + a] = ob[f][b];
    }
    elem_sync<P>();
  }
}

// h_k = sum_d C_dk u_d at the points of the thread's xi_3 line (C = w |J| J^{-T}: w |J| times
// the reference-direction components of the vector field u), from its three nodal fields in
// buf.  Ends without a barrier (buf has been read).
template <int P, int Q>
__device__ __forceinline__ void contravariant(double *buf, int t, const double *sg, double (&h)[3][Q]) {
  constexpr int N = P + 1, Q2 = Q * Q;
  constexpr rules::GaussRule<Q> gr = rules::gauss<Q>();
  using VB = TabEO<P, Q, 0>;
  fwd_val3_xy<P, Q>(buf, t);
  const double x1 = kGaussRule<Q>.x[t % Q], x2 = kGaussRule<Q>.x[t / Q];
  const double wab = kGaussRule<Q>.w[t % Q] * kGaussRule<Q>.w[t / Q];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    double z[N];
#pragma unroll
    for (int k = 0; k < N; ++k) z[k] = buf[d * N * Q2 + k * Q2 + t];
    const auto sv = eo::split(z);
    LineAdjComp L;
    L.init(sg, d, x1, x2);
    auto point = [&](int c, double v) {
      double r1, r2, r3;
      L.at(gr.x[c], r1, r2, r3);
      const double wv = (wab * gr.w[c]) * v;
      h[0][c] = (d == 0 ? 0.0 : h[0][c]) + r1 * wv;
      h[1][c] = (d == 0 ? 0.0 : h[1][c]) + r2 * wv;
      h[2][c] = (d == 0 ? 0.0 : h[2][c]) + r3 * wv;
    };
#pragma unroll
    for (int c = 0; c < Q / 2; ++c) {
      double v0, v1;
      eo::out_pair<VB>(sv, c, v0, v1);
      point(c, v0);
      point(Q - 1 - c, v1);
    }
    if constexpr (Q % 2 == 1) point(Q / 2, eo::out_mid<VB>(sv));
  }
}

// What the element kernels below begin with: the nodes' map entries and destinations and the
// element's trilinear coefficients (loads in flight together; no barrier).  values() loads what
// the map leads to, before the destinations are waited for.
template <int P, bool POS, typename F>
__device__ __forceinline__ void begin_vel(Nodes<P> &nd, const int32_t *vmap, const int32_t *vpos,
                                          int vcompact, const double *geo, int64_t e0, uint32_t rel, int t,
                                          double *sg, int32_t *smap, F values) {
  const ElemTab z = elem_tab<P>(vmap, vpos, vcompact, e0);
  nd.load_map(z, t, rel);
  nd.load_rank(z, t);
  load_geo<P>(sg, geo, e0, rel, t);
  values();
  nd.template load_dest<POS>(z, rel);
  nd.keep(smap, t);
}

// The three nodal components of u (essential DoFs included), loaded, and put into buf
// (component f at f n^3).
template <int P>
struct Vec3 {
  double v[3][Nodes<P>::NL];
  __device__ __forceinline__ void load(const Nodes<P> &nd, const double *u, int64_t nv) {
#pragma unroll
    for (int r = 0; r < 3; ++r) nd.load_values(u + r * nv, v[r]);
  }
  // ends with a barrier
  __device__ __forceinline__ void put(double *buf, int t, bool active, const Nodes<P> &nd) {
#pragma unroll
    for (int r = 0; r < 3; ++r) nd.pin(v[r]);
#pragma unroll
    for (int r = 0; r < 3; ++r) put_nodal<P, true>(buf + r * Dims<P>::N3, t, active, nd, v[r]);
    elem_sync<P>();
  }
};

// Convection term N(u) (eq. nonlinear) on the velocity space: n_c = sum_d u_d w |J| d u_c / d x_d
// = sum_k h_k d_ref_k u_c with h = contravariant(u), so that the geometric factors are needed
// once per point and not per component, and a component's gradient lines live only while it is
// processed and the loop over components stays rolled.  What bounds it: VALU issue and LDS.
// (With 9 stored factors read per point and the three components' lines held together it took
// 230 registers at p = 4 and twice the HBM bytes: 28 x 27 x 29 p = 5 291 -> 186 us, 84 x 85 x 83
// p = 1 361 -> 224 us.  Unrolled over the components: 202 registers, 21 x 22 x 20 p = 4 58 us
// against 52.)
template <int P, bool POS>
__global__ void __launch_bounds__(Dims<P>::THREADS, SDims<P>::CONV_OCC)
convection_kernel(const int32_t *__restrict__ vmap, const int32_t *__restrict__ vpos,
                  int vcompact, const double *__restrict__ geo, int64_t nelem,
                  const double *__restrict__ u, int64_t nv, double *__restrict__ Yv,
                  int64_t vestride, double *__restrict__ yv) {
  using S = SDims<P>;
  constexpr int N = S::N, Q = S::Q, TPE = S::TPE, E = S::E, N3 = N * N * N;
  using VB = TabEO<P, Q, 0>;
  using VG = TabEO<P, Q, 1>;
  __shared__ __align__(16) double smem[E * Lds<P>::FULL];
  __shared__ __align__(16) double sgeo[E * kGeoStride];
  __shared__ int32_t smap_all[E * N3];
  const int le = threadIdx.x / TPE;
  const int t = threadIdx.x - le * TPE;
  const int64_t e0 = (int64_t)xcd_block() * E;
  const bool active = e0 + le < nelem;
  double *buf = smem + le * Lds<P>::FULL;
  double *sg = sgeo + le * kGeoStride;
  int32_t *smap = smap_all + le * N3;
  Nodes<P> nd;
  Vec3<P> u3;
  begin_vel<P, POS>(nd, vmap, vpos, vcompact, geo, e0, active ? le : 0, t, sg, smap,
                    [&] { u3.load(nd, u, nv); });
  u3.put(buf, t, active, nd);
  double v[Nodes<P>::NL];  // the next component's nodal values
  nd.load_values(u, v);
  double h[3][Q];
  contravariant<P, Q>(buf, t, sg, h);
  // (one component at a time, not unrolled: fewer live registers)
#pragma unroll 1
  for (int r = 0; r < 3; ++r) {
    elem_sync<P>();  // buf has been read
    put_nodal<P, true>(buf + VelLay<P>::NOD, t, active, nd, v);
    elem_sync<P>();
    if (r < 2) nd.load_values(u + (r + 1) * nv, v);
    fwd_grad_xy<P, Q, VelLay<P>>(buf, t);
    double p[1][N];
    {
      eo::Split<N, double> bb, gb, bg;
      read_z3<P, Q, VelLay<P>>(buf, t, bb, gb, bg);
      eo::Acc<N, double> A;
      A.zero();
#pragma unroll
      for (int c = 0; c < Q / 2; ++c) {
        double x0, x1, y0, y1, z0, z1;
        eo::out_pair<VB>(bg, c, x0, x1);
        eo::out_pair<VB>(gb, c, y0, y1);
        eo::out_pair<VG>(bb, c, z0, z1);
        A.template add_pair<VB>(c, h[0][c] * x0 + h[1][c] * y0 + h[2][c] * z0,
                                h[0][Q - 1 - c] * x1 + h[1][Q - 1 - c] * y1 + h[2][Q - 1 - c] * z1);
      }
      if constexpr (Q % 2 == 1) {
        constexpr int M = Q / 2;
        A.template add_mid<VB>(h[0][M] * eo::out_mid<VB>(bg) + h[1][M] * eo::out_mid<VB>(gb) +
                               h[2][M] * eo::out_mid<VG>(bb));
      }
      A.finish(p[0]);
    }
    bwd_mass_xy<P, Q, 1, VelLay<P>>(buf, t, p);
    emit_e<P, double>(buf + VelLay<P>::NOD, t, active, smap, Yv + r * vestride, yv + r * nv);
  }
}

// Weak curl (CURL) or weak gradient of the projection step, tested against phi: with
// Gamma_dr = sum_k C_dk d_ref_k u_r = w |J| d u_r / d x_d,
//   curl      n_c = eps_cde Gamma_de                (w |J| (curl u)_c)
//   gradient  n_c = Gamma_c0 (one input field s)    (w |J| (grad s)_c)
// One input component after the other, its derivatives added into the three outputs at the
// points (rolled loop; the outputs' roles rotate with it).  21 x 22 x 20 p = 4 against 9 stored
// factors per point: curl 79 -> 49 us, gradient 61 -> 32 us.
template <int P, bool POS, bool CURL>
__global__ void __launch_bounds__(Dims<P>::THREADS, SDims<P>::OCC)
weak_phi_kernel(const int32_t *__restrict__ vmap, const int32_t *__restrict__ vpos,
                int vcompact, const double *__restrict__ geo, int64_t nelem,
                const double *__restrict__ u, int64_t nv, double *__restrict__ Yv,
                int64_t vestride, double *__restrict__ yv) {
  using S = SDims<P>;
  constexpr int N = S::N, Q = S::Q, TPE = S::TPE, E = S::E, N3 = N * N * N;
  constexpr int NIN = CURL ? 3 : 1;
  constexpr rules::GaussRule<Q> gr = rules::gauss<Q>();
  using VB = TabEO<P, Q, 0>;
  using VG = TabEO<P, Q, 1>;
  __shared__ __align__(16) double smem[E * Lds<P>::FULL];
  __shared__ __align__(16) double sgeo[E * kGeoStride];
  __shared__ int32_t smap_all[E * N3];
  const int le = threadIdx.x / TPE;
  const int t = threadIdx.x - le * TPE;
  const int64_t e0 = (int64_t)xcd_block() * E;
  const bool active = e0 + le < nelem;
  double *buf = smem + le * Lds<P>::FULL;
  double *sg = sgeo + le * kGeoStride;
  int32_t *smap = smap_all + le * N3;
  Nodes<P> nd;
  double v[Nodes<P>::NL];  // the next component's nodal values
  begin_vel<P, POS>(nd, vmap, vpos, vcompact, geo, e0, active ? le : 0, t, sg, smap,
                    [&] { nd.load_values(u, v); });
  nd.pin(v);
  // n[k]: output r + 1 + k of the current input component r (curl), output k (gradient)
  double n[3][Q];
#pragma unroll
  for (int d = 0; d < 3; ++d)
#pragma unroll
    for (int c = 0; c < Q; ++c) n[d][c] = 0.0;
  const double x1 = kGaussRule<Q>.x[t % Q], x2 = kGaussRule<Q>.x[t / Q];
  // (one component at a time, not unrolled: fewer live registers)
#pragma unroll 1
  for (int r = 0; r < NIN; ++r) {
    if (r > 0) elem_sync<P>();  // buf has been read
    put_nodal<P, true>(buf + VelLay<P>::NOD, t, active, nd, v);
    elem_sync<P>();
    if (r + 1 < NIN) nd.load_values(u + (r + 1) * nv, v);
    fwd_grad_xy<P, Q, VelLay<P>>(buf, t);
    eo::Split<N, double> bb, gb, bg;
    read_z3<P, Q, VelLay<P>>(buf, t, bb, gb, bg);
    // curl: d u_r / d x_d enters output r + 1 for d = r + 2 and, negated, output r + 2 for d = r + 1
    constexpr int ND = CURL ? 2 : 3;
    LineAdjComp L[ND];
#pragma unroll
    for (int k = 0; k < ND; ++k) {
      const int d = CURL ? (r + 2 - k < 3 ? r + 2 - k : r - 1 - k) : k;
      L[k].init(sg, d, x1, x2);
    }
    auto point = [&](int c, double dx, double dy, double dz) {
#pragma unroll
      for (int k = 0; k < ND; ++k) {
        double r1, r2, r3;
        L[k].at(gr.x[c], r1, r2, r3);
        const double g = r1 * dx + r2 * dy + r3 * dz;
        if (CURL) n[k][c] += k == 0 ? g : -g;
        else n[k][c] = g;
      }
    };
#pragma unroll
    for (int c = 0; c < Q / 2; ++c) {
      double x0, x1c, y0, y1, z0, z1;
      eo::out_pair<VB>(bg, c, x0, x1c);
      eo::out_pair<VB>(gb, c, y0, y1);
      eo::out_pair<VG>(bb, c, z0, z1);
      point(c, x0, y0, z0);
      point(Q - 1 - c, x1c, y1, z1);
    }
    if constexpr (Q % 2 == 1) point(Q / 2, eo::out_mid<VB>(bg), eo::out_mid<VB>(gb), eo::out_mid<VG>(bb));
    if constexpr (CURL) {
#pragma unroll
      for (int c = 0; c < Q; ++c) {
        const double first = n[0][c];
        n[0][c] = n[1][c];
        n[1][c] = n[2][c];
        n[2][c] = first;
      }
    }
  }
  // (curl: after r = 0, 1, 2 the outputs are in the order 1, 2, 0)
  const double wab = kGaussRule<Q>.w[t % Q] * kGaussRule<Q>.w[t / Q];
  double p[3][N];
#pragma unroll
  for (int f = 0; f < 3; ++f) {
    eo::Acc<N, double> A;
    A.zero();
#pragma unroll
    for (int c = 0; c < Q / 2; ++c)
      A.template add_pair<VB>(c, (wab * gr.w[c]) * n[f][c], (wab * gr.w[c]) * n[f][Q - 1 - c]);
    if constexpr (Q % 2 == 1) A.template add_mid<VB>((wab * gr.w[Q / 2]) * n[f][Q / 2]);
    A.finish(p[f]);
  }
  bwd_mass_xy<P, Q, 3>(buf, t, p);
#pragma unroll
  for (int f = 0; f < 3; ++f) {
    const int o = CURL ? (f + 1) % 3 : f;
    emit_e<P, double>(buf + f * N3, t, active, smap, Yv + o * vestride, yv + o * nv);
  }
}

// Transposed reference-gradient contraction: from the three channels v_k at the points
// of the thread's xi_3 line (the components of the field to be tested against the
// reference gradient d_ref_k phi), the element vector sum_Q sum_k d_ref_k phi_l(Q) v_k(Q)
// in buf[0 .. n^3).  Channel k carries G along xi_k and B along the other two directions.
template <int PO, int Q>
__device__ __forceinline__ void bwd_grad(double *buf, int t, const double (&v)[3][Q]) {
  constexpr int NO = PO + 1;
  constexpr int NQ2 = NO * Q * Q, N2Q = NO * NO * Q;
  using BT = TabEO<PO, Q, 0>;
  using GT = TabEO<PO, Q, 1>;
  // out[i] += sum_c T(c, i) in[c] for c over the q points (T = B or G)
  auto line = [](auto tag, const double (&in)[Q], eo::Acc<NO, double> &A) {
    using TB = decltype(tag);
#pragma unroll
    for (int c = 0; c < Q / 2; ++c) A.template add_pair<TB>(c, in[c], in[Q - 1 - c]);
    if constexpr (Q % 2 == 1) A.template add_mid<TB>(in[Q / 2]);
  };
  {  // xi_3: channels 0, 1 with B, channel 2 with G: [c] -> [k][b][a]
    double r[3][NO];
#pragma unroll
    for (int f = 0; f < 3; ++f) {
      eo::Acc<NO, double> A;
      A.zero();
      if (f == 2) line(GT{}, v[f], A);
      else line(BT{}, v[f], A);
      A.finish(r[f]);
    }
    __syncthreads();
#pragma unroll
    for (int f = 0; f < 3; ++f)
#pragma unroll
      for (int k = 0; k < NO; ++k) buf[f * NQ2 + k * Q * Q + t] = r[f][k];
    __syncthreads();
  }
  {  // xi_2: [k][b][a] -> [k][j][a]; s0 = B^T ch0 (G along xi_1 pending), s1 = G^T ch1 + B^T ch2
    const bool w = t < Q * NO;
    const int a = t % Q, k = t / Q;
    double r[2][NO];
    if (w) {
      double in0[Q], in1[Q], in2[Q];
#pragma unroll
      for (int b = 0; b < Q; ++b) {
        in0[b] = buf[(k * Q + b) * Q + a];
        in1[b] = buf[NQ2 + (k * Q + b) * Q + a];
        in2[b] = buf[2 * NQ2 + (k * Q + b) * Q + a];
      }
      eo::Acc<NO, double> A0, A1;
      A0.zero();
      A1.zero();
      line(BT{}, in0, A0);
      line(GT{}, in1, A1);
      line(BT{}, in2, A1);
      A0.finish(r[0]);
      A1.finish(r[1]);
    }
    __syncthreads();
    if (w) {
#pragma unroll
      for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int j = 0; j < NO; ++j) buf[f * N2Q + (k * NO + j) * Q + a] = r[f][j];
    }
    __syncthreads();
  }
  {  // xi_1: [k][j][a] -> [k][j][i]; out = G^T s0 + B^T s1
    const bool w = t < NO * NO;
    const int j = t % NO, k = t / NO;
    double r[NO];
    if (w) {
      double in0[Q], in1[Q];
#pragma unroll
      for (int a = 0; a < Q; ++a) {
        in0[a] = buf[(k * NO + j) * Q + a];
        in1[a] = buf[N2Q + (k * NO + j) * Q + a];
      }
      eo::Acc<NO, double> A;
      A.zero();
      line(GT{}, in0, A);
      line(BT{}, in1, A);
      A.finish(r);
    }
    __syncthreads();
    if (w) {
#pragma unroll
      for (int i = 0; i < NO; ++i) buf[(k * NO + j) * NO + i] = r[i];
    }
    __syncthreads();
  }
}

// Weak divergence of a nodal vector field V (the pressure right-hand side of the
// projection step, Section 4.2): r_l = sum_Q w |J| grad phi_l . V = sum_Q
// grad_ref phi_l . (C^T V) with C = w |J| J^{-T}: C^T V is formed per point and one backward
// reference-gradient pass gives the single output (member 0 of the E-vector and of y).
// 21 x 22 x 20 p = 4 against 9 stored factors per point: 54 -> 25 us.
template <int P, bool POS>
__global__ void __launch_bounds__(Dims<P>::THREADS, SDims<P>::OCC)
weak_div_kernel(const int32_t *__restrict__ vmap, const int32_t *__restrict__ vpos,
                int vcompact, const double *__restrict__ geo, int64_t nelem,
                const double *__restrict__ u, int64_t nv, double *__restrict__ Yv,
                double *__restrict__ yv) {
  using S = SDims<P>;
  using D = Dims<P>;
  constexpr int N = S::N, Q = S::Q, TPE = S::TPE, E = S::E, N3 = N * N * N;
  __shared__ __align__(16) double smem[E * D::BUF];
  __shared__ __align__(16) double sgeo[E * kGeoStride];
  __shared__ int32_t smap_all[E * N3];
  const int le = threadIdx.x / TPE;
  const int t = threadIdx.x - le * TPE;
  const int64_t e0 = (int64_t)xcd_block() * E;
  const bool active = e0 + le < nelem;
  double *buf = smem + le * D::BUF;
  double *sg = sgeo + le * kGeoStride;
  int32_t *smap = smap_all + le * N3;
  {
    Nodes<P> nd;
    Vec3<P> u3;
    begin_vel<P, POS>(nd, vmap, vpos, vcompact, geo, e0, active ? le : 0, t, sg, smap,
                      [&] { u3.load(nd, u, nv); });
    u3.put(buf, t, active, nd);
  }
  double h[3][Q];  // (C^T V)_k at the points of the line
  contravariant<P, Q>(buf, t, sg, h);
  bwd_grad<P, Q>(buf, t, h);
  emit_e<P, double>(buf, t, active, smap, Yv, yv);
}

template <int P>
hipError_t launch_stokes_pt(const StokesArgs &a, hipStream_t s) {
  if constexpr (P < 2) {
    return hipErrorInvalidValue;
  } else {
    using D = Dims<P>;
    if (a.nelem <= 0) return hipSuccess;
    constexpr bool POS = evec_dof_ordered(P);
    if ((a.vpos != nullptr) != POS) return hipErrorInvalidValue;
    dim3 grid((unsigned)((a.nelem + D::E - 1) / D::E));
    dim3 block(D::THREADS);
    hipLaunchKernelGGL((coupling_kernel<P, POS>), grid, block, 0, s, a.vmap, a.vpos, a.vcompact,
                       a.pmap, a.pcompact, a.geo, a.nelem, a.u, a.pres, a.nv, a.Yv, a.vestride,
                       a.yv, a.Yp, a.yp);
    return hipGetLastError();
  }
}

template <int P>
hipError_t launch_convection_pt(const ConvArgs &a, hipStream_t s) {
  using D = Dims<P>;
  if (a.nelem <= 0) return hipSuccess;
  constexpr bool POS = evec_dof_ordered(P);
  if ((a.vpos != nullptr) != POS) return hipErrorInvalidValue;
  dim3 grid((unsigned)((a.nelem + D::E - 1) / D::E));
  dim3 block(D::THREADS);
  switch (a.kind) {
    case kWeakConvection:
      hipLaunchKernelGGL((convection_kernel<P, POS>), grid, block, 0, s, a.vmap, a.vpos,
                         a.vcompact, a.geo, a.nelem, a.u, a.nv, a.Yv, a.vestride, a.yv);
      break;
    case kWeakCurl:
      hipLaunchKernelGGL((weak_phi_kernel<P, POS, true>), grid, block, 0, s, a.vmap, a.vpos,
                         a.vcompact, a.geo, a.nelem, a.u, a.nv, a.Yv, a.vestride, a.yv);
      break;
    case kWeakGradient:
      hipLaunchKernelGGL((weak_phi_kernel<P, POS, false>), grid, block, 0, s, a.vmap, a.vpos,
                         a.vcompact, a.geo, a.nelem, a.u, a.nv, a.Yv, a.vestride, a.yv);
      break;
    case kWeakDivergence:
      hipLaunchKernelGGL((weak_div_kernel<P, POS>), grid, block, 0, s, a.vmap, a.vpos, a.vcompact,
                         a.geo, a.nelem, a.u, a.nv, a.Yv, a.yv);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

__global__ void __launch_bounds__(256)
lincomb_kernel(LinComb lc, const double *__restrict__ scale, const uint8_t *__restrict__ mask,
               double *y, int64_t n, int64_t total) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * 256) {
    double v = 0.0;
    for (int j = 0; j < lc.nterm; ++j) v += lc.c[j] * lc.x[j][i];
    const int64_t g = i % n;
    if (scale) v /= scale[g];
    if (mask && mask[g]) v = 0.0;
    y[i] = v;
  }
}

}  // namespace

hipError_t launch_stokes(const StokesArgs &a, hipStream_t s) {
#define SFEM_CALL(P) launch_stokes_pt<P>(a, s)
  SFEM_DISPATCH_P(a.p, SFEM_CALL)
#undef SFEM_CALL
}

hipError_t launch_convection(const ConvArgs &a, hipStream_t s) {
#define SFEM_CALL(P) launch_convection_pt<P>(a, s)
  SFEM_DISPATCH_P(a.p, SFEM_CALL)
#undef SFEM_CALL
}

hipError_t launch_lincomb(const LinComb &lc, const double *scale, const uint8_t *mask, double *y,
                          int64_t n, int nb, hipStream_t s) {
  const int64_t total = n * nb;
  if (total <= 0) return hipSuccess;
  if (lc.nterm < 1 || lc.nterm > kMaxLinTerms) return hipErrorInvalidValue;
  int64_t blocks = (total + 1023) / 1024;
  if (blocks > 65535) blocks = 65535;
  hipLaunchKernelGGL(lincomb_kernel, dim3((unsigned)blocks), dim3(256), 0, s, lc, scale, mask, y, n,
                     total);
  return hipGetLastError();
}

}  // namespace sfem
