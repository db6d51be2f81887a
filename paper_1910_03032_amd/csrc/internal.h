// Internal declarations of the sfem library (host side + kernel launchers).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "cg_plan.h"
#include "plan.h"
#include "sfem.h"

namespace sfem {

// How the assembly sets essential DoFs: copy x (operator apply), 1 (diagonal), 0 (load)
// What the assembly kernel writes at the essential DoFs (kEssAdd: it adds the assembled
// sums to y at the other listed DoFs and leaves the essential entries as they are).
enum EssKind { kEssCopyX = 0, kEssOne = 1, kEssZero = 2, kEssAdd = 3 };

// 1D tables for order P (n = P + 1 GLL nodes, q = P + 2 Gauss points), row-major
// [q][n]: B(a, i) = phi_i(xi_a), G(a, i) = phi_i'(xi_a).
struct Rules1D {
  int p = 0, q = 0;
  std::vector<double> gll_x, gll_w, gauss_x, gauss_w;
  std::vector<double> B, G;
};
// Host computation of the rules (Newton iterations on Legendre recurrences,
// barycentric Lagrange weights).  Returns false if a Newton iteration fails.
bool make_rules(int p, int q, Rules1D &out);

// Per-member PCG scalars kept on the device.
struct PcgScalars {
  double rho;     // r^T z
  double rr;      // r^T r
  double bb;      // b^T b
  double pw;      // p^T A p
  double alpha, beta;
  double tol2;    // (rtol ||b||)^2
  int active;     // 1 while iterating
  int status;     // 0 ok, SFEM_E_BREAKDOWN, SFEM_E_NAN
  int iters;      // completed iterations
  int pad;
  double zshift;  // null-space solves: mean of dinv r, removed from the preconditioned residual
};

// ---------------------------------------------------------------------------
// Kernel launchers (implemented in the .hip files).  Every launcher enqueues on
// `s` and returns the hipError_t of the launch.  The 1D tables are compile-time
// constants of the kernels (rules.h).
// ---------------------------------------------------------------------------
struct ApplyArgs {
  int p;
  int op;                   // SFEM_MASS / SFEM_DIFFUSION / SFEM_HELMHOLTZ
  const int32_t *map;       // [nei][n^3] flagged map, internal element order
  const double *geo;        // trilinear coefficients of the elements, [nei][kGeoStride] (geom.h)
  const double *cw;         // w nu / |J| at the points, [nei][q^3], or null (nu = 1)
  int64_t cw_mstride;       // entries of cw between batch members (0 = shared)
  double alpha, beta;       // coefficients of the mass and diffusion terms
  int thin;                 // some element needs LineGeom's factors in float32 (geom.h)
  int64_t ndof;
  int nbatch;
  int64_t nelem;
  const void *x;
  void *y;                  // output at the sole DoFs
  void *evec;               // E-vector of the shared nodes, [nbatch][estride]
  int64_t estride;          // E-vector entries per member (contributions to shared DoFs)
  const int32_t *pos;       // DoF-ordered E-vector: [nelem][epe] entry of each element
                            // node; null: element-ordered, node r of element e -> e*epe + r
  int compact;              // nodes indexed by surface rank (1, epe = S) or local node (0)
  double *part;             // CG: the partials of p.Ap, [nb][part_mstride] (cg_parts)
  int64_t part_mstride;
};
// Element phase of the apply over all elements (writes the E-vector).
hipError_t launch_apply_f64(const ApplyArgs &a, hipStream_t s);
hipError_t launch_apply_f32(const ApplyArgs &a, hipStream_t s);
// The same as the first launch of a CG iteration (pcg.h): a.x is unused, a.part is required.  The
// direction is formed from the preconditioned residual -- dinv r (launch_apply_cg*: r and dinv in
// the apply's precision, [nb][ndof], dinv member stride dinv_mstride), or z given (launch_apply_cgz,
// float64 or, with z32, float32) -- and the old direction p.  sc: the state after the last update;
// unless ready (it already holds beta) the partials upart ([nb][4][unblk]) complete it; the
// completed state goes to sc_next and, if given, to host (device-visible host memory).
struct CgIn {
  const void *r, *dinv, *p;
  const void *z;
  int z32;
  int64_t dinv_mstride;
  const PcgScalars *sc;
  PcgScalars *sc_next, *host;
  const double *upart;
  int unblk, ready, nullspace;
};
hipError_t launch_apply_cg64(const ApplyArgs &a, const CgIn &g, hipStream_t s);
hipError_t launch_apply_cg32(const ApplyArgs &a, const CgIn &g, hipStream_t s);
hipError_t launch_apply_cgz(const ApplyArgs &a, const CgIn &g, hipStream_t s);
// elements per workgroup of the CG iteration's apply kernel
int apply_group_elems_f64(int p);
int apply_group_elems_f32(int p);
// Assembly list on the device (see HostPlan): the assembled DoFs, ascending, the CSR
// offsets of their contributions, and for the element-ordered E-vector the entries of
// those contributions (slot == null: DoF-ordered, the entries are [aoff[i], aoff[i+1])).
struct AsmPlan {
  const int32_t *alist;
  const int32_t *aoff;
  const int32_t *slot;
  int64_t na;
};
// Assembly phase over the list: y[g] = sum of g's E-vector entries in element order;
// essential DoFs get x[g], 1 or 0 per ess_kind.
constexpr int kMaxParts = 1024;  // cap of the partial sums of a dot product by the vector kernels
template <typename T>
hipError_t launch_assemble(const AsmPlan &pl, const T *evec, int64_t estride, const T *x, T *y,
                           int64_t n, int nb, int ess_kind, hipStream_t s);

struct DiagArgs {
  int p;
  const int32_t *map;
  const double *geo;        // trilinear coefficients (geom.h)
  const double *cw;         // w nu / |J|, [nelem][q^3], or null (nu = 1)
  double alpha, beta;       // coefficients of the mass and diffusion terms
  int64_t nelem;
  double *diag;             // [ndof], written at the sole DoFs
  double *evec;             // E-vector of the shared nodes
  const int32_t *pos;       // E-vector entry of each element node, or null (see ApplyArgs)
  int compact;
};
hipError_t launch_diag(const DiagArgs &a, hipStream_t s);

// bad[0] = 1 if |J| is not positive at some quadrature point, bad[1] = 1 if two columns of J are
// nearly parallel there (kMetricLimit of geom.h).
hipError_t launch_check_det(int q, const double *gx, const double *gw, const double *xyz, int64_t nei,
                            int *bad, hipStream_t s);
// Collocated (GLL-integrated) mass contributions of every element node: sole DoFs into
// diag, shared nodes into their E-vector entry (then assembled with ess rows = 1).
hipError_t launch_colloc_mass(int p, const double *gll_x, const double *gll_w, const double *xyz,
                              const int32_t *map, const int32_t *pos, int compact, int64_t nelem,
                              double *diag, double *evec, hipStream_t s);
hipError_t launch_qpoint_coords(int q, const double *gx, const double *gw, const double *xyz,
                                int64_t nei, double *xq, hipStream_t s);
// Trilinear coefficients of the elements (geom.h), [nei][kGeoStride].
hipError_t launch_geo_setup(const double *xyz, int64_t nei, double *geo, hipStream_t s);
// cw = w nu / |J| at the points of nfield coefficient fields, and the library's copy of nu.
hipError_t launch_fold(int q, const double *gx, const double *gw, const double *geo, const double *nu_user,
                       int64_t nei, int nfield, double *cw, double *nu64, hipStream_t s);
hipError_t launch_cast_f32(const double *src, float *dst, int64_t n, hipStream_t s);

struct GradArgs {
  int p;
  const int32_t *map;
  const double *geo;
  double beta;
  int64_t ndof, nei;
  int nbatch;
  const double *u, *lam;
  double *g;                // [nbatch][nelem][q^3] caller order
};
hipError_t launch_grad(const GradArgs &a, hipStream_t s);

struct LoadArgs {
  int p;
  const int32_t *map;
  const double *geo;
  int64_t ndof, nei;
  int nbatch;
  const double *f;          // [nbatch][nelem][q^3]
  double *b;                // written at the sole DoFs
  double *evec;             // E-vector of the shared nodes, [nbatch][estride]
  int64_t estride;
  const int32_t *pos;       // E-vector entry of each element node, or null (see ApplyArgs)
  int compact;
};
hipError_t launch_load(const LoadArgs &a, hipStream_t s);

// Where the update kernel of the CG finds (A p)_g: doff[g] holds the offset of g's E-vector
// entries (the next DoF's offset ends them) with the map's sole and essential flags; slot: as
// in AsmPlan.
struct CgDofs {
  const int32_t *doff;      // [ndof + 1]
  const int32_t *slot;
};

// Vector kernels of the PCG (T = double or float).  Partial-sum buffers hold
// [nb][nv][nblk] doubles.  dinv may be shared by all members (dms = 0) or per member
// (dms = n).
template <typename T>
struct VecOps {
  static hipError_t start(const T *b, const T *w, T *x, T *r, const T *dinv, int64_t dms, T *p,
                          double *part, int nblk, int64_t n, int nb, hipStream_t s);
  // per-member partial sums of a[m] . c[m] (a: [nb][n]; c: member stride c_mstride, 0 for
  // one vector shared by all members, or null for the all-ones vector)
  static hipError_t dot(const T *a, const T *c, int64_t c_mstride, double *part, int nblk,
                        int64_t n, int nb, hipStream_t s);
  // The second launch of a CG iteration (pcg.h) after the element kernel in CG mode: dpart[m *
  // dmstride + i], i < dcount, are its partials of p.Ap, y and evec its outputs; leaves the
  // partials of r.z, r.r, sum z, sum r in part ([nb][4][nblk], nblk = cg_update_nblk) and the
  // state with alpha in sc_next.
  static hipError_t update(const CgDofs &dofs, const T *evec, int64_t estride, const T *y, T *x, T *p, T *r,
                           const T *dinv, int64_t dms, const PcgScalars *sc, PcgScalars *sc_next,
                           const double *dpart, int64_t dmstride, int dcount, double *part, int nblk,
                           int64_t n, int nb, hipStream_t s);
  static hipError_t fill(T *p, T v, int64_t n, hipStream_t s);
  static hipError_t recip(const double *d, T *out, int64_t n, hipStream_t s);
};
int vec_nblk(int64_t n);
hipError_t launch_sub_norm(const double *b, const double *w, double *r, double *part, int nblk,
                           int64_t n, int nb, hipStream_t s);
// Scalar steps of the CG.  With nullspace != 0 (constants in the operator's null space,
// n unknowns per member) the preconditioned residual z = dinv r is orthogonalized,
// z - mean(z) 1, and rho = r^T z of that vector (Section 5.3).
hipError_t launch_pcg_init(const double *part, int nblk, int nb, double rtol, PcgScalars *sc,
                           hipStream_t s, int nullspace = 0, int64_t n = 0);
int cg_update_nblk(int64_t n, int nb);
// out[m][b] = sum of the b-th of nblk equal stretches of member m's dcount partials (cg_fold_nblk).
hipError_t launch_cg_fold(const double *dpart, int64_t dmstride, int dcount, double *out, int nblk, int nb,
                          hipStream_t s);
// The same update around a preconditioner applied between the launches (one member, z given in
// the preconditioner's precision TZ); no partials.  TZ = float: r32 = (float) r, its input.  With
// t also the preconditioner's first smoothing sweep, t = omega tdinv r.
template <typename TZ>
hipError_t launch_cgz_update(const CgDofs &dofs, const double *evec, const double *y, double *x, double *p,
                             double *r, const TZ *z, float *r32, TZ *t, const TZ *tdinv, TZ omega,
                             const PcgScalars *sc, PcgScalars *sc_next, const double *dpart, int dcount,
                             int64_t n, hipStream_t s);
// Partials of r.z, r.r, sum z, sum r ([4][nblk], nblk = cg_update_nblk); with b of r.z, r.r, b.b,
// sum z, sum r ([5][nblk], the input of launch_pcg_init).
template <typename TZ>
hipError_t launch_cgz_dots(const double *r, const TZ *z, const double *b, double *part, int nblk, int64_t n,
                           hipStream_t s);
// In place, the state of the next iteration from the update's partials; also written to host, if
// given (device-visible host memory, [nb]).
hipError_t launch_cg_finish(PcgScalars *sc, PcgScalars *host, const double *part, int nblk, int nb,
                            int nullspace, int64_t n, hipStream_t s);
// v[m][i] -= c[m] * scale (member-wise constant shift)
hipError_t launch_shift(double *v, const double *c, double scale, int64_t n, int nb, hipStream_t s);
hipError_t launch_reduce1(const double *part, int nblk, int nb, double *out, hipStream_t s);
hipError_t launch_ir_norm(const double *part, int nblk, int nb, int set_bb, double rtol, double *ir,
                          hipStream_t s);
hipError_t launch_ir_cast(const double *r, const double *ir, float *r32, int64_t n, int nb,
                          hipStream_t s);
hipError_t launch_ir_accum(double *x, const float *d, const double *ir, int64_t n, int nb,
                           hipStream_t s);

}  // namespace sfem
