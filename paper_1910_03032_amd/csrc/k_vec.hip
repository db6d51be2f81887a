// Vector kernels of the Jacobi-preconditioned CG (Section 5, Section 5.3) and of the
// FP64 iterative refinement around an FP32 inner CG.
//
// All dot products form and add their terms in float64, also for float32 vectors (p.Ap: energy.h).
// Reductions go by per-block partial sums in a fixed order, so every result is bitwise
// reproducible for a given size; in a CG iteration the partials are summed by every workgroup that
// needs them, a long list first and many members' by launches of their own (cg_plan.h).  The CG
// scalars (rho, alpha, beta, ...) stay on the device; the host only reads them at its convergence
// checks.
#include <hip/hip_runtime.h>

#include <cmath>

#include "internal.h"
#include "pcg.h"

namespace sfem {
namespace {

constexpr int VB = 256;

// Sums over a block of VB threads, in every thread: wave totals, then the waves in order.
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV]) {
  __shared__ double sh[NV][VB / 64];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const double t = wave_total(v[k]);
    if ((threadIdx.x & 63) == 0) sh[k][threadIdx.x >> 6] = t;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    v[k] = 0.0;
#pragma unroll
    for (int w = 0; w < VB / 64; ++w) v[k] += sh[k][w];
  }
}

template <int NV>
__device__ __forceinline__ void write_part(double (&v)[NV], double *part, int nblk) {
  block_sum<NV>(v);
  if (threadIdx.x == 0) {
    const int m = blockIdx.y;
#pragma unroll
    for (int k = 0; k < NV; ++k) part[((int64_t)m * NV + k) * nblk + blockIdx.x] = v[k];
  }
}

// Sum of the nblk partials of quantity k (NV quantities per member, part[(m NV + k) nblk
// + i]) of member m by a block of NT threads: each thread sums a fixed strided subset
// (4 independent loads per step), then wave totals and the waves in order.  The order
// depends only on nblk and NT.  Result broadcast to all threads.
template <int NV, int NT>
__device__ __forceinline__ void reduce_parts_m(const double *part, int nblk, int m, double (&v)[NV]) {
  __shared__ double sh[NV][NT / 64];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const double *pk = part + ((int64_t)m * NV + k) * nblk;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    for (int i = threadIdx.x; i < nblk; i += 4 * NT) {
      // clamped, not predicated: the four loads are in flight together also in the last step
      const int i1 = i + NT, i2 = i + 2 * NT, i3 = i + 3 * NT, last = nblk - 1;
      const double v0 = pk[i], v1 = pk[i1 < nblk ? i1 : last], v2 = pk[i2 < nblk ? i2 : last],
                   v3 = pk[i3 < nblk ? i3 : last];
      s0 += v0;
      s1 += i1 < nblk ? v1 : 0.0;
      s2 += i2 < nblk ? v2 : 0.0;
      s3 += i3 < nblk ? v3 : 0.0;
    }
    const double s = wave_total((s0 + s1) + (s2 + s3));
    if ((threadIdx.x & 63) == 0) sh[k][threadIdx.x >> 6] = s;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    double s = 0.0;
    for (int w = 0; w < NT / 64; ++w) s += sh[k][w];
    v[k] = s;
  }
}

// One block of RB threads per member (blockIdx.x = member).
constexpr int RB = 1024;
template <int NV>
__device__ __forceinline__ void reduce_parts(const double *part, int nblk, double (&v)[NV]) {
  reduce_parts_m<NV, RB>(part, nblk, blockIdx.x, v);
}

// r = b - w (w may be null: r = b); x = 0 if xzero; p = 0 (the first direction is z = dinv r);
// partials: r.z (rho), r.r, b.b, sum z, sum r
template <typename T>
__global__ void start_kernel(const T *__restrict__ b, const T *__restrict__ w, T *__restrict__ x,
                             T *__restrict__ r, const T *__restrict__ dinv, int64_t dinv_mstride,
                             T *__restrict__ p, double *__restrict__ part, int nblk, int64_t n) {
  const int64_t off = (int64_t)blockIdx.y * n;
  const T *dm = dinv + (int64_t)blockIdx.y * dinv_mstride;
  double v[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (int64_t i = (int64_t)blockIdx.x * VB + threadIdx.x; i < n; i += (int64_t)nblk * VB) {
    const T bi = b[off + i];
    const T ri = w ? (T)(bi - w[off + i]) : bi;
    const T pi = dm[i] * ri;
    r[off + i] = ri;
    p[off + i] = T(0);
    if (x) x[off + i] = T(0);
    v[0] += (double)ri * (double)pi;
    v[1] += (double)ri * (double)ri;
    v[2] += (double)bi * (double)bi;
    v[3] += (double)pi;
    v[4] += (double)ri;
  }
  write_part<5>(v, part, nblk);
}

template <typename T>
__global__ void dot_kernel(const T *__restrict__ a, const T *__restrict__ c, int64_t c_mstride,
                           double *__restrict__ part, int nblk, int64_t n) {
  const int64_t off = (int64_t)blockIdx.y * n;
  const T *cm = c ? c + (int64_t)blockIdx.y * c_mstride : nullptr;
  double v[1] = {0.0};
  for (int64_t i = (int64_t)blockIdx.x * VB + threadIdx.x; i < n; i += (int64_t)nblk * VB)
    v[0] += (double)a[off + i] * (cm ? (double)cm[i] : 1.0);
  write_part<1>(v, part, nblk);
}

// The second launch of a CG iteration (pcg.h): per DoF, w = (A p)_g -- the element kernel's y
// at a DoF of one element, p itself at an essential DoF, else the sum of the DoF's E-vector
// entries in element order (as assemble_kernel) -- then p, x += alpha p, r -= alpha w and the
// partials of r.z, r.r, sum z, sum r of the new r.  doff: per DoF the offset of its entries,
// with the map's flags (the count follows from the next DoF's offset).  Bound by HBM (or the
// last-level cache): 7 vector streams, the offsets and the entries, in one pass where an
// assembly, an update and a direction kernel made three.  Blocks of 512 threads, at most
// kCgUpdateMax of them: few partials for every block of the next launch to sum, and 16 waves per CU in flight.
constexpr int CU_NT = 512;

// With Z (one member) the preconditioned residual z is given instead of dinv r, there are no
// partials, and what the preconditioner starts from is written too (CgzOut).
template <typename TZ>
struct CgzOut {
  float *r32;       // (float) r, or null
  TZ *t;            // first smoothing sweep omega tdinv r, or null
  const TZ *tdinv;
  TZ omega;
};
template <typename T, typename TZ, bool Z>
__global__ void __launch_bounds__(CU_NT)
cg_update_kernel(CgDofs dofs, const T *__restrict__ Y, int64_t estride, const T *__restrict__ y,
                 T *__restrict__ x, T *__restrict__ p, T *__restrict__ r,
                 const TZ *__restrict__ dinv, int64_t dinv_mstride, const PcgScalars *__restrict__ sc,
                 PcgScalars *__restrict__ sc_next, const double *__restrict__ dpart, int64_t dmstride,
                 int dcount, double *__restrict__ part, int nblk, int64_t n, CgzOut<TZ> zo) {
  const int m = blockIdx.y;
  const int64_t off = (int64_t)m * n;
  const TZ *dm = dinv + (int64_t)m * dinv_mstride;  // (Z: the given z)
  const T *Ym = Y + (int64_t)m * estride, *ym = y + off;
  T *xm = x + off, *pm = p + off, *rm = r + off;
  // U entries per thread and pass, all their loads in flight together; those of the first
  // pass are requested before the partial sums are read
  constexpr int U = 2;
  int32_t o[U], o1[U];
  T ex[U], ep[U], er[U], ed[U];
  const int64_t stride = (int64_t)nblk * CU_NT;
  auto fetch = [&](int64_t i) {
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int64_t j = i + k * stride < n ? i + k * stride : n - 1;
      o[k] = dofs.doff[j];
      o1[k] = dofs.doff[j + 1];
      ex[k] = xm[j];
      ep[k] = pm[j];
      er[k] = rm[j];
      ed[k] = (T)dm[j];
    }
  };
  int64_t i = (int64_t)blockIdx.x * CU_NT + threadIdx.x;
  fetch(i);
  double pw[1];
  reduce_parts_m<1, CU_NT>(dpart + (int64_t)m * dmstride, dcount, 0, pw);
  PcgScalars s;
  copy_state(s, sc[m]);
  set_alpha(s, pw[0]);
  if (blockIdx.x == 0 && threadIdx.x == 0) copy_state(sc_next[m], s);
  const T alpha = (T)s.alpha, beta = (T)s.beta, zs = (T)s.zshift;
  double v[4] = {0.0, 0.0, 0.0, 0.0};
  for (; i < n; i += U * stride) {
    T w[U];
    int32_t a[U], cnt[U];
    {
      T val[U][8], yi[U];
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int64_t j = i + k * stride;
        a[k] = o[k] & kDofMask;
        cnt[k] = j < n ? (o1[k] & kDofMask) - a[k] : 0;
#pragma unroll
        for (int q = 0; q < 8; ++q)
          val[k][q] = (q < cnt[k]) ? Ym[dofs.slot ? dofs.slot[a[k] + q] : a[k] + q] : T(0);
        yi[k] = (j < n && (o[k] & kSoleBit)) ? ym[j] : T(0);
      }
#pragma unroll
      for (int k = 0; k < U; ++k) {
        w[k] = val[k][0];
#pragma unroll
        for (int q = 1; q < 8; ++q)
          if (q < cnt[k]) w[k] += val[k][q];
        for (int q = 8; q < cnt[k]; ++q) w[k] += Ym[dofs.slot ? dofs.slot[a[k] + q] : a[k] + q];
        if (o[k] & kSoleBit) w[k] = yi[k];
      }
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int64_t j = i + k * stride;
      if (j >= n) continue;
      const T pi = Z ? cg_dir(T(1), ed[k], zs, beta, ep[k]) : cg_dir(ed[k], er[k], zs, beta, ep[k]);
      if (o[k] < 0) w[k] = pi;  // essential
      const T ri = er[k] - alpha * w[k];
      pm[j] = pi;
      xm[j] = ex[k] + alpha * pi;
      rm[j] = ri;
      if constexpr (Z) {
        if (zo.r32) zo.r32[j] = (float)ri;
        if (zo.t) zo.t[j] = zo.omega * zo.tdinv[j] * (TZ)ri;
        continue;
      }
      const T zi = ed[k] * ri;
      v[0] += (double)ri * (double)zi;
      v[1] += (double)ri * (double)ri;
      v[2] += (double)zi;
      v[3] += (double)ri;
    }
    if (i + U * stride < n) fetch(i + U * stride);
  }
  if constexpr (Z) return;
  // block sums: wave totals, then the waves in order
  __shared__ double sh[4][CU_NT / 64];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    v[k] = wave_total(v[k]);
    if ((threadIdx.x & 63) == 0) sh[k][threadIdx.x >> 6] = v[k];
  }
  __syncthreads();
  if (threadIdx.x < 4) {
    double t = 0.0;
    for (int w = 0; w < CU_NT / 64; ++w) t += sh[threadIdx.x][w];
    part[((int64_t)m * 4 + threadIdx.x) * nblk + blockIdx.x] = t;
  }
}

// out[m][b] = sum of the b-th of nblk equal stretches of member m's dcount partials.
__global__ void __launch_bounds__(VB)
cg_fold_kernel(const double *__restrict__ dpart, int64_t dmstride, int dcount, double *__restrict__ out, int nblk) {
  const int len = (dcount + nblk - 1) / nblk, lo = blockIdx.x * len;
  const int n = dcount - lo < len ? dcount - lo : len;
  double v[1] = {0.0};
  if (n > 0) reduce_parts_m<1, VB>(dpart + (int64_t)blockIdx.y * dmstride + lo, n, 0, v);
  if (threadIdx.x == 0) out[(int64_t)blockIdx.y * nblk + blockIdx.x] = v[0];
}

// The state of the next iteration from the update's partials (a block per member), where the
// host reads it before the next element kernel runs.
__global__ void __launch_bounds__(256)
cg_finish_kernel(PcgScalars *__restrict__ sc, PcgScalars *__restrict__ host, const double *__restrict__ part,
                 int nblk, int nullspace, int64_t n) {
  const int m = blockIdx.x;
  __shared__ double sums[4][4];
  PcgScalars s;
  copy_state(s, sc[m]);
  const double *p = part + (int64_t)m * 4 * nblk;
  PartLoads<4, 4> up;
  up.load(p, nblk);
  up.parts(sums, nblk);
  __syncthreads();
  cg_next_from<4>(s, sums, nullspace, n);
  if (threadIdx.x == 0) {
    copy_state(sc[m], s);
    if (host) copy_state(host[m], s);
  }
}

// Partials of r.z, r.r, (BB: b.b,) sum z, sum r.
template <typename TZ, bool BB>
__global__ void __launch_bounds__(CU_NT)
cgz_dots_kernel(const double *__restrict__ r, const TZ *__restrict__ z, const double *__restrict__ b,
                double *__restrict__ part, int nblk, int64_t n) {
  constexpr int NV = BB ? 5 : 4, U = 2;
  double v[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = 0.0;
  const int64_t stride = (int64_t)nblk * CU_NT;
  for (int64_t i = (int64_t)blockIdx.x * CU_NT + threadIdx.x; i < n; i += U * stride) {
    double ri[U], zi[U], bi[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int64_t j = i + k * stride < n ? i + k * stride : n - 1;
      ri[k] = r[j];
      zi[k] = (double)z[j];
      bi[k] = BB ? b[j] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      if (i + k * stride >= n) continue;
      v[0] += ri[k] * zi[k];
      v[1] += ri[k] * ri[k];
      if constexpr (BB) v[2] += bi[k] * bi[k];
      v[NV - 2] += zi[k];
      v[NV - 1] += ri[k];
    }
  }
  __shared__ double sh[NV][CU_NT / 64];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    v[k] = wave_total(v[k]);
    if ((threadIdx.x & 63) == 0) sh[k][threadIdx.x >> 6] = v[k];
  }
  __syncthreads();
  if (threadIdx.x < NV) {
    double t = 0.0;
    for (int w = 0; w < CU_NT / 64; ++w) t += sh[threadIdx.x][w];
    part[(int64_t)threadIdx.x * nblk + blockIdx.x] = t;
  }
}

// r = b - w with partial r.r (w may be null: r = b); r may be null (norm only)
__global__ void sub_norm_kernel(const double *__restrict__ b, const double *__restrict__ w,
                                double *__restrict__ r, double *__restrict__ part, int nblk,
                                int64_t n) {
  const int64_t off = (int64_t)blockIdx.y * n;
  double v[1] = {0.0};
  for (int64_t i = (int64_t)blockIdx.x * VB + threadIdx.x; i < n; i += (int64_t)nblk * VB) {
    const double ri = w ? b[off + i] - w[off + i] : b[off + i];
    if (r) r[off + i] = ri;
    v[0] += ri * ri;
  }
  write_part<1>(v, part, nblk);
}

__global__ void __launch_bounds__(RB) init_scalars_kernel(const double *__restrict__ part, int nblk, double rtol,
                                    PcgScalars *__restrict__ sc, int nullspace, int64_t n) {
  double v[5];
  reduce_parts<5>(part, nblk, v);
  if (threadIdx.x == 0) {
    PcgScalars &s = sc[blockIdx.x];
    s.zshift = nullspace ? v[3] / (double)n : 0.0;
    s.rho = v[0] - s.zshift * v[4];
    s.rr = v[1];
    s.bb = v[2];
    s.pw = 0.0;
    s.alpha = 0.0;
    s.beta = 0.0;
    s.tol2 = rtol * rtol * v[2];
    s.iters = 0;
    const bool finite = isfinite(v[0]) && isfinite(v[1]) && isfinite(v[2]);
    s.status = finite ? 0 : SFEM_E_NAN;
    s.active = (finite && v[2] > 0.0 && v[1] > s.tol2) ? 1 : 0;
  }
}

// v[m][i] -= c[m] * scale
__global__ void shift_kernel(double *__restrict__ v, const double *__restrict__ c, double scale,
                             int64_t n) {
  const int m = blockIdx.y;
  const double d = c[m] * scale;
  for (int64_t i = (int64_t)blockIdx.x * VB + threadIdx.x; i < n; i += (int64_t)gridDim.x * VB)
    v[(int64_t)m * n + i] -= d;
}

// out[m * nv + k] = sum of partials
template <int NV>
__global__ void __launch_bounds__(RB) reduce_out_kernel(const double *__restrict__ part, int nblk,
                                  double *__restrict__ out) {
  double v[NV];
  reduce_parts<NV>(part, nblk, v);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < NV; ++k) out[(int64_t)blockIdx.x * NV + k] = v[k];
  }
}

// IR state per member: [0] = ||r||^2, [1] = ||b||^2, [2] = scale (||r|| while refining, else 0)
__global__ void __launch_bounds__(RB) ir_norm_kernel(const double *__restrict__ part, int nblk, int set_bb, double rtol,
                               double *__restrict__ ir) {
  double v[1];
  reduce_parts<1>(part, nblk, v);
  if (threadIdx.x == 0) {
    double *s = ir + 3 * (int64_t)blockIdx.x;
    s[0] = v[0];
    if (set_bb) s[1] = v[0];
    s[2] = (v[0] > rtol * rtol * s[1]) ? sqrt(v[0]) : 0.0;
  }
}

__global__ void ir_cast_kernel(const double *__restrict__ r, const double *__restrict__ ir,
                               float *__restrict__ r32, int64_t n) {
  const int m = blockIdx.y;
  const double sc = ir[3 * m + 2];
  const double inv = sc > 0.0 ? 1.0 / sc : 0.0;
  const int64_t off = (int64_t)m * n;
  for (int64_t i = (int64_t)blockIdx.x * VB + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * VB)
    r32[off + i] = (float)(r[off + i] * inv);
}

__global__ void ir_accum_kernel(double *__restrict__ x, const float *__restrict__ d,
                                const double *__restrict__ ir, int64_t n) {
  const int m = blockIdx.y;
  const double sc = ir[3 * m + 2];
  if (sc == 0.0) return;
  const int64_t off = (int64_t)m * n;
  for (int64_t i = (int64_t)blockIdx.x * VB + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * VB)
    x[off + i] += sc * (double)d[off + i];
}

// Assembly over the list of shared and essential DoFs: y[g] = sum of the E-vector
// entries of list entry i in element order -- [aoff[i], aoff[i+1]) for the DoF-ordered
// E-vector (consecutive threads then read consecutive runs), slot[aoff[i]..aoff[i+1])
// for the element-ordered one; essential DoFs (no entries) get x[g], 1 or 0 (kEssAdd:
// y[g] += the sum at the other DoFs, essential entries untouched).  The first KS entries of
// each are loaded together, longer lists fall back to a loop.  Index arithmetic is 32-bit
// (entries below 2^30, checked at set-up).
constexpr int KS = 8;

template <typename T>
__global__ void __launch_bounds__(VB)
assemble_kernel(AsmPlan pl, const T *__restrict__ Y, int64_t estride, const T *__restrict__ x,
                T *__restrict__ y, int64_t n, int ess_kind, int nblk) {
  const int mb = blockIdx.y;
  const T *Ym = Y + (int64_t)mb * estride;
  const T *xm = x ? x + (int64_t)mb * n : nullptr;
  T *ym = y + (int64_t)mb * n;
  const int na = (int)pl.na;
  for (int i = (int)blockIdx.x * VB + (int)threadIdx.x; i < na; i += nblk * VB) {
    const int32_t g = pl.alist[i], a = pl.aoff[i], d = pl.aoff[i + 1] - a;
    int32_t sl[KS];
#pragma unroll
    for (int j = 0; j < KS; ++j) sl[j] = (j < d) ? (pl.slot ? pl.slot[a + j] : a + j) : 0;
    T val[KS];
#pragma unroll
    for (int j = 0; j < KS; ++j) val[j] = (j < d) ? Ym[sl[j]] : T(0);
    T acc = val[0];
#pragma unroll
    for (int j = 1; j < KS; ++j)
      if (j < d) acc += val[j];
    for (int j = KS; j < d; ++j) acc += Ym[pl.slot ? pl.slot[a + j] : a + j];
    if (ess_kind == kEssAdd) {
      if (d > 0) ym[g] += acc;
      continue;
    }
    if (d == 0) acc = (ess_kind == kEssCopyX) ? xm[g] : (ess_kind == kEssOne ? T(1) : T(0));
    ym[g] = acc;
  }
}

template <typename T>
__global__ void fill_kernel(T *__restrict__ p, T v, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * VB + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * VB)
    p[i] = v;
}

template <typename T>
__global__ void recip_kernel(const double *__restrict__ d, T *__restrict__ out, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * VB + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * VB)
    out[i] = (T)(1.0 / d[i]);
}

unsigned grid_for(int64_t n) {
  int64_t b = (n + VB * 4 - 1) / (VB * 4);
  if (b < 1) b = 1;
  if (b > 4096) b = 4096;
  return (unsigned)b;
}

}  // namespace

int vec_nblk(int64_t n) {
  int64_t b = (n + VB * 2 - 1) / (VB * 2);
  if (b < 1) b = 1;
  if (b > kMaxParts) b = kMaxParts;
  return (int)b;
}

template <typename T>
hipError_t VecOps<T>::start(const T *b, const T *w, T *x, T *r, const T *dinv, int64_t dms, T *p,
                            double *part, int nblk, int64_t n, int nb, hipStream_t s) {
  hipLaunchKernelGGL((start_kernel<T>), dim3(nblk, nb), dim3(VB), 0, s, b, w, x, r, dinv, dms, p,
                     part, nblk, n);
  return hipGetLastError();
}

template <typename T>
hipError_t VecOps<T>::dot(const T *a, const T *c, int64_t c_mstride, double *part, int nblk,
                          int64_t n, int nb, hipStream_t s) {
  hipLaunchKernelGGL((dot_kernel<T>), dim3(nblk, nb), dim3(VB), 0, s, a, c, c_mstride, part, nblk, n);
  return hipGetLastError();
}

template <typename T>
hipError_t VecOps<T>::update(const CgDofs &dofs, const T *evec, int64_t estride, const T *y, T *x, T *p, T *r,
                             const T *dinv, int64_t dms, const PcgScalars *sc, PcgScalars *sc_next,
                             const double *dpart, int64_t dmstride, int dcount, double *part, int nblk,
                             int64_t n, int nb, hipStream_t s) {
  hipLaunchKernelGGL((cg_update_kernel<T, T, false>), dim3(nblk, nb), dim3(CU_NT), 0, s, dofs, evec, estride,
                     y, x, p, r, dinv, dms, sc, sc_next, dpart, dmstride, dcount, part, nblk, n, CgzOut<T>{});
  return hipGetLastError();
}

template <typename T>
hipError_t VecOps<T>::fill(T *p, T v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL((fill_kernel<T>), dim3(grid_for(n)), dim3(VB), 0, s, p, v, n);
  return hipGetLastError();
}

template <typename T>
hipError_t VecOps<T>::recip(const double *d, T *out, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL((recip_kernel<T>), dim3(grid_for(n)), dim3(VB), 0, s, d, out, n);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_assemble(const AsmPlan &pl, const T *evec, int64_t estride, const T *x, T *y,
                           int64_t n, int nb, int ess_kind, hipStream_t s) {
  if (pl.na <= 0 || nb <= 0) return hipSuccess;
  int64_t nblk = (pl.na + VB - 1) / VB;
  if (nblk > 8192) nblk = 8192;
  hipLaunchKernelGGL((assemble_kernel<T>), dim3((unsigned)nblk, nb), dim3(VB), 0, s, pl, evec, estride, x, y,
                     n, ess_kind, (int)nblk);
  return hipGetLastError();
}
template hipError_t launch_assemble<double>(const AsmPlan &, const double *, int64_t, const double *,
                                            double *, int64_t, int, int, hipStream_t);
template hipError_t launch_assemble<float>(const AsmPlan &, const float *, int64_t, const float *,
                                           float *, int64_t, int, int, hipStream_t);

template struct VecOps<double>;
template struct VecOps<float>;

template <typename TZ>
hipError_t launch_cgz_update(const CgDofs &dofs, const double *evec, const double *y, double *x, double *p,
                             double *r, const TZ *z, float *r32, TZ *t, const TZ *tdinv, TZ omega,
                             const PcgScalars *sc, PcgScalars *sc_next, const double *dpart, int dcount,
                             int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int nblk = cg_update_nblk(n, 1);
  hipLaunchKernelGGL((cg_update_kernel<double, TZ, true>), dim3(nblk), dim3(CU_NT), 0, s, dofs, evec, (int64_t)0,
                     y, x, p, r, z, (int64_t)0, sc, sc_next, dpart, (int64_t)0, dcount, (double *)nullptr, nblk, n,
                     CgzOut<TZ>{r32, t, tdinv, omega});
  return hipGetLastError();
}
template hipError_t launch_cgz_update<double>(const CgDofs &, const double *, const double *, double *, double *,
                                              double *, const double *, float *, double *, const double *, double,
                                              const PcgScalars *, PcgScalars *, const double *, int, int64_t,
                                              hipStream_t);
template hipError_t launch_cgz_update<float>(const CgDofs &, const double *, const double *, double *, double *,
                                             double *, const float *, float *, float *, const float *, float,
                                             const PcgScalars *, PcgScalars *, const double *, int, int64_t,
                                             hipStream_t);

template <typename TZ>
hipError_t launch_cgz_dots(const double *r, const TZ *z, const double *b, double *part, int nblk, int64_t n,
                           hipStream_t s) {
  if (b)
    hipLaunchKernelGGL((cgz_dots_kernel<TZ, true>), dim3(nblk), dim3(CU_NT), 0, s, r, z, b, part, nblk, n);
  else
    hipLaunchKernelGGL((cgz_dots_kernel<TZ, false>), dim3(nblk), dim3(CU_NT), 0, s, r, z, b, part, nblk, n);
  return hipGetLastError();
}
template hipError_t launch_cgz_dots<double>(const double *, const double *, const double *, double *, int, int64_t,
                                            hipStream_t);
template hipError_t launch_cgz_dots<float>(const double *, const float *, const double *, double *, int, int64_t,
                                           hipStream_t);

hipError_t launch_sub_norm(const double *b, const double *w, double *r, double *part, int nblk,
                           int64_t n, int nb, hipStream_t s) {
  hipLaunchKernelGGL(sub_norm_kernel, dim3(nblk, nb), dim3(VB), 0, s, b, w, r, part, nblk, n);
  return hipGetLastError();
}

hipError_t launch_pcg_init(const double *part, int nblk, int nb, double rtol, PcgScalars *sc,
                           hipStream_t s, int nullspace, int64_t n) {
  hipLaunchKernelGGL(init_scalars_kernel, dim3(nb), dim3(RB), 0, s, part, nblk, rtol, sc, nullspace, n);
  return hipGetLastError();
}

// (all members together fill the chip: every workgroup of the update reads all partials of its
// member's p.Ap, which number nb times those of one member, and every workgroup of the element
// kernel the update's partials of its members)
int cg_update_nblk(int64_t n, int nb) {
  const int64_t most = nb < kCgUpdateMax ? kCgUpdateMax / nb : 1;
  int64_t b = (n + CU_NT - 1) / CU_NT;
  if (b < 1) b = 1;
  if (b > most) b = most;
  return (int)b;
}

hipError_t launch_cg_fold(const double *dpart, int64_t dmstride, int dcount, double *out, int nblk, int nb,
                          hipStream_t s) {
  hipLaunchKernelGGL(cg_fold_kernel, dim3(nblk, nb), dim3(VB), 0, s, dpart, dmstride, dcount, out, nblk);
  return hipGetLastError();
}

hipError_t launch_cg_finish(PcgScalars *sc, PcgScalars *host, const double *part, int nblk, int nb,
                            int nullspace, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(cg_finish_kernel, dim3(nb), dim3(256), 0, s, sc, host, part, nblk, nullspace, n);
  return hipGetLastError();
}

hipError_t launch_shift(double *v, const double *c, double scale, int64_t n, int nb, hipStream_t s) {
  if (n <= 0 || nb <= 0) return hipSuccess;
  hipLaunchKernelGGL(shift_kernel, dim3(grid_for(n), nb), dim3(VB), 0, s, v, c, scale, n);
  return hipGetLastError();
}

hipError_t launch_reduce1(const double *part, int nblk, int nb, double *out, hipStream_t s) {
  hipLaunchKernelGGL((reduce_out_kernel<1>), dim3(nb), dim3(RB), 0, s, part, nblk, out);
  return hipGetLastError();
}

hipError_t launch_ir_norm(const double *part, int nblk, int nb, int set_bb, double rtol, double *ir,
                          hipStream_t s) {
  hipLaunchKernelGGL(ir_norm_kernel, dim3(nb), dim3(RB), 0, s, part, nblk, set_bb, rtol, ir);
  return hipGetLastError();
}

hipError_t launch_ir_cast(const double *r, const double *ir, float *r32, int64_t n, int nb,
                          hipStream_t s) {
  hipLaunchKernelGGL(ir_cast_kernel, dim3(grid_for(n), nb), dim3(VB), 0, s, r, ir, r32, n);
  return hipGetLastError();
}

hipError_t launch_ir_accum(double *x, const float *d, const double *ir, int64_t n, int nb,
                           hipStream_t s) {
  hipLaunchKernelGGL(ir_accum_kernel, dim3(grid_for(n), nb), dim3(VB), 0, s, x, d, ir, n);
  return hipGetLastError();
}

}  // namespace sfem
