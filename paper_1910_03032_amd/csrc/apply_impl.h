// Sum-factorized element kernels for Q_p hexahedra on gfx950.
//
// Per element (Section 3.1, eq. sumFactorized and L^K = G^T W G):
//   gather x_e -> contract xi_1 with B, G -> contract xi_2 -> contract xi_3
//   -> pointwise quadrature function (v = alpha w|J| u, g = beta nu w|J| J^-1 J^-T grad_ref u)
//      with the geometric factors formed from the element's trilinear map (geom.h)
//   -> transposed contractions xi_3 -> xi_2 -> xi_1 -> scatter into y.
//
// Work decomposition: one element is owned by q^2 threads; in every stage a thread
// owns one 1D line of the tensor along the direction being contracted, holds the
// n (or q) inputs of that line in registers and produces the whole output line, so
// LDS is read once per input value.  The 1D tables are compile-time constants and
// every contraction uses their symmetry (even-odd form: the nodes and the Gauss
// points are symmetric about 0, so B is centro-symmetric and G centro-antisymmetric),
// which halves the multiply-adds; the xi_3 stage walks the quadrature slices in
// symmetric pairs (c, q-1-c).  Intermediates between stages live in LDS, one buffer
// per element.  Several (element, batch member) pairs share a workgroup (E of ApplyCfg),
// the members of an element next to each other, so that a batched apply reads each
// element's coefficients from HBM once for all members.
//
// Assembly (no atomics, deterministic): one launch of the element kernel covers every
// element.  A DoF that belongs to this element only (the element-interior nodes of a
// conforming mesh) is written straight to y.  The value of a shared node (element
// surface) goes to its own entry of the E-vector, which is ordered by destination DoF
// (the entry comes from a position table read with the map); an assembly kernel then
// gives each shared DoF to one thread, which sums its contiguous E-vector entries in
// element order (owner computes) -- and sets the essential DoFs.
// Workgroups are mapped to elements so that each of the 8 XCDs works on one
// contiguous range of elements, which keeps the x values shared by neighbouring
// elements in that XCD's L2.
//
// LDS layouts inside an element buffer (a, b, c: quadrature indices along
// xi_1..3; i, j, k: node indices), with the strides of Lds<P>:
//   nodal         [k][j][i]
//   after xi_1    [k][j][a]      (two fields: B- and G-contracted)
//   after xi_2    [k][b][a]      (three fields)
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "energy.h"
#include "eo.h"
#include "geom.h"
#include "internal.h"
#include "pcg.h"
#include "rules.h"

namespace sfem {

template <int P>
struct Dims {
  static constexpr int N = P + 1, Q = P + 2;
  static constexpr int N2 = N * N, N3 = N * N * N, Q2 = Q * Q, Q3 = Q * Q * Q;
  static constexpr int QN2 = Q * N2, NQ2 = N * Q2;
  static constexpr int TPE = Q2;  // threads per element
  static constexpr int E = (256 / TPE) > 0 ? (256 / TPE) : 1;
  static constexpr int mx(int a, int b) { return a > b ? a : b; }
  static constexpr int BUF = mx(N3, mx(2 * Q * N2, 3 * Q2 * N));
  static constexpr int THREADS = E * TPE;
  // minimum waves per SIMD the element kernels are compiled for: the largest that
  // the Helmholtz kernels reach without spilling registers (p = 8 spills slightly)
  static constexpr int OCC = P <= 2 ? 4 : (P <= 6 ? 3 : 2);
};

// Layout of the apply kernels' element buffer.  A half-wave's 32 lanes are served in one
// cycle when they touch different banks, and the bank is the element index modulo 32 for
// 4- and 8-byte elements alike; with dense strides the stages' accesses took about twice
// the cycles of that (2.7 times at p = 6, where every stride is even).  LQ (line of
// [k][j][a]), SK (its plane), SP (plane of [k][b][a]) and BUF modulo 32 (element to element)
// are the strides with the fewest conflicts, counted over all accesses of a workgroup, that
// take at most 12 % more LDS than the dense ones and keep the workgroups per CU (p = 6, 7);
// mass kernels keep one field each (DIFF false).  24^3 p = 6 in float32: 65 -> 60 us; mass at
// 36^3 p = 4: 68 -> 61 us.  The nodal vectors have a place of their own past the [k][j][a]
// fields, so that the xi_1 stages need no barrier between their reads and writes.
template <int P, bool DIFF = true>
struct Lds {
  static constexpr int N = P + 1, Q = P + 2;
  static constexpr int pick(int a1, int a2, int a3, int a4, int a5, int a6, int a7, int a8) {
    return P == 1 ? a1 : P == 2 ? a2 : P == 3 ? a3 : P == 4 ? a4 : P == 5 ? a5 : P == 6 ? a6 : P == 7 ? a7 : a8;
  }
  static constexpr int LN = pick(2, 3, 5, 5, 7, 7, 9, 9);
  static constexpr int LQ = pick(3, 5, 6, 7, 7, 9, 9, 11);
  static constexpr int SK = pick(12, 20, 24, 38, 42, 72, 72, 103);
  static constexpr int SP = pick(11, 20, 25, 38, 56, 68, 81, 106);
  static constexpr int XF = N * SK, YF = N * SP;  // fields of [k][j][a] and of [k][b][a]
  static constexpr int NOD = DIFF ? 2 * XF : XF;
  static constexpr int FULL = pick(72, 188, 325, 580, 1009, 1428, 1952, 2884);
  static constexpr int MASS = NOD + N * N * LN > YF ? NOD + N * N * LN : YF;
  static constexpr int BUF = DIFF ? FULL : MASS + (FULL % 32 - MASS % 32 + 32) % 32;
  static_assert(LN >= N && LQ >= Q && SK >= N * LQ && SP >= Q * Q, "strides");
  static_assert(BUF >= NOD + N * N * LN && BUF >= (DIFF ? 3 : 1) * YF, "element buffer");
  static __device__ __forceinline__ int nodal(int l) { return NOD + (LN == N ? l : l + l / N); }
  static_assert(LN == N || LN == N + 1, "nodal()");
};
// The dense nodal vector at the start of a buffer.
struct DenseNodal {
  static __device__ __forceinline__ int nodal(int l) { return l; }
};

// Barrier between the stages of one element's threads.  Where a wave holds whole elements,
// they exchange data inside it only, and LDS keeps a wave's accesses in order (p = 2 and 6
// without the workgroup's barriers: 201 -> 185 us at 72^3 p = 2, float64).
// (TH: threads of the workgroup)
template <int P, int TH = Dims<P>::THREADS>
__device__ __forceinline__ void elem_sync() {
  if constexpr (64 % Dims<P>::TPE == 0 || TH <= 64) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// The 1D tables as compile-time constants of the order P (q = P + 2): after loop
// unrolling every table entry is a literal, so no table lives in registers or memory.
template <int P, typename T>
struct Tab {
  static constexpr rules::Tables<P, P + 2> c = rules::tables<P, P + 2>();
  __host__ __device__ static constexpr T B(int a, int i) { return (T)c.B[a][i]; }
  __host__ __device__ static constexpr T G(int a, int i) { return (T)c.G[a][i]; }
};

// Local nodes one thread handles in the gather and output loops (l = t + k TPE).
template <int P>
struct Per {
  static constexpr int NL = (Dims<P>::N3 + Dims<P>::TPE - 1) / Dims<P>::TPE;
};

// Rank of local node l among the element's surface nodes (a node with i, j or k in
// {0, p}): face k = 0, face k = p, then for each interior k the ring of the (i, j)
// square; -1 for an interior node.  The ranks of all local nodes of order P form a
// table in constant memory: one 2-byte load per node instead of index arithmetic.
template <int P>
struct RankTable {
  int16_t r[(P + 1) * (P + 1) * (P + 1)];
};
template <int P>
constexpr RankTable<P> make_rank_table() {
  RankTable<P> t{};
  constexpr int N = P + 1;
  for (int l = 0; l < N * N * N; ++l) {
    const int i = l % N, j = (l / N) % N, k = l / (N * N);
    int r = -1;
    if (k == 0) {
      r = i + N * j;
    } else if (k == P) {
      r = N * N + i + N * j;
    } else {
      const int base = 2 * N * N + (k - 1) * 4 * P;
      if (j == 0)
        r = base + i;
      else if (j == P)
        r = base + N + i;
      else if (i == 0 || i == P)
        r = base + 2 * N + 2 * (j - 1) + (i == 0 ? 0 : 1);
    }
    t.r[l] = (int16_t)r;
  }
  return t;
}
template <int P>
__constant__ RankTable<P> kRankTable = make_rank_table<P>();
template <int P>
constexpr RankTable<P> make_node_table() {
  RankTable<P> t{};
  for (int l = 0; l < (P + 1) * (P + 1) * (P + 1); ++l) t.r[l] = (int16_t)l;
  return t;
}
// The general layout's entry order: the node itself.
template <int P>
__constant__ RankTable<P> kNodeTable = make_node_table<P>();
template <int P>
__host__ __device__ constexpr int surf_count() {
  return 2 * (P + 1) * (P + 1) + (P - 1) * 4 * P;
}

// One value at a byte offset from a pointer that is the same in all lanes (scalar base and
// 32-bit lane offset, no 64-bit address arithmetic per lane).
template <typename T>
__device__ __forceinline__ T ld(const void *base, uint32_t byte) {
  return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + byte);
}

// Index tables of the elements of one workgroup, advanced to its first element (e0).
struct ElemTab {
  const int32_t *map;   // [..][n^3] flagged map
  const int32_t *pos;   // [..][epe] E-vector entries (DoF-ordered E-vector), or unused
  const int16_t *rank;  // node -> entry within the element's E-vector row (-1: none)
  uint32_t ebase;       // element-ordered E-vector: entry of e0's row
  uint32_t epe;         // entries per element
};
template <int P>
__device__ __forceinline__ ElemTab elem_tab(const int32_t *map, const int32_t *pos, int compact,
                                            int64_t e0) {
  ElemTab z;
  z.epe = compact ? surf_count<P>() : Dims<P>::N3;
  z.map = map + e0 * Dims<P>::N3;
  z.pos = pos ? pos + e0 * z.epe : nullptr;
  z.rank = compact ? kRankTable<P>.r : kNodeTable<P>.r;
  z.ebase = (uint32_t)(e0 * z.epe);
  return z;
}

// What one thread needs of its nodes l = t + k TPE: the map entry c and the destination d
// of the node's value (the map entry of a sole or essential DoF, the E-vector entry of a
// shared one).  A thread without a k-th node takes the last node, with the same values as
// that node's owner, so that no load or LDS store is predicated: all loads of a group are in
// flight together.
template <int P>
struct Nodes {
  static constexpr int NL = Per<P>::NL;
  int32_t c[NL], r[NL], d[NL];
  static __device__ __forceinline__ int node(int t, int k) {
    const int l = t + k * Dims<P>::TPE;
    return l < Dims<P>::N3 ? l : Dims<P>::N3 - 1;
  }
  // rel: the thread's element, relative to the workgroup's first
  __device__ __forceinline__ void load_map(const ElemTab &z, int t, uint32_t rel) {
#pragma unroll
    for (int k = 0; k < NL; ++k) c[k] = ld<int32_t>(z.map, (rel * Dims<P>::N3 + node(t, k)) * 4u);
  }
  __device__ __forceinline__ void load_rank(const ElemTab &z, int t) {
#pragma unroll
    for (int k = 0; k < NL; ++k) r[k] = ld<int16_t>(z.rank, node(t, k) * 2u);
  }
  // (after load_map and load_rank)
  template <bool POS>
  __device__ __forceinline__ void load_dest(const ElemTab &z, uint32_t rel) {
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const uint32_t w = rel * z.epe + (uint32_t)(r[k] > 0 ? r[k] : 0);
      d[k] = POS ? ld<int32_t>(z.pos, w * 4u) : (int32_t)(z.ebase + w);
    }
#pragma unroll
    for (int k = 0; k < NL; ++k) d[k] = (c[k] >= 0 && !(c[k] & kSoleBit)) ? d[k] : c[k];
  }
  template <typename T>
  __device__ __forceinline__ void load_values(const T *xm, T (&v)[NL]) const {
#pragma unroll
    for (int k = 0; k < NL; ++k) v[k] = xm[c[k] & kDofMask];
  }
  // Keep the loads of v where they were written: under the condition of their use, each would
  // be issued in a branch of its own after whatever is waited for before it.
  template <typename T>
  static __device__ __forceinline__ void pin(T (&v)[NL]) {
#pragma unroll
    for (int k = 0; k < NL; ++k) asm volatile("" : "+v"(v[k]));
  }
  __device__ __forceinline__ void keep(int32_t *smap, int t) const {
#pragma unroll
    for (int k = 0; k < NL; ++k) smap[node(t, k)] = d[k];
  }
};

// The trilinear coefficients of the thread's element into its place in LDS; no barrier.
template <int P>
__device__ __forceinline__ void load_geo(double *sg, const double *geo, int64_t e0, uint32_t rel, int t) {
  constexpr int TPE = Dims<P>::TPE;
#pragma unroll
  for (int k = 0; k * TPE < kGeoStride; ++k) {
    const int i = t + k * TPE < kGeoStride ? t + k * TPE : kGeoStride - 1;
    sg[i] = ld<double>(geo + e0 * kGeoStride, (rel * kGeoStride + i) * 8u);
  }
}

// Gather the element's nodal values (essential DoFs as 0) into the nodal vector of layout
// Lds<P>.  Ends with a barrier.
template <int P, typename T>
__device__ __forceinline__ void gather_e(T *buf, int t, bool active, const Nodes<P> &nd,
                                         const T *__restrict__ xm) {
  T v[Nodes<P>::NL];
  nd.load_values(xm, v);
  nd.pin(v);
#pragma unroll
  for (int k = 0; k < Nodes<P>::NL; ++k)
    buf[Lds<P>::nodal(Nodes<P>::node(t, k))] = (active && nd.c[k] >= 0) ? v[k] : T(0);
  elem_sync<P>();
}

// Output of the element vector at L::nodal: sole DoFs -> y, shared nodes -> their E-vector
// entry, essential -> nothing.  The destinations come from LDS, kept by the gather.
template <int P, typename T, class L = DenseNodal>
__device__ __forceinline__ void emit_e(const T *buf, int t, bool active, const int32_t *smap,
                                       T *__restrict__ Y, T *__restrict__ y) {
  using D = Dims<P>;
  constexpr int NL = Per<P>::NL;
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    const int l = Nodes<P>::node(t, k);
    const int32_t c = smap[l];
    const T v = buf[L::nodal(l)];
    // one predicated store per node: the destination is selected, not branched to
    if (active && t + k * D::TPE < D::N3 && c >= 0) ((c & kSoleBit) ? y : Y)[c & kDofMask] = v;
  }
}

// Deterministic sum over a block of THREADS threads, result on thread 0 (sh: THREADS / 64 + 1
// doubles): a wave total each (the last wave may be partial), then the waves in order.
template <int THREADS>
__device__ __forceinline__ double block_sum_d(double v, double *sh) {
  constexpr int NW = (THREADS + 63) / 64;
  const int wave = threadIdx.x >> 6;
  v = wave_total(v, wave == NW - 1 ? THREADS - 1 - 64 * (NW - 1) : 63);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[wave] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < NW; ++w) s += sh[w];
  return s;
}

// xi_1 contraction: [k][j][i] -> [k][j][a] with B (field 0) and, if DIFF, G (field 1).
template <int P, typename T, bool DIFF, int TH = Dims<P>::THREADS>
__device__ __forceinline__ void fwd_x(T *buf, int t) {
  using D = Dims<P>;
  using L = Lds<P, DIFF>;
  constexpr int N = D::N, Q = D::Q;
  const bool w = t < D::N2;
  const int j = t % N, k = t / N;
  T ob[Q], og[Q];
  if (w) {
    T in[N];
#pragma unroll
    for (int i = 0; i < N; ++i) in[i] = buf[L::NOD + (k * N + j) * L::LN + i];
    const auto sp = eo::split(in);
    eo::apply<eo::Tab1<P, 0>>(sp, ob);
    if constexpr (DIFF) eo::apply<eo::Tab1<P, 1>>(sp, og);
  }
  if (w) {
#pragma unroll
    for (int a = 0; a < Q; ++a) {
      buf[k * L::SK + j * L::LQ + a] = ob[a];
      if constexpr (DIFF) buf[L::XF + k * L::SK + j * L::LQ + a] = og[a];
    }
  }
  elem_sync<P, TH>();
}

// xi_2 contraction: [k][j][a] -> [k][b][a]: field 0 = B(B x), and if DIFF
// field 1 = G_y(B_x x) (for d/dxi_2), field 2 = B_y(G_x x) (for d/dxi_1).
template <int P, typename T, bool DIFF, int TH = Dims<P>::THREADS>
__device__ __forceinline__ void fwd_y(T *buf, int t) {
  using D = Dims<P>;
  using L = Lds<P, DIFF>;
  constexpr int N = D::N, Q = D::Q;
  const bool w = t < Q * N;
  const int a = t % Q, k = t / Q;
  T obb[Q], ogb[Q], obg[Q];
  if (w) {
    T ib[N], ig[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      ib[j] = buf[k * L::SK + j * L::LQ + a];
      if constexpr (DIFF) ig[j] = buf[L::XF + k * L::SK + j * L::LQ + a];
    }
    const auto sb = eo::split(ib);
    eo::apply<eo::Tab1<P, 0>>(sb, obb);
    if constexpr (DIFF) {
      eo::apply<eo::Tab1<P, 1>>(sb, ogb);
      eo::apply<eo::Tab1<P, 0>>(eo::split(ig), obg);
    }
  }
  elem_sync<P, TH>();
  if (w) {
#pragma unroll
    for (int b = 0; b < Q; ++b) {
      buf[k * L::SP + b * Q + a] = obb[b];
      if constexpr (DIFF) {
        buf[L::YF + k * L::SP + b * Q + a] = ogb[b];
        buf[2 * L::YF + k * L::SP + b * Q + a] = obg[b];
      }
    }
  }
  elem_sync<P, TH>();
}

// Read the xi_3 lines of thread t = a + q b (no barrier).
template <int P, typename T, bool DIFF>
__device__ __forceinline__ void load_z(const T *buf, int t, T (&zbb)[P + 1], T (&zgb)[P + 1],
                                       T (&zbg)[P + 1]) {
  using L = Lds<P, DIFF>;
#pragma unroll
  for (int k = 0; k < L::N; ++k) {
    zbb[k] = buf[k * L::SP + t];
    if constexpr (DIFF) {
      zgb[k] = buf[L::YF + k * L::SP + t];
      zbg[k] = buf[2 * L::YF + k * L::SP + t];
    }
  }
}

// Transposed xi_2: [k][b][a] (fields p1, p2, p3) -> [k][j][a] (fields r1, r2) with
// r1 = B^T p1 + G^T p2 and r2 = B^T p3.
template <int P, typename T, bool DIFF, int TH = Dims<P>::THREADS>
__device__ __forceinline__ void bwd_y(T *buf, int t) {
  using D = Dims<P>;
  using L = Lds<P, DIFF>;
  using BT = eo::Tab1<P, 0>;
  using GT = eo::Tab1<P, 1>;
  constexpr int N = D::N, Q = D::Q;
  const bool w = t < Q * N;
  const int a = t % Q, k = t / Q;
  T r1[N], r2[N];
  if (w) {
    T i1[Q], i2[Q], i3[Q];
#pragma unroll
    for (int b = 0; b < Q; ++b) {
      i1[b] = buf[k * L::SP + b * Q + a];
      if constexpr (DIFF) {
        i2[b] = buf[L::YF + k * L::SP + b * Q + a];
        i3[b] = buf[2 * L::YF + k * L::SP + b * Q + a];
      }
    }
    eo::Acc<N, T> A1, A2;
    A1.zero();
    A2.zero();
#pragma unroll
    for (int b = 0; b < Q / 2; ++b) {
      A1.template add_pair<BT>(b, i1[b], i1[Q - 1 - b]);
      if constexpr (DIFF) {
        A1.template add_pair<GT>(b, i2[b], i2[Q - 1 - b]);
        A2.template add_pair<BT>(b, i3[b], i3[Q - 1 - b]);
      }
    }
    if constexpr (Q % 2 == 1) {
      A1.template add_mid<BT>(i1[Q / 2]);
      if constexpr (DIFF) {
        A1.template add_mid<GT>(i2[Q / 2]);
        A2.template add_mid<BT>(i3[Q / 2]);
      }
    }
    A1.finish(r1);
    if constexpr (DIFF) A2.finish(r2);
  }
  elem_sync<P, TH>();
  if (w) {
#pragma unroll
    for (int j = 0; j < N; ++j) {
      buf[k * L::SK + j * L::LQ + a] = r1[j];
      if constexpr (DIFF) buf[L::XF + k * L::SK + j * L::LQ + a] = r2[j];
    }
  }
  elem_sync<P, TH>();
}

// Transposed xi_1: [k][j][a] (r1, r2) -> nodal [k][j][i] = B^T r1 + G^T r2.
template <int P, typename T, bool DIFF, int TH = Dims<P>::THREADS>
__device__ __forceinline__ void bwd_x(T *buf, int t) {
  using D = Dims<P>;
  using L = Lds<P, DIFF>;
  using BT = eo::Tab1<P, 0>;
  using GT = eo::Tab1<P, 1>;
  constexpr int N = D::N, Q = D::Q;
  const bool w = t < D::N2;
  const int j = t % N, k = t / N;
  T yo[N];
  if (w) {
    T i1[Q], i2[Q];
#pragma unroll
    for (int a = 0; a < Q; ++a) {
      i1[a] = buf[k * L::SK + j * L::LQ + a];
      if constexpr (DIFF) i2[a] = buf[L::XF + k * L::SK + j * L::LQ + a];
    }
    eo::Acc<N, T> A;
    A.zero();
#pragma unroll
    for (int a = 0; a < Q / 2; ++a) {
      A.template add_pair<BT>(a, i1[a], i1[Q - 1 - a]);
      if constexpr (DIFF) A.template add_pair<GT>(a, i2[a], i2[Q - 1 - a]);
    }
    if constexpr (Q % 2 == 1) {
      A.template add_mid<BT>(i1[Q / 2]);
      if constexpr (DIFF) A.template add_mid<GT>(i2[Q / 2]);
    }
    A.finish(yo);
  }
  if (w) {
#pragma unroll
    for (int i = 0; i < N; ++i) buf[L::NOD + (k * N + j) * L::LN + i] = yo[i];
  }
  elem_sync<P, TH>();
}

// Index of the element batch of this workgroup such that XCD k (workgroups are
// dispatched round-robin over the 8 XCDs) gets one contiguous range of batches.
__device__ __forceinline__ int xcd_block() {
  const unsigned nblk = gridDim.x, b = blockIdx.x;
  const unsigned xcd = b & 7u, k = b >> 3;
  const unsigned q8 = nblk >> 3, r8 = nblk & 7u;
  return (int)(xcd * q8 + (xcd < r8 ? xcd : r8) + k);
}

// How the element kernel of order P and precision T is built (chosen by measurement on
// MI355X):
//   ZLDS   the xi_3 stage's input lines are read from LDS again for every slice pair, one at
//          a time, instead of being held in registers for the whole stage: where that decides
//          the waves per SIMD.  Float64 p = 7 has two either way and holds them (243 registers
//          of 256, LDS busy a third: three members at 24^3 377 -> 350 us);
//   OCC    minimum waves per SIMD the kernel is compiled for (launch bound): three float64
//          ones at p = 5 and 6 as well (29^3 p = 5 115 -> 100 us, 24^3 p = 6 101 -> 82 us,
//          Helmholtz with nu).  Four at p = 3 and 4, and three at p = 7, would spill 44 to
//          100 bytes (1.00, 0.85 and 0.85 times as fast);
//   REFORM the output's addresses are formed anew: kept since the gather they cost the stages
//          up to 15 registers, and with them spills, whose stores wait for the prologue's
//          loads (12^3 p = 5 16.8 -> 16.3 us, float32 18^3 p = 8 61 -> 59 us with four waves;
//          without a spill to save 0.5 to 3 % slower);
//   E      elements per workgroup (q^2 threads each).  The applies take as many as fill one
//          wave at p = 1, whose stages then need no barriers, and two waves at p = 3 (1.05
//          and 1.03 - 1.06 times as fast as four waves); one to three waves were slower at
//          p = 4, 5 and 8 (0.90 - 0.98), and the CG iteration's kernels read the partial sums
//          once per workgroup.  Eight waves at p = 8, which leave few lanes idle: 0.94
//          (float32 0.79).
template <int P, typename T, int CG>
struct ApplyCfg {
  static constexpr bool F64 = sizeof(T) == 8;
  static constexpr int E = CG ? Dims<P>::E : P == 1 ? 7 : P == 3 ? 5 : Dims<P>::E;
  static constexpr int THREADS = E * Dims<P>::TPE;
  static constexpr bool ZLDS = F64 ? (P == 5 || P == 6 || P == 8) : (P == 6 || P == 8 || (CG && P >= 4));
  static constexpr int OCC = F64 ? Dims<P>::OCC : (P <= 6 || (P == 8 && !CG) ? 4 : 3);
  static constexpr bool REFORM = CG != 0 || P == (F64 ? 5 : 8);
};

// The plain applies pass no CG inputs (half of the launch's argument bytes).
struct NoCg {};

// OP: 0 mass, 1 diffusion, 2 helmholtz (matches sfem_op).  Writes y at the sole DoFs
// and the E-vector Y[m] at the shared nodes.
//
// The geometric factors are formed from the element's trilinear coefficients (geom.h) along
// each thread's xi_3 line; with NU the kernel reads one value per point, cw = w nu / |J|
// ([nelem][q^3] per field, float64 for both precisions), and without (nu = 1) none.  The
// float64 operators multiply by adj(J) twice.  The float32 ones form the six factors in
// float64 and round each once, so that they are those a stored float32 copy would hold
// (forming them in float32 rounds adj(J) twice each: 5-15 % more error of the apply), THIN from
// adj(J) where the metric would lose digits (kMetricLimit).
//
// Reading the factors (7 values per point) bound the kernel by HBM: of the 553 MB of an apply
// at 32^3 p = 4 in float64, 396 MB were factors.  Formed, they cost 35 to 40 operations a
// point, and the kernel is bound by VALU issue, LDS and the latency between its barriers:
// 120.3 -> 77.3 us there, 212 -> 126 us for nu = 1 at 63 x 61 x 59 p = 2, float32 32^3 p = 8
// 341 -> 290 us.  With the layouts of Lds, eight barriers a workgroup instead of eleven, and
// every load of the prologue issued before the first wait for the map's followers: 69, 100 and
// 264 us.  Of 107 us at 36^3 p = 4 the loads, stores and the assembly alone took 68 and the
// quadrature function 20; of a workgroup's 20000 cycles, its loads took 7000 and VALU issue 3900.
//
// Work items are (element, member) pairs, pair v = e * nbatch + m, E per workgroup: the
// members of one element run side by side (in the same workgroup or in neighbouring
// ones, on one XCD) and read the element's coefficients, which all members share unless
// cw_mstride != 0, from the same cache lines.
// CG = 1: the first launch of a CG iteration (pcg.h) with z = dinv r; CG = 2: with z given; x is
// unused and part required.  The partials
// of p.Ap are then the element energies at the quadrature points, sum v u + g . grad_ref u, plus
// p^2 of the essential DoFs at the element that carries their flag (kEssOwnerBit).
template <int P, typename T, int OP, bool NU, int CG, bool THIN>
__global__ void __launch_bounds__((ApplyCfg<P, T, CG>::THREADS), (ApplyCfg<P, T, CG>::OCC))
apply_kernel(const int32_t *__restrict__ map, const double *__restrict__ geo,
             const double *__restrict__ cw, int64_t cw_mstride, double alpha, double beta, int64_t nelem,
             int nbatch, int64_t ndof, const T *__restrict__ x, T *__restrict__ Y,
             int64_t estride, const int32_t *__restrict__ pos, int compact, T *__restrict__ y,
             double *__restrict__ part,
             int64_t part_mstride, std::conditional_t<CG != 0, CgIn, NoCg> cg) {
  using D = Dims<P>;
  constexpr int N = D::N, Q = D::Q, Q2 = D::Q2, Q3 = D::Q3, N3 = D::N3;
  using C = ApplyCfg<P, T, CG>;
  constexpr int TPE = D::TPE, E = C::E, THREADS = C::THREADS;
  constexpr bool MASS = (OP == 0) || (OP == 2);
  constexpr bool DIFF = (OP == 1) || (OP == 2);
  using LD = Lds<P, DIFF>;

  constexpr bool POS = evec_dof_ordered(P);
  // element buffers; after the output step also the block sum of the fused dot product
  static_assert(E * LD::BUF * sizeof(T) >= 8 * sizeof(double), "block sum space");
  __shared__ __align__(16) T smem[E * LD::BUF];
  __shared__ __align__(16) double sgeo[E * kGeoStride];  // the elements' trilinear coefficients
  __shared__ __align__(16) double sgauss[E * 2 * Q];     // the Gauss rule, for each element's threads
  __shared__ int32_t smap_all[E * N3];  // the elements' map entries, kept for the output
  const int le = threadIdx.x / TPE;
  const int t = threadIdx.x - le * TPE;
  // the grid has one workgroup per E (element, member) pairs (nelem * nbatch pairs); the
  // workgroup's first pair is (e0, r0), the thread's is (e0 + rel, m)
  const int64_t npair = nelem * (int64_t)nbatch;
  const int64_t v_lo = (int64_t)xcd_block() * E;
  const int count = (int)((npair - v_lo) < E ? (npair - v_lo) : E);
  const bool active = le < count;
  int64_t e0 = v_lo;
  uint32_t r0 = 0, rel = active ? le : 0, m = 0;  // (inactive slots redo e0's data)
  if (nbatch != 1) {
    e0 = v_lo / nbatch;
    r0 = (uint32_t)(v_lo - e0 * nbatch);
    const uint32_t rr = r0 + rel;
    rel = rr / (uint32_t)nbatch;
    m = rr - rel * (uint32_t)nbatch;
  }
  T *buf = smem + le * LD::BUF;
  double dot = 0.0;  // CG: the thread's part of p.Ap

  {
    const T *xm = CG ? nullptr : x + (int64_t)m * ndof;
    // first group of loads: the map, the entry order, the coefficients of the element and
    // of the thread's points; then what the map leads to
    const ElemTab z = elem_tab<P>(map, pos, compact, e0);
    Nodes<P> nd;
    nd.load_map(z, t, rel);
    nd.load_rank(z, t);
    constexpr int NW = CG ? THREADS / 64 : 1;
    // CG: the update's partials of the workgroup's first member and the state; also when the
    // state is ready, for loads under a condition are waited for where it ends
    std::conditional_t<CG != 0, PartLoads<NW, 2>, NoCg> up;
    PcgScalars s;
    if constexpr (CG) {
      up.load(cg.upart + (int64_t)r0 * 4 * cg.unblk, cg.unblk);
      copy_state(s, cg.sc[m]);
    }
    constexpr int NG = (kGeoStride + TPE - 1) / TPE;
    double gv[NG];
#pragma unroll
    for (int k = 0; k < NG; ++k) {
      const int i = t + k * TPE < kGeoStride ? t + k * TPE : kGeoStride - 1;
      gv[k] = ld<double>(geo + e0 * kGeoStride, (rel * kGeoStride + i) * 8u);
    }
    double cv[Q];  // w nu / |J| at the points of the thread's line
    if constexpr (NU) {
      const double *ce = cw + (int64_t)m * cw_mstride + e0 * (int64_t)Q3 + (rel * Q3 + t);
#pragma unroll
      for (int c = 0; c < Q; ++c) cv[c] = ce[c * Q2];
    }
    static_assert(sizeof(rules::GaussRule<Q>) == 2 * Q * sizeof(double) && TPE >= 2 * Q, "points, then weights");
    const int gi = t < 2 * Q ? t : 2 * Q - 1;
    const double gq = ld<double>(&kGaussRule<Q>, (uint32_t)gi * 8u);
    int32_t *smap = smap_all + le * N3;
    constexpr int NL = Nodes<P>::NL;
    T v[CG ? 1 : NL];
    T zr[CG ? NL : 1], zd[CG ? NL : 1], zp[CG ? NL : 1];
    if constexpr (!CG) {
      nd.load_values(xm, v);
    } else {
      if constexpr (CG == 1) {
        nd.load_values((const T *)cg.r + (int64_t)m * ndof, zr);
        nd.load_values((const T *)cg.dinv + (int64_t)m * cg.dinv_mstride, zd);
      } else {
        if (cg.z32) {
#pragma unroll
          for (int j = 0; j < NL; ++j) zr[j] = (T)((const float *)cg.z)[nd.c[j] & kDofMask];
        } else {
          nd.load_values((const T *)cg.z, zr);
        }
#pragma unroll
        for (int j = 0; j < NL; ++j) zd[j] = T(1);
      }
      nd.load_values((const T *)cg.p + (int64_t)m * ndof, zp);
    }
    nd.template load_dest<POS>(z, rel);
#pragma unroll
    for (int k = 0; k < NG; ++k)
      sgeo[le * kGeoStride + (t + k * TPE < kGeoStride ? t + k * TPE : kGeoStride - 1)] = gv[k];
    double *sgq = sgauss + le * 2 * Q;
    sgq[gi] = gq;
    if constexpr (!CG) {
      nd.pin(v);
      nd.keep(smap, t);
#pragma unroll
      for (int k = 0; k < NL; ++k)
        buf[LD::nodal(Nodes<P>::node(t, k))] = (active && nd.c[k] >= 0) ? v[k] : T(0);
      elem_sync<P, THREADS>();
    } else {
      // the states of the workgroup's members: here distinct ones, the k-th (r0 + k) mod nbatch
      __shared__ double sums[E][4][NW];
      const int here = nbatch < count ? nbatch : count;
      const int k = le < here ? le : le % here;
      auto other_parts = [&](double (&sh)[4][NW], int64_t mm, bool all) {
        const double *p = cg.upart + mm * 4 * cg.unblk;
        PartLoads<NW, 2> q;
        if (all) {
          q.load(p, cg.unblk);
          q.parts(sh, cg.unblk);
        }
        if (cg.nullspace) {
          q.load(p + 2 * (int64_t)cg.unblk, cg.unblk);
          q.parts(*reinterpret_cast<double(*)[4][NW]>(&sh[2]), cg.unblk);
        }
      };
      if (!cg.ready) {
        up.parts(sums[0], cg.unblk);
        other_parts(sums[0], r0, false);
        for (int i = 1; i < here; i += 2) {  // two members' loads together
          const int i1 = i + 1 < here ? i + 1 : i;
          const uint32_t ma = (r0 + (uint32_t)i) % (uint32_t)nbatch, mb = (r0 + (uint32_t)i1) % (uint32_t)nbatch;
          PartLoads<NW, 2> qa, qb;
          qa.load(cg.upart + (int64_t)ma * 4 * cg.unblk, cg.unblk);
          qb.load(cg.upart + (int64_t)mb * 4 * cg.unblk, cg.unblk);
          qa.parts(sums[i], cg.unblk);
          qb.parts(sums[i1], cg.unblk);
          other_parts(sums[i], ma, false);
          if (i1 > i) other_parts(sums[i1], mb, false);
        }
        __syncthreads();
        cg_next_from<NW>(s, sums[k], cg.nullspace, ndof);
      }
      if (blockIdx.x == 0) {  // the first workgroup passes the states on (r0 = 0)
        if (t == 0 && le < here) {
          copy_state(cg.sc_next[m], s);
          if (cg.host) copy_state(cg.host[m], s);
        }
        for (int mm = here; mm < nbatch; ++mm) {
          PcgScalars o;
          copy_state(o, cg.sc[mm]);
          if (!cg.ready) {
            __syncthreads();
            other_parts(sums[0], mm, true);
            __syncthreads();
            cg_next_from<NW>(o, sums[0], cg.nullspace, ndof);
          }
          if (threadIdx.x == 0) {
            copy_state(cg.sc_next[mm], o);
            if (cg.host) copy_state(cg.host[mm], o);
          }
        }
      }
      nd.pin(zr);
      if constexpr (CG == 1) nd.pin(zd);
      nd.pin(zp);
      nd.keep(smap, t);
      const T beta = (T)s.beta, zs = (T)s.zshift;
#pragma unroll
      for (int j = 0; j < NL; ++j) {
        const T pv = cg_dir(zd[j], zr[j], zs, beta, zp[j]);
        buf[LD::nodal(Nodes<P>::node(t, j))] = (active && nd.c[j] >= 0) ? pv : T(0);
        if (active && t + j * TPE < N3 && nd.c[j] < 0 && (nd.c[j] & kEssOwnerBit)) dot += (double)pv * (double)pv;
      }
      elem_sync<P, THREADS>();
    }
    fwd_x<P, T, DIFF, THREADS>(buf, t);
    fwd_y<P, T, DIFF, THREADS>(buf, t);

    // xi_3 contraction, quadrature function, transposed xi_3: thread = line (a, b),
    // processed by symmetric slice pairs (c, q-1-c).
    {
      using BT = eo::Tab1<P, 0>;
      using GT = eo::Tab1<P, 1>;
      constexpr rules::GaussRule<Q> gr = rules::gauss<Q>();
      std::conditional_t<sizeof(T) == 8 || THIN, LineGeom, LineMetric> L;
      const int la = t % Q, lb = t / Q;
      L.init(sgeo + le * kGeoStride, sgq[la], sgq[lb]);
      const double wab = sgq[Q + la] * sgq[Q + lb];
      const double wm = alpha * wab;             // mass weight of the line
      const double ws = NU ? beta : beta * wab;  // diffusion weight (cw holds w)
      // the stage's input lines (split into even and odd parts), held in registers or,
      // with ZLDS, read from LDS again for every slice pair
      eo::Split<N, T> held[DIFF ? 3 : 1];
      auto read_line = [&](int f) {
        T z[N];
#pragma unroll
        for (int k = 0; k < N; ++k) z[k] = buf[f * LD::YF + k * LD::SP + t];
        return eo::split(z);
      };
      if constexpr (!C::ZLDS) {
#pragma unroll
        for (int f = 0; f < (DIFF ? 3 : 1); ++f) held[f] = read_line(f);
      }
      auto zline = [&](int f) {
        if constexpr (C::ZLDS) {
          asm volatile("" ::: "memory");  // a fresh LDS read, not a reuse of the last one
          return read_line(f);
        } else {
          return held[f];
        }
      };
      eo::Acc<N, T> A1, A2, A3;
      A1.zero();
      A2.zero();
      A3.zero();
      // v = alpha w |J| u and g = beta nu w |J| J^-1 J^-T grad_ref u at slice c
      auto qfun = [&](int c, T u, T dx, T dy, T dz, T &v, T &g1, T &g2, T &g3) {
        const double xc = gr.x[c], wc = gr.w[c];
        v = g1 = g2 = g3 = T(0);
        double det = 0.0;
        if constexpr (MASS || !NU) det = L.det(xc);
        if constexpr (MASS) v = (T)((wm * wc) * det) * u;
        if constexpr (DIFF) {
          const double s = NU ? cv[c] * ws : (ws * wc) * recip(det);
          if constexpr (sizeof(T) == 8) {
            double r1[3], r2[3], r3[3], f[3];
            L.adj(xc, r1, r2, r3);
#pragma unroll
            for (int r = 0; r < 3; ++r) f[r] = s * (r1[r] * dx + r2[r] * dy + r3[r] * dz);
            g1 = r1[0] * f[0] + r1[1] * f[1] + r1[2] * f[2];
            g2 = r2[0] * f[0] + r2[1] * f[1] + r2[2] * f[2];
            g3 = r3[0] * f[0] + r3[1] * f[1] + r3[2] * f[2];
          } else {
            float G[6];
            L.factors(xc, s, G);
            g1 = G[0] * dx + G[3] * dy + G[4] * dz;
            g2 = G[3] * dx + G[1] * dy + G[5] * dz;
            g3 = G[4] * dx + G[5] * dy + G[2] * dz;
          }
        }
        if constexpr (CG) {
          if constexpr (sizeof(T) == 8) {
            dot += v * u + g1 * dx + g2 * dy + g3 * dz;
          } else {
            if constexpr (MASS) dot = add_energy(dot, v, u);
            if constexpr (DIFF) dot = add_energy(dot, g1, dx, g2, dy, g3, dz);
          }
          asm volatile("" : "+v"(dot));  // summed here: postponed, its operands would stay live
        }
      };
#pragma unroll
      for (int c = 0; c < Q / 2; ++c) {
        T u0 = 0, u1 = 0, dx0 = 0, dx1 = 0, dy0 = 0, dy1 = 0, dz0 = 0, dz1 = 0;
        const eo::Split<N, T> sbb = zline(0);
        if constexpr (MASS) eo::out_pair<BT>(sbb, c, u0, u1);
        if constexpr (DIFF) {
          eo::out_pair<GT>(sbb, c, dz0, dz1);
          eo::out_pair<BT>(zline(1), c, dy0, dy1);
          eo::out_pair<BT>(zline(2), c, dx0, dx1);
        }
        T v0, g10, g20, g30, v1, g11, g21, g31;
        qfun(c, u0, dx0, dy0, dz0, v0, g10, g20, g30);
        qfun(Q - 1 - c, u1, dx1, dy1, dz1, v1, g11, g21, g31);
        if constexpr (MASS) A1.template add_pair<BT>(c, v0, v1);
        if constexpr (DIFF) {
          A1.template add_pair<GT>(c, g30, g31);
          A2.template add_pair<BT>(c, g20, g21);
          A3.template add_pair<BT>(c, g10, g11);
        }
      }
      if constexpr (Q % 2 == 1) {
        T u = 0, dx = 0, dy = 0, dz = 0;
        const eo::Split<N, T> sbb = zline(0);
        if constexpr (MASS) u = eo::out_mid<BT>(sbb);
        if constexpr (DIFF) {
          dz = eo::out_mid<GT>(sbb);
          dy = eo::out_mid<BT>(zline(1));
          dx = eo::out_mid<BT>(zline(2));
        }
        T v, g1, g2, g3;
        qfun(Q / 2, u, dx, dy, dz, v, g1, g2, g3);
        if constexpr (MASS) A1.template add_mid<BT>(v);
        if constexpr (DIFF) {
          A1.template add_mid<GT>(g3);
          A2.template add_mid<BT>(g2);
          A3.template add_mid<BT>(g1);
        }
      }
      T p1[N], p2[N], p3[N];
      A1.finish(p1);
      if constexpr (DIFF) {
        A2.finish(p2);
        A3.finish(p3);
      }
      // a thread's lines replace those it read: no barrier before the stores
#pragma unroll
      for (int k = 0; k < N; ++k) {
        buf[k * LD::SP + t] = p1[k];
        if constexpr (DIFF) {
          buf[LD::YF + k * LD::SP + t] = p2[k];
          buf[2 * LD::YF + k * LD::SP + t] = p3[k];
        }
      }
      elem_sync<P, THREADS>();
    }

    bwd_y<P, T, DIFF, THREADS>(buf, t);
    bwd_x<P, T, DIFF, THREADS>(buf, t);
    T *Ym = Y + (int64_t)m * estride, *ym = y + (int64_t)m * ndof;
    int te = t;
    if constexpr (C::REFORM) asm volatile("" : "+v"(te));
    emit_e<P, T, LD>(buf, te, active, smap, Ym, ym);
    if constexpr (CG) {
      // one sum per member, or per pair where a workgroup holds a member once at most
      // (cg_parts); the workgroup's pairs k < count hold the members (r0 + k) mod nbatch
      double *sh = reinterpret_cast<double *>(smem);
      if (nbatch == 1) {
        const double sum = block_sum_d<THREADS>(active ? dot : 0.0, sh);
        if (threadIdx.x == 0) part[blockIdx.x] = sum;
      } else {
        static_assert(E * LD::BUF * sizeof(T) >= THREADS * sizeof(double), "the threads' parts");
        __syncthreads();
        sh[threadIdx.x] = active ? dot : 0.0;
        __syncthreads();
        constexpr int NWF = THREADS / 64;  // full waves, each takes the next sum
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nsum = cg_sums(nbatch, E, count);
        for (int i = wave; wave < NWF && i < nsum; i += NWF) {
          const CgSum c = cg_sum(i, nbatch, E, blockIdx.x, e0, (int)r0);
          double sum = 0.0;
          for (int k = c.first; k < count; k += c.step)
            for (int j = lane; j < TPE; j += 64) sum += sh[k * TPE + j];
          sum = wave_total(sum);
          if (lane == 0) part[(int64_t)c.member * part_mstride + c.slot] = sum;
        }
      }
    }
  }
}

// The float32 apply of several members with one coefficient: a workgroup takes E elements and
// all their members in turn.  The six factors and the mass weight of the thread's points are
// formed in float64 once, rounded, and kept in 7 q registers, which the coefficients of the
// line's metric and w nu / |J| took; formed for each member they are a quarter of the vector
// instructions at p = 4: three members at 29^3 p = 2 30 -> 23.5 us, 29^3 p = 4 100 -> 81 us,
// 114^3 p = 1 617 -> 388 us (Helmholtz with nu; by pairs at the left).
// CG = 1: the first launch of a CG iteration as in apply_kernel, with a partial of p.Ap per
// workgroup and member (refined solves of three members: 30^3 p = 4 43.8 -> 36.8 ms, 54^3 p = 1
// 9.8 -> 5.7 ms).
template <int P, int OP, bool NU, int CG>
__global__ void __launch_bounds__((ApplyCfg<P, float, CG>::THREADS), (ApplyCfg<P, float, CG>::OCC))
apply_members_kernel(const int32_t *__restrict__ map, const double *__restrict__ geo, const double *__restrict__ cw,
                     double alpha, double beta, int64_t nelem, int nbatch, int64_t ndof,
                     const float *__restrict__ x, float *__restrict__ Y, int64_t estride,
                     const int32_t *__restrict__ pos, int compact, float *__restrict__ y, double *__restrict__ part,
                     int64_t part_mstride, std::conditional_t<CG != 0, CgIn, NoCg> cg) {
  using D = Dims<P>;
  using C = ApplyCfg<P, float, CG>;
  using LD = Lds<P, true>;
  using T = float;
  constexpr int N = D::N, Q = D::Q, Q2 = D::Q2, Q3 = D::Q3, N3 = D::N3, TPE = D::TPE, E = C::E, THREADS = C::THREADS;
  constexpr int NL = Nodes<P>::NL;
  constexpr bool MASS = OP == 2, POS = evec_dof_ordered(P);
  static_assert(OP == 1 || OP == 2, "diffusion or Helmholtz");
  constexpr rules::GaussRule<Q> gr = rules::gauss<Q>();
  using BT = eo::Tab1<P, 0>;
  using GT = eo::Tab1<P, 1>;
  __shared__ __align__(16) T smem[E * LD::BUF];
  __shared__ __align__(16) double sgeo[E * kGeoStride];
  __shared__ int32_t smap_all[E * N3];
  const int le = threadIdx.x / TPE;
  const int t = threadIdx.x - le * TPE;
  const int64_t e0 = (int64_t)xcd_block() * E;
  const bool active = e0 + le < nelem;
  const uint32_t rel = active ? le : 0;
  T *buf = smem + le * LD::BUF;
  int32_t *smap = smap_all + le * N3;
  const ElemTab z = elem_tab<P>(map, pos, compact, e0);
  Nodes<P> nd;
  nd.load_map(z, t, rel);
  nd.load_rank(z, t);
  constexpr int NG = (kGeoStride + TPE - 1) / TPE;
  double gv[NG];
#pragma unroll
  for (int k = 0; k < NG; ++k) {
    const int i = t + k * TPE < kGeoStride ? t + k * TPE : kGeoStride - 1;
    gv[k] = ld<double>(geo + e0 * kGeoStride, (rel * kGeoStride + i) * 8u);
  }
  double cv[Q];  // w nu / |J| at the points of the thread's line
  if constexpr (NU) {
#pragma unroll
    for (int c = 0; c < Q; ++c) cv[c] = ld<double>(cw + e0 * Q3, (rel * Q3 + t + c * Q2) * 8u);
  }
  // CG: the members' states, member m's by thread m (the update's partials summed first)
  constexpr int NW = CG ? THREADS / 64 : 1, MM = CG ? kCgMembersMax : 1;
  __shared__ double sums[MM][4][NW], sdir[MM][2], sdot[CG ? (THREADS + 63) / 64 + 1 : 1];
  PcgScalars st;
  if constexpr (CG) copy_state(st, cg.sc[(int)threadIdx.x < nbatch ? (int)threadIdx.x : nbatch - 1]);
  T v[NL];
  if constexpr (!CG) nd.load_values(x, v);
  nd.template load_dest<POS>(z, rel);
  if constexpr (CG) {
    if (!cg.ready) {
      for (int i = 0; i < nbatch; i += 2) {  // two members' loads together
        const int i1 = i + 1 < nbatch ? i + 1 : i;
        const double *pa = cg.upart + (int64_t)i * 4 * cg.unblk, *pb = cg.upart + (int64_t)i1 * 4 * cg.unblk;
        PartLoads<NW, 2> qa, qb;
        qa.load(pa, cg.unblk);
        qb.load(pb, cg.unblk);
        qa.parts(sums[i], cg.unblk);
        qb.parts(sums[i1], cg.unblk);
        if (cg.nullspace) {
          qa.load(pa + 2 * (int64_t)cg.unblk, cg.unblk);
          qb.load(pb + 2 * (int64_t)cg.unblk, cg.unblk);
          qa.parts(*reinterpret_cast<double(*)[4][NW]>(&sums[i][2]), cg.unblk);
          qb.parts(*reinterpret_cast<double(*)[4][NW]>(&sums[i1][2]), cg.unblk);
        }
      }
      __syncthreads();
    }
    if ((int)threadIdx.x < nbatch) {
      const int m = threadIdx.x;
      if (!cg.ready) cg_next_from<NW>(st, sums[m], cg.nullspace, ndof);
      sdir[m][0] = st.beta;
      sdir[m][1] = st.zshift;
      if (blockIdx.x == 0) {
        copy_state(cg.sc_next[m], st);
        if (cg.host) copy_state(cg.host[m], st);
      }
    }
    __syncthreads();
  }
  double dot = 0.0;
  // the member's direction (pcg.h) into the nodal vector
  auto put_dir = [&](int m) {
    if constexpr (CG) {
      T zr[NL], zd[NL], zp[NL];
      nd.load_values((const T *)cg.r + (int64_t)m * ndof, zr);
      nd.load_values((const T *)cg.dinv + (int64_t)m * cg.dinv_mstride, zd);
      nd.load_values((const T *)cg.p + (int64_t)m * ndof, zp);
      nd.pin(zr);
      nd.pin(zd);
      nd.pin(zp);
      const T bt = (T)sdir[m][0], zs = (T)sdir[m][1];
      dot = 0.0;
#pragma unroll
      for (int k = 0; k < NL; ++k) {
        const T pv = cg_dir(zd[k], zr[k], zs, bt, zp[k]);
        buf[LD::nodal(Nodes<P>::node(t, k))] = (active && nd.c[k] >= 0) ? pv : T(0);
        if (active && t + k * TPE < N3 && nd.c[k] < 0 && (nd.c[k] & kEssOwnerBit)) dot += (double)pv * (double)pv;
      }
    }
  };
#pragma unroll
  for (int k = 0; k < NG; ++k)
    sgeo[le * kGeoStride + (t + k * TPE < kGeoStride ? t + k * TPE : kGeoStride - 1)] = gv[k];
  if constexpr (!CG) nd.pin(v);
  nd.keep(smap, t);
  if constexpr (CG) {
    put_dir(0);
  } else {
#pragma unroll
    for (int k = 0; k < NL; ++k) buf[LD::nodal(Nodes<P>::node(t, k))] = (active && nd.c[k] >= 0) ? v[k] : T(0);
  }
  elem_sync<P, THREADS>();
  T G[Q][6], wd[Q];
  {
    LineMetric L;
    const int la = t % Q, lb = t / Q;
    L.init(sgeo + le * kGeoStride, kGaussRule<Q>.x[la], kGaussRule<Q>.x[lb]);
    const double wab = kGaussRule<Q>.w[la] * kGaussRule<Q>.w[lb];
    const double wm = alpha * wab, ws = NU ? beta : beta * wab;
#pragma unroll
    for (int c = 0; c < Q; ++c) {
      double det = 0.0;
      if constexpr (MASS || !NU) det = L.det(gr.x[c]);
      wd[c] = MASS ? (T)((wm * gr.w[c]) * det) : T(0);
      L.factors(gr.x[c], NU ? cv[c] * ws : (ws * gr.w[c]) * recip(det), G[c]);
    }
  }
  for (int m = 0; m < nbatch; ++m) {
    if (!CG && m + 1 < nbatch) nd.load_values(x + (int64_t)(m + 1) * ndof, v);
    fwd_x<P, T, true, THREADS>(buf, t);
    fwd_y<P, T, true, THREADS>(buf, t);
    {
      auto line = [&](int f) {
        T u[N];
#pragma unroll
        for (int k = 0; k < N; ++k) u[k] = buf[f * LD::YF + k * LD::SP + t];
        return eo::split(u);
      };
      // held in registers, or from p = 5 on read again for every slice pair
      constexpr bool AGAIN = P >= 5;
      const eo::Split<N, T> held[3] = {line(0), line(1), line(2)};
      auto zline = [&](int f) {
        if constexpr (AGAIN) {
          asm volatile("" ::: "memory");  // a fresh LDS read, not a reuse of the last one
          return line(f);
        } else {
          return held[f];
        }
      };
      eo::Acc<N, T> A1, A2, A3;
      A1.zero();
      A2.zero();
      A3.zero();
      auto flux = [&](int c, T dx, T dy, T dz, T &g1, T &g2, T &g3) {
        g1 = G[c][0] * dx + G[c][3] * dy + G[c][4] * dz;
        g2 = G[c][3] * dx + G[c][1] * dy + G[c][5] * dz;
        g3 = G[c][4] * dx + G[c][5] * dy + G[c][2] * dz;
      };
#pragma unroll
      for (int c = 0; c < Q / 2; ++c) {
        T u0 = 0, u1 = 0, dx0, dx1, dy0, dy1, dz0, dz1, a1, a2, a3, b1, b2, b3;
        // (CG: each energy is summed at once; postponed, its operands would stay live)
        if constexpr (MASS) {
          eo::out_pair<BT>(zline(0), c, u0, u1);
          const T v0 = wd[c] * u0, v1 = wd[Q - 1 - c] * u1;
          if constexpr (CG) {
            dot = add_energy(add_energy(dot, v0, u0), v1, u1);
            asm volatile("" : "+v"(dot));
          }
          A1.template add_pair<BT>(c, v0, v1);
        }
        eo::out_pair<GT>(zline(0), c, dz0, dz1);
        eo::out_pair<BT>(zline(1), c, dy0, dy1);
        eo::out_pair<BT>(zline(2), c, dx0, dx1);
        flux(c, dx0, dy0, dz0, a1, a2, a3);
        if constexpr (CG) {
          dot = add_energy(dot, a1, dx0, a2, dy0, a3, dz0);
          asm volatile("" : "+v"(dot));
        }
        flux(Q - 1 - c, dx1, dy1, dz1, b1, b2, b3);
        if constexpr (CG) {
          dot = add_energy(dot, b1, dx1, b2, dy1, b3, dz1);
          asm volatile("" : "+v"(dot));
        }
        A1.template add_pair<GT>(c, a3, b3);
        A2.template add_pair<BT>(c, a2, b2);
        A3.template add_pair<BT>(c, a1, b1);
      }
      if constexpr (Q % 2 == 1) {
        T g1, g2, g3, u = 0;
        if constexpr (MASS) {
          u = eo::out_mid<BT>(zline(0));
          A1.template add_mid<BT>(wd[Q / 2] * u);
        }
        const T dx = eo::out_mid<BT>(zline(2)), dy = eo::out_mid<BT>(zline(1)), dz = eo::out_mid<GT>(zline(0));
        flux(Q / 2, dx, dy, dz, g1, g2, g3);
        if constexpr (CG) dot = add_energy(add_energy(dot, wd[Q / 2] * u, u), g1, dx, g2, dy, g3, dz);
        A1.template add_mid<GT>(g3);
        A2.template add_mid<BT>(g2);
        A3.template add_mid<BT>(g1);
      }
      T p1[N], p2[N], p3[N];
      A1.finish(p1);
      A2.finish(p2);
      A3.finish(p3);
      // a thread's lines replace those it read: no barrier before the stores
#pragma unroll
      for (int k = 0; k < N; ++k) {
        buf[k * LD::SP + t] = p1[k];
        buf[LD::YF + k * LD::SP + t] = p2[k];
        buf[2 * LD::YF + k * LD::SP + t] = p3[k];
      }
      elem_sync<P, THREADS>();
    }
    bwd_y<P, T, true, THREADS>(buf, t);
    bwd_x<P, T, true, THREADS>(buf, t);
    int te = t;
    if constexpr (P >= 5) asm volatile("" : "+v"(te));  // addresses formed anew (REFORM of ApplyCfg)
    emit_e<P, T, LD>(buf, te, active, smap, Y + (int64_t)m * estride, y + (int64_t)m * ndof);
    if constexpr (CG) {
      const double sum = block_sum_d<THREADS>(active ? dot : 0.0, sdot);
      if (threadIdx.x == 0) part[(int64_t)m * part_mstride + blockIdx.x] = sum;
    }
    if (m + 1 < nbatch) {
      elem_sync<P, THREADS>();  // the nodal vector has been read
      if constexpr (CG) {
        put_dir(m + 1);
      } else {
#pragma unroll
        for (int k = 0; k < NL; ++k) buf[LD::nodal(Nodes<P>::node(t, k))] = (active && nd.c[k] >= 0) ? v[k] : T(0);
      }
      elem_sync<P, THREADS>();
    }
  }
}

template <int P, typename T, int CG>
hipError_t launch_apply_pt(const ApplyArgs &a, const CgIn &g, hipStream_t s) {
  if (a.nelem <= 0 || a.nbatch <= 0) return hipSuccess;
  if ((a.pos != nullptr) != evec_dof_ordered(P)) return hipErrorInvalidValue;
  if (CG && !a.part) return hipErrorInvalidValue;
  using C = ApplyCfg<P, T, CG>;
  dim3 grid((unsigned)((a.nelem * a.nbatch + C::E - 1) / C::E));
  dim3 block(C::THREADS);
  // (up to p = 6 and, in CG iterations, 4, where the members kernel's registers fit four waves per SIMD:
  // f32_by_members)
  if constexpr (sizeof(T) == 4 && CG <= 1 && P <= (CG ? kCgMembersMaxP : kMembersMaxP)) {
    if (f32_by_members(P, a.op, a.nbatch, !a.cw || a.cw_mstride == 0, a.thin != 0, CG != 0,
                       (a.nelem + C::E - 1) / C::E, C::THREADS)) {
      std::conditional_t<CG != 0, CgIn, NoCg> cg;
      if constexpr (CG != 0) cg = g;
      dim3 eg((unsigned)((a.nelem + C::E - 1) / C::E));
#define SFEM_MEMBERS(OP, NU)                                                                             \
  hipLaunchKernelGGL((apply_members_kernel<P, OP, NU, CG>), eg, block, 0, s, a.map, a.geo, a.cw, a.alpha,    \
                     a.beta, a.nelem, a.nbatch, a.ndof, (const float *)a.x, (float *)a.evec, a.estride,  \
                     a.pos, a.compact, (float *)a.y, a.part, a.part_mstride, cg)
      if (a.op == SFEM_DIFFUSION && a.cw) SFEM_MEMBERS(1, true);
      else if (a.op == SFEM_DIFFUSION) SFEM_MEMBERS(1, false);
      else if (a.cw) SFEM_MEMBERS(2, true);
      else SFEM_MEMBERS(2, false);
#undef SFEM_MEMBERS
      return hipGetLastError();
    }
  }
  std::conditional_t<CG != 0, CgIn, NoCg> cg;
  if constexpr (CG != 0) cg = g;
#define SFEM_APPLY_GEO(OP, NU, THIN)                                                                    \
  hipLaunchKernelGGL((apply_kernel<P, T, OP, NU, CG, THIN>), grid, block, 0, s, a.map, a.geo, a.cw,     \
                     a.cw_mstride, a.alpha, a.beta, a.nelem, a.nbatch, a.ndof, (const T *)a.x,          \
                     (T *)a.evec, a.estride, a.pos, a.compact, (T *)a.y, a.part, a.part_mstride, cg)
#define SFEM_APPLY(OP, NU)                                            \
  do {                                                                \
    if constexpr (sizeof(T) == 4 && OP != SFEM_MASS) {                \
      if (a.thin) SFEM_APPLY_GEO(OP, NU, true);                       \
      else SFEM_APPLY_GEO(OP, NU, false);                             \
    } else {                                                          \
      SFEM_APPLY_GEO(OP, NU, false);                                  \
    }                                                                 \
  } while (0)
  if (a.op == SFEM_MASS) SFEM_APPLY(0, false);
  else if (a.op == SFEM_DIFFUSION && a.cw) SFEM_APPLY(1, true);
  else if (a.op == SFEM_DIFFUSION) SFEM_APPLY(1, false);
  else if (a.cw) SFEM_APPLY(2, true);
  else SFEM_APPLY(2, false);
#undef SFEM_APPLY
#undef SFEM_APPLY_GEO
  return hipGetLastError();
}

// Elements per workgroup of the CG iteration's apply kernel for order P and precision T.
template <int P, typename T>
int apply_group_elems_pt() {
  return ApplyCfg<P, T, 1>::E;
}

#define SFEM_DISPATCH_P(p, CALL) \
  switch (p) {                   \
    case 1: return CALL(1);      \
    case 2: return CALL(2);      \
    case 3: return CALL(3);      \
    case 4: return CALL(4);      \
    case 5: return CALL(5);      \
    case 6: return CALL(6);      \
    case 7: return CALL(7);      \
    case 8: return CALL(8);      \
    default: return hipErrorInvalidValue; \
  }

}  // namespace sfem
