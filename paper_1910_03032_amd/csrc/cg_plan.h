// Sizes and rules of the applies and of the CG iteration's two launches that need no GPU: where
// members are taken in turn, the places of the partials of p.Ap, when a long list of them is folded
// first, and when the states are formed apart.
#pragma once

#include <stdint.h>

#include "eo.h"
#include "sfem.h"

namespace sfem {

// The float32 kernels that take an element's members in turn (apply_impl.h): the orders whose
// factors fit the registers, members with one coefficient, elements whose factors the metric gives
// (thin: geom.h), and enough waves without the members to fill the chip; in a CG iteration at most
// as many members as the kernel keeps states of.  groups: workgroups of the elements alone, of
// threads threads each.  Times by pairs over times in turn, of two, three and eight members: applies
// of 1250 waves (p = 4) 0.97, 0.90, 0.87, of 1600 to 1750 (p = 2, 3, 4) 1.02 - 1.05, 1.00 - 1.09, 1.03 -
// 1.10, of 1100 and 880 (p = 3) 0.98, 0.95, 0.94 and 0.94, 0.95, 0.85, and of 1100 to 1500 (p = 1, where
// a workgroup is one wave) 1.00 - 1.03, 1.03 - 1.05, 1.03; CG iterations of 1600 to 2000 waves (p = 1 to 4)
// 1.05 - 1.21, 0.94 - 1.17, 0.93 - 1.32, of 1100 to 1250 0.98 - 1.13, 0.89 - 1.04, 0.80 - 0.99.
// At p = 5 and 6, where an apply reads its lines again to fit the registers, from twice as many: 2200
// (p = 5, 6) 0.98 and 0.97, 0.97 and 0.95, 0.97 and 0.98, 3300 1.02 and 1.01, 1.00 and 1.00, 1.07 and 1.08,
// 4100 to 4700 1.03 - 1.05, 1.04 - 1.08, 1.11 - 1.16; with their factors stored, which three members read
// from cache, 18^3 p = 5 (4700 waves) had taken 44.7 us, 47.1 now in turn and 49.0 by pairs, 23^3 94.3,
// 82.0 and 91.2.  At p = 7 the gain was 1.01 - 1.03 from 6500 waves, in CG iterations 1.00 - 1.15.
constexpr int kMembersMaxP = 6, kCgMembersMaxP = 4, kCgMembersMax = 8, kMembersMinWaves = 1600;
inline bool f32_by_members(int p, int op, int nb, bool one_coef, bool thin, bool cg, int64_t groups, int threads) {
  return p <= (cg ? kCgMembersMaxP : kMembersMaxP) && nb > 1 && op != SFEM_MASS && one_coef && !thin &&
         groups * ((threads + 63) / 64) >= (p <= 4 ? 1 : 2) * kMembersMinWaves && (!cg || nb <= kCgMembersMax);
}

// Workgroups of the update, and so partials of its sums, at most: every kernel that sums them in one
// group of loads (PartLoads) is checked against it.
constexpr int kCgUpdateMax = 512;

// Partials of p.Ap per member that the element kernel leaves, E elements per workgroup: one per
// workgroup, and where it takes (element, member) pairs of more members than it has pairs, one
// per element (every other workgroup's partial would be 0).
SFEM_HD int64_t cg_parts(int64_t nelem, int nb, int E, bool by_members) {
  if (by_members) return (nelem + E - 1) / E;
  return nb > E ? nelem : (nelem * nb + E - 1) / E;
}

// By pairs a workgroup whose first pair is (e0, r0), with count <= E pairs, leaves cg_sums of them:
// the i-th is the sum of its pairs first, first + step, .. of one member, at slot of that member.
struct CgSum {
  int first, step, member;
  int64_t slot;
};
SFEM_HD int cg_sums(int nb, int E, int count) { return nb > E ? count : nb; }
SFEM_HD CgSum cg_sum(int i, int nb, int E, int64_t block, int64_t e0, int r0) {
  if (nb > E) return CgSum{i, E, (r0 + i) % nb, e0 + (r0 + i) / nb};
  return CgSum{(i - r0 + nb) % nb, nb, i, block};
}

// More than kCgFoldMin partials of a member are summed to cg_fold_nblk(count) before the update, all
// of whose workgroups read them (0: no fold).  An iteration with and without, float64: 9400 partials
// (64^3 p = 1) 70 and 71 us, 3.6e4 233 and 233, 7.5e4 (eight members) 531 and 540, 2.1e5 (180^3 p = 1)
// 1351 and 1401.
constexpr int64_t kCgFoldMin = 32768;
constexpr int kCgFoldLen = 1024, kCgFoldMax = 256;
SFEM_HD int cg_fold_nblk(int64_t count) {
  if (count <= kCgFoldMin) return 0;
  const int64_t b = (count + kCgFoldLen - 1) / kCgFoldLen;
  return (int)(b < kCgFoldMax ? b : kCgFoldMax);
}

// Whether a launch of its own forms the states of the next iteration, which otherwise every
// workgroup of the element kernel forms for its members (up to E of them by pairs, all of them in
// turn; the first workgroup for the rest too).  That launch takes 1 to 2 us; the sums at the head of
// a workgroup cost more where many workgroups follow each other on a CU, or one has many members to
// go through.  An iteration with the launch and without, float64: one member 36^3 p = 1 22.5 and
// 22.0 us, 28^3 p = 3 42.6 and 42.7, 48^3 p = 4 315 and 325, 100^3 p = 1 228 and 254; three members
// 20^3 p = 1 19.8 and 19.1, 20^3 p = 2 27.8 and 29.1, 64^3 p = 1 196 and 251; eight 6^3 p = 1 15.9 and
// 15.7, 4^3 p = 2 15.6 and 16.8, 64^3 p = 1 530 and 980; 32 members 40^3 p = 1 621 and 1950.
constexpr int64_t kCgStatesApart = 2600;
constexpr int kCgStatesApartNb = 8;
SFEM_HD bool cg_states_apart(int64_t nelem, int nb, int E, bool by_members) {
  const int64_t groups = by_members ? (nelem + E - 1) / E : (nelem * nb + E - 1) / E;
  const int here = by_members || nb < E ? nb : E;
  return nb >= kCgStatesApartNb || groups * here >= kCgStatesApart;
}

}  // namespace sfem
