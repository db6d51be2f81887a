// Host check of the CG iteration's partials: every (element, member) pair of a launch enters exactly
// one of the sums that its workgroup leaves, every slot of every member is written exactly once, and
// no list that the update reads is longer than its bound.
#include <cstdio>
#include <vector>

#include "cg_plan.h"

using namespace sfem;

// Where float32 members are taken in turn: elements per workgroup, threads and sizes on both sides of
// the measured crossover of the applies (E) and of the CG iterations (E of 4 waves each).
static void check_members() {
  auto rule = [](int p, bool cg, int E, int n) {
    return f32_by_members(p, SFEM_HELMHOLTZ, 3, true, false, cg, (n * n * n + E - 1) / E, E * (p + 2) * (p + 2));
  };
  const bool ok = !rule(1, false, 7, 18) && rule(1, false, 7, 26) && !rule(2, false, 16, 16) && rule(2, false, 16, 19) &&
                  !rule(3, false, 5, 14) && rule(3, false, 5, 16) && !rule(4, false, 7, 13) && rule(4, false, 7, 15) &&
                  !rule(5, false, 5, 15) && rule(5, false, 5, 18) && !rule(6, false, 4, 13) && rule(6, false, 4, 16) &&
                  !rule(7, false, 3, 20) && !rule(5, true, 5, 18) && !rule(3, true, 10, 14) && rule(3, true, 10, 17) && !rule(4, true, 7, 13) && rule(4, true, 7, 19);
  if (!ok) std::printf("FAIL members in turn\n");
  if (f32_by_members(2, SFEM_MASS, 3, true, false, false, 1 << 20, 256) ||
      f32_by_members(2, SFEM_HELMHOLTZ, 3, false, false, false, 1 << 20, 256) ||
      f32_by_members(2, SFEM_HELMHOLTZ, 3, true, true, false, 1 << 20, 256) ||
      f32_by_members(2, SFEM_HELMHOLTZ, 9, true, false, true, 1 << 20, 256) ||
      f32_by_members(8, SFEM_HELMHOLTZ, 3, true, false, false, 1 << 20, 200))
    std::printf("FAIL members that go by pairs\n");
}

int main() {
  check_members();
  for (int E : {2, 3, 4, 5, 7, 10, 16, 28})
    for (int64_t nelem : {1, 2, 3, 7, 27, 64, 125, 1000})
      for (int nb : {1, 2, 3, 4, 5, 8, 16, 27, 28, 29, 33, 64}) {
        const int64_t parts = cg_parts(nelem, nb, E, false), npair = nelem * nb;
        std::vector<int> written((size_t)(parts * nb), 0), used((size_t)npair, 0);
        if (nb > 1)
          for (int64_t blk = 0; blk * E < npair; ++blk) {
            const int64_t v = blk * E, e0 = v / nb;
            const int r0 = (int)(v - e0 * nb), count = (int)(npair - v < E ? npair - v : E);
            for (int i = 0; i < cg_sums(nb, E, count); ++i) {
              const CgSum c = cg_sum(i, nb, E, blk, e0, r0);
              if (c.member < 0 || c.member >= nb || c.slot < 0 || c.slot >= parts) {
                std::printf("FAIL range E=%d nelem=%d nb=%d\n", E, (int)nelem, nb);
                return 0;
              }
              ++written[(size_t)(c.member * parts + c.slot)];
              for (int k = c.first; k < count; k += c.step) {
                if ((r0 + k) % nb != c.member) std::printf("FAIL member E=%d nelem=%d nb=%d\n", E, (int)nelem, nb);
                ++used[(size_t)(v + k)];
              }
            }
          }
        else if (parts != (nelem + E - 1) / E)
          std::printf("FAIL parts E=%d nelem=%d\n", E, (int)nelem);
        for (int w : written)
          if (nb > 1 && w != 1) std::printf("FAIL written %d times E=%d nelem=%d nb=%d\n", w, E, (int)nelem, nb);
        for (int u : used)
          if (nb > 1 && u != 1) std::printf("FAIL used %d times E=%d nelem=%d nb=%d\n", u, E, (int)nelem, nb);
        if (parts > nelem) std::printf("FAIL %d parts of %d elements\n", (int)parts, (int)nelem);
      }
  for (int64_t count = 1; count < 4000000; count = count * 5 / 4 + 1) {
    const int f = cg_fold_nblk(count);
    if ((f ? f : count) > kCgFoldMin || f > kCgFoldMax) std::printf("FAIL fold of %d\n", (int)count);
    if (f) {  // the stretches of cg_fold_kernel
      const int64_t len = (count + f - 1) / f;
      if (len * f < count) std::printf("FAIL stretches of %d\n", (int)count);
    }
  }
  return 0;
}
