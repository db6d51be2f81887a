// Instantiations of the CG element kernel (pcg.h) in double for p = 1..8, q = p + 2.
#include "apply_impl.h"

namespace sfem {

hipError_t launch_apply_cg64(const ApplyArgs &a, const CgIn &g, hipStream_t s) {
#define SFEM_CALL(P) launch_apply_pt<P, double, 1>(a, g, s)
  SFEM_DISPATCH_P(a.p, SFEM_CALL)
#undef SFEM_CALL
}

}  // namespace sfem
