// Instantiations of the CG element kernel (pcg.h) with the preconditioned residual given, in
// double for p = 1..8, q = p + 2.
#include "apply_impl.h"

namespace sfem {

hipError_t launch_apply_cgz(const ApplyArgs &a, const CgIn &g, hipStream_t s) {
  if (a.nbatch != 1) return hipErrorInvalidValue;
#define SFEM_CALL(P) launch_apply_pt<P, double, 2>(a, g, s)
  SFEM_DISPATCH_P(a.p, SFEM_CALL)
#undef SFEM_CALL
}

}  // namespace sfem
