// Many-row GEMM instantiations: 32-row chunks (2 x 4 waves of 1 row tiles).
#include "gemm_mr.h"

namespace jf {

hipError_t launch_mr_rt2(const void* X, size_t xplane, const void* Wp, const MrPlan& m, const Epi& ep, hipStream_t st) {
  switch (m.CT) {
    case 4: return launch_mr_cfg<1, 1, 2, 4, 150>(X, xplane, Wp, m, ep, st);
    case 8: return launch_mr_cfg<1, 2, 2, 4, 150>(X, xplane, Wp, m, ep, st);
    case 12: return launch_mr_cfg<1, 3, 2, 4, 150>(X, xplane, Wp, m, ep, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace jf
