// Many-row GEMM instantiations: 192-row chunks (4 x 2 waves of 3 row tiles).
#include "gemm_mr.h"

namespace jf {

hipError_t launch_mr_rt12(const void* X, size_t xplane, const void* Wp, const MrPlan& m, const Epi& ep, hipStream_t st) {
  switch (m.CT) {
    case 2: return launch_mr_cfg<3, 1, 4, 2, 156>(X, xplane, Wp, m, ep, st);
    case 4: return launch_mr_cfg<3, 2, 4, 2, 156>(X, xplane, Wp, m, ep, st);
    case 6: return launch_mr_cfg<3, 3, 4, 2, 156>(X, xplane, Wp, m, ep, st);
    case 8: return launch_mr_cfg<3, 4, 4, 2, 156>(X, xplane, Wp, m, ep, st);
    case 10: return launch_mr_cfg<3, 5, 4, 2, 156>(X, xplane, Wp, m, ep, st);
    case 12: return launch_mr_cfg<3, 6, 4, 2, 156>(X, xplane, Wp, m, ep, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace jf
