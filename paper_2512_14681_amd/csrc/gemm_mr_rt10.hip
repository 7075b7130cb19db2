// Many-row GEMM instantiations: 160-row chunks (2 x 4 waves of 5 row tiles).
#include "gemm_mr.h"

namespace jf {

hipError_t launch_mr_rt10(const void* X, size_t xplane, const void* Wp, const MrPlan& m, const Epi& ep, hipStream_t st) {
  switch (m.CT) {
    case 4: return launch_mr_cfg<5, 1, 2, 4, 156>(X, xplane, Wp, m, ep, st);
    case 8: return launch_mr_cfg<5, 2, 2, 4, 156>(X, xplane, Wp, m, ep, st);
    case 12: return launch_mr_cfg<5, 3, 2, 4, 156>(X, xplane, Wp, m, ep, st);
    case 16: return launch_mr_cfg<5, 4, 2, 4, 156>(X, xplane, Wp, m, ep, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace jf
