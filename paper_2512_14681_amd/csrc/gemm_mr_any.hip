// Many-row GEMM instantiations for operands off a 16-byte boundary: 64-, 96-
// and 128-row chunks.
#include "gemm_mr.h"

namespace jf {

hipError_t launch_mr_any(const void* X, size_t xplane, const void* Wp, const MrPlan& m, const Epi& ep, hipStream_t st) {
  switch (16 * m.RT + m.CT) {
    case 16 * 4 + 2: return launch_mr_cfg<1, 1, 4, 2, 150, true>(X, xplane, Wp, m, ep, st);
    case 16 * 4 + 4: return launch_mr_cfg<1, 2, 4, 2, 150, true>(X, xplane, Wp, m, ep, st);
    case 16 * 4 + 6: return launch_mr_cfg<1, 3, 4, 2, 150, true>(X, xplane, Wp, m, ep, st);
    case 16 * 4 + 8: return launch_mr_cfg<1, 4, 4, 2, 150, true>(X, xplane, Wp, m, ep, st);
    case 16 * 4 + 10: return launch_mr_cfg<1, 5, 4, 2, 150, true>(X, xplane, Wp, m, ep, st);
    case 16 * 4 + 12: return launch_mr_cfg<1, 6, 4, 2, 150, true>(X, xplane, Wp, m, ep, st);
    case 16 * 6 + 4: return launch_mr_cfg<3, 1, 2, 4, 150, true>(X, xplane, Wp, m, ep, st);
    case 16 * 6 + 8: return launch_mr_cfg<3, 2, 2, 4, 150, true>(X, xplane, Wp, m, ep, st);
    case 16 * 6 + 12: return launch_mr_cfg<3, 3, 2, 4, 150, true>(X, xplane, Wp, m, ep, st);
    case 16 * 8 + 2: return launch_mr_cfg<2, 1, 4, 2, 150, true>(X, xplane, Wp, m, ep, st);
    case 16 * 8 + 4: return launch_mr_cfg<2, 2, 4, 2, 150, true>(X, xplane, Wp, m, ep, st);
    case 16 * 8 + 6: return launch_mr_cfg<2, 3, 4, 2, 150, true>(X, xplane, Wp, m, ep, st);
    case 16 * 8 + 8: return launch_mr_cfg<2, 4, 4, 2, 150, true>(X, xplane, Wp, m, ep, st);
    case 16 * 8 + 10: return launch_mr_cfg<2, 5, 4, 2, 150, true>(X, xplane, Wp, m, ep, st);
    case 16 * 8 + 12: return launch_mr_cfg<2, 6, 4, 2, 150, true>(X, xplane, Wp, m, ep, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace jf
