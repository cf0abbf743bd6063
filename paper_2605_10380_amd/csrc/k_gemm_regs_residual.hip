#include "k_gemm_regs.h"

namespace ax {

void launch_regs_residual(const GemmArgs& g, int shape, hipStream_t s) {
    if (g.a_lo_off) launch_regs_shape<EPI_RESIDUAL, true, false>(g, shape, s);
    else launch_regs_shape<EPI_RESIDUAL, false, false>(g, shape, s);
}

}  // namespace ax
