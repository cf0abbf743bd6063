#include "k_gemm_regs.h"

namespace ax {

void launch_regs_slices(const GemmArgs& g, int shape, hipStream_t s) {
    if (g.a_lo_off) launch_regs_shape<EPI_RESIDUAL, true, true>(g, shape, s);
    else launch_regs_shape<EPI_RESIDUAL, false, true>(g, shape, s);
}

}  // namespace ax
