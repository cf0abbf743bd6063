#include "k_gemm_regs.h"

namespace ax {

void launch_regs_qkv(const GemmArgs& g, int shape, hipStream_t s) {
    if (g.a_lo_off) launch_regs_shape<EPI_QKV, true, false>(g, shape, s);
    else launch_regs_shape<EPI_QKV, false, false>(g, shape, s);
}

}  // namespace ax
