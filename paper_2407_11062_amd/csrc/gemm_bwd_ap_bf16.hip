// dX and dW in one launch: Block-AP, bf16 weights.
#include "gemm_bwd.h"

namespace eqat {

void launch_bwd_ap_bf16(int bits, int dx, const GemmQArgs &q, const MidArgs &m, const GemmDwArgs &d, int n_dx, int n_dw, hipStream_t st)
{
    launch_bwd_types<bf16_t, true>(bits, dx, q, m, d, n_dx, n_dw, st);
}

}  // namespace eqat
