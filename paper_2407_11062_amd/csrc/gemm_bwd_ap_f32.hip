// dX and dW in one launch: Block-AP, fp32 weights.
#include "gemm_bwd.h"

namespace eqat {

void launch_bwd_ap_f32(int bits, int dx, const GemmQArgs &q, const MidArgs &m, const GemmDwArgs &d, int n_dx, int n_dw, hipStream_t st)
{
    launch_bwd_types<float, true>(bits, dx, q, m, d, n_dx, n_dw, st);
}

}  // namespace eqat
