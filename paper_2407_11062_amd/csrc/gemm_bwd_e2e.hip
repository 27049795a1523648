// dX and dW in one launch: E2E-QP.
#include "gemm_bwd.h"

namespace eqat {

void launch_bwd_e2e(int bits, int dx, const GemmQArgs &q, const MidArgs &m, const GemmDwArgs &d, int n_dx, int n_dw, hipStream_t st)
{
    launch_bwd_types<bf16_t, false>(bits, dx, q, m, d, n_dx, n_dw, st);
}

}  // namespace eqat
