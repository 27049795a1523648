// dX and dW of one backward in one launch: workgroups of eight waves, one per compute unit, first those of dX, then those of dW.
//
// Alone, each of the two ends with a last round that leaves compute units idle (320 tiles of dX and 400 of dW, 13B at 4096 tokens: 1.25 and 1.56
// rounds; 192 workgroups of dX and 256 tiles, 515 tokens), starts with a chip that waits for its first operands and ends with one that stores.  The two
// need nothing of each other; in one launch the tiles of dW start as those of dX end.  Both are the code that their own launches run (the
// register budget, 256 for either, and the LDS, one workgroup per compute unit, are the same).  When it is taken and what it gains: bwd_together().
#pragma once
#include "mid_dx.h"
#include "tile_gemm.h"

#include <algorithm>
#include <atomic>

namespace eqat {

constexpr int kBwdBig = 0, kBwdBigRagged = 1;       // what computes dX: 256 x 256 tiles, the same for any contraction length; 64, 96, 128: mid_dx_body with such token tiles

// CUT: tiles of dW that are cut along T where dW has a launch of its own are cut alike here, with a workgroup per item (n_dw: workgroups of that launch).
// Only plans that split tiles (SkPlan::split): a workgroup number has dp_rounds + 1 items at most and one part, and nobody waits for anybody.  The second
// contributor of a run waits for the first one, which may not have been dispatched here: the grid is larger than what is resident.
template <int BITS, typename WT, bool AP, int DX, bool CUT>
__global__ __launch_bounds__(512) void k_gemm_bwd(const GemmQArgs q, const MidArgs m, const GemmDwArgs d, const int n_dx, const int n_dw)
{
    typedef DwTileBig D;
    typedef TileBig Q;
    const int bid = (int)blockIdx.x, pad = (n_dx + 7) & ~7;          // every workgroup of dW stays on the XCD that its number asks for
    if (bid < pad) {
        if (bid >= n_dx) return;
        if constexpr (DX >= 64) mid_dx_body<BITS, DX>(m, (uint32_t)bid, (uint32_t)n_dx);
        else gemm_q_body<BITS, true, DX == kBwdBig ? kWhole : kRagged, Q::BM, Q::BN, Q::BK, Q::WGM, Q::WGN>(q, bid, n_dx);
    } else {
        gemm_dw_body<BITS, WT, AP, D::BM, D::BN, D::BK, D::NS, D::WGM, D::WGN, CUT, true>(d, CUT ? (bid - pad) % n_dw : bid - pad, n_dw, CUT ? (bid - pad) / n_dw : 0);
    }
}

template <int BITS, typename WT, bool AP, int DX, bool CUT = false>
void launch_bwd_t(const GemmQArgs &q, const MidArgs &m, const GemmDwArgs &d, int n_dx, int n_dw, hipStream_t st)
{
    typedef DwTileBig D;
    constexpr size_t dw = dw_smem_bytes<WT, AP, D::BM, D::BN, D::BK, D::NS, D::WGM, D::WGN>();
    constexpr size_t smem = std::max(dw, [] { if constexpr (DX >= 64) return (size_t)DxLds<BITS, DX>::TOTAL; else return q_smem_bytes<true, TileBig>(); }());
    static_assert(smem + (CUT ? 64 : 0) <= 160 * 1024, "LDS of one CU; tiles that are cut have a word of their own");
    static_assert(!CUT || DX < 64, "cut tiles of dW come with big tiles of dX (bwd_together)");
    auto kern = k_gemm_bwd<BITS, WT, AP, DX, CUT>;
    static std::atomic<uint64_t> allowed{0};          // more dynamic LDS than the default limit: once per device
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev > 63) dev = 0;
    if (!((allowed.load(std::memory_order_relaxed) >> dev) & 1u)) {
        (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        allowed.fetch_or((uint64_t)1 << dev, std::memory_order_relaxed);
    }
    kern<<<dim3((unsigned)(((n_dx + 7) & ~7) + n_dw * (CUT ? d.sk.dp_rounds + 1 : 1))), dim3(512), smem, st>>>(q, m, d, n_dx, n_dw);
}

template <typename WT, bool AP>
void launch_bwd_types(int bits, int dx, const GemmQArgs &q, const MidArgs &m, const GemmDwArgs &d, int n_dx, int n_dw, hipStream_t st)
{
#define EQAT_BWD(B)                                                                                        \
    do {                                                                                                   \
        if (d.sk.walk && dx == kBwdBig) launch_bwd_t<B, WT, AP, kBwdBig, true>(q, m, d, n_dx, n_dw, st);     \
        else if (d.sk.walk) launch_bwd_t<B, WT, AP, kBwdBigRagged, true>(q, m, d, n_dx, n_dw, st);          \
        else if (dx == kBwdBig) launch_bwd_t<B, WT, AP, kBwdBig>(q, m, d, n_dx, n_dw, st);                  \
        else if (dx == kBwdBigRagged) launch_bwd_t<B, WT, AP, kBwdBigRagged>(q, m, d, n_dx, n_dw, st);      \
        else if (dx == 64) launch_bwd_t<B, WT, AP, 64>(q, m, d, n_dx, n_dw, st);                            \
        else if (dx == 96) launch_bwd_t<B, WT, AP, 96>(q, m, d, n_dx, n_dw, st);                            \
        else launch_bwd_t<B, WT, AP, 128>(q, m, d, n_dx, n_dw, st);                                         \
    } while (0)
    if (bits == 2) EQAT_BWD(2); else if (bits == 3) EQAT_BWD(3); else EQAT_BWD(4);
#undef EQAT_BWD
}

void launch_bwd_ap_bf16(int bits, int dx, const GemmQArgs &q, const MidArgs &m, const GemmDwArgs &d, int n_dx, int n_dw, hipStream_t st);
void launch_bwd_ap_f32(int bits, int dx, const GemmQArgs &q, const MidArgs &m, const GemmDwArgs &d, int n_dx, int n_dw, hipStream_t st);
void launch_bwd_e2e(int bits, int dx, const GemmQArgs &q, const MidArgs &m, const GemmDwArgs &d, int n_dx, int n_dw, hipStream_t st);

}  // namespace eqat
