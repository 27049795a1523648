// dX for few output tiles in a launch of its own (what the kernel does and what bounds it: mid_dx.h).
#include "common.h"
#include "kernels.h"
#include "mid_dx.h"

#include <algorithm>
#include <atomic>

namespace eqat {

namespace {

template <int BITS, int BM>
__global__ __launch_bounds__(kMidNT) void k_gemm_mid_dx(const MidArgs a)
{
    mid_dx_body<BITS, BM>(a, blockIdx.x, gridDim.x);
}

template <int BITS, int BM> void launch_t(const MidArgs &a, hipStream_t st)
{
    constexpr int smem = (int)DxLds<BITS, BM>::TOTAL;
    auto kern = k_gemm_mid_dx<BITS, BM>;
    static std::atomic<uint64_t> allowed{0};          // more dynamic LDS than the default limit: once per device
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev > 63) dev = 0;
    if (!((allowed.load(std::memory_order_relaxed) >> dev) & 1u)) {
        (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
        allowed.fetch_or((uint64_t)1 << dev, std::memory_order_relaxed);
    }
    kern<<<dim3((unsigned)(a.tiles_m * a.tiles_n)), dim3(kMidNT), smem, st>>>(a);
}

}  // namespace

// Rounds of workgroups (one per compute unit) at 0.73 (64 tokens), 0.93 (96) or 1.2 us (128) a step, 3 us between rounds.
double mid_dx_us(const Problem &p, int cus, int *tokens)
{
    double best = 1e30;
    for (const int bm : {64, 96, 128}) {
        const int64_t rounds = (((p.T + bm - 1) / bm) * ((p.I + kMidBN - 1) / kMidBN) + cus - 1) / cus;
        if (rounds > 2) continue;
        const double us = 2.7 + (double)rounds * (3.0 + (double)((p.O + 127) / 128) * (bm == 64 ? 0.73 : bm == 96 ? 0.93 : 1.2));
        if (us < best) { best = us; *tokens = bm; }
    }
    return best;
}

MidArgs mid_dx_args(const Problem &p, int tokens, const void *dY, const void *codes, const void *sz, void *dX)
{
    MidArgs a{};
    a.X = (const bf16_t *)dY; a.codes = (const uint32_t *)codes; a.s = (const float *)sz; a.Y = (bf16_t *)dX;
    a.T = (int)p.T; a.I = (int)p.O; a.O = (int)p.I; a.G = (int)p.G; a.group = (int)p.g;
    a.x_bytes = (uint32_t)(p.T * p.O * 2);
    a.code_row_bytes = (uint32_t)(work_code_bytes(p) / p.O);
    a.codes_bytes = (uint32_t)work_code_bytes(p);
    a.s_bytes = (uint32_t)(p.O * p.G * 8);
    a.tiles_m = (a.T + tokens - 1) / tokens;
    a.tiles_n = (a.O + kMidBN - 1) / kMidBN;
    a.band = band_of(a.tiles_m, tokens);
    return a;
}

void launch_mid_dx(const Problem &p, int tokens, const void *dY, const void *codes, const void *sz, void *dX, hipStream_t st)
{
    const MidArgs a = mid_dx_args(p, tokens, dY, codes, sz, dX);
#define EQAT_DX(B) do { if (tokens == 128) launch_t<B, 128>(a, st); else if (tokens == 96) launch_t<B, 96>(a, st); else launch_t<B, 64>(a, st); } while (0)
    if (p.bits == 2) EQAT_DX(2); else if (p.bits == 3) EQAT_DX(3); else EQAT_DX(4);
#undef EQAT_DX
}

}  // namespace eqat
