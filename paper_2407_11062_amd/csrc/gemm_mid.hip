// Forward for few output tiles (prompt processing, short training batches: more than 32 tokens, at most 512 tiles of 128 x 128
// and two rounds of workgroups here, see mid_applies): Y[T,O] = X[T,I] * What[O,I]^T.
//
// The 256 x 256 and 128 x 128 tile kernels have too few tiles here (333 tokens x 4096 rows: 96 on 256 compute units) and
// every workgroup walks the whole contraction: 64 K tiles of 0.55 us whatever the fill.  This kernel puts the spare
// parallelism into the contraction INSIDE a workgroup: eight waves are 2 (64 weight rows each) x 4 (a quarter of every
// 256-wide K step each), and their sums meet in LDS at the end, in a fixed order, without a trip through memory.
// A wave owns its weights alone, so they go from codes to MFMA operands in its registers (a lane holds one 32-code
// segment per 32-row block and K step; weights are the A operand) and only tokens and codes pass through LDS.  Because
// nothing re-lays the weights, the caller's dense stream is read as it is (no pass of its own before the GEMM); the working
// layout is the same kernel with another segment load, bitwise the same results.
// Everything a K step needs is fetched a step ahead straight into LDS: tokens as a [BM][256] bf16 tile (the 16-byte chunk c
// of row r at position c ^ (r & 7), so that the 8 lanes a read serves together, 8 rows of one chunk, hit different banks),
// codes as whole row pieces.  (Codes and step sizes loaded by the lanes that use them touch 32 cache lines per
// instruction: 1.5 instead of 1.2 us per K step.)
// What bounds it is the rebuild.  Beside a 32x32x16 product (33 cycles) a SIMD issues some 4.9 arithmetic instructions, every
// further one costs 4 cycles (two waves, measured with independent instructions; max(33, 13.5 + 4 n) fits), and here a
// product goes with 5 (96 tokens, 2 bit, working layout) to 14 (64 tokens, 4 bit) of them.  Switched off one at a time (2 bit,
// 64 tokens, 4096 x 4096, 24.5 us): the rebuild 15.4, all loads 21.5, the LDS reads 24.1; everything but the products 11.8.  So
//   - the rebuild of slice t + 1 is spread between the products of slice t, and everything a step starts with is read in the
//     last slice of the step before, behind the barrier that sits in front of that slice (333 tokens, 4096 x 11008, us:
//     2 bit 63 -> 60, 3 bit, working layout 70 -> 65; 4 bit 66 -> 64).
// Measured, us: 2 bit, 333 tokens: 4096 x 4096 41 -> 28 (and the re-layout of the codes, 6, gone), 4096 x 11008 104 -> 60
// (14 gone); 4 bit, 150 tokens, 11008 x 4096 45 -> 38 (10 gone).
#include "common.h"
#include "dense_codes.h"
#include "kernels.h"

#include <algorithm>
#include <atomic>

namespace eqat {

namespace {

struct MidArgs {
    const bf16_t *X; const uint32_t *codes; const float *s; const uint32_t *zp; const float *zf; bf16_t *Y;
    int T, I, O, G;
    uint32_t spg_magic;            // ceil(2^32 / (g/32)), 0 for g = 32: group of a segment
    uint32_t code_row_bytes, z_row_words;
    uint32_t x_bytes, codes_bytes, s_bytes, z_bytes;
    int tiles_m, tiles_n;
};

constexpr int kMidBN = 128, kMidBK = 256, kMidKG = 4, kMidNT = 512;

// LDS of one K step: token tile, codes, and per weight row and segment a word with the step size and one (3-bit packed zero
// points: two) with the zero point.
template <int BITS, int SRC, int BM> struct MidLds {
    static constexpr int WPS = SRC == kWorking ? WorkCodes<BITS>::kWords : BITS;      // words per segment
    static constexpr int NCH = 2 * WPS;                                               // 16-byte chunks of a row's codes
    static constexpr int ZW = SRC == kPackedZ && BITS == 3 ? 2 : 1;
    static constexpr uint32_t TOK = BM * kMidBK * 2, CODES = kMidBN * NCH * 16, ROWW = kMidBN * 8 * 4;
    static constexpr uint32_t STEP = TOK + CODES + (1 + ZW) * ROWW, TOTAL = 2 * STEP;
    static_assert(TOTAL <= 160 * 1024, "LDS of one CU");
};
// position of the 16-byte chunk c of a row's codes: the lanes of a read (32 rows, one segment) spread over the banks
template <int NCH> __device__ __forceinline__ int code_chunk_swz(int row, int c)
{
    return NCH == 4 ? c ^ ((row >> 1) & 3) : NCH == 8 ? c ^ (row & 7) : c;            // rows of 96 bytes spread by themselves
}

template <int BITS, int SRC, int BM>
__global__ __launch_bounds__(kMidNT) void k_gemm_mid(const MidArgs a)
{
    typedef MidLds<BITS, SRC, BM> L;
    constexpr int MI = BM / 32, WPS = L::WPS, NCH = L::NCH;
    constexpr int A_LOADS = BM / 16;                  // direct-to-LDS instructions per wave and K step (two rows each)
    constexpr int C_INSTR = kMidBN * NCH / 64;        // ... for the codes, in all
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave & 1, kg = wave >> 1, r = lane & 31, h = lane >> 5;

    // Every XCD gets a contiguous range of tiles, token tiles of one weight tile next to each other: the codes are fetched
    // into one L2 only.
    const int nb = (int)gridDim.x, xcd = (int)(blockIdx.x & 7), rem = nb & 7;
    const int pid = xcd * (nb >> 3) + (xcd < rem ? xcd : rem) + (int)(blockIdx.x >> 3);
    const int m0 = (pid % a.tiles_m) * BM, n0 = (pid / a.tiles_m) * kMidBN;

    const RawRsrc rX = make_raw_rsrc(a.X, a.x_bytes);
    const RawRsrc rW = make_raw_rsrc(a.codes, a.codes_bytes);
    const RawRsrc rS = make_raw_rsrc(a.s, a.s_bytes);
    const RawRsrc rZ = make_raw_rsrc(SRC == kFloatZ ? (const void *)a.zf : (const void *)a.zp, a.z_bytes);
    const int n_segs = a.I >> 5, steps = (a.I + kMidBK - 1) / kMidBK;
    const uint32_t lds0 = lds_addr_of(smem_raw);

    // ---- loads of one K step.  Rows past T or O are out of range of their buffers (zeros); columns past I: tokens and
    // step sizes come as zeros, the codes there are whatever follows the row.
    uint32_t off[A_LOADS];
    int col[A_LOADS];
#pragma unroll
    for (int it = 0; it < A_LOADS; ++it) {
        const int row = (wave * A_LOADS + it) * 2 + h;
        col[it] = (r ^ (row & 7)) * 8;
        off[it] = m0 + row < a.T ? ((uint32_t)(m0 + row) * (uint32_t)a.I + (uint32_t)col[it]) * 2u : kOobOffset;
    }
    uint32_t coff[(C_INSTR + 7) / 8];
#pragma unroll
    for (int it = 0; it < (C_INSTR + 7) / 8; ++it) {
        const int e = (it * 8 + wave) * 64 + lane, row = e / NCH;
        coff[it] = (uint32_t)(n0 + row) * a.code_row_bytes + (uint32_t)code_chunk_swz<NCH>(row, e % NCH) * 16u;
    }
    const uint32_t srow = (uint32_t)(n0 + wave * 16 + (lane >> 3));        // rows of the step sizes: 8 per instruction, two instructions
    // Load number d of those a wave issues per K step: codes, step sizes and zero points, then tokens.
    constexpr int C_LOADS = (C_INSTR + 7) / 8, S_LOADS = 2 * (1 + L::ZW), LOADS = C_LOADS + S_LOADS + A_LOADS;
    auto load = [&](int d, int step, int buf) {
        const uint32_t base = lds0 + (uint32_t)buf * L::STEP;
        if (d < C_LOADS) {
            if (C_INSTR % 8 == 0 || d * 8 + wave < C_INSTR)
                load_to_lds16_at(rW, base + L::TOK + (uint32_t)((d * 8 + wave) * 1024), coff[d] + (uint32_t)step * (NCH * 16));
        } else if (d < C_LOADS + S_LOADS) {
            const int e = d - C_LOADS, it = e / (1 + L::ZW), what = e % (1 + L::ZW);           // what: step size, zero point (, its second word)
            const int seg = step * 8 + (lane & 7);
            const uint32_t j = a.spg_magic ? __umulhi((uint32_t)seg, a.spg_magic) : (uint32_t)seg;
            const bool ok = seg < n_segs;
            const uint32_t gi = (srow + 8 * it) * (uint32_t)a.G + j;
            const uint32_t at = base + L::TOK + L::CODES + (uint32_t)((wave * 2 + it) * 256) + (uint32_t)what * L::ROWW;
            if constexpr (SRC == kWorking) load_to_lds4_at(rS, at, ok ? gi * 8u + 4u * what : kOobOffset);
            else if (what == 0) load_to_lds4_at(rS, at, ok ? gi * 4u : kOobOffset);
            else if constexpr (SRC == kFloatZ) load_to_lds4_at(rZ, at, ok ? gi * 4u : kOobOffset);
            else load_to_lds4_at(rZ, at, ((srow + 8 * it) * a.z_row_words + ((j * BITS) >> 5)) * 4u + 4u * (what - 1));
        } else {
            const int it = d - C_LOADS - S_LOADS;
            load_to_lds16_at(rX, base + (uint32_t)((wave * A_LOADS + it) * 1024),
                             step * kMidBK + col[it] < a.I ? off[it] + (uint32_t)step * (kMidBK * 2) : kOobOffset);
        }
    };
    // part P of 3 of a step's loads
    auto load_part = [&](auto part, int step, int buf) {
        constexpr int P = decltype(part)::value;
#pragma unroll
        for (int d = 0; d < LOADS; ++d)
            if (d * 3 / LOADS == P) load(d, step, buf);
    };
    struct Seg { uint32_t w[WPS]; };
    auto eight = [&](const WhatTable<BITS> &tab, const Seg &sg, auto t) -> bf16x8 {
        constexpr int T4 = decltype(t)::value;
        if constexpr (SRC == kWorking) {
            WorkCodes<BITS> c;
#pragma unroll
            for (int k = 0; k < WPS; ++k) c.w[k] = sg.w[k];
            return tab.template eight<T4>(c);
        } else {
            CodeWords<BITS> c;
#pragma unroll
            for (int k = 0; k < WPS; ++k) c.w[k] = sg.w[k];
            return unslot_of<BITS>(eight_of<BITS, T4>(tab, c));
        }
    };

    floatx16 acc[2][MI];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[b][i][q] = 0.0f;

    Seg cur[2];
    WhatTable<BITS> tab[2];
    bf16x8 x[2][MI], w[2][2];
    // this lane's segment (number 2 kg + h of the step) of both 32-row blocks, with what it takes to rebuild the weights
    float ws[2];
    uint32_t wz[2][L::ZW];
    auto read_codes = [&](int buf) {
        const unsigned char *const here = smem_raw + (uint32_t)buf * L::STEP;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int row = wn * 64 + b * 32 + r;
            const uint32_t *const sw = reinterpret_cast<const uint32_t *>(here + L::TOK + L::CODES) + row * 8 + 2 * kg + h;
            ws[b] = __uint_as_float(sw[0]);
#pragma unroll
            for (int k = 0; k < L::ZW; ++k) wz[b][k] = sw[(k + 1) * (L::ROWW / 4)];
            const unsigned char *const codes = here + L::TOK + row * (NCH * 16);
            if constexpr (WPS == 2) {
                const uintx2 v = *reinterpret_cast<const uintx2 *>(codes + code_chunk_swz<NCH>(row, kg) * 16 + h * 8);
                cur[b].w[0] = v[0]; cur[b].w[1] = v[1];
            } else if constexpr (WPS == 3) {
                const uint32_t *const v = reinterpret_cast<const uint32_t *>(codes + (2 * kg + h) * 12);
                cur[b].w[0] = v[0]; cur[b].w[1] = v[1]; cur[b].w[2] = v[2];
            } else {
                const uintx4 v = *reinterpret_cast<const uintx4 *>(codes + code_chunk_swz<NCH>(row, 2 * kg + h) * 16);
                cur[b].w[0] = v[0]; cur[b].w[1] = v[1]; cur[b].w[2] = v[2]; cur[b].w[3] = v[3];
            }
        }
    };
    auto build = [&](int step, int b) {
        float z = __uint_as_float(wz[b][0]);
        if constexpr (SRC == kPackedZ) {
            const uint32_t seg = (uint32_t)(step * 8 + 2 * kg + h);
            const uint32_t zshift = ((a.spg_magic ? __umulhi(seg, a.spg_magic) : seg) * BITS) & 31u;
            const uint32_t v = L::ZW == 2 ? __builtin_amdgcn_alignbit(wz[b][L::ZW - 1], wz[b][0], zshift) : wz[b][0] >> zshift;
            z = (float)(v & ((1u << BITS) - 1u));
        }
        tab[b].build(ws[b], z);
    };
    const unsigned char *const tile = smem_raw + r * 512;
    auto read_x = [&](int slot, int buf, int t) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
            x[slot][i] = *reinterpret_cast<const bf16x8 *>(tile + (uint32_t)buf * L::STEP + i * (32 * 512) + (((kg * 8 + h * 4 + t) ^ (r & 7)) * 16));
    };
    auto products = [&](int slot) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int b = 0; b < 2; ++b)
                acc[b][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[slot][b], x[slot][i], acc[b][i], 0, 0, 0);
    };
    // one product, one LDS read, a share of the arithmetic, repeated
    auto weave = [&](auto valu) {
#pragma unroll
        for (int q = 0; q < 2 * MI; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, decltype(valu)::value, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr int kVal = (BITS == 4 ? 52 : 40) / (2 * MI) + 1;

#pragma unroll
    for (int d = 0; d < LOADS; ++d) load(d, 0, 0);
    wait_all_and_barrier();
    if (steps > 1) load_part(IC<0>{}, 1, 1);
    read_codes(0);
    read_x(0, 0, 0);
    build(0, 0); build(0, 1);
    w[0][0] = eight(tab[0], cur[0], IC<0>{}); w[0][1] = eight(tab[1], cur[1], IC<0>{});
    __builtin_amdgcn_sched_barrier(0);
    for (int step = 0; step < steps; ++step) {
        const int buf = step & 1;
        if (step + 1 < steps) load_part(IC<1>{}, step + 1, buf ^ 1);
        __builtin_amdgcn_sched_barrier(0);
        read_x(1, buf, 1);
        products(0);
        w[1][0] = eight(tab[0], cur[0], IC<1>{}); w[1][1] = eight(tab[1], cur[1], IC<1>{});
        weave(IC<kVal>{});
        if (step + 1 < steps) load_part(IC<2>{}, step + 1, buf ^ 1);
        __builtin_amdgcn_sched_barrier(0);
        read_x(0, buf, 2);
        products(1);
        w[0][0] = eight(tab[0], cur[0], IC<2>{}); w[0][1] = eight(tab[1], cur[1], IC<2>{});
        weave(IC<kVal>{});
        read_x(1, buf, 3);
        products(0);
        w[1][0] = eight(tab[0], cur[0], IC<3>{}); w[1][1] = eight(tab[1], cur[1], IC<3>{});
        weave(IC<kVal>{});
        wait_all_and_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if (step + 2 < steps) load_part(IC<0>{}, step + 2, buf);
        __builtin_amdgcn_sched_barrier(0);
        read_codes(buf ^ 1);
        read_x(0, buf ^ 1, 0);
        products(1);
        build(step + 1, 0); build(step + 1, 1);
        w[0][0] = eight(tab[0], cur[0], IC<0>{}); w[0][1] = eight(tab[1], cur[1], IC<0>{});
        weave(IC<kVal + 4>{});
    }

    // ---- sums: acc[b][i][q] is row 8 (q / 4) + 4 h + q % 4 of block b, token 32 i + r.  One 32-row block of every wave at a
    // time passes through LDS as [wave][token][32 rows] (the 16-byte chunk c of a token at c ^ (token & 7)); wave (wn, kg) then
    // adds the four K quarters, in order, for the kg-th quarter of the tokens and stores 64 bytes of a row per 8 lanes.
    constexpr uint32_t WAVE_BYTES = BM * 32 * 4;
    static_assert(8 * WAVE_BYTES <= L::TOTAL, "the sums go where the tiles were");
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                floatx4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = acc[b][i][4 * q + e];
                *reinterpret_cast<floatx4 *>(smem_raw + wave * WAVE_BYTES + (i * 32 + r) * 128 + (((2 * q + h) ^ (r & 7)) * 16)) = v;
            }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < BM / 4 / 8; ++k) {
            const int tok = kg * (BM / 4) + k * 8 + (lane >> 3), ch = lane & 7;
            floatx4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int g = 0; g < kMidKG; ++g) {
                const floatx4 v = *reinterpret_cast<const floatx4 *>(smem_raw + (g * 2 + wn) * WAVE_BYTES + tok * 128 + ((ch ^ (tok & 7)) * 16));
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[e] += v[e];
            }
            const int o = n0 + wn * 64 + b * 32 + ch * 4;
            if (m0 + tok < a.T && o < a.O) {           // O is a multiple of 8
                bf16x4 y;
#pragma unroll
                for (int e = 0; e < 4; ++e) y[e] = (bf16_t)sum[e];
                *reinterpret_cast<bf16x4 *>(a.Y + (size_t)(m0 + tok) * a.O + o) = y;
            }
        }
    }
}


template <int BITS, int SRC, int BM> void launch_t(MidArgs a, hipStream_t st)
{
    constexpr int smem = (int)MidLds<BITS, SRC, BM>::TOTAL;
    auto kern = k_gemm_mid<BITS, SRC, BM>;
    static std::atomic<uint64_t> allowed{0};          // more dynamic LDS than the default limit: once per device
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev > 63) dev = 0;
    if (!((allowed.load(std::memory_order_relaxed) >> dev) & 1u)) {
        (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
        allowed.fetch_or((uint64_t)1 << dev, std::memory_order_relaxed);
    }
    a.tiles_m = (a.T + BM - 1) / BM;
    a.tiles_n = (a.O + kMidBN - 1) / kMidBN;
    kern<<<dim3((unsigned)(a.tiles_m * a.tiles_n)), dim3(kMidNT), smem, st>>>(a);
}

// What a launch with token tiles of `bm` takes, in us: rounds of workgroups (one per compute unit), each 6 us and 1.2 (64
// tokens) or 1.45 (96) us per 256-wide K step; fitted at 4096, 8192 and 11008 inputs.
int64_t rounds_of(const Problem &p, int bm) { return (((p.T + bm - 1) / bm) * ((p.O + kMidBN - 1) / kMidBN) + 255) / 256; }
double launch_us(const Problem &p, int bm)
{
    return (double)rounds_of(p, bm) * (6.0 + (double)((p.I + kMidBK - 1) / kMidBK) * (bm == 64 ? 1.2 : 1.45));
}

int token_tile(const Problem &p) { return launch_us(p, 96) < launch_us(p, 64) ? 96 : 64; }

template <int SRC> void launch_src(const Problem &p, const MidArgs &a, hipStream_t st)
{
    const bool tall = token_tile(p) == 96;
#define EQAT_MID(B) do { if (tall) launch_t<B, SRC, 96>(a, st); else launch_t<B, SRC, 64>(a, st); } while (0)
    if (p.bits == 2) EQAT_MID(2); else if (p.bits == 3) EQAT_MID(3); else EQAT_MID(4);
#undef EQAT_MID
}

MidArgs mid_args(const Problem &p, const void *X, const void *codes, const void *s, void *Y)
{
    MidArgs a{};
    a.X = (const bf16_t *)X; a.codes = (const uint32_t *)codes; a.s = (const float *)s; a.Y = (bf16_t *)Y;
    a.T = (int)p.T; a.I = (int)p.I; a.O = (int)p.O; a.G = (int)p.G;
    a.spg_magic = p.g == 32 ? 0u : (uint32_t)((((uint64_t)1 << 32) + (uint64_t)(p.g / 32) - 1) / (uint64_t)(p.g / 32));
    a.x_bytes = (uint32_t)(p.T * p.I * 2);
    return a;
}

}  // namespace

// From 3-bit codes as packed, which have no byte alignment, a K step takes 0.45 us longer than from the working layout.  With two
// rounds of workgroups and three token tiles or more that is more than the re-layout costs, and even the 128 x 128 tiles
// behind a re-layout are faster then (g = 128, us, as packed / tiles / re-laid: 1300 tokens, 4096 x 11008 198 / 181 / 167;
// 384 tokens, 11008 x 8192 148 / 136 / 122; 640 tokens, 8192 x 5120 95 / 90 / 83).  With two token tiles every weight is
// rebuilt twice only: 160 tokens, 28672 x 4096 76 as packed, 81 re-laid.
FwdRoute mid_route(const Problem &p, bool from_packed)
{
    const int tokens = token_tile(p);
    return FwdRoute{from_packed && p.bits == 3 && p.T > 2 * tokens && rounds_of(p, tokens) > 1 ? FWD_RELAY_MID : FWD_MID, tokens, kMidBN};
}

double mid_us(const Problem &p) { return std::min(launch_us(p, 96), launch_us(p, 64)); }

// Against the 128 x 128-tile kernel, which takes 0.55 us per 64-wide K tile while a compute unit has one tile at most and
// 0.9 or more beyond that (11008 x 4096: 256 tokens, 172 tiles: 43 us there, 46-49 here in two rounds; 288 tokens, 258
// tiles: 61 and 47; 400 tokens: 63 and 57).  More than two rounds here, or more than two tiles per compute unit there: the
// 256 x 256 tiles are the better kernel (11008 x 4096, 515 tokens: 68 us in tiles, 84 here).  The GEMMs alone are compared:
// a forward from the packed arrays saves the re-layout as well and would gain a little earlier, but every forward entry point
// shares the rule, so that their results stay bitwise equal.
bool mid_applies(const Problem &p)
{
    if (!p.act_bf16 || !group_by_magic(p) || p.T <= 32) return false;
    if (p.T <= 64) return !gemv_work_applies(p);
    const int64_t tiles = ((p.T + 127) / 128) * ((p.O + 127) / 128);
    return tiles <= 512 && mid_us(p) < 4.0 + (double)((p.I + 63) / 64) * (tiles <= 256 ? 0.55 : 0.9);
}

void launch_mid(const Problem &p, const void *X, const void *Wpacked, const float *s, const void *zpacked, const float *zfloat,
                void *Y, hipStream_t st)
{
    MidArgs a = mid_args(p, X, Wpacked, s, Y);
    a.zp = (const uint32_t *)zpacked; a.zf = zfloat;
    a.code_row_bytes = (uint32_t)(p.I * p.bits / 8);
    a.z_row_words = (uint32_t)((p.G * p.bits + 31) / 32);
    a.codes_bytes = (uint32_t)(p.O * p.I * p.bits / 8);
    a.s_bytes = (uint32_t)(p.O * p.G * 4);
    a.z_bytes = zfloat != nullptr ? a.s_bytes : (uint32_t)(p.O * a.z_row_words * 4);
    if (zfloat != nullptr) launch_src<kFloatZ>(p, a, st); else launch_src<kPackedZ>(p, a, st);
}

void launch_mid_work(const Problem &p, const void *X, const void *codes, const void *sz, void *Y, hipStream_t st)
{
    MidArgs a = mid_args(p, X, codes, sz, Y);
    a.code_row_bytes = (uint32_t)(work_code_bytes(p) / p.O);
    a.codes_bytes = (uint32_t)work_code_bytes(p);
    a.s_bytes = (uint32_t)(p.O * p.G * 8);
    launch_src<kWorking>(p, a, st);
}

}  // namespace eqat
