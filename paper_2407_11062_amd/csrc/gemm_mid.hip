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
// product goes with 5.5 (96 tokens, 2 bit, working layout) to 13 (64 tokens, 4 bit) of them.  Switched off one at a time (2 bit,
// 64 tokens, 4096 x 4096, 24.5 us): the rebuild 15.4, all loads 21.5, the LDS reads 24.1; everything but the products 11.8.  So
//   - a K step is four slices of 16 per wave; the barrier sits in the middle of a step, behind the reads of all its tokens: in
//     the third slice the next step's codes are read, in the fourth its tables and first weights are made, so that no slice waits
//     for LDS, and every slice's rebuild is spread evenly between the products of the slice before;
//   - addresses are scalar work: the buffers move along K, the lanes' offsets stay;
//   - where the tiles still fill the chip, 128 tokens share a rebuilt weight (k_gemm_mid_tall below).
// Measured, us, 333 tokens, from the packed arrays (the chain of a step behind its barrier / this): 4096 x 4096 2 bit 26.4 -> 23.2,
// 3 bit 35 -> 31.4, 4 bit 30.9 -> 25.2; 4096 x 11008 61 -> 54, 70 -> 60, 72 -> 58.
#include "common.h"
#include "dense_codes.h"
#include "kernels.h"
#include "mid_tiles.h"

#include <algorithm>
#include <atomic>

namespace eqat {

namespace {

constexpr int kMidBK = 256;

// A prepared layer's forward reads the step sizes as the caller has them and the zero points as the layer holds them.  The backward wants them as pairs: where
// it follows, this launch leaves them as well, a share per workgroup, read before the sums meet and written behind the tile.
struct PairsShare {
    uint32_t at;
    intx4 s, z;
    static __device__ __forceinline__ uint32_t fours(const MidArgs &a) { return a.pairs != nullptr ? a.s_bytes / 16 : 0u; }      // the rows are a multiple of 8
    __device__ __forceinline__ void read(const MidArgs &a)
    {
        at = blockIdx.x * (uint32_t)kMidNT + threadIdx.x;
        if (at < fours(a)) { s = reinterpret_cast<const intx4 *>(a.s)[at]; z = reinterpret_cast<const intx4 *>(a.zf)[at]; }
    }
    __device__ __forceinline__ void write(const MidArgs &a)
    {
        while (at < fours(a)) {
            intx4 *const to = reinterpret_cast<intx4 *>(a.pairs) + 2 * (size_t)at;
            to[0] = intx4{s[0], z[0], s[1], z[1]};
            to[1] = intx4{s[2], z[2], s[3], z[3]};
            at += gridDim.x * (uint32_t)kMidNT;
            if (at < fours(a)) { s = reinterpret_cast<const intx4 *>(a.s)[at]; z = reinterpret_cast<const intx4 *>(a.zf)[at]; }
        }
    }
};

// LDS of one K step: token tile, codes, and per weight row and segment a word with the step size and one (3-bit packed zero
// points: two) with the zero point.
template <int BITS, int SRC, int BM> struct MidLds {
    static constexpr int WPS = kRelaid<SRC> ? WorkCodes<BITS>::kWords : BITS;      // words per segment
    static constexpr int NCH = 2 * WPS;                                               // 16-byte chunks of a row's codes
    static constexpr int ZW = SRC == kPackedZ && BITS == 3 ? 2 : 1;
    static constexpr uint32_t WAVE_CODES = NCH == 4 ? 1024 : 2048;                    // the 16 rows that a wave fetches
    static constexpr uint32_t TOK = BM * kMidBK * 2, CODES = 8 * WAVE_CODES, ROWW = kMidBN * 8 * 4;
    static constexpr uint32_t STEP = TOK + CODES + (1 + ZW) * ROWW, TOTAL = 2 * STEP;
    static_assert(TOTAL <= 160 * 1024, "LDS of one CU");
};
// position of the 16-byte chunk c of a row's codes: the lanes of a read (32 rows, one segment) spread over the banks
template <int NCH> __device__ __forceinline__ int code_chunk_swz(int row, int c)
{
    return NCH == 2 ? c ^ ((row >> 2) & 1) : NCH == 4 ? c ^ ((row >> 1) & 3) : NCH == 8 ? c ^ (row & 7) : c;            // rows of 96 bytes spread by themselves
}

template <int BITS, int SRC, int BM>
__global__ __launch_bounds__(kMidNT) void k_gemm_mid(const MidArgs a)
{
    typedef MidLds<BITS, SRC, BM> L;
    constexpr int MI = BM / 32, WPS = L::WPS, NCH = L::NCH;
    constexpr int A_LOADS = BM / 16;                  // direct-to-LDS instructions per wave and K step (two rows each)
    constexpr int C_LOADS = NCH == 4 ? 1 : 2;         // ... for the codes
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave & 1, kg = wave >> 1, r = lane & 31, h = lane >> 5;

    int m0, n0;
    tile_of(a, BM, blockIdx.x, gridDim.x, m0, n0);

    const int n_segs = a.I >> 5, steps = (a.I + kMidBK - 1) / kMidBK;
    const uint32_t lds0 = lds_addr_of(smem_raw);

    // ---- loads of one K step.  Rows past T or O are out of range of their buffers (zeros); columns past I: tokens and
    // step sizes come as zeros, the codes there are whatever follows the row.  The lanes' byte offsets into tokens and codes
    // stay as they are, the buffers move along K.
    uint32_t off[A_LOADS];
#pragma unroll
    for (int it = 0; it < A_LOADS; ++it) {
        const int row = (wave * A_LOADS + it) * 2 + h;
        off[it] = m0 + row < a.T ? ((uint32_t)(m0 + row) * (uint32_t)a.I + (uint32_t)((r ^ (row & 7)) * 8)) * 2u : kOobOffset;
    }
    uint32_t coff[C_LOADS];
#pragma unroll
    for (int it = 0; it < C_LOADS; ++it) {
        const int e = it * 64 + lane, row = wave * 16 + e / NCH;
        coff[it] = e < 16 * NCH ? (uint32_t)(n0 + row) * a.code_row_bytes + (uint32_t)code_chunk_swz<NCH>(row, e % NCH) * 16u : kOobOffset;
    }
    const uint32_t srow = (uint32_t)(n0 + wave * 16 + (lane >> 3));        // rows of the step sizes: 8 per instruction, two instructions
    const uint32_t each = a.spg_magic == 0u ? ~0u : 0u;                    // groups of 32: every segment is one
    auto group_of = [&](uint32_t seg) { return __umulhi(seg, a.spg_magic) + (seg & each); };
    Moving bX(a.X, a.x_bytes), bW(a.codes, a.codes_bytes);
    RawRsrc rX, rW;
    uint32_t s_left = 0;
    [[maybe_unused]] uint32_t z_left = 0;            // floats: as many as step sizes
    uint32_t sgroup = 0;                 // of this lane's segment
    uint32_t soff = 0;                   // 0, or out of range where the segment lies past the end of the rows
    int to_aim = steps;                  // counters of their own: a step number that lanes compute with ends up in a vector register, and
    uint32_t seg = (uint32_t)(lane & 7); // with it the descriptors
    auto aim = [&]() {                   // at the next step; past the last one nothing is in range (zeros)
        const bool live = to_aim-- > 0;
        rX = bX.at(live); rW = bW.at(live);
        bX.by(kMidBK * 2); bW.by(NCH * 16);
        s_left = live ? a.s_bytes : 0u;
        if constexpr (!kTwoFloats<SRC>) z_left = live ? a.z_bytes : 0u;
        sgroup = group_of(seg);
        soff = (int)seg < n_segs ? 0u : kOobOffset;
        seg += 8;
    };
    // in front of the loads of every step
    auto mask_last = [&](int step) {
        if (step == steps - 1 && a.I % kMidBK != 0) {
#pragma unroll
            for (int it = 0; it < A_LOADS; ++it) {
                const int row = (wave * A_LOADS + it) * 2 + h;
                if ((r ^ (row & 7)) * 8 >= a.I % kMidBK) off[it] = kOobOffset;
            }
        }
    };
    // Load number d of those a wave issues per K step: codes, step sizes and zero points, then tokens.
    constexpr int S_LOADS = 2 * (1 + L::ZW), LOADS = C_LOADS + S_LOADS + A_LOADS;
    auto load = [&](int d, int buf) {
        const uint32_t base = lds0 + (uint32_t)buf * L::STEP;
        const RawRsrc rS = make_raw_rsrc(a.s, s_left), rZ = make_raw_rsrc(kTwoFloats<SRC> ? (const void *)a.zf : (const void *)a.zp, kTwoFloats<SRC> ? s_left : z_left);
        if (d < C_LOADS) {
            load_to_lds16_at(rW, base + L::TOK + (uint32_t)wave * L::WAVE_CODES + (uint32_t)(d * 1024), coff[d]);
        } else if (d < C_LOADS + S_LOADS) {
            const int e = d - C_LOADS, it = e / (1 + L::ZW), what = e % (1 + L::ZW);           // what: step size, zero point (, its second word)
            const uint32_t gi = (srow + 8 * it) * (uint32_t)a.G + sgroup;
            const uint32_t at = base + L::TOK + L::CODES + (uint32_t)((wave * 2 + it) * 256) + (uint32_t)what * L::ROWW;
            if constexpr (SRC == kWorking) load_to_lds4_at(rS, at, (gi * 8u + 4u * what) | soff);
            else if (what == 0) load_to_lds4_at(rS, at, (gi * 4u) | soff);
            else if constexpr (kTwoFloats<SRC>) load_to_lds4_at(rZ, at, (gi * 4u) | soff);
            else load_to_lds4_at(rZ, at, ((srow + 8 * it) * a.z_row_words + ((sgroup * BITS) >> 5)) * 4u + 4u * (what - 1));
        } else {
            const int it = d - C_LOADS - S_LOADS;
            load_to_lds16_at(rX, base + (uint32_t)((wave * A_LOADS + it) * 1024), off[it]);
        }
    };
    // part P of 2 of a step's loads
    auto load_part = [&](auto part, int buf) {
        constexpr int P = decltype(part)::value;
#pragma unroll
        for (int d = 0; d < LOADS; ++d)
            if (d * 2 / LOADS == P) load(d, buf);
        __builtin_amdgcn_sched_barrier(0);
    };

    floatx16 acc[2][MI];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[b][i][q] = 0.0f;

    // This lane's segment (number 2 kg + h of the step) of both 32-row blocks, with what it takes to rebuild the weights: read
    // from LDS a slice before it is needed.
    struct Raw { uint32_t c[2][WPS], s[2], z[2][L::ZW], zshift; };
    Raw raw;
    uint32_t cur[2][WPS];
    WhatTable<BITS> tab[2];
    constexpr bool kShared = BITS == 2 && !kRelaid<SRC>;     // 2-bit codes as packed: the lookups of a word serve two slices
    uint32_t lo[2][4], hi[2][4];
    bf16x8 x[4][MI], w[2][2];
    uint32_t raw_seg = (uint32_t)(2 * kg);        // of the lanes h = 0
    auto read_raw = [&](int buf) {        // the steps in order
        const unsigned char *const here = smem_raw + (uint32_t)buf * L::STEP;
        if constexpr (SRC == kPackedZ) raw.zshift = ((h ? group_of(raw_seg + 1) : group_of(raw_seg)) * BITS) & 31u;
        raw_seg += 8;
        const int row = wn * 64 + r;                  // row + 32 lies a constant further on everywhere
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const uint32_t *const sw = reinterpret_cast<const uint32_t *>(here + L::TOK + L::CODES) + (row + b * 32) * 8 + 2 * kg + h;
            raw.s[b] = sw[0];
#pragma unroll
            for (int k = 0; k < L::ZW; ++k) raw.z[b][k] = sw[(k + 1) * (L::ROWW / 4)];
            const unsigned char *const codes = here + L::TOK + (uint32_t)((row >> 4) + 2 * b) * L::WAVE_CODES + (row & 15) * (NCH * 16);
            if constexpr (WPS == 2) {
                const uintx2 v = *reinterpret_cast<const uintx2 *>(codes + code_chunk_swz<NCH>(row, kg) * 16 + h * 8);
                raw.c[b][0] = v[0]; raw.c[b][1] = v[1];
            } else if constexpr (WPS == 3) {
                const uint32_t *const v = reinterpret_cast<const uint32_t *>(codes + (2 * kg + h) * 12);
                raw.c[b][0] = v[0]; raw.c[b][1] = v[1]; raw.c[b][2] = v[2];
            } else {
                const uintx4 v = *reinterpret_cast<const uintx4 *>(codes + code_chunk_swz<NCH>(row, 2 * kg + h) * 16);
                raw.c[b][0] = v[0]; raw.c[b][1] = v[1]; raw.c[b][2] = v[2]; raw.c[b][3] = v[3];
            }
        }
    };
    auto build = [&]() {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            float z = __uint_as_float(raw.z[b][0]);
            if constexpr (SRC == kPackedZ) {
                const uint32_t v = L::ZW == 2 ? __builtin_amdgcn_alignbit(raw.z[b][L::ZW - 1], raw.z[b][0], raw.zshift) : raw.z[b][0] >> raw.zshift;
                z = (float)(v & ((1u << BITS) - 1u));
            }
            tab[b].build(__uint_as_float(raw.s[b]), z);
#pragma unroll
            for (int k = 0; k < WPS; ++k) cur[b][k] = raw.c[b][k];
        }
    };
    auto look_up = [&](int word) {                // bytes of the codes k, k + 4, k + 8 and k + 12 of a word
        if constexpr (kShared) {
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t c = (cur[b][word] >> (2 * k)) & 0x03030303u;
                    lo[b][k] = __builtin_amdgcn_perm(tab[b].lo[0], tab[b].lo[0], c);
                    hi[b][k] = __builtin_amdgcn_perm(tab[b].hi[0], tab[b].hi[0], c);
                }
        }
    };
    auto eight = [&](int b, auto t) -> bf16x8 {
        constexpr int T4 = decltype(t)::value;
        if constexpr (kShared) {
            uintx4 u;
#pragma unroll
            for (int k = 0; k < 4; ++k) u[k] = __builtin_amdgcn_perm(hi[b][k], lo[b][k], T4 % 2 ? 0x07030602u : 0x05010400u);
            return unslot_of<BITS>(__builtin_bit_cast(bf16x8, u));
        } else if constexpr (kRelaid<SRC>) {
            WorkCodes<BITS> c;
#pragma unroll
            for (int k = 0; k < WPS; ++k) c.w[k] = cur[b][k];
            return tab[b].template eight<T4>(c);
        } else {
            CodeWords<BITS> c;
#pragma unroll
            for (int k = 0; k < WPS; ++k) c.w[k] = cur[b][k];
            return unslot_of<BITS>(eight_of<BITS, T4>(tab[b], c));
        }
    };
    auto rebuild = [&](int slot, auto t) { w[slot][0] = eight(0, t); w[slot][1] = eight(1, t); };
    const unsigned char *const tile = smem_raw + r * 512;
    auto read_x = [&](int t, int buf) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
            x[t][i] = *reinterpret_cast<const bf16x8 *>(tile + (uint32_t)buf * L::STEP + i * (32 * 512) + (((kg * 8 + h * 4 + t) ^ (r & 7)) * 16));
    };
    auto products = [&](int t) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int b = 0; b < 2; ++b)
                acc[b][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[t & 1][b], x[t][i], acc[b][i], 0, 0, 0);
    };
    // What a slice rebuilds from is not used before it, and what it rebuilds is there at its end; between the two one product, a few
    // LDS reads and a share of the arithmetic (`n` instructions) in turns.
    auto begin = [&]() {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
#pragma unroll
            for (int k = 0; k < WPS; ++k) asm volatile("" : "+v"(cur[b][k]));
            if constexpr (kShared) {
#pragma unroll
                for (int k = 0; k < 4; ++k) asm volatile("" : "+v"(lo[b][k]), "+v"(hi[b][k]));
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto weave = [&](auto n) {
#pragma unroll
        for (int q = 0; q < 2 * MI; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, decltype(n)::value / (2 * MI) + 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x004, 5, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto end = [&](int slot) { asm volatile("" : "+v"(w[slot][0]), "+v"(w[slot][1])); };
    constexpr int kRebuild = BITS == 2 ? (kShared ? 16 : 24) : BITS == 3 ? (kRelaid<SRC> ? 24 : 40) : 46;      // of one slice
    constexpr int kTables = BITS == 2 ? 26 : BITS == 3 ? 42 : 12, kLook = kShared ? 30 : 0;

    mask_last(0); aim();
    load_part(IC<0>{}, 0); load_part(IC<1>{}, 0);
    wait_all_and_barrier();
    mask_last(1); aim();
    load_part(IC<0>{}, 1); load_part(IC<1>{}, 1);
    read_raw(0);
    read_x(0, 0);
    build(); look_up(0);
    rebuild(0, IC<0>{});
    __builtin_amdgcn_sched_barrier(0);
    auto one_step = [&](int step, auto par) __attribute__((always_inline)) {
        constexpr int buf = decltype(par)::value;
        mask_last(step + 2);
        begin();
        read_x(1, buf); read_x(2, buf);
        products(0);
        rebuild(1, IC<1>{}); look_up(1);
        weave(IC<kRebuild + kLook + 10>{}); end(1);
        begin();
        read_x(3, buf);
        products(1);
        rebuild(0, IC<2>{});
        aim();
        weave(IC<kRebuild + 6>{}); end(0);
        wait_all_and_barrier();           // the next step is in LDS; everyone has this one's tokens in registers
        load_part(IC<0>{}, buf);
        begin();
        read_raw(buf ^ 1); read_x(0, buf ^ 1);
        products(2);
        rebuild(1, IC<3>{});
        weave(IC<kRebuild + 6>{}); end(1);
        load_part(IC<1>{}, buf);
        products(3);
        build(); look_up(0);
        rebuild(0, IC<0>{});
        weave(IC<kRebuild + kTables + kLook>{}); end(0);
    };
    for (int step = 0;;) {
        one_step(step, IC<0>{}); if (++step >= steps) break;
        one_step(step, IC<1>{}); if (++step >= steps) break;
    }
    wait_all_and_barrier();

    [[maybe_unused]] PairsShare pairs;
    if constexpr (SRC == kPrepared) pairs.read(a);
    store_sums<BM, L::TOTAL>(a, acc, smem_raw, m0, n0, wave, lane);
    if constexpr (SRC == kPrepared) pairs.write(a);
}

// ---- 128 tokens per tile -----------------------------------------------------------------------------------
// Four products per rebuilt fragment instead of two or three, so the matrix cores have less arithmetic to wait for (6.7
// instructions a product at 2 bit, 7 at 4; 7.1 and 9.5 with 96 tokens).  Two stages of 256-wide K steps would take 176 KB
// of LDS, so a step is 128 wide: a wave multiplies one segment of it, and the lanes h = 0 and 1 of a row take 16 of its codes
// each.  With the room that leaves, tokens are fetched two steps ahead (three stages), codes four; step sizes and zero points
// come four steps at a time, 16 bytes a lane.  A lane's byte offsets never change: the buffers move along K, which is scalar work
// (offsets per lane and load were 30 of 123 instructions a step).  Every wave issues the same number of loads a step, so
// the barrier waits for a count and not for the loads of the step after next.
// Measured, us, 1000 tokens, 4096 x 4096, from the packed arrays (128 x 128 tiles behind a re-layout / here): 2 bit 57 / 40, 3 bit
// 60 / 45, 4 bit 61 / 41; from the working layout 47 / 35, 48 / 36, 50 / 38.  What bounds it: 1940 cycles a step, of which the
// products need 1056, the arithmetic beside them 1290; without the loads of a step 1500.
constexpr int kTallBM = 128;
template <int BITS, int SRC> struct TallLds {
    static constexpr int WPS = kRelaid<SRC> ? WorkCodes<BITS>::kWords : BITS;
    static constexpr int NCH = WPS;
    static constexpr int ZW = SRC == kPackedZ && BITS == 3 ? 2 : 1;
    // tokens: three stages; codes: four, 1 KB per wave and its 16 rows; step sizes and zero points of four steps: two
    static constexpr uint32_t TOK = kTallBM * 128 * 2, CODES = 8 * 1024, SUPER = 16 * 1024;
    static constexpr uint32_t CODES_AT = 3 * TOK, SUPERS = CODES_AT + 4 * CODES, TOTAL = SUPERS + 2 * SUPER;
    static_assert(TOTAL <= 160 * 1024, "LDS of one CU");
};

template <int BITS, int SRC>
__global__ __launch_bounds__(kMidNT) void k_gemm_mid_tall(const MidArgs a)
{
    typedef TallLds<BITS, SRC> L;
    constexpr int BM = kTallBM, MI = BM / 32, WPS = L::WPS, NCH = L::NCH, BK = 128;
    constexpr int N = 1 + MI;                 // loads a wave issues per K step: codes, tokens
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave & 1, kg = wave >> 1, r = lane & 31, h = lane >> 5;

    int m0, n0;
    tile_of(a, BM, blockIdx.x, gridDim.x, m0, n0);

    const int steps = (a.I + BK - 1) / BK;
    const uint32_t lds0 = lds_addr_of(smem_raw);

    // ---- loads of one K step: every lane keeps one byte offset per instruction for good, the buffers move along (scalar work)
    uint32_t off[MI];
#pragma unroll
    for (int it = 0; it < MI; ++it) {
        const int row = (wave * MI + it) * 4 + (lane >> 4);
        off[it] = m0 + row < a.T ? ((uint32_t)(m0 + row) * (uint32_t)a.I + (uint32_t)(((lane & 15) ^ (row & 7)) * 8)) * 2u : kOobOffset;
    }
    const int crow = wave * 16 + lane / NCH;
    const uint32_t coff = lane < 16 * NCH ? (uint32_t)(n0 + crow) * a.code_row_bytes + (uint32_t)code_chunk_swz<NCH>(crow, lane % NCH) * 16u : kOobOffset;
    // Step sizes and zero points of four steps (a superstep) at a time, 16-byte chunks of a row's groups: 64 bytes a row of each,
    // (s, z) pairs 128, packed zero points 16 that hold them all.  Chunk c of a row sits at position c ^ (row / 2) (pairs: row).
    const int dshift = a.group == 32 ? 0 : a.group == 64 ? 1 : 2;          // segment of a step -> group of a step
    uint32_t soff[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        if constexpr (SRC == kWorking) {
            const int row = wave * 16 + e * 8 + (lane >> 3), c = (lane & 7) ^ (row & 7);
            soff[e] = c < (8 >> dshift) ? (uint32_t)(n0 + row) * (uint32_t)a.G * 8u + (uint32_t)c * 16u : kOobOffset;
        } else if (kTwoFloats<SRC> || e == 0) {
            const int row = wave * 16 + (lane >> 2), c = (lane & 3) ^ ((row >> 1) & 3);
            soff[e] = c < (4 >> dshift) ? (uint32_t)(n0 + row) * (uint32_t)a.G * 4u + (uint32_t)c * 16u : kOobOffset;
        } else {
            soff[e] = lane < 16 ? (uint32_t)(n0 + wave * 16 + lane) * a.z_row_words * 4u : kOobOffset;
        }
    }
    // number of the first group of a step, carried from step to step: a group ends every `per` steps, or 4 >> dshift end in one
    const int per = a.group > 128 ? a.group / 128 : 1, inc = 4 >> dshift;
    struct Group {
        int j, at;
        __device__ __forceinline__ void next(int per, int inc) { ++at; const bool wrap = at == per; j += wrap ? inc : 0; at = wrap ? 0 : at; }
    };
    auto load_super = [&](int step) {              // the superstep that begins with this step
        const bool live = step < steps;
        const uint32_t j = live ? (uint32_t)(a.group >= 128 ? step / per : step * inc) : 0u;
        const uint32_t to = lds0 + L::SUPERS + (uint32_t)((step >> 2) & 1) * L::SUPER;
        constexpr uint32_t SB = SRC == kWorking ? 8u : 4u;
        const RawRsrc rS = make_raw_rsrc((const char *)a.s + j * SB, live ? a.s_bytes - j * SB : 0u);
        if constexpr (SRC == kWorking) {
            load_to_lds16_at(rS, to + (uint32_t)(wave * 2048), soff[0]);
            load_to_lds16_at(rS, to + (uint32_t)(wave * 2048 + 1024), soff[1]);
        } else {
            load_to_lds16_at(rS, to + (uint32_t)(wave * 1024), soff[0]);
            const uint32_t zat = kTwoFloats<SRC> ? j * 4u : ((j * BITS) >> 5) * 4u;
            const RawRsrc rZ = make_raw_rsrc((kTwoFloats<SRC> ? (const char *)a.zf : (const char *)a.zp) + zat, live ? a.z_bytes - zat : 0u);
            load_to_lds16_at(rZ, to + 8192u + (uint32_t)(wave * 1024), soff[1]);
        }
    };
    Moving bX(a.X, a.x_bytes), bW(a.codes, a.codes_bytes);
    RawRsrc rX, rW;
    auto aim_x = [&](int step) { rX = bX.at(step < steps); bX.by(BK * 2); };            // the steps in order
    auto aim_codes = [&](int step) { rW = bW.at(step < steps); bW.by(NCH * 16); };
    // tokens past the end of the rows come as zeros; called in front of the loads of every step
    auto mask_last = [&](int step) {
        if (step == steps - 1 && a.I % BK != 0) {
#pragma unroll
            for (int it = 0; it < MI; ++it) {
                const int row = (wave * MI + it) * 4 + (lane >> 4);
                if (((lane & 15) ^ (row & 7)) * 8 >= a.I % BK) off[it] = kOobOffset;
            }
        }
    };
    auto load_codes = [&](int step) {
        load_to_lds16_at(rW, lds0 + L::CODES_AT + (uint32_t)(step & 3) * L::CODES + (uint32_t)(wave * 1024), coff);
    };
    constexpr int MH = (MI + 1) / 2;       // token loads issued in the last slice of the step before
    auto load_x = [&](int from, int to, uint32_t stage) {
#pragma unroll
        for (int it = 0; it < MI; ++it)
            if (it >= from && it < to) load_to_lds16_at(rX, lds0 + stage + (uint32_t)((wave * MI + it) * 1024), off[it]);
    };

    floatx16 acc[2][MI];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[b][i][q] = 0.0f;

    // A wave multiplies the segment kg of a step; the lanes h = 0 and 1 of a row take 16 of its codes each, eight per product.
    // Codes, step size and zero point of a step are read from LDS a slice before they are rebuilt.
    constexpr int HW = WPS == 2 ? 1 : 2;
    constexpr bool kShared = BITS == 2 && !kRelaid<SRC>;     // 2-bit codes as packed: the lookups of a word serve both products
    struct Raw { uint32_t c[2][HW], s[2], z[2][L::ZW], zshift, keep; };
    Raw raw;
    uint32_t cur[2][HW], lo[2][4], hi[2][4];
    WhatTable<BITS> tab[2];
    bf16x8 x[2][MI], w[2][2];
    Group gr{0, 0};                       // of the step that is read next
    int super_j = 0, seg_left = (a.I >> 5) - kg;       // first group of its superstep; segments from this wave's on to the end of the row
    auto read_raw = [&](int step) {       // the steps in order
        super_j = (step & 3) == 0 ? gr.j : super_j;
        const unsigned char *const sup = smem_raw + L::SUPERS + (uint32_t)((step >> 2) & 1) * L::SUPER;
        const unsigned char *const here = smem_raw + L::CODES_AT + (uint32_t)(step & 3) * L::CODES;
        const int slot = gr.j - super_j + (kg >> dshift);           // of the segment's group among those of the superstep
        const uint32_t zbit = (uint32_t)(gr.j + (kg >> dshift)) * BITS - (((uint32_t)super_j * BITS) & ~31u);
        const int row = wn * 64 + r;      // row + 32 lies a constant further on everywhere
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const unsigned char *const codes = here + b * 2048 + (row >> 4) * 1024 + (row & 15) * (NCH * 16);
            if constexpr (WPS == 2) {
                raw.c[b][0] = *reinterpret_cast<const uint32_t *>(codes + code_chunk_swz<NCH>(row, kg >> 1) * 16 + (kg & 1) * 8 + h * 4);
            } else if constexpr (WPS == 3) {
                const uint32_t *const v = reinterpret_cast<const uint32_t *>(codes + kg * 12 + h * 4);
                raw.c[b][0] = v[0]; raw.c[b][1] = v[1];
            } else {
                const uintx2 v = *reinterpret_cast<const uintx2 *>(codes + code_chunk_swz<NCH>(row, kg) * 16 + h * 8);
                raw.c[b][0] = v[0]; raw.c[b][1] = v[1];
            }
            if constexpr (SRC == kWorking) {
                const uintx2 v = *reinterpret_cast<const uintx2 *>(sup + b * 4096 + row * 128 + (((slot >> 1) ^ (row & 7)) * 16) + (slot & 1) * 8);
                raw.s[b] = v[0]; raw.z[b][0] = v[1];
            } else {
                const uint32_t at = (uint32_t)(b * 2048 + row * 64 + (((slot >> 2) ^ ((row >> 1) & 3)) * 16) + (slot & 3) * 4);
                raw.s[b] = *reinterpret_cast<const uint32_t *>(sup + at);
                if constexpr (kTwoFloats<SRC>) {
                    raw.z[b][0] = *reinterpret_cast<const uint32_t *>(sup + 8192 + at);
                } else {
                    const uint32_t *const p = reinterpret_cast<const uint32_t *>(sup + 8192 + b * 2048 + (row >> 4) * 1024 + (row & 15) * 16) + (zbit >> 5);
#pragma unroll
                    for (int k = 0; k < L::ZW; ++k) raw.z[b][k] = p[k];
                }
            }
        }
        raw.zshift = zbit & 31u;
        raw.keep = seg_left > 0 ? ~0u : 0u;
        seg_left -= 4;
        gr.next(per, inc);
    };
    auto build = [&]() {                  // from raw
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            // segments past the end of the rows: the step size and the zero point are what follows the row, the weights have to be zeros
            float z;
            if constexpr (SRC == kPackedZ) {
                const uint32_t v = L::ZW == 2 ? __builtin_amdgcn_alignbit(raw.z[b][L::ZW - 1], raw.z[b][0], raw.zshift) : raw.z[b][0] >> raw.zshift;
                z = (float)(v & ((1u << BITS) - 1u));
            } else {
                z = __uint_as_float(raw.z[b][0] & raw.keep);
            }
            tab[b].build(__uint_as_float(raw.s[b] & raw.keep), z);
            if constexpr (WPS == 3) {     // 16 codes are 48 bits: the second half of a segment starts in the middle of a word
                cur[b][0] = __builtin_amdgcn_alignbit(raw.c[b][1], raw.c[b][0], (uint32_t)h * 16u);
                cur[b][1] = raw.c[b][1] >> ((uint32_t)h * 16u);
            } else {
#pragma unroll
                for (int k = 0; k < HW; ++k) cur[b][k] = raw.c[b][k];
            }
        }
    };
    auto look_up = [&]() {                // bytes of the codes k, k + 4, k + 8 and k + 12
        if constexpr (kShared) {
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t c = (cur[b][0] >> (2 * k)) & 0x03030303u;
                    lo[b][k] = __builtin_amdgcn_perm(tab[b].lo[0], tab[b].lo[0], c);
                    hi[b][k] = __builtin_amdgcn_perm(tab[b].hi[0], tab[b].hi[0], c);
                }
        }
    };
    auto eight = [&](int b, auto t) -> bf16x8 {
        constexpr int T4 = decltype(t)::value;
        if constexpr (kShared) {
            uintx4 u;
#pragma unroll
            for (int k = 0; k < 4; ++k) u[k] = __builtin_amdgcn_perm(hi[b][k], lo[b][k], T4 ? 0x07030602u : 0x05010400u);
            return unslot_of<BITS>(__builtin_bit_cast(bf16x8, u));
        } else if constexpr (kRelaid<SRC>) {
            WorkCodes<BITS> c;
#pragma unroll
            for (int k = 0; k < HW; ++k) c.w[k] = cur[b][k];
            return tab[b].template eight<T4>(c);
        } else {
            CodeWords<BITS> c;
#pragma unroll
            for (int k = 0; k < HW; ++k) c.w[k] = cur[b][k];
            return unslot_of<BITS>(eight_of<BITS, T4>(tab[b], c));
        }
    };
    auto read_x = [&](int slot, const unsigned char *here, int t) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
            x[slot][i] = *reinterpret_cast<const bf16x8 *>(here + (i * 32 + r) * 256 + (((kg * 4 + h * 2 + t) ^ (r & 7)) * 16));
    };
    auto products = [&](int slot) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int b = 0; b < 2; ++b)
                acc[b][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[slot][b], x[slot][i], acc[b][i], 0, 0, 0);
    };
    auto weave = [&](auto valu) {
#pragma unroll
        for (int q = 0; q < 2 * MI; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, decltype(valu)::value, 0);
            __builtin_amdgcn_sched_group_barrier(0x004, 5, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // instructions of arithmetic in the two slices of a step
    constexpr int kV0 = (BITS == 2 ? (kShared ? 52 : 54) : BITS == 3 ? (kRelaid<SRC> ? 70 : 88) : 68) / (2 * MI) + 1;
    constexpr int kV1 = (BITS == 2 ? (kShared ? 60 : 44) : BITS == 3 ? (kRelaid<SRC> ? 48 : 60) : 60) / (2 * MI) + 1;
    auto wait_and_barrier = [&](auto left) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(decltype(left)::value));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    auto pin = [&]() {          // what the rebuild reads is not to be used before this point
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int k = 0; k < (kShared ? 4 : HW); ++k) {
                if constexpr (kShared) asm volatile("" : "+v"(lo[b][k]), "+v"(hi[b][k]));
                else asm volatile("" : "+v"(cur[b][k]));
            }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto keep = [&](int slot) {        // ... and what it yields is there by now
        asm volatile("" : "+v"(w[slot][0]), "+v"(w[slot][1]));
    };
    auto pin_tables = [&]() {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int k = 0; k < HW; ++k) asm volatile("" : "+v"(cur[b][k]));
    };

    load_super(0);
    aim_codes(0); load_codes(0); aim_codes(1); load_codes(1);
    mask_last(0); aim_x(0); load_x(0, MI, 0);
    aim_codes(2); load_codes(2);
    mask_last(1); aim_x(1); load_x(0, MI, L::TOK);
    aim_codes(3); load_codes(3);
    mask_last(2); aim_x(2); load_x(0, MH, 2 * L::TOK);
    wait_and_barrier(IC<N + 1 + MH>{});
    read_raw(0);
    read_x(0, smem_raw, 0);
    build(); look_up();
    w[0][0] = eight(0, IC<0>{}); w[0][1] = eight(1, IC<0>{});
    read_raw(1);
    __builtin_amdgcn_sched_barrier(0);
    auto one_step = [&](int step, auto stage) __attribute__((always_inline)) {
        constexpr uint32_t S0 = decltype(stage)::value * L::TOK, S1 = (decltype(stage)::value + 1) % 3 * L::TOK,
                           S2 = (decltype(stage)::value + 2) % 3 * L::TOK;
        load_x(MH, MI, S2);
        mask_last(step + 3);
        if ((step & 3) == 0) load_super(step + 4);
        pin();
        aim_x(step + 3); aim_codes(step + 4);
        read_x(1, smem_raw + S0, 1);
        products(0);
        w[1][0] = eight(0, IC<1>{}); w[1][1] = eight(1, IC<1>{});
        build();
        weave(IC<kV0>{});
        keep(1);
        pin_tables();
        wait_and_barrier(IC<N>{});
        load_codes(step + 4);
        load_x(0, MH, S0);
        __builtin_amdgcn_sched_barrier(0);
        read_raw(step + 2);
        read_x(0, smem_raw + S1, 0);
        products(1);
        look_up();
        w[0][0] = eight(0, IC<0>{}); w[0][1] = eight(1, IC<0>{});
        weave(IC<kV1>{});
        keep(0);
    };
    for (int step = 0;;) {
        one_step(step, IC<0>{}); if (++step >= steps) break;
        one_step(step, IC<1>{}); if (++step >= steps) break;
        one_step(step, IC<2>{}); if (++step >= steps) break;
    }
    wait_and_barrier(IC<0>{});

    [[maybe_unused]] PairsShare pairs;
    if constexpr (SRC == kPrepared) pairs.read(a);
    store_sums<BM, L::TOTAL>(a, acc, smem_raw, m0, n0, wave, lane);
    if constexpr (SRC == kPrepared) pairs.write(a);
}

template <int BITS, int SRC, int BM> void launch_t(MidArgs a, hipStream_t st)
{
    int smem;
    void (*kern)(MidArgs);
    if constexpr (BM == kTallBM) { kern = k_gemm_mid_tall<BITS, SRC>; smem = (int)TallLds<BITS, SRC>::TOTAL; }
    else { kern = k_gemm_mid<BITS, SRC, BM>; smem = (int)MidLds<BITS, SRC, BM>::TOTAL; }
    static std::atomic<uint64_t> allowed{0};          // more dynamic LDS than the default limit: once per device
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev > 63) dev = 0;
    if (!((allowed.load(std::memory_order_relaxed) >> dev) & 1u)) {
        (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
        allowed.fetch_or((uint64_t)1 << dev, std::memory_order_relaxed);
    }
    a.tiles_m = (a.T + BM - 1) / BM;
    a.tiles_n = (a.O + kMidBN - 1) / kMidBN;
    a.band = band_of(a.tiles_m, BM);
    kern<<<dim3((unsigned)(a.tiles_m * a.tiles_n)), dim3(kMidNT), smem, st>>>(a);
}

// What a launch with token tiles of `bm` takes, in us: rounds of workgroups (one per compute unit), each 6 us and 1.2 (64
// tokens), 1.45 (96) or 1.95 (128) us per 256-wide K step: an upper figure for the first two, which have become faster since
// (1.08 and 1.4 at 192 workgroups), so that the lines to the other kernels stay where both sides were measured.
int64_t rounds_of(const Problem &p, int bm) { return (((p.T + bm - 1) / bm) * ((p.O + kMidBN - 1) / kMidBN) + 255) / 256; }
double launch_us(const Problem &p, int bm)
{
    return (double)rounds_of(p, bm) * (6.0 + (double)((p.I + kMidBK - 1) / kMidBK) * (bm == 64 ? 1.2 : bm == 96 ? 1.45 : 1.95));
}

// The tall kernel finds the groups of a 128-wide step by counting: groups of 32 or 64, or whole steps.  One round only: in two
// the 96-token tiles (or the tile kernels) are faster (2000 tokens, 4096 x 4096, 2 bit: 82 us, the tile kernel 75).
bool tall_applies(const Problem &p) { return (p.g == 32 || p.g == 64 || p.g % 128 == 0) && rounds_of(p, 128) == 1; }

int token_tile(const Problem &p)
{
    const int low = launch_us(p, 96) < launch_us(p, 64) ? 96 : 64;
    return tall_applies(p) && launch_us(p, 128) < launch_us(p, low) ? 128 : low;
}

template <int SRC> void launch_src(const Problem &p, const MidArgs &a, hipStream_t st)
{
    const int bm = token_tile(p);
#define EQAT_MID(B) do { if (bm == 128) launch_t<B, SRC, 128>(a, st); else if (bm == 96) launch_t<B, SRC, 96>(a, st); else launch_t<B, SRC, 64>(a, st); } while (0)
    if (p.bits == 2) EQAT_MID(2); else if (p.bits == 3) EQAT_MID(3); else EQAT_MID(4);
#undef EQAT_MID
}

MidArgs mid_args(const Problem &p, const void *X, const void *codes, const void *s, void *Y)
{
    MidArgs a{};
    a.X = (const bf16_t *)X; a.codes = (const uint32_t *)codes; a.s = (const float *)s; a.Y = (bf16_t *)Y;
    a.T = (int)p.T; a.I = (int)p.I; a.O = (int)p.O; a.G = (int)p.G; a.group = (int)p.g;
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

double mid_us(const Problem &p) { return launch_us(p, token_tile(p)); }

// The small launch that pairs step sizes and zero points takes 2 us beside the forward.  Without it the forward fetches twice the cache lines of them a K step, with groups of 64 and
// more: 200 random sizes of 256 to 16000 inputs, 65 to 2000 tokens, us, with that launch / without:
// - one group to a row: 288 -> 544 8.6 / 6.6, 7360 -> 1144 38.1 / 36.1, 14624 -> 1880 91.5 / 89.7; with the backward, 14880 -> 1408 193.9 / 191.9;
// - groups of 32: 8160 -> 1856 54.8 / 46.7, 13856 -> 3640 97.8 / 95.2.  A forward that leaves many pairs for few workgroups to write loses, though: with the backward 4928 -> 7368
//   107.5 / 104.3, 14016 -> 1272, 82 tokens 117.9 / 126.4;
// - others gain up to 24 steps of 256 inputs, counted over the rounds of workgroups: 3200 -> 2360 19.4 / 17.7, 4992 -> 4096 37.5 / 36.1, 6592 -> 208 32.0 / 32.4, 9216 -> 1096 40.5 / 41.2, 14464 -> 544
//   70.2 / 77.9; two rounds, 7424 -> 3672 with the backward 218.6 / 222.3.
bool mid_pairs_itself(const Problem &p, bool keep)
{
    if (mid_us(p) > 120.0) return false;
    return p.G == 1 || (p.g == 32 && !keep) || rounds_of(p, token_tile(p)) * ((p.I + kMidBK - 1) / kMidBK) <= 24;
}

// Against k_gemm_ksplit while there are at most 256 tiles of 128 x 128 (with one workgroup per tile 4.8 us and 0.8 to 1.1, with
// the fill, a pair of 64-wide K tiles; 1024 inputs, 2000 tokens, 2048 rows: 12 us there, 14 here).  With more than 640 inputs one
// round of 64- or 96-token tiles runs here whatever these estimates say.  Where the contraction is short they leave out what a
// launch there costs beside its K tiles: us, here / there, from the packed arrays 443 tokens, 832 x 552 10.1 / 15.2, from a prepared
// layer 109 tokens, 896 x 1680 12.0 / 14.3, and in all of 64 sizes between 672 and 1280 inputs by 1 to 80 %.  Where it is long
// and the tiles are few, several workgroups share a tile there, which this rule does not weigh: from the packed arrays / prepared,
// 128 tokens, 28672 x 8192 121 here and 127 there / 113 and 106; 256 tokens, 11008 x 4096 49 and 51 / 48 and 46; 256 tokens, 8192 x 1024
// 36 and 31 / 35 and 27.
// Against the 128 x 128-tile kernel with two tiles per compute unit beyond 256 tiles (0.9 us per K tile; 11008 x 4096: 288 tokens,
// 258 tiles 61 us there and 42 here; 400 tokens 63 and 51).  More than two rounds here, or more than two tiles per compute unit there: the 256 x 256 tiles are the better kernel.  The GEMMs
// alone are compared: a forward from the packed arrays saves the re-layout as well and would gain a little earlier, but every
// forward entry point shares the rule, so that their results stay bitwise equal.
bool mid_applies(const Problem &p)
{
    if (!p.act_bf16 || !group_by_magic(p) || p.T <= 32) return false;
    if (p.T <= 64) return !gemv_work_applies(p);
    const int64_t tiles = ((p.T + 127) / 128) * ((p.O + 127) / 128);
    const int bm = token_tile(p);
    if (tiles <= 256 && p.I > 640 && bm < 128 && rounds_of(p, bm) == 1) return true;
    const double other = tiles <= 256 ? 4.8 + (double)((p.I + 127) / 128) * (0.8 + 0.3 * (double)tiles / 256.0)
                                      : 4.0 + (double)((p.I + 63) / 64) * 0.9;
    return tiles <= 512 && mid_us(p) < other;
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

void launch_mid_prepared(const Problem &p, const void *X, const void *codes, const float *s, const float *z, void *pairs, void *Y, hipStream_t st)
{
    MidArgs a = mid_args(p, X, codes, s, Y);
    a.zf = z;
    a.code_row_bytes = (uint32_t)(work_code_bytes(p) / p.O);
    a.codes_bytes = (uint32_t)work_code_bytes(p);
    a.s_bytes = a.z_bytes = (uint32_t)(p.O * p.G * 4);
    a.pairs = (float *)pairs;
    launch_src<kPrepared>(p, a, st);
}

}  // namespace eqat
