// dX for few output tiles (short training batches): dX[T,I] = dY[T,O] * What[O,I].
//
// The forward's kernel for these sizes (gemm_mid.hip) with the weights turned round: eight waves are 2 (64 in-features each) x 4 (a
// quarter of every 128-wide step along O each), a wave owns its weights alone, tokens come two steps ahead straight into LDS (three
// stages) and the barrier of a step, in its middle, waits for a count and not for the loads of the steps to come.
// The contraction runs along O, the codes and the groups along I: a lane rebuilds one 32-code segment per step, with the step size of its own
// row o, and what it holds then are 32 columns of one k.  MFMA operands want eight k of one column, so the 32 x 64 weights of a wave and
// step pass through a patch of LDS of the wave's own (4 KB, [k][64 columns], 16-byte stores) and come back by transpose reads; LDS accesses
// of a wave complete in order, so the patch needs no barrier and, as both slices' fragments are in registers before the next step is stored, no
// second copy.  Codes and (s, zbar) pairs are the wave's own as well: every lane fetches what it will read.
// What bounds it: at 128 tokens a step is 1056 cycles of products per SIMD beside 530 (2 bit) to 1060 (4 bit) of rebuild and some 1100 of LDS traffic
// (32 KB of tokens in and 64 out, 32 KB of weights in and out), and takes 2100 to 2500; without its loads 1600 to 2050, without the rebuild as well 1050.
// So the loads of a step are spread over it (all behind the barrier: 87 us where 81 are taken, 515 tokens, 11008 -> 4096, 3 bit), and what touches many
// cache lines is fetched in as few instructions as possible (pairs in two 4-byte loads a lane: 120 -> 113, 1000 tokens, 4 bit, g = 128).
// Measured, us, k_gemm_ksplit / here (operands cold): 4096 -> 4096, 515 tokens, 3 bit 37.7 / 31.8, 11008 -> 4096 99 / 74; 11008 -> 4096, 1000 tokens,
// 4 bit 128 / 107; 128 x 128 tiles of k_gemm_q / here: 891 tokens, 3816 -> 5632, 4 bit 88 / 65.
#pragma once
#include "common.h"
#include "kernels.h"
#include "mid_tiles.h"

namespace eqat {

template <int BITS, int BM> struct DxLds {
    static constexpr uint32_t TOK = BM * 128 * 2, PATCH = 4096, CODES = 1024, SZ = 1024;
    static constexpr uint32_t PATCHES_AT = 3 * TOK, RAW_AT = PATCHES_AT + 8 * PATCH;
    // stages of codes and pairs, two steps ahead of what is rebuilt or, with room, three
    static constexpr int NC = RAW_AT + 3 * 8 * (CODES + SZ) <= 160 * 1024 ? 3 : 2;
    static constexpr uint32_t SUMS = 8 * BM * 32 * 4, LOOP = RAW_AT + NC * 8 * (CODES + SZ), TOTAL = LOOP > SUMS ? LOOP : SUMS;
    static_assert(TOTAL <= 160 * 1024, "LDS of one CU");
};

// Row k of a patch has eight 16-byte chunks of columns; chunk c sits at c ^ patch_swz(k): the rows that a store or a transpose read serves
// together lie on different banks.
__device__ __forceinline__ int patch_swz(int k) { return ((k >> 1) & 1) * 4 + ((k ^ (k >> 3)) & 1) * 2 + ((k >> 2) & 1); }

// As Moving, in 32-bit steps: the 64-bit sum of two buffers more lands in vector registers, and with it the descriptors.
struct Moving32 {
    uint32_t lo, hi, left;
    __device__ __forceinline__ Moving32(const void *p, uint32_t bytes) : lo((uint32_t)(uint64_t)p), hi((uint32_t)((uint64_t)p >> 32) & 0xFFFFu), left(bytes) {}
    __device__ __forceinline__ void by(uint32_t n)
    {
        const uint64_t to = (uint64_t)lo + n;
        lo = __builtin_amdgcn_readfirstlane((uint32_t)to);
        hi = __builtin_amdgcn_readfirstlane(hi + (uint32_t)(to >> 32)); left -= n;
    }
    __device__ __forceinline__ RawRsrc at(bool live) const
    {
        RawRsrc r;
        r.w[0] = (int)lo; r.w[1] = (int)hi; r.w[2] = live ? (int)left : 0; r.w[3] = 0x00020000;
        return r;
    }
};

// (bid, grid): this workgroup's number among those of dX, which may share its launch with another GEMM
template <int BITS, int BM>
__device__ __forceinline__ void mid_dx_body(const MidArgs &a, const uint32_t bid, const uint32_t grid)
{
    typedef DxLds<BITS, BM> L;
    constexpr int MI = BM / 32, BK = 128, NC = L::NC, WPS = WorkCodes<BITS>::kWords;
    constexpr int C_LOADS = 2, N = C_LOADS + MI;          // loads a wave issues per step: codes, pairs; tokens
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave & 1, kg = wave >> 1, r = lane & 31, h = lane >> 5;

    int m0, n0;
    tile_of(a, BM, bid, grid, m0, n0);

    const int steps = (a.I + BK - 1) / BK;
    const uint32_t lds0 = lds_addr_of(smem_raw);

    // ---- loads of one step: every lane keeps its byte offsets, the buffers move along K (scalar work)
    uint32_t off[MI];
#pragma unroll
    for (int it = 0; it < MI; ++it) {
        const int row = (wave * MI + it) * 4 + (lane >> 4);
        off[it] = m0 + row < a.T ? ((uint32_t)(m0 + row) * (uint32_t)a.I + (uint32_t)(((lane & 15) ^ (row & 15)) * 8)) * 2u : kOobOffset;
    }
    // this lane's row o (of the 32 of its wave and step) and segment; rows past O are out of range (zeros: weights of exactly zero), segments past
    // the end of a row are those of the next, and their columns are never stored
    const uint32_t seg = (uint32_t)(n0 >> 5) + 2u * wn + h;
    const uint32_t coff = WPS == 2 ? h ? kOobOffset : (uint32_t)(kg * 32 + r) * a.code_row_bytes + (seg - h) * 8u            // both segments of row `lane`, from lanes 0 .. 31
                                   : (uint32_t)(kg * 32 + r) * a.code_row_bytes + seg * 16u;
    // (s, zbar) of the groups of both segments, side by side if they are two: 16 bytes of row `lane`, from lanes 0 .. 31
    const uint32_t grp0 = (seg - h) * 32u / (uint32_t)a.group, at_pair = (uint32_t)(r * 16) + (seg * 32u / (uint32_t)a.group - grp0) * 8u;
    const uint32_t soff = h ? kOobOffset : ((uint32_t)(kg * 32 + r) * (uint32_t)a.G + grp0) * 8u;
    Moving32 bX(a.X, a.x_bytes), bW(a.codes, a.codes_bytes), bS(a.s, a.s_bytes);
    RawRsrc rX, rW, rS;
    // the steps in order, with counters of their own: a step number that lanes compute with ends up in a vector register, and with it the descriptors
    int x_left = steps, codes_left = steps;
    auto aim_x = [&]() { rX = bX.at(x_left-- > 0); bX.by(BK * 2); };
    auto aim_codes = [&]() {
        const bool live = codes_left-- > 0;
        rW = bW.at(live); bW.by(BK * a.code_row_bytes);
        rS = bS.at(live); bS.by(BK * 8u * (uint32_t)a.G);
    };
    // tokens past the end of the rows come as zeros; called in front of the loads of every step
    auto mask_last = [&](int step) {
        if (step == steps - 1 && a.I % BK != 0) {
#pragma unroll
            for (int it = 0; it < MI; ++it) {
                const int row = (wave * MI + it) * 4 + (lane >> 4);
                if (((lane & 15) ^ (row & 15)) * 8 >= a.I % BK) off[it] = kOobOffset;
            }
        }
    };
    auto raw_at = [&](int slot) { return L::RAW_AT + (uint32_t)((slot * 8 + wave) * (int)(L::CODES + L::SZ)); };
    auto load_codes = [&](int slot) {
        const uint32_t to = __builtin_amdgcn_readfirstlane(lds0 + raw_at(slot));
        load_to_lds16_at(rW, to, coff);
        load_to_lds16_at(rS, to + L::CODES, soff);
    };
    // a step's token loads, in four parts (see one_step)
    constexpr int X1 = MI >= 2 ? 1 : MI, X2 = MI >= 3 ? 2 : X1, X3 = MI >= 4 ? 3 : X2 + (MI == 2 ? 1 : MI - X2);
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

    // ---- codes -> patch
    WorkCodes<BITS> raw, cur;
    float raw_s, raw_z;
    WhatTable<BITS> tab;
    auto read_raw = [&](int slot) {
        const unsigned char *const here = smem_raw + raw_at(slot);
        if constexpr (WPS == 2) {
            const uintx2 v = *reinterpret_cast<const uintx2 *>(here + r * 16 + h * 8);
            raw.w[0] = v[0]; raw.w[1] = v[1];
        } else {
            const uintx4 v = *reinterpret_cast<const uintx4 *>(here + lane * 16);
            raw.w[0] = v[0]; raw.w[1] = v[1]; raw.w[2] = v[2]; raw.w[3] = v[3];
        }
        const floatx2 pair = *reinterpret_cast<const floatx2 *>(here + L::CODES + at_pair);
        raw_s = pair[0]; raw_z = pair[1];
    };
    auto build = [&]() {
        tab.build(raw_s, raw_z);
        cur = raw;
    };
    auto pin = [&]() {
        if constexpr (BITS <= 3) asm volatile("" : "+v"(tab.lo[0]), "+v"(tab.hi[0]));
        else asm volatile("" : "+v"(tab.b));
#pragma unroll
        for (int k = 0; k < WPS; ++k) asm volatile("" : "+v"(cur.w[k]));
    };
    unsigned char *const patch = smem_raw + L::PATCHES_AT + wave * L::PATCH;
    unsigned char *put[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) put[q] = patch + r * 128 + (((h * 4 + q) ^ patch_swz(r)) * 16);
    auto store_piece = [&](auto piece) {
        constexpr int Q = decltype(piece)::value;
        *reinterpret_cast<bf16x8 *>(put[Q]) = tab.template eight<Q>(cur);
    };
    // block b (32 columns), slice t (16 k): two transpose reads of four k each
    typedef short4v __attribute__((address_space(3))) * lds_p;
    const unsigned char *get[2][2];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int i = lane & 15, blk = lane >> 4, k = (blk >> 1) * 8 + (i >> 2) + 4 * e, col = b * 32 + (blk & 1) * 16 + (i & 3) * 4;
            get[b][e] = patch + k * 128 + (((col >> 3) ^ patch_swz(k)) * 16) + (col & 7) * 2;
        }
    bf16x8 x[2][MI], w[2][2];
    auto read_w = [&](auto slice) {
        constexpr int t = decltype(slice)::value;         // patch_swz(k + 16) = patch_swz(k)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(get[b][0] + t * 2048));
            const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(get[b][1] + t * 2048));
            typedef short short8v __attribute__((ext_vector_type(8)));
            short8v v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            w[t][b] = __builtin_bit_cast(bf16x8, v);
        }
    };
    auto read_x = [&](int slot, const unsigned char *here, int t) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
            x[slot][i] = *reinterpret_cast<const bf16x8 *>(here + (i * 32 + r) * 256 + (((kg * 4 + t * 2 + h) ^ (r & 15)) * 16));
    };
    // the products of half the token blocks
    constexpr int MH = (MI + 1) / 2;
    auto products = [&](int slot, auto half) {
        constexpr int H = decltype(half)::value;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int b = 0; b < 2; ++b)
                if ((i < MH) == (H == 0)) acc[b][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[slot][b], x[slot][i], acc[b][i], 0, 0, 0);
    };
    // reads and writes of the patch keep their order
    auto in_order = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_wave_barrier();
    };
    // `n` products, between them their share of LDS reads, arithmetic and stores
    auto weave = [&](auto n, auto reads, auto valu, auto writes) {
        constexpr int NP = decltype(n)::value;
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, (decltype(reads)::value + NP - 1) / NP, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, decltype(valu)::value / NP + 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x200, (decltype(writes)::value + NP - 1) / NP, 0);
            __builtin_amdgcn_sched_group_barrier(0x004, 6, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // `stores`: LDS operations (of a wave they complete in order) that may still be under way: the pieces just stored, in a patch that nobody else reads
    auto wait_and_barrier = [&](auto left, auto stores) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(decltype(left)::value) | decltype(stores)::value << 8);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr int kEight = BITS == 4 ? 24 : 10, kBuild = BITS == 2 ? 14 : BITS == 3 ? 22 : 4;

    // Order of the loads: codes c0 c1, tokens x0 (three stages of codes: c2), x1; then per step, behind its barrier the first X2 loads of the tokens
    // three steps on, at its end the codes NC steps after those just read, in front of the next barrier the rest of those tokens.  What the
    // barrier of step s waits for ends with the last of the tokens s + 1; the N loads behind them may be under way.
    aim_codes(); load_codes(0);
    aim_codes(); load_codes(1);
    mask_last(0); aim_x(); load_x(0, MI, 0);
    if constexpr (NC == 3) { aim_codes(); load_codes(2); }
    mask_last(1); aim_x(); load_x(0, MI, L::TOK);
    wait_and_barrier(IC<(NC - 2) * C_LOADS + MI>{}, IC<0>{});
    read_raw(0);
    build();
    __builtin_amdgcn_s_waitcnt(0xC07F);               // lgkmcnt(0): stage 0 has been read
    aim_codes(); load_codes(0);
    mask_last(2); aim_x(); load_x(0, X2, 2 * L::TOK);
    store_piece(IC<0>{}); store_piece(IC<1>{}); store_piece(IC<2>{}); store_piece(IC<3>{});
    in_order();
    read_w(IC<0>{});
    read_raw(1);
    read_x(0, smem_raw, 0);
    build();
    __builtin_amdgcn_s_waitcnt(0xC07F);
    aim_codes(); load_codes(1);
    __builtin_amdgcn_sched_barrier(0);
    int slot = 2 % NC;                                // of the codes that are read next
    // A wave's loads are spread over the step: eight waves that issue all of theirs behind the barrier wait for each other.
    auto one_step = [&](int step, auto stage) __attribute__((always_inline)) {
        constexpr uint32_t S0 = decltype(stage)::value * L::TOK, S1 = (decltype(stage)::value + 1) % 3 * L::TOK, S2 = (decltype(stage)::value + 2) % 3 * L::TOK;
        // first slice; the second one's fragments are read, then three quarters of the next step's weights go where they were
        load_x(X2, X3, S2);
        __builtin_amdgcn_sched_barrier(0);
        read_w(IC<1>{});
        read_x(1, smem_raw + S0, 1);
        in_order();
        products(0, IC<0>{});
        store_piece(IC<0>{});
        weave(IC<2 * MH>{}, IC<4 + MI>{}, IC<kEight>{}, IC<1>{});
        load_x(X3, MI, S2);
        __builtin_amdgcn_sched_barrier(0);
        products(0, IC<1>{});
        store_piece(IC<1>{}); store_piece(IC<2>{});
        aim_x(); aim_codes();
        weave(IC<2 * (MI - MH)>{}, IC<0>{}, IC<2 * kEight>{}, IC<2>{});
        mask_last(step + 3);
        wait_and_barrier(IC<N>{}, IC<3>{});           // tokens of the next step, codes of the one after; everyone has read stage S0
        load_x(0, X1, S0);
        __builtin_amdgcn_sched_barrier(0);
        read_raw(slot);
        products(1, IC<0>{});
        store_piece(IC<3>{});
        weave(IC<2 * MH>{}, IC<3>{}, IC<kEight>{}, IC<1>{});
        load_x(X1, X2, S0);
        __builtin_amdgcn_sched_barrier(0);
        in_order();
        read_w(IC<0>{});
        read_x(0, smem_raw + S1, 0);
        products(1, IC<1>{});
        build();
        weave(IC<2 * (MI - MH)>{}, IC<4 + MI>{}, IC<kBuild>{}, IC<0>{});
        pin();                                        // what build() makes of them is there: the codes have been read
        load_codes(slot);
        __builtin_amdgcn_sched_barrier(0);
        slot = slot + 1 == NC ? 0 : slot + 1;
    };
    for (int step = 0;;) {
        one_step(step, IC<0>{}); if (++step >= steps) break;
        one_step(step, IC<1>{}); if (++step >= steps) break;
        one_step(step, IC<2>{}); if (++step >= steps) break;
    }
    wait_and_barrier(IC<0>{}, IC<0>{});

    store_sums<BM, L::TOTAL>(a, acc, smem_raw, m0, n0, wave, lane);
}

MidArgs mid_dx_args(const Problem &p, int tokens, const void *dY, const void *codes, const void *sz, void *dX);       // tiles of `tokens` tokens

}  // namespace eqat
