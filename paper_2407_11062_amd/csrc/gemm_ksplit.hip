// fwd / dX with at most as many 128 x 128 output tiles as the chip has compute units: C[M,N] = A[M,K] * What (see k_gemm_q).
//
// The tile kernel gives such a launch one workgroup of four waves per compute unit, one wave per SIMD: 0.55 us per 64-wide K
// tile however few tokens there are (64 to 1000 tokens, 11008 x 4096: dX 97 us).  Here a workgroup is two groups of four
// waves, each with LDS tiles of its own, that take the K tiles in turns; their sums meet in LDS at the end.  So every SIMD
// has two waves to switch between and a pair of K tiles takes 0.75 us (few workgroups) to 1.1 (256, the clock gives way).  And a
// tile may be shared by up to four workgroups, a stretch of K each, where there are that many to spare: all write their sums,
// the last to arrive adds them up in order (nobody waits for anybody).
// Activations come two K tiles ahead straight into LDS, codes three ahead into registers; the rebuild of the next K tile and
// the fragment reads of the next slice are spread between the products of a slice.
// Measured, dX, us, tile kernel / here: 11008 -> 4096, 256 tokens: 2 bit 96 / 38, 4 bit 103 / 39; 4096 -> 4096: 256 tokens 36 / 23
// and 38 / 24, 1000 tokens 42 / 40 and 46 / 44; 5504 -> 2048: 515 tokens 52 / 29 (the same call again and again, operands in the last
// cache; the costs below and those of ksplit_parts come from such calls as well.  Among the other launches of a training pass 1000
// tokens, 4096 -> 4096, 4 bit took 58; dX comes here only where k_gemm_mid_dx is not faster).  What bounds it: a pair of K tiles is 1024
// cycles of products beside 192 KB of LDS traffic (1536 cycles); the parts, written through to memory, cost 3 us and 0.045 each.
#include "common.h"
#include "gemm_tiles.h"
#include "kernels.h"

#include <algorithm>
#include <atomic>

namespace eqat {

namespace {

constexpr int kKsBM = 128, kKsBN = 128, kKsBK = 64, kKsNT = 512;      // per K group and K tile; threads of both groups
constexpr int kKsMaxParts = 4;                                        // workgroups per tile: the last one has all their parts in flight
constexpr size_t kKsPartBytes = (size_t)kKsBM * kKsBN * sizeof(float);


struct KsArgs {
    const bf16_t *A; const uint32_t *codes; const floatx2 *sz; bf16_t *C; float *parts; uint32_t *counters;
    int M, N, K, I, G;
    uint32_t spg_magic;
    uint32_t a_bytes, codes_bytes, sz_bytes, c_bytes;
    int tiles_m, tiles_n, parts_per_tile, pairs;       // pairs of K tiles, one for each group
};

template <bool BT> constexpr int ks_ldb() { return BT ? kKsBN + kPadKM : kKsBK + kPadKC; }
template <bool BT> constexpr uint32_t ks_group_bytes()
{
    return 2u * (uint32_t)(kKsBM * kKsBK + (BT ? kKsBK * ks_ldb<BT>() : kKsBN * ks_ldb<BT>())) * 2u;
}

// The 32 x 64 outputs of a wave (lane order of the 32 x 32 MFMA) through its 2 KB patch of LDS, 64 bytes of a row from four lanes.
__device__ __forceinline__ void ks_store(const floatx16 (&v)[2], unsigned char *stg, const __amdgpu_buffer_rsrc_t &rC, int m0, int n0, int M, int N, int lane)
{
    bf16_t *const cell = reinterpret_cast<bf16_t *>(stg) + (lane >> 5) * (4 * 32) + (lane & 31);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
#pragma unroll
        for (int r = 0; r < 16; ++r) cell[(8 * (r >> 2) + (r & 3)) * 32] = (bf16_t)v[j][r];
        asm volatile("" ::: "memory");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const intx4 w = *reinterpret_cast<const intx4 *>(stg + k * 1024 + lane * 16);
            const int m = m0 + k * 16 + (lane >> 2), n = n0 + j * 32 + (lane & 3) * 8;
            __builtin_amdgcn_raw_buffer_store_b128(w, rC, (m < M && n < N) ? (int)(((uint32_t)m * (uint32_t)N + (uint32_t)n) * 2u) : (int)kOobOffset, 0, 0);
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_wave_barrier();
    }
}

// What workgroup `bid` of `nb` computes: a stretch of K-tile pairs of one tile.  Every XCD gets a contiguous range of (part, tile)
// numbers, tiles in bands of four tile rows.
struct KsItem { int number, tile, part, tm, tn, first_pair, pairs; };
__host__ __device__ __forceinline__ KsItem ks_item(int bid, int nb, int tiles_m, int tiles_n, int parts, int pairs)
{
    KsItem it;
    const int xcd = bid & 7, rem = nb & 7, ntiles = tiles_m * tiles_n;
    it.number = xcd * (nb >> 3) + (xcd < rem ? xcd : rem) + (bid >> 3);
    it.part = it.number / ntiles;
    it.tile = it.number - it.part * ntiles;
    constexpr int band_rows = 4;
    const int width = band_rows * tiles_n, band = it.tile / width, first = band * band_rows;
    const int rows = tiles_m - first < band_rows ? tiles_m - first : band_rows, in = it.tile - band * width;
    it.tm = first + in % rows;
    it.tn = in / rows;
    const int base = pairs / parts, extra = pairs % parts;
    it.first_pair = it.part * base + (it.part < extra ? it.part : extra);
    it.pairs = base + (it.part < extra ? 1 : 0);
    return it;
}

template <int BITS, bool BT>
__global__ __launch_bounds__(kKsNT) void k_gemm_ksplit(const KsArgs a)
{
    constexpr int LDB = ks_ldb<BT>(), A_ELEMS = kKsBM * kKsBK, B_ELEMS = BT ? kKsBK * LDB : kKsBN * LDB;
    constexpr int SEGB = 4 * WorkCodes<BITS>::kWords;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave >> 2, w4 = wave & 3, wm = w4 >> 1, wn = w4 & 1, gt = tid & 255;
    bf16_t *const sA = reinterpret_cast<bf16_t *>(smem_raw + (uint32_t)kg * ks_group_bytes<BT>());
    bf16_t *const sB = sA + 2 * A_ELEMS;

    const KsItem item = ks_item((int)blockIdx.x, (int)gridDim.x, a.tiles_m, a.tiles_n, a.parts_per_tile, a.pairs);
    const int pid = item.number, ntiles = a.tiles_m * a.tiles_n, tile = item.tile;
    const int m0 = item.tm * kKsBM, n0 = item.tn * kKsBN, n = item.pairs;
    const int k_first = (2 * item.first_pair + kg) * kKsBK;

    const __amdgpu_buffer_rsrc_t rCodes = make_rsrc(a.codes, a.codes_bytes);
    const __amdgpu_buffer_rsrc_t rS = make_rsrc(a.sz, a.sz_bytes);

    // activations
    const uint32_t ldsA = lds_addr_of(sA);
    uint32_t offA[4];
    int kA[4];
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int row = (w4 * 4 + it) * 8 + (lane >> 3);
        kA[it] = kc_swz(row, lane & 7) * 8;
        offA[it] = m0 + row < a.M ? ((uint32_t)(m0 + row) * (uint32_t)a.K + (uint32_t)kA[it]) * 2u : kOobOffset;
    }
    RawRsrc rA;
    // aims rA at K tile t of this group; past the last one nothing is in range (zeros)
    auto aim_a = [&](int t) {
        const int k0 = __builtin_amdgcn_readfirstlane(k_first + t * 2 * kKsBK);
        const bool live = t < n && k0 < a.K;
        rA = make_raw_rsrc(a.A + (live ? k0 : 0), live ? a.a_bytes - (uint32_t)k0 * 2u : 0u);
    };
    // in the tile that K ends in, what lies past the end comes as zeros; called in front of its loads
    auto mask_a = [&](int t) {
        const int k0 = k_first + t * 2 * kKsBK;
        if (t < n && k0 < a.K && k0 + kKsBK > a.K) {
#pragma unroll
            for (int it = 0; it < 4; ++it) offA[it] = k0 + kA[it] < a.K ? offA[it] : kOobOffset;
        }
    };
    auto load_a = [&](int it, int buf) {
        load_to_lds16_at(rA, ldsA + (uint32_t)((buf * A_ELEMS + (w4 * 4 + it) * 8 * 64) * 2), offA[it]);
    };
    // codes and (s, z) pairs: a thread owns one 32-code segment of its group's weight tile; past K, and past the last column, step
    // size and zero point come as zeros and the weights are exactly zero
    const uint32_t code_row_bytes = (uint32_t)a.I / 32u * SEGB;
    const int b_r = BT ? gt >> 2 : gt >> 1, b_s = BT ? gt & 3 : gt & 1;         // row and segment inside the weight tile
    uint32_t offC, offS, seg;
    if constexpr (BT) {
        seg = (uint32_t)(n0 >> 5) + b_s;
        const uint32_t grp = a.spg_magic ? __umulhi(seg, a.spg_magic) : seg;
        offC = (uint32_t)(k_first + b_r) * code_row_bytes + seg * SEGB;
        offS = (int)seg * 32 < a.I ? ((uint32_t)(k_first + b_r) * (uint32_t)a.G + grp) * 8u : kOobOffset;
    } else {
        seg = (uint32_t)(k_first >> 5) + b_s;
        offC = (uint32_t)(n0 + b_r) * code_row_bytes + seg * SEGB;
        offS = (uint32_t)(n0 + b_r) * (uint32_t)a.G * 8u;
    }
    WorkCodes<BITS> stC[2];
    floatx2 stS[2];
    WhatTable<BITS> tab;
    auto load_codes = [&](auto set) {
        constexpr int S = decltype(set)::value;
        stC[S] = load_work_codes<BITS>(rCodes, offC);
        intx2 v;
        if constexpr (BT) {
            v = buf_load8(rS, offS);
            offC += 2u * kKsBK * code_row_bytes;
            offS += 2u * kKsBK * (uint32_t)a.G * 8u;
        } else {
            const uint32_t grp = a.spg_magic ? __umulhi(seg, a.spg_magic) : seg;
            v = buf_load8(rS, (int)seg * 32 < a.I ? offS + grp * 8u : kOobOffset);
            seg += 2 * kKsBK / 32;
            offC += 2 * kKsBK / 32 * SEGB;
        }
        stS[S][0] = __int_as_float(v[0]); stS[S][1] = __int_as_float(v[1]);
    };
    const int sw = BT ? km_chunk_swz(b_r, b_s) : 0;
    bf16x8 *dstB[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) dstB[q] = reinterpret_cast<bf16x8 *>(sB + b_r * LDB + b_s * 32) + (q ^ sw);
    auto commit = [&](auto set, auto piece, int buf) {
        constexpr int S = decltype(set)::value, P = decltype(piece)::value;
        if constexpr (P == 0) tab.build(stS[S][0], stS[S][1]);
        *reinterpret_cast<bf16x8 *>(reinterpret_cast<bf16_t *>(dstB[P]) + buf * B_ELEMS) = tab.template eight<P>(stC[S]);
    };

    floatx16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    bf16x8 fa[2][2], fb[2][2];
    auto read_a = [&](int slot, int buf, int kk) {
#pragma unroll
        for (int i = 0; i < 2; ++i) fa[slot][i] = frag_kc_swz(sA + buf * A_ELEMS, wm * 64 + i * 32, kk, lane);
    };
    auto read_b = [&](int slot, int buf, int kk) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if constexpr (!BT) fb[slot][j] = frag_kc<LDB>(sB + buf * B_ELEMS, wn * 64 + j * 32, kk, lane);
            else fb[slot][j] = frag_km<LDB>(sB + buf * B_ELEMS, wn * 64 + j * 32, kk, lane);
        }
    };
    auto mfma = [&](int slot, int i, int j) {
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[slot][i], fb[slot][j], acc[i][j], 0, 0, 0);
    };
    auto slice = [&](int slot) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) mfma(slot, i, j);
    };
    auto weave = [&]() {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, BT ? 2 : 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, BITS == 4 ? 8 : 6, 0);
            __builtin_amdgcn_sched_group_barrier(0x004, 5, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
#define EQAT_FENCE __builtin_amdgcn_sched_barrier(0)
    // K tile t, in buffer PAR = t & 1
    auto step = [&](auto par, int t) __attribute__((always_inline)) {
        constexpr int PAR = decltype(par)::value;
        typedef IC<PAR ^ 1> Next;
        load_a(2, PAR ^ 1); load_a(3, PAR ^ 1);
        mask_a(t + 2);
        EQAT_FENCE;
        read_b(1, PAR, 1); read_a(1, PAR, 1);
        slice(0);
        commit(Next{}, IC<1>{}, PAR ^ 1);
        weave();
        read_b(0, PAR, 2); read_a(0, PAR, 2);
        slice(1);
        commit(Next{}, IC<2>{}, PAR ^ 1);
        aim_a(t + 2);
        weave();
        read_b(1, PAR, 3); read_a(1, PAR, 3);
        slice(0);
        commit(Next{}, IC<3>{}, PAR ^ 1);
        weave();
        wait_all_and_barrier();
        load_a(0, PAR); load_a(1, PAR);
        EQAT_FENCE;
        read_b(0, PAR ^ 1, 0); read_a(0, PAR ^ 1, 0);
        slice(1);
        commit(par, IC<0>{}, PAR);
        weave();
        load_codes(Next{});
        EQAT_FENCE;
    };

    load_codes(IC<0>{});
    mask_a(0); aim_a(0);
#pragma unroll
    for (int it = 0; it < 4; ++it) load_a(it, 0);
    load_codes(IC<1>{});
    commit(IC<0>{}, IC<0>{}, 0); commit(IC<0>{}, IC<1>{}, 0); commit(IC<0>{}, IC<2>{}, 0); commit(IC<0>{}, IC<3>{}, 0);
    wait_all_and_barrier();
    load_codes(IC<0>{});
    mask_a(1); aim_a(1);
    load_a(0, 1); load_a(1, 1);
    commit(IC<1>{}, IC<0>{}, 1);
    read_a(0, 0, 0);
    read_b(0, 0, 0);
    for (int t = 0;;) {
        step(IC<0>{}, t);
        if (++t >= n) break;
        step(IC<1>{}, t);
        if (++t >= n) break;
    }
    wait_all_and_barrier();

    // ---- sums of the two K groups: each keeps one of the wave's two block rows and hands the other over (32 x 64 outputs a wave)
    {
        unsigned char *const mine = smem_raw + wave * 8192 + lane * 16;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                floatx4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = kg ? acc[0][j][4 * q + e] : acc[1][j][4 * q + e];
                *reinterpret_cast<floatx4 *>(mine + (j * 4 + q) * 1024) = v;
            }
    }
    __syncthreads();
    floatx16 sum[2];
    {
        const unsigned char *const theirs = smem_raw + (wave ^ 4) * 8192 + lane * 16;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const floatx4 v = *reinterpret_cast<const floatx4 *>(theirs + (j * 4 + q) * 1024);
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[j][4 * q + e] = (kg ? acc[1][j][4 * q + e] : acc[0][j][4 * q + e]) + v[e];
            }
    }
    if (a.parts_per_tile > 1) {
        // Parts and counter are written and read at device scope (the contributors sit on different XCDs), no cache is flushed:
        // every wave waits for its stores, the workgroup meets, then one lane counts it in.
        __shared__ uint32_t s_last;
        constexpr uint32_t kPart = kKsBM * kKsBN * 4;
        const uint32_t at = (uint32_t)(wave * 8192 + lane * 16);
        const __amdgpu_buffer_rsrc_t mine = make_rsrc(a.parts + (size_t)pid * (kPart / 4), kPart);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            intx4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = __float_as_int(sum[q >> 2][(q & 3) * 4 + e]);
            __builtin_amdgcn_raw_buffer_store_b128(v, mine, (int)(at + q * 1024u), 0, kAuxDeviceScope);
        }
        wait_all_and_barrier();
        if (tid == 0) {
            const uint32_t before = __hip_atomic_fetch_add(a.counters + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_last = before == (uint32_t)(a.parts_per_tile - 1) ? 1u : 0u;
            if (s_last) __hip_atomic_store(a.counters + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (s_last == 0u) return;
        auto fetch = [&](int k, intx4 (&v)[8]) {
            const __amdgpu_buffer_rsrc_t r = make_rsrc(a.parts + (size_t)(k * ntiles + tile) * (kPart / 4), k < a.parts_per_tile ? kPart : 0u);
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = __builtin_amdgcn_raw_buffer_load_b128(r, (int)(at + q * 1024u), 0, kAuxDeviceScope);
        };
        auto add = [&](const intx4 (&v)[8]) {
#pragma unroll
            for (int q = 0; q < 8; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[q >> 2][(q & 3) * 4 + e] += __int_as_float(v[q][e]);
        };
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) sum[j][e] = 0.0f;
        intx4 v[kKsMaxParts][8];
#pragma unroll
        for (int k = 0; k < kKsMaxParts; ++k) fetch(k, v[k]);
#pragma unroll
        for (int k = 0; k < kKsMaxParts; ++k) add(v[k]);
    }
    __syncthreads();
    ks_store(sum, smem_raw + wave * kStoreStageBytes, make_rsrc(a.C, a.c_bytes), m0 + wm * 64 + kg * 32, n0 + wn * 64, a.M, a.N, lane);
}

template <int BITS, bool BT> void launch_t(const KsArgs &a, hipStream_t st)
{
    constexpr int smem = 2 * (int)ks_group_bytes<BT>();
    static_assert(smem <= 160 * 1024, "LDS of one CU");
    auto kern = k_gemm_ksplit<BITS, BT>;
    static std::atomic<uint64_t> allowed{0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev > 63) dev = 0;
    if (!((allowed.load(std::memory_order_relaxed) >> dev) & 1u)) {
        (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
        allowed.fetch_or((uint64_t)1 << dev, std::memory_order_relaxed);
    }
    kern<<<dim3((unsigned)(a.tiles_m * a.tiles_n * a.parts_per_tile)), dim3(kKsNT), smem, st>>>(a);
}

struct Shape { int M, N, K, tiles, pairs; };
Shape shape_of(const Problem &p, bool bt)
{
    Shape s{};
    s.M = (int)p.T; s.N = (int)(bt ? p.I : p.O); s.K = (int)(bt ? p.O : p.I);
    s.tiles = (int)std::min<int64_t>((int64_t)((s.M + kKsBM - 1) / kKsBM) * ((s.N + kKsBN - 1) / kKsBN), 1 << 20);
    s.pairs = (s.K + 2 * kKsBK - 1) / (2 * kKsBK);
    return s;
}

}  // namespace

// One round of workgroups (more tiles: the tile kernel has two workgroups per compute unit and is level or ahead, 1280 tokens, 4096 x
// 4096: 62 us there, two rounds here 66).  A launch takes 4.5 us, 0.95 a pair of K tiles and, where a tile has several
// contributors, 2.5 us and 0.045 per part; a part is at least four pairs.  Two or four whole K tiles are too few for two groups: the
// tile kernel needs no sum of theirs (forward on a prepared layer, us, there / here: 128 inputs, 150 tokens, 3224 rows 9.1 / 9.8, 3546
// tokens, 880 rows 10.0 / 10.8; 256 inputs, 617 tokens, 3480 rows 10.8 / 11.6; dX, 128 rows, 74 tokens, 24128 inputs 18.5 / 19.2).
// Lengths up to four K tiles that are no multiple of two stay here: the forward is level (71 random sizes 32 to 224 inputs, 1 to 4000 tokens, within 2 % but for one), dX 1 %
// faster with one pair of K tiles and 5 % with two (69 sizes; 477 tokens, 216 -> 5088 7.5 us here, 8.4 there).
int ksplit_parts(const Problem &p, bool bt, const SkScratch &sk)
{
    if (!p.act_bf16 || p.T < 1 || !group_by_magic(p)) return 0;
    const Shape s = shape_of(p, bt);
    if (s.tiles > 256 || (s.K <= 4 * kKsBK && s.K % (2 * kKsBK) == 0)) return 0;
    const int room = sk.partials == nullptr || sk.counters == nullptr ? 1 : (int)std::min<size_t>(sk.bytes / (s.tiles * kKsPartBytes), kKsMaxParts);
    const int most = std::min(std::min(room, 256 / s.tiles), s.pairs / 4);
    int best = 1;
    double best_us = 4.5 + 0.95 * s.pairs;
    for (int c = 2; c <= most; ++c) {
        const double us = 7.0 + 0.95 * ((s.pairs + c - 1) / c) + 0.045 * s.tiles * c;
        if (us < best_us) { best = c; best_us = us; }
    }
    return best;
}

size_t ksplit_bytes(const Problem &p, bool bt, int parts)
{
    return parts > 1 ? (size_t)shape_of(p, bt).tiles * parts * kKsPartBytes : 0;
}

bool ksplit_item_for_test(const Problem &p, bool bt, const SkScratch &sk, int block, int32_t item[10])
{
    const int parts = ksplit_parts(p, bt, sk);
    if (parts == 0) return false;
    const Shape s = shape_of(p, bt);
    const int tiles_m = (s.M + kKsBM - 1) / kKsBM, tiles_n = (s.N + kKsBN - 1) / kKsBN, grid = s.tiles * parts;
    if (block >= grid) return false;
    const KsItem it = ks_item(block, grid, tiles_m, tiles_n, parts, s.pairs);
    const int32_t v[10] = {it.tm, it.tn, it.first_pair, it.first_pair + it.pairs, it.part, parts, grid, s.pairs, tiles_m, tiles_n};
    for (int k = 0; k < 10; ++k) item[k] = v[k];
    return true;
}

void launch_ksplit(const Problem &p, bool bt, const void *A, const void *codes, const void *sz, void *C, const SkScratch &sk, int parts,
                   hipStream_t st)
{
    const Shape s = shape_of(p, bt);
    KsArgs a{};
    a.A = (const bf16_t *)A; a.codes = (const uint32_t *)codes; a.sz = (const floatx2 *)sz; a.C = (bf16_t *)C;
    a.parts = sk.partials; a.counters = sk.counters;
    a.M = s.M; a.N = s.N; a.K = s.K; a.I = (int)p.I; a.G = (int)p.G;
    a.spg_magic = p.g == 32 ? 0u : (uint32_t)((((uint64_t)1 << 32) + (uint64_t)(p.g / 32) - 1) / (uint64_t)(p.g / 32));
    a.a_bytes = (uint32_t)(p.T * a.K * 2); a.codes_bytes = (uint32_t)work_code_bytes(p); a.sz_bytes = (uint32_t)(p.O * p.G * 8);
    a.c_bytes = (uint32_t)(p.T * a.N * 2);
    a.tiles_m = (a.M + kKsBM - 1) / kKsBM; a.tiles_n = (a.N + kKsBN - 1) / kKsBN;
    a.pairs = s.pairs;
    a.parts_per_tile = parts;
#define EQAT_GO(B) do { if (bt) launch_t<B, true>(a, st); else launch_t<B, false>(a, st); } while (0)
    if (p.bits == 2) EQAT_GO(2); else if (p.bits == 3) EQAT_GO(3); else EQAT_GO(4);
#undef EQAT_GO
}

}  // namespace eqat
