// The 256 x 256 and 128 x 128 tile kernels of the bf16 GEMMs: bodies that gemm_mfma.hip launches by themselves and gemm_bwd.h side by side.
//
// Two LDS tile formats feed the MFMA operands:
//   KC  "K contiguous"  [row][BK + 8]      fragment = one ds_read_b128 per lane
//   KM  "K major"       [k][cols + 32]     fragment = two ds_read_b64_tr_b16 (LDS transpose reads)
// The paddings make both read patterns bank-conflict free.
#pragma once
#include "common.h"
#include "gemm_tiles.h"
#include "kernels.h"

namespace eqat {

// ---- workgroup -> tile mapping ---------------------------------------------------------------------------
// Consecutive workgroup ids go round-robin over the 8 XCDs, each with its own L2.  Give every XCD a
// contiguous range of tile ids, then walk the tiles in bands of kBand tile-rows so that the tiles resident on
// one XCD at a time share their operand panels.
// nb = number of tiles; (xcd, loc) = the loc-th tile of XCD xcd.  Returns false past the end of that XCD's range.
__host__ __device__ __forceinline__ bool tile_of_xcd_slot(int nb, int xcd, int loc, int tiles_m, int tiles_n, int &tm, int &tn, int kBand)
{
    const int per = nb >> 3, rem = nb & 7;
    if (loc >= per + (xcd < rem ? 1 : 0)) return false;
    const int pid = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + loc;
    const int width = kBand * tiles_n, band = pid / width, first = band * kBand;
    const int rows = tiles_m - first < kBand ? tiles_m - first : kBand, in = pid - band * width;
    tm = first + in % rows;
    tn = in / rows;
    return true;
}
// ---- work of one workgroup: whole tiles, then a share of the tiles that do not fill a round ---------------
// A grid of G workgroups (all resident at once, G / 8 per XCD) covers nb tiles.  When nb is between one and two rounds
// of G (the 13B-shaped linears at 4096 tokens give 1.25 rounds of 256 x 256 tiles) the second round would run on a
// fraction of the chip.  Instead the tiles beyond the last whole round but one are cut along K: their K-tile pairs,
// laid end to end per XCD, are dealt out in equal contiguous runs, so a workgroup's run may begin and end in the middle
// of a tile.  A run is at least one tile long, so a tile has at most two contributors.  The contributor that arrives
// first writes its fp32 accumulators to memory and raises the tile's flag; the one that arrives second waits for the
// flag (a wait for a workgroup that is already running and itself waits for nobody), adds that part to its own
// accumulators (a + b = b + a: the result does not depend on who came first) and runs the tile's epilogue.  Counter
// and flag of a tile are back at zero when its second contributor is done, so a launch leaves them as it found them.
// Whether cutting pays is a measured matter (host side, plan_tiles): a partly filled round costs less than its share
// of a full one on this power-limited chip, and every part costs a trip of 256 KB through memory.
// When the tiles beyond the first round are few (at most half a round), dealing out runs would cut nearly every tile of
// the launch (1.25 rounds: 31 of 40 per XCD).  Then (`split`) every workgroup first computes one whole tile, and each
// of the remaining tiles is shared by c = W / n_sk workgroups (at most kSkMaxSplit), a c-th of its K range each; all
// write their parts and the one that arrives last adds them up in their order (a fixed order: reproducible).
constexpr int kSkMaxSplit = 8;
struct SkPlan {
    int walk;              // 0: the grid has one workgroup per tile and none of the below applies
    int dp_rounds;         // whole tiles per workgroup: tiles loc0 + r * (G / 8) of its XCD, r < dp_rounds
    int split;             // 1: the tiles beyond the whole rounds are split among groups of workgroups (see above)
    int pairs;             // K-tile pairs per output tile
    int slots;             // parts per workgroup: 1 where tiles are split, 2 for runs
    float *partials;       // [G][2] accumulator tiles (a run has at most a head and a tail piece), [G] where tiles are split
    uint32_t *counters;    // [2][2 G], zero: arrivals, then flags, one each per tile that may be cut (at most 2 G / 8 per XCD)
};
struct SkItem {
    int tm, tn, ctr;       // tile, and the index of its counter when it is cut
    int kb, ke;            // K-tile pairs [kb, ke) of the tile
    int parts, first;      // number of contributors (1: the whole tile is mine) and the first one's index in the XCD
    int first_slot;        // which of its two buffers the first contributor used (all others use buffer 0)
    int fixed;             // 1: a split tile (all contributors write, the last one to arrive sums all parts); 0: a run's tile
};
__host__ __device__ __forceinline__ int sk_owner_of_pair(int p, int base, int extra)
{
    const int cut = extra * (base + 1);
    return p < cut ? p / (base + 1) : extra + (p - cut) / (base > 0 ? base : 1);
}
// item number j of workgroup `bid` of a grid of `grid`; false past its last one
__host__ __device__ __forceinline__ bool sk_item_of(const SkPlan &sk, int nb, int tiles_m, int tiles_n, int band, int bid, int grid,
                                                   int j, SkItem &it)
{
    const int xcd = bid & 7, loc0 = bid >> 3;
    it.kb = 0; it.ke = sk.pairs; it.parts = 1; it.first = 0; it.first_slot = 0; it.ctr = 0; it.fixed = 0;
    if (!sk.walk) return j == 0 && tile_of_xcd_slot(grid, xcd, loc0, tiles_m, tiles_n, it.tm, it.tn, band);
    const int W = grid >> 3;
    if (j < sk.dp_rounds) return tile_of_xcd_slot(nb, xcd, loc0 + j * W, tiles_m, tiles_n, it.tm, it.tn, band);
    const int n_sk = (nb >> 3) + (xcd < (nb & 7) ? 1 : 0) - sk.dp_rounds * W;
    if (n_sk <= 0) return false;
    if (sk.split) {
        if (j != sk.dp_rounds) return false;                       // one piece per workgroup
        const int c = W / n_sk < kSkMaxSplit ? W / n_sk : kSkMaxSplit;                   // contributors per tile (at least 2: the host's choice)
        const int t = loc0 / c, me = loc0 - t * c;
        if (t >= n_sk) return false;
        const int base = sk.pairs / c, extra = sk.pairs % c;
        it.kb = me * base + (me < extra ? me : extra);
        it.ke = it.kb + base + (me < extra ? 1 : 0);
        it.parts = c; it.first = t * c; it.fixed = 1;
        it.ctr = xcd * 2 * W + t;
        return tile_of_xcd_slot(nb, xcd, sk.dp_rounds * W + t, tiles_m, tiles_n, it.tm, it.tn, band);
    }
    const int P = sk.pairs, total = n_sk * P, base = total / W, extra = total % W;
    const int start = loc0 * base + (loc0 < extra ? loc0 : extra), end = start + base + (loc0 < extra ? 1 : 0);
    const int t = start / P + (j - sk.dp_rounds);
    if (start >= end || t * P >= end) return false;
    it.kb = (start > t * P ? start : t * P) - t * P;
    it.ke = (end < (t + 1) * P ? end : (t + 1) * P) - t * P;
    if (it.kb > 0 || it.ke < P) {
        it.first = sk_owner_of_pair(t * P, base, extra);
        it.parts = sk_owner_of_pair((t + 1) * P - 1, base, extra) - it.first + 1;
        const int fstart = it.first * base + (it.first < extra ? it.first : extra);
        it.first_slot = fstart / P == t ? 0 : 1;
        it.ctr = xcd * 2 * W + t;          // t < n_sk <= 2 W: the plan never cuts more than two rounds
    }
    return tile_of_xcd_slot(nb, xcd, sk.dp_rounds * W + t, tiles_m, tiles_n, it.tm, it.tn, band);
}

// A contributor of a tile cut along K is done with its K range.  Returns true in the one that holds the sum of all
// parts in `acc` afterwards and runs the tile's epilogue, false in the others (their part is in memory, their work on
// the tile done).
//   Two contributors of a run: the one that arrives first writes its part and raises the tile's flag, the one that
//   arrives second waits for the flag (for a workgroup that is already running and itself waits for nobody) and adds
//   that part to its own accumulators (a + b = b + a).
//   A split tile (it.fixed): every contributor writes its part and counts itself in; the one that finds itself last
//   adds up ALL parts from memory, its own included, in the order of the contributors.  Nobody waits for anybody, and
//   the sum does not depend on who came last.
// Layout of a part: the float4 number q of accumulator block (i, j) of thread t at ((i * NI + j) * 4 + q) * NT + t.
// The contributors may sit on different XCDs, each with its own L2, so parts and flag are written and read with
// device-scope accesses (cache policy sc1: written through to memory, read from memory); no cache is flushed or
// invalidated as a whole (a device-scope fence writes back and invalidates the entire L2 of the XCD, operand panels
// included: measured, that alone cost more than cutting the tiles gained).  Order on the writing side: every wave
// waits for its stores to complete, the workgroup meets, then one thread signals.
constexpr int kSkSpinLimit = 1 << 22;    // polls of ~1 us: a bound that is never reached, so that no wave can spin for ever
// register r of block (i, j), whichever way a kernel keeps its accumulators
template <int MI, int NI> __device__ __forceinline__ float acc_get(const floatx16 (&acc)[MI][NI], int i, int j, int r) { return acc[i][j][r]; }
template <int MI, int NI> __device__ __forceinline__ float acc_get(const floatx4 (&acc)[MI][NI][4], int i, int j, int r) { return acc[i][j][r >> 2][r & 3]; }
template <int MI, int NI> __device__ __forceinline__ void acc_set(floatx16 (&acc)[MI][NI], int i, int j, int r, float v) { acc[i][j][r] = v; }
template <int MI, int NI> __device__ __forceinline__ void acc_set(floatx4 (&acc)[MI][NI][4], int i, int j, int r, float v) { acc[i][j][r >> 2][r & 3] = v; }
// NB = 32 x 32 blocks of a part that are fetched together (16 registers each)
template <int MI, int NI, int NT, int NB = 2, typename ACC>
__device__ __forceinline__ bool sk_hand_in(const SkPlan &sk, const SkItem &it, ACC &acc, int tid, int bid, int grid)
{
    static_assert((MI * NI) % NB == 0, "whole batches");
    __shared__ uint32_t s_sums;
    constexpr size_t kTile = (size_t)MI * NI * 16 * NT;          // floats per part
    constexpr uint32_t kTileBytes = (uint32_t)(kTile * sizeof(float));
    const int xcd = bid & 7, me = (bid >> 3) - it.first;       // 0 .. parts - 1
    const bool split = it.fixed != 0;
    uint32_t *arrivals = sk.counters + it.ctr, *flag = sk.counters + 2 * grid + it.ctr;
    if (tid == 0) s_sums = split ? 0u : atomicInc(arrivals, 1u);                          // run: 0 -> 1 -> 0
    __syncthreads();
    const bool second = s_sums != 0u;              // of a run
    // Straight-line code for all roles (branches around the accumulators make the register allocator spill them): the
    // stores of the contributor that keeps its part in registers go to an out-of-range offset, where they are dropped.
    const uint32_t st_base = second ? kOobOffset : (uint32_t)tid * 16u;
    const __amdgpu_buffer_rsrc_t mine =
        make_rsrc(sk.partials + ((size_t)bid * sk.slots + (!split && me == 0 ? it.first_slot : 0)) * kTile, kTileBytes);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                intx4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = __float_as_int(acc_get<MI, NI>(acc, i, j, 4 * q + e));
                __builtin_amdgcn_raw_buffer_store_b128(v, mine, st_base + (uint32_t)(((i * NI + j) * 4 + q) * NT * 16), 0, kAuxDeviceScope);
            }
            __builtin_amdgcn_sched_barrier(0);      // one 32 x 32 block at a time: few register copies
        }
    wait_all_and_barrier();                // every store of the workgroup has completed
    if (tid == 0) {
        if (split) {
            const uint32_t before = __hip_atomic_fetch_add(arrivals, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const bool last = before == (uint32_t)(it.parts - 1);
            if (last) __hip_atomic_store(arrivals, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_sums = last ? 1u : 0u;
        } else if (!second) {
            __hip_atomic_store(flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            int polls = 0;
            while (__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u && ++polls < kSkSpinLimit)
                __builtin_amdgcn_s_sleep(32);
            __hip_atomic_store(flag, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __syncthreads();
    const bool sums = s_sums != 0u;
    // the last contributor of a split tile starts from zero and takes every part, its own too, from memory (bitwise AND
    // instead of a branch, see above)
    const uint32_t keep = (split && sums) ? 0u : ~0u;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc_set<MI, NI>(acc, i, j, r, __uint_as_float(__float_as_uint(acc_get<MI, NI>(acc, i, j, r)) & keep));
    // parts to add, in the order of the contributors (a trip count of zero for those that do not sum)
    const int n_take = !sums ? 0 : split ? it.parts : 1;
    for (int k = 0; k < n_take; ++k) {
        const int from = split ? it.first + k : it.first + (1 - me);                  // contributor whose part this is
        const int slot = (!split && me == 1) ? it.first_slot : 0;
        const __amdgpu_buffer_rsrc_t theirs = make_rsrc(sk.partials + (((size_t)from * 8 + xcd) * sk.slots + slot) * kTile, kTileBytes);
        // NB blocks in flight at a time.  In the fwd / dX kernels two (32 registers): with more (two parts together, 64
        // registers) they spilled or lost their second workgroup per CU, because the pipeline state of the next tile is
        // alive here.
#pragma unroll
        for (int b0 = 0; b0 < MI * NI; b0 += NB) {
            intx4 v[NB][4];
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    v[b][q] = __builtin_amdgcn_raw_buffer_load_b128(theirs, (uint32_t)tid * 16u + (uint32_t)(((b0 + b) * 4 + q) * NT * 16), 0, kAuxDeviceScope);
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc_set<MI, NI>(acc, (b0 + b) / NI, (b0 + b) % NI, 4 * q + e,
                                        acc_get<MI, NI>(acc, (b0 + b) / NI, (b0 + b) % NI, 4 * q + e) + __int_as_float(v[b][q][e]));
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    return sums;
}

// ======================================================================================================
// fwd / dX:  C[M,N] = A[M,K] * B,  A plain bf16 (K contiguous), B = What rebuilt from codes.
//   BT = false (fwd): B element (k, n) = What[n][k]   -> weight tile is KC  [BN][BK]
//   BT = true  (dX) : B element (k, n) = What[k][n]   -> weight tile is KM  [BK][BN]
// ======================================================================================================
struct GemmQArgs {
    const bf16_t *A; const uint32_t *codes; const floatx2 *sz; bf16_t *C;
    int M, N, K;           // problem
    int I, G, g;           // weight matrix geometry: row length, groups per row, group size
    uint32_t a_bytes, codes_bytes, sz_bytes, c_bytes;
    int tiles_m, tiles_n;
    int band;              // tile rows walked together by one XCD (see tile_of_xcd_slot)
    SkPlan sk;             // which tiles, or parts of tiles, a workgroup computes
};

// f(IC<0>{}), f(IC<1>{}), ..., f(IC<N - 1>{}): a loop whose index is a compile-time constant inside the body
template <int N, int I = 0, typename F> __device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (I < N) { f(IC<I>{}); static_for<N, I + 1>(f); }
}

// With more than 128 accumulator registers per lane the accumulators must live in AGPRs (the MFMA "acd" form);
// the compiler only picks that form when it believes the kernel needs AGPRs, which this empty statement asserts.
template <int ACC_REGS> __device__ __forceinline__ void want_agpr_accumulators()
{
    if constexpr (ACC_REGS > 128) { float zero = 0.0f; asm volatile("" ::"a"(zero)); }
}

// Software pipeline of the main loop (one workgroup, K tile kt, LDS buffer kt & 1):
//   - behind the barrier of tile kt (which sits before its last 16-wide slice) the activation tile kt+2 starts to
//     stream from global memory straight into LDS buffer kt & 1, whose last fragments are in registers by then;
//   - the weight codes and (s, zbar) pairs of tile kt+3 are fetched into registers (two staging sets);
//   - while the MFMAs consume buffer kt & 1, the staged codes of tile kt+1 become bf16 What in the other weight
//     buffer, a quarter after each slice, so that this VALU / LDS-write work hides under the MFMAs of the same
//     wave; fragments of slice kk+1 are read while slice kk multiplies.
// K tiles past the end of K multiply zeros: the weights there are exactly zero (see load_a below).
// A workgroup may own several output tiles; the pipeline then runs on through the tile boundaries.
// MODE kCut: for launches that cut tiles along K (SkPlan::dp_rounds == 0, or split, with walk), any contraction length; kRagged: whole tiles,
// any contraction length; kWhole: whole tiles, a contraction of a multiple of two K tiles, and none of that code (the main loop is sensitive to it).
// (bid, grid): this workgroup's number among those of the GEMM, which may share its launch with another one.
enum QMode { kWhole, kCut, kRagged };
template <int BITS, bool BT, int MODE, int BM, int BN, int BK, int WGM, int WGN>
__device__ __forceinline__ void gemm_q_body(const GemmQArgs &a, const int bid, const int grid)
{
    constexpr bool CUT = MODE == kCut;
    constexpr int NT = 64 * WGM * WGN, NW = WGM * WGN, WTM = BM / WGM, WTN = BN / WGN, MI = WTM / 32, NI = WTN / 32;
    constexpr int LDB = BT ? BN + kPadKM : BK + kPadKC;
    constexpr uint32_t kRingBytes = 2u * (uint32_t)(BM * BK + (BT ? BK * LDB : BN * LDB)) * 2u;    // the two K-tile buffers
    constexpr int A_ELEMS = BM * BK, B_ELEMS = BT ? BK * LDB : BN * LDB;
    constexpr int A_LOADS = BM / 8 / NW;              // direct-to-LDS instructions per wave (8 rows each)
    constexpr int B_SEGS = BN * BK / 32 / NT;         // 32-code segments per thread
    constexpr int KK = BK / 16;
    static_assert(BK == 64 && BM % (8 * NW) == 0 && BN * BK / 32 % NT == 0, "tile / thread mismatch");

    want_agpr_accumulators<MI * NI * 16>();
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    bf16_t *sA = reinterpret_cast<bf16_t *>(smem_raw);            // [2][A_ELEMS]
    bf16_t *sB = sA + 2 * A_ELEMS;                                // [2][B_ELEMS]

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;

    // Items of this workgroup (see SkPlan): whole tiles, then possibly pieces of tiles cut along K.  The K loop runs
    // THROUGH the item boundaries: the loaders below each keep their own position in that sequence, two (activations)
    // and three (codes) K tiles ahead of the MFMAs, so that the first K tiles of the next item are in LDS and in
    // registers when the last MFMA of the current one issues.
    const int ntiles = a.tiles_m * a.tiles_n;
    const int nk = (a.K + BK - 1) / BK, nk2 = (nk + 1) & ~1;              // K tiles per output tile, two per trip
    // item j: origin of its tile, first K tile and number of K tiles (even); past the last item: rows and columns out
    // of range (the loaders then fetch zeros)
    const int xcd = bid & 7, loc0 = bid >> 3;
    const int loc_step = a.sk.walk ? grid >> 3 : ntiles;          // no second tile without a.sk.walk
    auto item_of = [&](int j, SkItem &it, int &m0, int &n0) -> bool {
        bool ok;
        if constexpr (CUT) {
            ok = sk_item_of(a.sk, ntiles, a.tiles_m, a.tiles_n, a.band, bid, grid, j, it);
            if (!ok) { it.kb = 0; it.ke = nk2 / 2; it.parts = 1; }
        } else {
            // whole tiles only: tile loc0 + j * (G / 8) of this XCD's range (walk), or the one tile of this workgroup
            ok = tile_of_xcd_slot(a.sk.walk ? ntiles : grid, xcd, loc0 + j * loc_step, a.tiles_m, a.tiles_n, it.tm, it.tn, a.band);
            it.kb = 0; it.ke = nk2 / 2; it.parts = 1;
        }
        m0 = ok ? it.tm * BM : a.tiles_m * BM;
        n0 = ok ? it.tn * BN : a.tiles_n * BN;
        return ok;
    };

    const RawRsrc rA = make_raw_rsrc(a.A, a.a_bytes);
    const __amdgpu_buffer_rsrc_t rCst = make_rsrc(a.C, a.c_bytes);
    const __amdgpu_buffer_rsrc_t rC = make_rsrc(a.codes, a.codes_bytes);
    const __amdgpu_buffer_rsrc_t rS = make_rsrc(a.sz, a.sz_bytes);
    const uint32_t code_row_bytes = (uint32_t)a.I / 32u * (4u * WorkCodes<BITS>::kWords);

    WorkCodes<BITS> stC[2][B_SEGS];
    floatx2 stS[2][B_SEGS];
    WhatTable<BITS> tabs[2][B_SEGS];

    // Activation tiles stream into LDS strictly in order (k0 = 0, BK, 2 BK, ... of one output tile, then of the next):
    // every direct-to-LDS instruction keeps a running byte offset that advances by one tile row segment per call, and
    // M0 comes from wave-uniform scalars.  Columns past K of a row would read the start of the next row; they meet weights
    // that are exactly zero (step size and zero point of a column past the end load as 0), and are not loaded at all when
    // K is ragged (see k_ragged below).
    const uint32_t ldsA = lds_addr_of(sA);
    uint32_t offA[A_LOADS];
    int a_tile = 0, a_left = 0;                     // loader position: tile ordinal, K tiles left in it
    // When K is not a multiple of two K tiles, the last K tile of an output tile reaches past the end of its rows (and a
    // padding K tile lies past it altogether).  The weights there are zero, but 0 * Inf is NaN: a non-finite value in
    // row t + 1 must not leak into row t, so the chunks past K of those tiles are loaded from out of range (zeros).
    const bool k_ragged = MODE != kWhole && a.K % (2 * BK) != 0;      // wave-uniform; the host sends every such K to these instantiations
    int a_kt = 0;                                   // K tile (within its output tile) that the next load_a fetches
    uint32_t a_past_k = 0;                          // bit `it`: in K tile nk - 1, this lane's chunk of load `it` lies past K
    if (k_ragged) {
        const int tail_cols = a.K - (nk - 1) * BK;  // 8 .. 64 valid columns in K tile nk - 1
#pragma unroll
        for (int it = 0; it < A_LOADS; ++it) {
            const int row = (wave * A_LOADS + it) * 8 + (lane >> 3);
            if (kc_swz(row, lane & 7) * 8 >= tail_cols) a_past_k |= 1u << it;
        }
    }
    auto a_enter_tile = [&]() {
        int m0, n0;
        SkItem si;
        (void)item_of(a_tile, si, m0, n0);
#pragma unroll
        for (int it = 0; it < A_LOADS; ++it) {
            const int row = (wave * A_LOADS + it) * 8 + (lane >> 3);
            const uint64_t o = ((uint64_t)(m0 + row) * (uint64_t)a.K + (uint64_t)((CUT ? si.kb * 2 * BK : 0) + kc_swz(row, lane & 7) * 8)) * 2u;
            offA[it] = o < kOobOffset ? (uint32_t)o : kOobOffset;   // rows past the matrix stay out of range for good
        }
        a_left = CUT ? 2 * (si.ke - si.kb) : nk2;
        a_kt = CUT ? 2 * si.kb : 0;
        ++a_tile;
    };
    auto load_a = [&](int buf) {
        --a_left;
        if (k_ragged && a_kt >= nk - 1) {            // rare: the last (and the padding) K tile of a ragged K
            const uint32_t past = a_kt >= nk ? ~0u : a_past_k;
#pragma unroll
            for (int it = 0; it < A_LOADS; ++it) {
                load_to_lds16_at(rA, ldsA + (uint32_t)((buf * A_ELEMS + (wave * A_LOADS + it) * 8 * 64) * 2),
                                 (past >> it) & 1u ? kOobOffset : offA[it]);
                offA[it] += BK * 2;
            }
        } else {
#pragma unroll
            for (int it = 0; it < A_LOADS; ++it) {
                load_to_lds16_at(rA, ldsA + (uint32_t)((buf * A_ELEMS + (wave * A_LOADS + it) * 8 * 64) * 2), offA[it]);
                offA[it] += BK * 2;
            }
        }
        ++a_kt;
    };
    // Weight codes and (s, zbar) pairs, in the same order.  Forward: a segment's group index wcol / g is carried from
    // call to call (a K tile advances wcol by BK <= 2 g, so two conditional steps replace a division per K tile).
    int grp[B_SEGS], rem[B_SEGS];
    int c_tile = 0, c_left = 0, c_n0 = 0, c_k0 = 0;
    auto c_enter_tile = [&]() {
        int m0;
        SkItem si;
        (void)item_of(c_tile, si, m0, c_n0);
        c_k0 = CUT ? si.kb * 2 * BK : 0;
#pragma unroll
        for (int it = 0; it < B_SEGS; ++it) {
            const int sidx = it * NT + tid;
            const int wcol = BT ? c_n0 + (sidx % (BN / 32)) * 32 : c_k0 + (sidx % (BK / 32)) * 32;
            grp[it] = wcol / (int)a.g;
            rem[it] = wcol % (int)a.g;
        }
        c_left = CUT ? 2 * (si.ke - si.kb) : nk2;
        ++c_tile;
    };
    auto load_codes = [&](auto set) {
        constexpr int S = decltype(set)::value;
        --c_left;
#pragma unroll
        for (int it = 0; it < B_SEGS; ++it) {
            const int sidx = it * NT + tid;
            int wrow, wcol;   // position in the weight matrix [O][I]
            if (!BT) { wrow = c_n0 + sidx / (BK / 32); wcol = c_k0 + (sidx % (BK / 32)) * 32; }
            else     { wrow = c_k0 + sidx / (BN / 32); wcol = c_n0 + (sidx % (BN / 32)) * 32; }
            const bool ok = wcol < a.I;
            stC[S][it] = load_work_codes<BITS>(rC, (uint32_t)wrow * code_row_bytes + (uint32_t)(wcol >> 5) * (4u * WorkCodes<BITS>::kWords));
            const intx2 sv = buf_load8(rS, ok ? ((uint32_t)wrow * (uint32_t)a.G + (uint32_t)grp[it]) * 8u : kOobOffset);
            stS[S][it][0] = __int_as_float(sv[0]);
            stS[S][it][1] = __int_as_float(sv[1]);
            if (!BT) {
#pragma unroll
                for (int h = 0; h < BK / 32; ++h) {
                    rem[it] += 32;
                    const bool wrap = rem[it] >= (int)a.g;
                    rem[it] = wrap ? rem[it] - (int)a.g : rem[it];
                    grp[it] += wrap ? 1 : 0;
                }
            }
        }
        c_k0 += BK;
    };
    // A loader steps into the next output tile BETWEEN K steps (and between the loads of the start-up sequence): a
    // branch inside a K step would cut the instruction schedule of the step in two.
    auto loaders_advance = [&]() {
        if (a_left == 0) a_enter_tile();
        if (c_left == 0) c_enter_tile();
    };
    // piece P of KK: every KK-th 16-byte store of the staged weight tile
    auto commit_piece = [&](auto set, auto piece, int buf) {
        constexpr int S = decltype(set)::value, P = decltype(piece)::value;
        bf16_t *dB = sB + buf * B_ELEMS;
#pragma unroll
        for (int it = 0; it < B_SEGS; ++it) {
            const int sidx = it * NT + tid;
            int r, c;
            if (!BT) { r = sidx / (BK / 32); c = (sidx % (BK / 32)) * 32; }
            else     { r = sidx / (BN / 32); c = (sidx % (BN / 32)) * 32; }
            WhatTable<BITS> &tab = tabs[S][it];
            if constexpr (P == 0) tab.build(stS[S][it][0], stS[S][it][1]);     // piece 0 of a tile always runs first
            bf16x8 *dst = reinterpret_cast<bf16x8 *>(dB + r * LDB + c);
            const int sw = BT ? km_chunk_swz(r, c >> 5) : 0;                    // KM tile: see km_chunk_swz
            if ((it * 4 + 0) % KK == P) dst[0 ^ sw] = tab.template eight<0>(stC[S][it]);
            if ((it * 4 + 1) % KK == P) dst[1 ^ sw] = tab.template eight<1>(stC[S][it]);
            if ((it * 4 + 2) % KK == P) dst[2 ^ sw] = tab.template eight<2>(stC[S][it]);
            if ((it * 4 + 3) % KK == P) dst[3 ^ sw] = tab.template eight<3>(stC[S][it]);
        }
    };

    floatx16 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    bf16x8 fa[2][MI], fb[2][NI];
    // B fragments first: the MFMAs run i-major, so both B fragments and A0 are needed by the first two MFMAs of a
    // slice and A3 only by the seventh; issued in that order, one read per MFMA of the previous slice, every read gets
    // about a slice of latency budget.
    auto read_frags = [&](int slot, const bf16_t *cA, const bf16_t *cB, int kk) {
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            if (!BT) fb[slot][j] = frag_kc<LDB>(cB, wn * WTN + j * 32, kk, lane);
            else     fb[slot][j] = frag_km<LDB>(cB, wn * WTN + j * 32, kk, lane);
        }
#pragma unroll
        for (int i = 0; i < MI; ++i) fa[slot][i] = frag_kc_swz(cA, wm * WTM + i * 32, kk, lane);
    };
    // One K tile.  PAR = kt & 1 is the LDS buffer being multiplied.  On entry the fragments of slice 0 are already
    // in registers.  The barrier sits BEFORE the MFMAs of the last slice: by then every wave has issued all its LDS
    // reads of this tile and finished writing the next one, so after the barrier the next tile's first fragments and
    // the global loads for later tiles are started and their latency hides under the last slice's MFMAs.
    auto mfma_slice = [&](int slot) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[slot][i], fb[slot][j], acc[i][j], 0, 0, 0);
    };
    auto step = [&](auto par) {
        constexpr int PAR = decltype(par)::value;
        const bf16_t *cA = sA + PAR * A_ELEMS, *cB = sB + PAR * B_ELEMS;
        // stage kk: start the reads of slice kk+1, multiply slice kk, convert a quarter of the next weight tile
        auto interleave = [&]() {
            // pipeline hint for the scheduler: one MFMA, one fragment read of the next slice, a few VALU ops of the
            // conversion, repeated (LDS reads spread over the slice measure 2-5 % faster than a burst in front of it)
#pragma unroll
            for (int q = 0; q < MI * NI; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
            }
        };
        read_frags(1, cA, cB, 1);
        mfma_slice(0);
        commit_piece(IC<PAR ^ 1>{}, IC<1>{}, PAR ^ 1);
        interleave();
        __builtin_amdgcn_sched_barrier(0);
        read_frags(0, cA, cB, 2);
        mfma_slice(1);
        commit_piece(IC<PAR ^ 1>{}, IC<2>{}, PAR ^ 1);
        interleave();
        __builtin_amdgcn_sched_barrier(0);
        read_frags(1, cA, cB, 3);
        mfma_slice(0);
        commit_piece(IC<PAR ^ 1>{}, IC<3>{}, PAR ^ 1);
        interleave();
        __builtin_amdgcn_sched_barrier(0);
        wait_all_and_barrier();   // next activation tile landed, my LDS traffic done
        // last slice of this tile, overlapped with the start of the next two tiles.  (The codes fetched here are first
        // used behind the next barrier, so the compiler never needs a vmcnt wait while the activation loads fly.)
        load_a(PAR);
        read_frags(0, sA + (PAR ^ 1) * A_ELEMS, sB + (PAR ^ 1) * B_ELEMS, 0);
        mfma_slice(1);
        commit_piece(IC<PAR>{}, IC<0>{}, PAR);
        interleave();
        load_codes(IC<PAR ^ 1>{});
        __builtin_amdgcn_sched_barrier(0);
    };

    // start-up of the first tile: K tiles 0 and 1 of the activations, 0, 1 and 2 of the codes, weight tile 0 rebuilt
    loaders_advance();
    load_codes(IC<0>{});
    load_a(0);
    loaders_advance();
    load_codes(IC<1>{});
    commit_piece(IC<0>{}, IC<0>{}, 0);
    commit_piece(IC<0>{}, IC<1>{}, 0);
    commit_piece(IC<0>{}, IC<2>{}, 0);
    commit_piece(IC<0>{}, IC<3>{}, 0);
    wait_all_and_barrier();
    loaders_advance();
    load_codes(IC<0>{});
    load_a(1);
    commit_piece(IC<1>{}, IC<0>{}, 1);
    read_frags(0, sA, sB, 0);

    for (int jt = 0;; ++jt) {
        int m0, n0;
        SkItem si;
        if (!item_of(jt, si, m0, n0)) break;
        // Two K tiles per trip, unconditionally (the register staging sets alternate at compile time, and a branch
        // between the two halves makes the accumulators flow through a merge that costs hundreds of copies).  With an
        // odd K-tile count the extra tile lies past K and multiplies zeros.  The last trips of this loop already fetch
        // (and rebuild) the first K tiles of the next item.
        for (int kt = CUT ? 2 * si.kb : 0; kt < (CUT ? 2 * si.ke : nk2); kt += 2) {
            loaders_advance();
            step(IC<0>{});
            loaders_advance();
            step(IC<1>{});
        }
        // a tile cut along K: only the contributor that arrives last stores it, from the sum of all parts
        bool mine_to_store = true;
        if constexpr (CUT) mine_to_store = si.parts == 1 || sk_hand_in<MI, NI, NT>(a.sk, si, acc, tid, bid, grid);
        if (!mine_to_store) {
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
            continue;
        }

        // C[m][n]: lane holds column n = l % 32 and rows 8*(r/4) + 4*(l/32) + r%4 of each 32x32 block.  Stored from
        // the registers that is sixteen 2-byte stores per block, each to two rows; instead the block goes through a
        // 2 KB patch of LDS of the wave's own (behind the tile ring, which the loads of the next tile are filling) and
        // leaves as two 16-byte stores per lane, 64 bytes of a row from four neighbouring lanes.
        {
            unsigned char *const stg = smem_raw + kRingBytes + wave * kStoreStageBytes;
            bf16_t *const cell = reinterpret_cast<bf16_t *>(stg) + (lane >> 5) * (4 * 32) + (lane & 31);
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        cell[(8 * (r >> 2) + (r & 3)) * 32] = (bf16_t)acc[i][j][r];
                        acc[i][j][r] = 0.0f;
                    }
                    asm volatile("" ::: "memory");
                    __builtin_amdgcn_wave_barrier();       // LDS accesses of a wave complete in order
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const intx4 v = *reinterpret_cast<const intx4 *>(stg + k * 1024 + lane * 16);
                        const int m = m0 + wm * WTM + i * 32 + k * 16 + (lane >> 2), n = n0 + wn * WTN + j * 32 + (lane & 3) * 8;
                        const uint32_t off = (m < a.M && n < a.N) ? ((uint32_t)m * (uint32_t)a.N + (uint32_t)n) * 2u : kOobOffset;
                        __builtin_amdgcn_raw_buffer_store_b128(v, rCst, (int)off, 0, 0);
                    }
                    asm volatile("" ::: "memory");
                    __builtin_amdgcn_sched_barrier(0);     // one 32x32 block at a time: keeps the accumulator copies few
                }
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0070);       // the loads issued past the last tile (all zeros) have landed too
}

// ======================================================================================================
// dW:  D[i][o] = sum_t X[t][i] * dY[t][o]   (M <-> i, N <-> o, K = T; both operand tiles KM)
// and, on the accumulators, for every weight (o, i):
//   Block-AP:  clamped = bit of the clamp plane; q = code; r = q - zbar
//              cs = clamped ? r : r - w/s ;  dW = clamped ? 0 : D ;  ds += D*cs ;  dz += clamped ? -s*D : 0
//   E2E-QP  :  ds += D * (q - z) ;  dz += -s*D  (dz only when asked for: zero points trained end to end)
// M <-> i puts the 32 columns of a group segment into the registers of one lane pair, so the group sums
// need one cross-lane exchange per 32x32 block.
// ======================================================================================================
struct GemmDwArgs {
    const bf16_t *X, *dY; const void *W; const uint32_t *codes; const uint8_t *clampbits; const floatx2 *sz;
    void *dW; float *ds, *dz, *part_ds, *part_dz;
    int T, I, O, G, g;
    uint32_t x_bytes, dy_bytes, w_bytes, codes_bytes, clamp_bytes, sz_bytes;
    int tiles_m, tiles_n;
    int direct;           // 1: every group lies inside one tile -> final ds/dz; 0: per-32-column partials
    SkPlan sk;            // which tiles, or parts of tiles, a workgroup computes (kernels that cut tiles along T)
};

// The epilogue of the Block-AP kernel reads W and writes dW through LDS.  In the accumulator layout a lane holds one
// weight ROW (out-feature) and four consecutive in-features per quad, so straight from the registers every load or
// store instruction would touch 32 different rows, 8 or 16 bytes of each.  Instead a wave moves the W rows it needs as
// whole 128- or 256-byte row pieces (16 bytes per lane, straight into LDS), picks its quads out of LDS, puts the dW
// quads back in their place and writes the rows out the way they came in.
// dW goes past the caches (non-temporal): it is not touched again before the update, and in the L2s it drives out the X and dY panels that the tiles still to come
// share.  So does W where there is more of it than they keep from the pass that read it last.  Backward, us, neither past them / dW / both: 300 tokens, 768 -> 4568, bf16 (7 MB of W)
// 29.2 / 28.6 / 28.6; 276 tokens, 1536 -> 1208, fp32 (7 MB) 25.9 / 25.3 / 27.8; 409 tokens, 5120 -> 752, fp32 (15 MB) 35.0 / 30.4 / 35.0; 78 tokens, 6240 -> 1648, bf16 (21 MB) 30.1 / 25.8 / 27.0;
// 514 tokens, 6016 -> 1248, fp32 (30 MB) 49.9 / 47.0 / 44.3; 748 tokens, 4224 -> 3952, fp32 (67 MB) 86.0 / 85.2 / 82.6.  (Y and dX, which the next call reads, lose 0.2-0.7 % that way.)
constexpr uint32_t kRowsOnceBytes = 24u << 20;
// A unit = 32 rows x UB blocks of 32 in-features, RBY bytes per row; a wave owns two unit-sized LDS slots.  The 16-byte
// chunks of a row are XOR-swizzled with (row >> 1) so that the 32 lanes of a quad read (32 rows, same chunk) spread
// over all banks (two rows share a chunk position: the 2-way conflict of an 8-byte access by 32 lanes is the minimum).
template <typename WT, int MI> struct DwStage {
    static constexpr int kEB = (int)sizeof(WT);
    static constexpr int UB = (8 / kEB) < MI ? (8 / kEB) : MI;       // blocks per unit: rows of at most 256 bytes
    static constexpr int RBY = UB * 32 * kEB;                         // 128 or 256
    static constexpr int CPR = RBY / 16, RPI = 64 / CPR, NIU = 32 / RPI;   // chunks per row, rows per instruction, instructions
    static constexpr int UNIT_BYTES = 32 * RBY;
    static constexpr int UPJ = MI / UB;                               // units per 32-row block column of the wave
    static_assert(MI % UB == 0 && RBY <= 256 && UNIT_BYTES == NIU * 1024, "unit geometry");
    // byte offset (inside a slot) of chunk 0 of this lane's row, with the row's swizzle and the lane's half folded in:
    // the 16-byte chunk c (bf16: the 8-byte half h of it) is at  lane_base ^ (c * 16)
    static __device__ __forceinline__ uint32_t lane_base(int lane)
    {
        const uint32_t ol = (uint32_t)lane & 31u, h = (uint32_t)lane >> 5, xo = ((ol >> 1) & (uint32_t)(CPR - 1)) << 4;
        return kEB == 2 ? (ol * RBY + 8u * h) | xo : (ol * RBY) | (xo ^ (h << 4));
    }
    // chunk of quad q of block ii of the unit (for fp32 the lane's half is a chunk of its own, folded into lane_base)
    static constexpr uint32_t quad_chunk_bytes(int ii, int q) { return (uint32_t)(kEB == 2 ? ii * 4 + q : ii * 8 + 2 * q) * 16u; }
};

template <typename WT> struct WQuad;     // four consecutive weights of one row, to and from LDS
template <> struct WQuad<bf16_t> {
    static __device__ __forceinline__ void read(const unsigned char *p, float (&v)[4])
    {
        const uintx2 u = *reinterpret_cast<const uintx2 *>(p);
        v[0] = __uint_as_float(u[0] << 16); v[1] = __uint_as_float(u[0] & 0xFFFF0000u);
        v[2] = __uint_as_float(u[1] << 16); v[3] = __uint_as_float(u[1] & 0xFFFF0000u);
    }
    static __device__ __forceinline__ void write(unsigned char *p, const float (&d)[4])
    {
        floatx2 lo, hi;
        lo[0] = d[0]; lo[1] = d[1]; hi[0] = d[2]; hi[1] = d[3];
        const bf16x2 a = __builtin_convertvector(lo, bf16x2), b = __builtin_convertvector(hi, bf16x2);   // one packed convert each
        uintx2 o;
        o[0] = __builtin_bit_cast(uint32_t, a); o[1] = __builtin_bit_cast(uint32_t, b);
        *reinterpret_cast<uintx2 *>(p) = o;
    }
};
template <> struct WQuad<float> {
    static __device__ __forceinline__ void read(const unsigned char *p, float (&v)[4])
    {
        const floatx4 u = *reinterpret_cast<const floatx4 *>(p);
        v[0] = u[0]; v[1] = u[1]; v[2] = u[2]; v[3] = u[3];
    }
    static __device__ __forceinline__ void write(unsigned char *p, const float (&d)[4])
    {
        *reinterpret_cast<floatx4 *>(p) = floatx4{d[0], d[1], d[2], d[3]};
    }
};

// K-major tiles ([k][COLS] bf16, filled by direct-to-LDS loads of 1 KB = kmRowsPerLoad rows each): in the operand layout
// of the 16x16x32 MFMA the two groups of sixteen lanes that the LDS serves together read the same 32 bytes of columns
// eight rows apart, and rows of 256 or 512 bytes all start on the same bank, so the two groups collided on every read
// (SQ_LDS_BANK_CONFLICT: 45 M cycles per launch at the 7B shapes).  Every eight rows are therefore followed by a gap of 32
// bytes: the second group's pieces land in the other half of each 64-byte unit (counter back to what the epilogue
// leaves, 1.6 M).  Gaps of 128 or 256 bytes do not help (the banks repeat every 256 bytes and the swizzle of the 64-byte
// units already uses all four positions), and swapping the halves by a swizzle of the columns reorders the 16-byte
// chunks that four neighbouring lanes fetch from memory, which costs far more than the conflicts did (-19 %).
template <int COLS> constexpr int kmRowsPerLoad = 64 / (COLS / 8);
constexpr int kmGapElems = 16;
template <int COLS> __host__ __device__ constexpr int km_row_elems(int k) { return k * COLS + (k >> 3) * kmGapElems; }
template <int COLS> constexpr int kmTileElems(int rows) { return rows * COLS + (rows / 8) * kmGapElems; }

// LDS the dW kernel asks for: the K loop's tile ring, or (Block-AP) the epilogue's stage plus the group-sum partials.
template <typename WT, bool BLOCK_AP, int BM, int BN, int BK, int NS, int WGM, int WGN>
constexpr size_t dw_stage_bytes()
{
    return BLOCK_AP ? (size_t)WGM * WGN * 2 * DwStage<WT, BM / WGM / 32>::UNIT_BYTES : 0;
}
template <typename WT, bool BLOCK_AP, int BM, int BN, int BK, int NS, int WGM, int WGN>
constexpr size_t dw_smem_bytes()
{
    const size_t ring = (size_t)NS * (kmTileElems<BM>(BK) + kmTileElems<BN>(BK)) * sizeof(bf16_t);
    const size_t epi = dw_stage_bytes<WT, BLOCK_AP, BM, BN, BK, NS, WGM, WGN>() + (size_t)2 * (BM / 32) * BN * sizeof(float);
    return ring > epi ? ring : epi;
}

// ---- KM tile filled by direct-to-LDS loads ------------------------------------------------------------------
// Tile [BK][COLS] bf16, rows unpadded.  A transpose read touches four consecutive k rows, 64 bytes of each, so
// the 64-byte units of a row are XOR-swizzled with (k & 3) to spread those rows over the banks.
template <int COLS>
__device__ __forceinline__ int km_swz_col(int k, int col) { return (((col >> 5) ^ (k & 3)) << 5) | (col & 31); }

// A fragment of the tile as an operand of v_mfma_f32_16x16x32_bf16: the lane holds column col0 + lane % 16 and the eight
// k values 32 ks + 8 (lane / 16) + 0 .. 7.  Every group of 16 lanes reads a patch of 4 k rows x 16 columns per instruction
// (the transpose read hands lane i of the group four k-consecutive values of column i).
template <int COLS>
__device__ __forceinline__ bf16x8 frag_km16_swz(const bf16_t *tile, int col0, int ks, int lane)
{
    const int i = lane & 15, b = lane >> 4;
    const int k = ks * 32 + b * 8 + (i >> 2), col = col0 + (i & 3) * 4;
    const int c = km_swz_col<COLS>(k, col);                                               // (k + 4) & 3 == k & 3
    typedef short4v __attribute__((address_space(3))) * lds_p;
    const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(tile + km_row_elems<COLS>(k) + c));
    const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(tile + km_row_elems<COLS>(k + 4) + c));
    typedef short short8v __attribute__((ext_vector_type(8)));
    short8v r = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, r);
}

// Streams consecutive [BK][COLS] row blocks of a row-major [rows][ld] bf16 matrix into LDS tiles, one direct-to-LDS
// instruction at a time (LOADS per wave and tile, RPI rows each).  Every instruction keeps its own running byte offset,
// so issuing one costs a scalar move to M0, the load and one add.  Columns past `ld` start at an out-of-range offset and
// advance like the others: tensors are smaller than 2 GiB, so 2 GiB plus any offset into one stays out of range (no
// wrap-around); rows past the end of the matrix fail the buffer's range check.
// RUNNING: the offsets stay such.  Left to itself the compiler keeps, for a loop of two tiles a trip, an offset for either tile and adds a scalar to them:
// twice the registers.
template <int BK, int COLS, int NW, bool RUNNING = false>
struct KmLoader {
    static constexpr int CPR = COLS / 8, RPI = kmRowsPerLoad<COLS>, LOADS = BK / RPI / NW;   // chunks per row, rows per instruction
    static_assert(BK % (RPI * NW) == 0 && CPR <= 64, "tile / wave mismatch");
    uint32_t off[LOADS], adv;                 // adv: bytes from one K tile to the next, the same for every lane
    __device__ __forceinline__ void init(int ld, int col0, int wave, int lane)
    {
#pragma unroll
        for (int it = 0; it < LOADS; ++it) {
            const int rb = (wave * LOADS + it) * RPI;                 // wave-uniform first row
            const int k = rb + lane / CPR, p = lane % CPR;
            const int col = col0 + (((p >> 2) ^ (k & 3)) << 5) + (p & 3) * 8;
            off[it] = col < ld ? ((uint32_t)k * (uint32_t)ld + (uint32_t)col) * 2u : kOobOffset;
        }
        adv = (uint32_t)BK * (uint32_t)ld * 2u;
    }
    // start n tiles further along K
    __device__ __forceinline__ void skip_tiles(int n)
    {
#pragma unroll
        for (int it = 0; it < LOADS; ++it) off[it] += (uint32_t)n * adv;
    }
    // instruction `it` of the next tile for this instruction slot; tile_lds = LDS address of the destination tile
    __device__ __forceinline__ void issue(const RawRsrc &r, int it, uint32_t tile_lds, int wave)
    {
        load_to_lds16_at(r, tile_lds + (uint32_t)(km_row_elems<COLS>((wave * LOADS + it) * RPI) * 2), off[it]);
        off[it] += adv;
        if constexpr (RUNNING) asm("" : "+v"(off[it]));
    }
};


// CUT: the grid is as large as the chip holds at once and a workgroup works through the items that a.sk deals it: whole
// tiles, and parts (along T) of tiles that it shares with others (ONE: item number `first` of them and no other) (see SkPlan; the accumulators of the parts meet in
// sk_hand_in, and the contributor that ends up with their sum runs the tile's epilogue).  Otherwise one tile per workgroup.
template <int BITS, typename WT, bool BLOCK_AP, int BM, int BN, int BK, int NS, int WGM, int WGN, bool CUT, bool ONE = !CUT>
__device__ __forceinline__ void gemm_dw_body(const GemmDwArgs &a, const int bid, const int grid, const int first = 0)
{
    constexpr int NT = 64 * WGM * WGN, NW = WGM * WGN, WTM = BM / WGM, WTN = BN / WGN, MI = WTM / 32, NI = WTN / 32;
    constexpr int A_ELEMS = kmTileElems<BM>(BK), B_ELEMS = kmTileElems<BN>(BK);      // with the gaps between the 1 KB pieces
    static_assert(NS >= 2, "at least two LDS stages");
    static_assert(NS * (A_ELEMS + B_ELEMS) * 2 >= 2 * (BM / 32) * BN * 4, "partials must fit in the tile buffers");

    want_agpr_accumulators<MI * NI * 16>();
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    bf16_t *sA = reinterpret_cast<bf16_t *>(smem_raw);            // [NS][A_ELEMS]
    bf16_t *sB = sA + NS * A_ELEMS;                               // [NS][B_ELEMS]

    int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave / WGN, wn = wave % WGN;
    const RawRsrc rX = make_raw_rsrc(a.X, a.x_bytes);
    const RawRsrc rY = make_raw_rsrc(a.dY, a.dy_bytes);
    const uint32_t ldsA = lds_addr_of(sA), ldsB = lds_addr_of(sB);

  for ([[maybe_unused]] int item = first;; ++item) {
    // What depends on the lane alone would otherwise be worked out once, in front of this loop, and kept in registers
    // through every phase of every item; the main loop has none to spare.
    if constexpr (CUT) asm volatile("" : "+v"(tid));
    int lane = tid & 63;
    int tm, tn;
    [[maybe_unused]] SkItem si;
    if constexpr (CUT) {
        if (!sk_item_of(a.sk, a.tiles_m * a.tiles_n, a.tiles_m, a.tiles_n, 8, bid, grid, item, si)) break;
        tm = si.tm; tn = si.tn;
    } else {
        // (bid < grid, the number of tiles: there is always one.  A return here would put the loads of the kernel's arguments behind its branch, one after
        // another: 155 tokens, 1920 -> 304, ds 8.15 us of kernel without, 8.45 with)
        (void)tile_of_xcd_slot(grid, bid & 7, bid >> 3, a.tiles_m, a.tiles_n, tm, tn, 8);
    }
    const int m0 = tm * BM, n0 = tn * BN;      // m0: first in-feature i, n0: first out-feature o
    // K tiles (of BK tokens) of this item: all of them, or the pairs [kb, ke) of a part (an even number of tiles, except
    // that the last pair of all may lack its second tile)
    int kt0 = 0, nk = (a.T + BK - 1) / BK;
    if constexpr (CUT) {
        kt0 = 2 * si.kb;
        nk = (2 * si.ke < nk ? 2 * si.ke : nk) - kt0;
    }
    // fp32 weights, whole tiles: the loop is two registers short, and each reload (a vector-memory operation) waits for all loads under way.  dW, ds and
    // dz, 3 bit, us so / with running offsets: 8192 tokens, 4096 x 4096 245 / 212; 1000 tokens, 11008 -> 4096 164 / 156; 2 bit 241 / 214 and 171 / 162.
    // (In the instantiation that cuts tiles running offsets cost 30 registers in scratch, in tiles of 128, which lack none, 3 %.)
    constexpr bool RUNNING = BLOCK_AP && sizeof(WT) == 4 && !CUT && BM == 256;
    KmLoader<BK, BM, NW, RUNNING> ldX;
    KmLoader<BK, BN, NW, RUNNING> ldY;
    ldX.init((int)a.I, m0, wave, lane);
    ldY.init((int)a.O, n0, wave, lane);
    if constexpr (CUT) { ldX.skip_tiles(kt0); ldY.skip_tiles(kt0); }
    constexpr int LA = decltype(ldX)::LOADS, LB = decltype(ldY)::LOADS, ND = LA + LB;
    // load number d (0 .. ND-1) of the NEXT K tile (tiles are fetched strictly in order) into LDS buffer `buf`
    auto issue_load = [&](int d, int buf) {
        if (d < LA) ldX.issue(rX, d, ldsA + (uint32_t)(buf * A_ELEMS * 2), wave);
        else ldY.issue(rY, d - LA, ldsB + (uint32_t)(buf * B_ELEMS * 2), wave);
    };
    auto load_tiles = [&](int buf) {
#pragma unroll
        for (int d = 0; d < ND; ++d) issue_load(d, buf);
    };

    floatx4 acc[MI][NI][4];      // [q] = registers 4 q .. 4 q + 3 of the block
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r >> 2][r & 3] = 0.0f;

    // The contraction runs on v_mfma_f32_16x16x32_bf16 (measured 4-7 % ahead of the 32x32x16 form in this loop, which
    // moves twice the accumulator registers per flop): the 32 x 32 block (i, j) of the wave is four 16 x 16 products, and
    // product (ii, jj) lives in acc[i][j][2 ii + jj] until the end of the K loop, where the blocks
    // are brought into the lane order of the 32 x 32 form that the epilogue is written for (see the start of the epilogue).
    // A K tile is KS slices of 32.  Per slice a wave needs MA = 2 MI fragments of X and NB = 2 NI of dY (4 registers
    // each).  The dY fragments are double-buffered; an X fragment is used by NB consecutive MFMAs only, so the fragment
    // of the next slice takes its registers as soon as those have been issued.
    constexpr int KS = BK / 32, MA = 2 * MI, NB = 2 * NI;
    static_assert(BK % 32 == 0 && KS >= 2 && MA >= NB, "slices of 32, at least two per tile; B fragments ride along with the first A fragments");
    bf16x8 fa[MA], fb[2][NB];
    auto frag_a = [&](int buf, int ks, int ia) { return frag_km16_swz<BM>(sA + buf * A_ELEMS, wm * WTM + ia * 16, ks, lane); };
    auto frag_b = [&](int buf, int ks, int jb) { return frag_km16_swz<BN>(sB + buf * B_ELEMS, wn * WTN + jb * 16, ks, lane); };
    auto mfma16 = [&](auto ia_, auto jb_, int pb) __attribute__((always_inline)) {
        constexpr int ia = decltype(ia_)::value, jb = decltype(jb_)::value;
        floatx4 &c = acc[ia >> 1][jb >> 1][(ia & 1) * 2 + (jb & 1)];
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[ia], fb[pb][jb], c, 0, 0, 0);
    };
    // One K tile.  Same pipeline as the forward kernel: the barrier sits before the last slice, whose MFMAs then cover
    // the first fragment reads of the next tile and the issue of the loads for a later tile.  The K tiles go round a ring
    // of NS LDS stages: behind the barrier of tile kt the stage of tile kt itself is free (its last fragments are in
    // registers) and takes tile kt + NS, so a load has NS - 1 tile times to land; the barrier waits only for the loads
    // of tile kt + 1 (vector-memory operations complete in order: "all but the newest (NS - 2) batches").
    // P = dY fragment buffer that holds slice 0 of this tile; slices alternate, so the next tile starts in (P + KS) & 1.
    auto step = [&](auto par, int buf, int nxt) __attribute__((always_inline)) {
        constexpr int P = decltype(par)::value;
        // MFMAs of X fragment ia, then, in their shadow, the fragments that replace it (and one dY fragment of the next
        // slice), from slice `ks_next` of stage `src`; in the last slice also one or two loads for tile kt + NS.
        auto run_slice = [&](auto pb_, auto last_, int src, int ks_next) __attribute__((always_inline)) {
            constexpr int pb = decltype(pb_)::value;
            constexpr bool last = decltype(last_)::value;
            static_for<MA>([&](auto ia_) __attribute__((always_inline)) {
                constexpr int ia = decltype(ia_)::value;
                static_for<NB>([&](auto jb_) __attribute__((always_inline)) { mfma16(ia_, jb_, pb); });
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (last) {
#pragma unroll
                    for (int d = 0; d < ND; ++d)
                        if (d * MA / ND == ia) issue_load(d, buf);
                }
                fa[ia] = frag_a(src, ks_next, ia);
                if constexpr (ia < NB) fb[pb ^ 1][ia] = frag_b(src, ks_next, ia);
                __builtin_amdgcn_sched_barrier(0);
            });
        };
        static_for<KS - 1>([&](auto ks_) __attribute__((always_inline)) {
            constexpr int ks = decltype(ks_)::value;
            run_slice(IC<((P + ks) & 1)>{}, IC<0>{}, buf, ks + 1);
        });
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((NS - 2) * ND));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        run_slice(IC<((P + KS - 1) & 1)>{}, IC<1>{}, nxt, 0);
    };

    if (nk > 0) {
#pragma unroll
        for (int st = 0; st < NS; ++st) load_tiles(st);            // tiles 0 .. NS-1 (past T: zeros)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((NS - 1) * ND));      // tile 0 has landed
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
#pragma unroll
        for (int jb = 0; jb < NB; ++jb) fb[0][jb] = frag_b(0, 0, jb);
#pragma unroll
        for (int ia = 0; ia < MA; ++ia) fa[ia] = frag_a(0, 0, ia);
        // Two tiles per trip, so that the fragment buffers alternate at compile time when a tile has an odd number of
        // slices; with an odd tile count the extra tile lies past T and multiplies zeros.
        int buf = 0;
        for (int kt = 0; kt < nk; kt += 2) {
            int nxt = buf + 1 == NS ? 0 : buf + 1;
            step(IC<0>{}, buf, nxt);
            buf = nxt; nxt = buf + 1 == NS ? 0 : buf + 1;
            step(IC<(KS & 1)>{}, buf, nxt);
            buf = nxt;
        }
    }
    wait_all_and_barrier();   // tile buffers become the partial-sum arrays
    if constexpr (CUT) {
        // a tile cut along T: only the contributor that ends up with the sum of all parts goes on to the epilogue
        asm volatile("" : "+v"(tid));
        if (si.parts > 1 && !sk_hand_in<MI, NI, NT, 4>(a.sk, si, acc, tid, bid, grid)) { if constexpr (ONE) break; else continue; }      // nothing else is alive here: four blocks at a time
    }
    // what the epilogue derives from the lane is worked out here, not in front of the K loop (see the top of the loop)
    asm volatile("" : "+v"(tid));
    lane = tid & 63;

    // ---- epilogue ----------------------------------------------------------------------------------
    using SG = DwStage<WT, MI>;
    constexpr uint32_t kStageBytes = (uint32_t)dw_stage_bytes<WT, BLOCK_AP, BM, BN, BK, NS, WGM, WGN>();
    float *p_ds = reinterpret_cast<float *>(smem_raw + kStageBytes);      // [BM/32][BN]
    float *p_dz = p_ds + (BM / 32) * BN;
    const __amdgpu_buffer_rsrc_t rC = make_rsrc(a.codes, a.codes_bytes);
    const __amdgpu_buffer_rsrc_t rS = make_rsrc(a.sz, a.sz_bytes);
    const __amdgpu_buffer_rsrc_t rB = make_rsrc(a.clampbits, a.clamp_bytes);
    const __amdgpu_buffer_rsrc_t rDW = make_rsrc(a.dW, a.dW != nullptr ? a.w_bytes : 0u);    // no dW wanted: stores dropped
    const RawRsrc rWraw = make_raw_rsrc(a.W, a.w_bytes);
    const uint32_t code_row_bytes = (uint32_t)a.I / 32u * (4u * WorkCodes<BITS>::kWords);
    const int h = lane >> 5;
    const int ibw = m0 + wm * WTM;                             // first in-feature of this wave

    // What a lane needs of its weight row for the MI blocks of one block column j, fetched with few, wide loads: the
    // codes and the clamp bits of the MI blocks lie side by side in memory.  (Blocks past the end of a row read what
    // follows, or zeros past the buffer; their accumulators and their W are zero, so whatever the codes are the sums
    // come out as zero, and nothing of such a block is stored.)
    constexpr int CODE_WORDS = MI * WorkCodes<BITS>::kWords, CODE_LOADS = (CODE_WORDS + 3) / 4;
    struct RowOps { uint32_t cw[CODE_LOADS * 4]; intx2 sv[MI]; uint32_t ncl[MI]; };
    auto load_row_ops = [&](int j, RowOps &r) {
        const int o = n0 + wn * WTN + j * 32 + (lane & 31);
        const bool row_ok = o < a.O && ibw < a.I;
        const uint32_t c0 = (uint32_t)o * code_row_bytes + (uint32_t)(ibw >> 5) * (4u * WorkCodes<BITS>::kWords);
#pragma unroll
        for (int q = 0; q < CODE_LOADS; ++q) {
            if constexpr (CODE_WORDS % 4 == 0) {
                const intx4 v = buf_load16(rC, row_ok ? c0 + 16u * q : kOobOffset);
                r.cw[4 * q] = v[0]; r.cw[4 * q + 1] = v[1]; r.cw[4 * q + 2] = v[2]; r.cw[4 * q + 3] = v[3];
            } else {
                static_assert(CODE_WORDS % 4 == 0 || CODE_WORDS == 2, "code words per wave row");
                const intx2 v = buf_load8(rC, row_ok ? c0 : kOobOffset);
                r.cw[0] = v[0]; r.cw[1] = v[1]; r.cw[2] = 0u; r.cw[3] = 0u;
            }
        }
        if constexpr (BLOCK_AP) {
            const uint32_t b0 = (uint32_t)o * (uint32_t)(a.I >> 3) + (uint32_t)(ibw >> 3);
            if constexpr (MI == 4) {
                const intx4 v = buf_load16(rB, row_ok ? b0 : kOobOffset);
                r.ncl[0] = v[0]; r.ncl[1] = v[1]; r.ncl[2] = v[2]; r.ncl[3] = v[3];
            } else if constexpr (MI == 2) {
                const intx2 v = buf_load8(rB, row_ok ? b0 : kOobOffset);
                r.ncl[0] = v[0]; r.ncl[1] = v[1];
            } else {
#pragma unroll
                for (int i = 0; i < MI; ++i) r.ncl[i] = (uint32_t)buf_load4(rB, row_ok ? b0 + 4u * i : kOobOffset);
            }
        }
        // (s, zbar) of each block's group: one load per group the wave's blocks touch (wave-uniform branches)
        int grp_prev = -1;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int ib = ibw + i * 32, grp = ib < a.I ? ib / a.g : -1 - i;
            if (i > 0 && grp == grp_prev) r.sv[i] = r.sv[i - 1];
            else r.sv[i] = buf_load8(rS, (o < a.O && ib < a.I) ? ((uint32_t)o * (uint32_t)a.G + (uint32_t)grp) * 8u : kOobOffset);
            grp_prev = grp;
        }
    };

    // W rows of unit u = (j, v): global byte offset of this lane's 16-byte chunk, per instruction
    auto unit_offsets = [&](int u, uint32_t (&off)[SG::NIU]) {
        const int j = u / SG::UPJ, v = u % SG::UPJ;
#pragma unroll
        for (int k = 0; k < SG::NIU; ++k) {
            const int r = k * SG::RPI + lane / SG::CPR, c = (lane % SG::CPR) ^ ((r >> 1) & (SG::CPR - 1));
            const int o = n0 + wn * WTN + j * 32 + r, i0 = ibw + v * SG::UB * 32 + c * (16 / SG::kEB);
            off[k] = (o < a.O && i0 < a.I) ? ((uint32_t)o * (uint32_t)a.I + (uint32_t)i0) * (uint32_t)SG::kEB : kOobOffset;
        }
    };
    const uint32_t stage_lds = lds_addr_of(smem_raw);
    auto slot_bytes = [&](int slot) { return (uint32_t)((wave * 2 + slot) * SG::UNIT_BYTES); };
    auto issue_unit = [&](int slot, const uint32_t (&off)[SG::NIU]) {
#pragma unroll
        for (int k = 0; k < SG::NIU; ++k) load_row_to_lds16_at(rWraw, stage_lds + slot_bytes(slot) + (uint32_t)(k * 1024), off[k], kRowsOnceBytes);
    };

    constexpr int NU = BLOCK_AP ? NI * SG::UPJ : 0;
    uint32_t goff[2][SG::NIU];
    if constexpr (BLOCK_AP) {
        // the first unit starts to stream in at once; the second follows below, a later one when its slot has been written out
        unit_offsets(0, goff[0]);
        issue_unit(0, goff[0]);
    }
    RowOps rops[2];
    load_row_ops(0, rops[0]);

    // ---- accumulators into the lane order of the 32 x 32 MFMA (while the loads above are under way) ----------------
    // From the K loop a lane holds, of block (i, j), product (ii, jj) in registers 4 (2 ii + jj) + b: row 16 ii +
    // 4 (lane / 16) + b, column 16 jj + lane % 16.  What follows wants register 4 q + b to be row 8 q + 4 (lane / 32) + b
    // of column lane % 32.  Rows 16 ii .. 16 ii + 15 are quads q = 2 ii and 2 ii + 1, so each half of a block is
    // converted by itself: every lane puts its two quads (16 bytes each) into a 2 KB patch of LDS that belongs to its
    // wave, [column][row quad] with the quad's place rotated by column / 4 against bank conflicts, and takes the two
    // quads it owns in the other order.  LDS accesses of a wave complete in order; nothing else touches the patch.
    {
        // Block-AP: the wave's second W slot, which is still empty; else the tile ring behind the partial sums
        const uint32_t patch = BLOCK_AP ? slot_bytes(1) : (uint32_t)(2 * (BM / 32) * BN * sizeof(float)) + (uint32_t)(wave * 2048);
        static_assert(BLOCK_AP ? SG::UNIT_BYTES >= 2048 : NS * (A_ELEMS + B_ELEMS) * 2 >= 2 * (BM / 32) * BN * 4 + NW * 2048, "room for the patch");
        const int c16 = lane & 15, rq_in = lane >> 4, c32 = lane & 31, h32 = lane >> 5;
        uint32_t at_in[2], at_out[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int col = 16 * t + c16, rq = 2 * t + h32;
            at_in[t] = patch + (uint32_t)(col * 64 + ((rq_in + (col >> 2)) & 3) * 16);
            at_out[t] = patch + (uint32_t)(c32 * 64 + ((rq + (c32 >> 2)) & 3) * 16);
        }
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) {
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        *reinterpret_cast<floatx4 *>(smem_raw + at_in[t]) = acc[i][j][2 * hh + t];
                    }
                    asm volatile("" ::: "memory");
                    __builtin_amdgcn_wave_barrier();
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        acc[i][j][2 * hh + t] = *reinterpret_cast<const floatx4 *>(smem_raw + at_out[t]);
                    }
                    asm volatile("" ::: "memory");
                    __builtin_amdgcn_wave_barrier();
                }
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);            // lgkmcnt(0): the patch has been read out, its place may take W rows
    asm volatile("" ::: "memory");
    if constexpr (NU > 1) {
        unit_offsets(1, goff[1]);
        issue_unit(1, goff[1]);
    }
    // The compiler does not see the loads into LDS: wait for them here.  The second unit was requested last and may
    // still be under way; its block column waits for it below.
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(NU > 1 ? SG::NIU : 0));
    asm volatile("" ::: "memory");
    const uint32_t lane_base = SG::lane_base(lane);

#pragma unroll
    for (int j = 0; j < NI; ++j) {
        const int ol = wn * WTN + j * 32 + (lane & 31), o = n0 + ol;
        if (j + 1 < NI) load_row_ops(j + 1, rops[(j + 1) & 1]);      // under this column's arithmetic
        const RowOps &ro = rops[j & 1];
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int ib = ibw + i * 32;                           // first of 32 in-features; whole block valid or not
            const bool valid = (o < a.O) && (ib < a.I);
            [[maybe_unused]] const int u = j * SG::UPJ + i / SG::UB, ii = i % SG::UB, slot = u & 1;
            if constexpr (BLOCK_AP) {
                if (ii == 0 && u >= 1) {       // requested after the first unit, or when its slot became free (below)
                    asm volatile("" ::: "memory");
                    __builtin_amdgcn_s_waitcnt(0x0070);
                    asm volatile("" ::: "memory");
                }
            }
            WorkCodes<BITS> cw;
#pragma unroll
            for (int k = 0; k < WorkCodes<BITS>::kWords; ++k) cw.w[k] = ro.cw[i * WorkCodes<BITS>::kWords + k];
            // this lane owns codes 8a + 4h + b (a, b in 0..3): four consecutive codes per a, h fields further along
            const uint32_t pre = (uint32_t)h * WorkCodes<BITS>::kField;
            uint32_t cq[4] = {cw.four(0, pre), cw.four(8, pre), cw.four(16, pre), cw.four(24, pre)};
            // keep the four masked words as they are: folded into one bit-field extract per code, the byte-to-float
            // conversions (v_cvt_f32_ubyte0..3, one instruction per code) would each need an extract in front
#pragma unroll
            for (int q = 0; q < 4; ++q) asm volatile("" : "+v"(cq[q]));
            const float s = __int_as_float(ro.sv[i][0]), zb = __int_as_float(ro.sv[i][1]);
            float sum_s = 0.0f, sum_z = 0.0f;
            if constexpr (BLOCK_AP) {
                // keep-bits: 1 where Eq.(1) did NOT clamp the weight
                const uint32_t ncl = ~(ro.ncl[i] >> (4 * h));
                const float rinv = valid ? 1.0f / s : 0.0f;
                const uint32_t quads = slot_bytes(slot) + lane_base;       // chunk bits are clear in slot_bytes
                // Per weight, with keep = all ones where it was not clamped (one bit-field extract) and bitwise ANDs
                // in place of selects:  du = D & keep (this is dW),  cs = (q - (w & keep) / s) - zbar, which is
                // r - w/s in range and r = q - zbar where clamped,  sum over clamped D = sum D - sum du.
                float sum_d = 0.0f, sum_u = 0.0f;
#define EQAT_ELEM(Q, B)                                                                                   \
    {                                                                                                     \
        const float d = acc[i][j][Q][B];                                                         \
        const uint32_t keep = (uint32_t)((int32_t)(ncl << (31 - ((Q) * 8 + (B)))) >> 31);                 \
        const float du = __uint_as_float(__float_as_uint(d) & keep);                                      \
        const float wm = __uint_as_float(__float_as_uint(wv[B]) & keep);                                  \
        const float cs = __builtin_fmaf(-wm, rinv, byte_to_float(cq[Q], B)) - zb;                         \
        sum_s = __builtin_fmaf(d, cs, sum_s);                                                             \
        sum_d += d;                                                                                       \
        sum_u += du;                                                                                      \
        dwv[B] = du;                                                                                      \
    }
#define EQAT_QUAD(Q)                                                                                      \
    {                                                                                                     \
        unsigned char *const cell = smem_raw + (quads ^ SG::quad_chunk_bytes(ii, (Q)));                   \
        float wv[4], dwv[4];                                                                              \
        WQuad<WT>::read(cell, wv);                                                                        \
        EQAT_ELEM(Q, 0) EQAT_ELEM(Q, 1) EQAT_ELEM(Q, 2) EQAT_ELEM(Q, 3)                                   \
        WQuad<WT>::write(cell, dwv);                                                                      \
    }
                EQAT_QUAD(0) EQAT_QUAD(1) EQAT_QUAD(2) EQAT_QUAD(3)
#undef EQAT_QUAD
#undef EQAT_ELEM
                sum_z = sum_d - sum_u;
            } else {
#define EQAT_ELEM(Q, B)                                                                                   \
    {                                                                                                     \
        const float d = acc[i][j][Q][B];                                                         \
        sum_s = __builtin_fmaf(d, byte_to_float(cq[Q], B) - zb, sum_s);                                   \
        sum_z += d;                                                                                       \
    }
#define EQAT_QUAD(Q) EQAT_ELEM(Q, 0) EQAT_ELEM(Q, 1) EQAT_ELEM(Q, 2) EQAT_ELEM(Q, 3)
                EQAT_QUAD(0) EQAT_QUAD(1) EQAT_QUAD(2) EQAT_QUAD(3)
#undef EQAT_QUAD
#undef EQAT_ELEM
            }
            sum_s += __shfl_xor(sum_s, 32);
            sum_z += __shfl_xor(sum_z, 32);
            if (h == 0) {
                p_ds[(wm * MI + i) * BN + ol] = sum_s;
                p_dz[(wm * MI + i) * BN + ol] = sum_z;
            }
            if constexpr (BLOCK_AP) {
                if (ii == SG::UB - 1) {
                    // The unit is complete: dW sits where W sat.  Rows go out the way they came in.  LDS accesses of a
                    // wave complete in order, so the reads below see the quads every lane of the wave has written.
                    asm volatile("" ::: "memory");
                    __builtin_amdgcn_wave_barrier();
#pragma unroll
                    for (int k = 0; k < SG::NIU; ++k) {
                        const intx4 v = *reinterpret_cast<const intx4 *>(smem_raw + slot_bytes(slot) + (uint32_t)(k * 1024 + lane * 16));
                        __builtin_amdgcn_raw_buffer_store_b128(v, rDW, (int)goff[slot][k], 0, kAuxOnce);
                    }
                    if (u + 2 < NU) {
                        asm volatile("" ::: "memory");
                        __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0): the slot has been read out
                        asm volatile("" ::: "memory");
                        unit_offsets(u + 2, goff[slot]);
                        issue_unit(slot, goff[slot]);
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);     // one 32x32 block at a time
        }
    }
    __syncthreads();
    if (a.direct) {
        // every group of this tile's rows is complete here: sum its g/32 block partials in order
        const int bpg = a.g >> 5, gpt = BM / a.g;
        for (int e = tid; e < gpt * BN; e += NT) {
            const int ol = e % BN, gi = e / BN, o = n0 + ol, i0 = m0 + gi * a.g;
            if (o >= a.O || i0 >= a.I) continue;
            float vs = 0.0f, vz = 0.0f;
            for (int k = 0; k < bpg; ++k) {
                vs += p_ds[(gi * bpg + k) * BN + ol];
                vz += p_dz[(gi * bpg + k) * BN + ol];
            }
            const size_t gidx = (size_t)o * a.G + i0 / a.g;
            if (a.ds != nullptr) a.ds[gidx] = vs;
            if (a.dz != nullptr) a.dz[gidx] = -a.sz[gidx][0] * vz;
        }
    } else {
        const int nb32 = a.I >> 5;
        for (int e = tid; e < (BM / 32) * BN; e += NT) {
            const int ol = e % BN, blk = e / BN, o = n0 + ol, i0 = m0 + blk * 32;
            if (o >= a.O || i0 >= a.I) continue;
            a.part_ds[(size_t)o * nb32 + (i0 >> 5)] = p_ds[blk * BN + ol];
            if (a.dz != nullptr) a.part_dz[(size_t)o * nb32 + (i0 >> 5)] = p_dz[blk * BN + ol];
        }
    }
    if constexpr (ONE) break;
    __syncthreads();          // the next item's tiles go where the sums were
  }
}

template <int BM_, int BN_, int BK_, int WGM_, int WGN_> struct Tile {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, WGM = WGM_, WGN = WGN_;
};
typedef Tile<128, 128, 64, 2, 2> TileSmall;   // 4 waves, 64x64 per wave: problems with few big tiles
typedef Tile<256, 256, 64, 2, 4> TileBig;     // 8 waves, 128x64 per wave
// dW: same output tiles.  The kernel takes any number of LDS stages NS and any K-tile width; measured, two stages of 64
// win: the big tile fits three stages only with 48-wide K tiles (3 x 48 KB), whose extra barriers cost what the deeper
// prefetch gains (-1 %); the small tile with three stages (96 KB) loses the second workgroup per CU (-17 %).
template <int BM_, int BN_, int BK_, int NS_, int WGM_, int WGN_> struct DwTile {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, NS = NS_, WGM = WGM_, WGN = WGN_;
};
typedef DwTile<128, 128, 64, 2, 2, 2> DwTileSmall;
typedef DwTile<256, 256, 64, 2, 2, 4> DwTileBig;
static_assert(DwTileSmall::BM == TileSmall::BM && DwTileBig::BM == TileBig::BM, "group-fits-in-tile tests use Tile*::BM");

template <bool BT, typename TS> constexpr size_t q_smem_bytes()
{
    constexpr int LDB = BT ? TS::BN + kPadKM : TS::BK + kPadKC;
    return 2 * (size_t)(TS::BM * TS::BK + (BT ? TS::BK * LDB : TS::BN * LDB)) * sizeof(bf16_t) + (size_t)TS::WGM * TS::WGN * kStoreStageBytes;
}
}  // namespace eqat
