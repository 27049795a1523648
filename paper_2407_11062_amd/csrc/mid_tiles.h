// Tiles of the kernels for few output tiles (gemm_mid.hip: forward, gemm_mid_dx.hip: dX): a workgroup of eight waves, 2 (64 weight rows each) x 4
// (a quarter of every K step each), computes 128 weight rows for a tile of tokens.
#pragma once
#include "common.h"
#include "gemm_tiles.h"

#include <hip/hip_runtime.h>

namespace eqat {

// Y[T,O] = X[T,I] * weights, I the contraction: the forward as it is; dX with dY as X, the out-features as I and the in-features as O.
struct MidArgs {
    const bf16_t *X; const uint32_t *codes; const float *s; const uint32_t *zp; const float *zf; bf16_t *Y;
    int T, I, O, G;
    int group;
    uint32_t spg_magic;            // ceil(2^32 / (g/32)), 0 for g = 32: group of a segment
    uint32_t code_row_bytes, z_row_words;
    uint32_t x_bytes, codes_bytes, s_bytes, z_bytes;
    int tiles_m, tiles_n, band;    // band: token tiles that an XCD walks together, 0: all of them
    // The tiles from number `whole` on, `shared` of them, are computed by `parts` workgroups each, a part of the contraction apiece (see share_sums).
    int whole, shared, parts;
    float *part_sums; unsigned long long *arrivals, launch;
    float *pairs;                        // the launch of a prepared layer leaves the (s, z) pairs here; NULL: does not
};

constexpr int kMidBN = 128, kMidKG = 4, kMidNT = 512;

// Every XCD gets a contiguous range of tiles, token tiles of one weight tile next to each other: the codes are fetched into one
// L2 only.  With many token tiles that has every XCD read all of X for a weight tile or two: they are walked in bands instead.
__device__ __forceinline__ uint32_t in_xcd_order(uint32_t bid, uint32_t nb)
{
    const uint32_t xcd = bid & 7, rem = nb & 7;
    return xcd * (nb >> 3) + (xcd < rem ? xcd : rem) + (bid >> 3);
}
__device__ __forceinline__ void place_of(const MidArgs &a, int bm, uint32_t pid, int &m0, int &n0)
{
    uint32_t first = 0, rows = (uint32_t)a.tiles_m;
    if (a.band > 0) {
        const uint32_t band = (uint32_t)a.band, width = band * (uint32_t)a.tiles_n, which = pid / width;
        pid -= which * width;
        first = which * band;
        rows = rows - first < band ? rows - first : band;
    }
    m0 = (int)(first + pid % rows) * bm;
    n0 = (int)(pid / rows) * kMidBN;
}
__device__ __forceinline__ void tile_of(const MidArgs &a, int bm, uint32_t bid, uint32_t nb, int &m0, int &n0) { place_of(a, bm, in_xcd_order(bid, nb), m0, n0); }

// A buffer that moves along K instead of the lanes' offsets into it: scalar work.  Past the last step nothing is in range.
struct Moving {
    uint64_t base; uint32_t left;
    __device__ __forceinline__ Moving(const void *p, uint32_t bytes) : base((uint64_t)p & 0xFFFFFFFFFFFFull), left(bytes) {}
    __device__ __forceinline__ void by(uint32_t n) { base += n; left -= n; }
    __device__ __forceinline__ RawRsrc at(bool live) const
    {
        RawRsrc r;
        r.w[0] = (int)(uint32_t)base; r.w[1] = (int)(uint32_t)(base >> 32); r.w[2] = live ? (int)left : 0; r.w[3] = 0x00020000;
        return r;
    }
};

// Sums of the four K quarters: acc[b][i][q] is row 8 (q / 4) + 4 h + q % 4 of block b, token 32 i + r.  One 32-row block of every wave
// at a time passes through LDS as [wave][token][32 rows] (the 16-byte chunk c of a token at c ^ (token & 7)); wave (wn, kg) then
// adds the four K quarters, in order, for the kg-th quarter of the tokens.  take(b, k, sum): four rows of block b for token 8 k + lane / 8 of that quarter.
template <int BM, uint32_t TOTAL, typename F>
__device__ __forceinline__ void quarter_sums(const floatx16 (&acc)[2][BM / 32], unsigned char *smem_raw, int wave, int lane, F &&take)
{
    const int wn = wave & 1, kg = wave >> 1, r = lane & 31, h = lane >> 5;
    constexpr uint32_t WAVE_BYTES = BM * 32 * 4;
    static_assert(8 * WAVE_BYTES <= TOTAL, "the sums go where the tiles were");
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < BM / 32; ++i)
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
            take(b, k, sum);
        }
    }
}
// 64 bytes of a row per 8 lanes
template <int BM> __device__ __forceinline__ void store_four(const MidArgs &a, int m0, int n0, int wave, int lane, int b, int k, const floatx4 &sum)
{
    const int tok = (wave >> 1) * (BM / 4) + k * 8 + (lane >> 3), o = n0 + (wave & 1) * 64 + b * 32 + (lane & 7) * 4;
    if (m0 + tok < a.T && o < a.O) {           // O is a multiple of 8
        bf16x4 y;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = (bf16_t)sum[e];
        *reinterpret_cast<bf16x4 *>(a.Y + (size_t)(m0 + tok) * a.O + o) = y;
    }
}
template <int BM, uint32_t TOTAL>
__device__ __forceinline__ void store_sums(const MidArgs &a, const floatx16 (&acc)[2][BM / 32], unsigned char *smem_raw, int m0, int n0, int wave, int lane)
{
    quarter_sums<BM, TOTAL>(acc, smem_raw, wave, lane, [&](int b, int k, const floatx4 &sum) { store_four<BM>(a, m0, n0, wave, lane, b, k, sum); });
}

// The same for one part of a shared tile.  The workgroup that arrived last, which is counted at its start, keeps its sums, adds the others' parts to them,
// all in the order of the parts, and stores the tile; the others write theirs and leave.  It waits only for workgroups that are running already, and they
// wait for nobody.  Parts and arrivals are written and read at device scope (the contributors may sit on different XCDs).
// The word that counts arrivals (bits 0..3) and parts written (4..7) lies in the caller's workspace and may hold anything before the first arrival: it
// counts for this launch only where its upper 56 bits are the launch's number, and the last to arrive clears it, so that a graph may replay the launch
// under the same number.
constexpr int kMidMaxParts = 4;
constexpr int kMidSpinLimit = 1 << 22;      // polls: a bound that is never reached
// by one lane; true in the last one
__device__ __forceinline__ bool arrive(const MidArgs &a, int tile)
{
    unsigned long long *const word = a.arrivals + tile;
    unsigned long long seen = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), next;
    do next = (seen & ~0xFFull) == a.launch ? seen + 1 : a.launch + 1;
    while (!__hip_atomic_compare_exchange_strong(word, &seen, next, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    return (int)(next & 0xF) == a.parts;
}
template <int BM, uint32_t TOTAL>
__device__ __forceinline__ void share_sums(const MidArgs &a, const floatx16 (&acc)[2][BM / 32], unsigned char *smem_raw, int m0, int n0, int wave, int lane, int tile, int part,
                                           const uint32_t &s_last)
{
    constexpr uint32_t kPart = BM * kMidBN * 4;
    constexpr int NK = BM / 4 / 8;
    const uint32_t at = (uint32_t)(wave * 64 + lane) * 16u;
    unsigned long long *const word = a.arrivals + tile;
    const bool first_lane = wave == 0 && lane == 0;
    floatx4 own[2 * NK];
    quarter_sums<BM, TOTAL>(acc, smem_raw, wave, lane, [&](int b, int k, const floatx4 &sum) { own[b * NK + k] = sum; });       // (a barrier and more)
    if (s_last == 0u) {
        const __amdgpu_buffer_rsrc_t mine = make_rsrc(a.part_sums + (size_t)(part * a.shared + tile) * (kPart / 4), kPart);
#pragma unroll
        for (int q = 0; q < 2 * NK; ++q)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(intx4, own[q]), mine, (int)(at + (uint32_t)q * (kMidNT * 16u)), 0, kAuxDeviceScope);
        wait_all_and_barrier();             // every store of the workgroup has completed
        if (first_lane) __hip_atomic_fetch_add(word, 0x10ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    if (first_lane) {
        const unsigned long long all = a.launch + (unsigned long long)(a.parts + (a.parts - 1) * 16);
        for (int polls = 0; polls < kMidSpinLimit && __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != all; ++polls) __builtin_amdgcn_s_sleep(1);
        __hip_atomic_store(word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    intx4 v[kMidMaxParts][2 * NK];
#pragma unroll
    for (int p = 0; p < kMidMaxParts; ++p) {          // its own place, and past the last part: nothing is in range (zeros)
        const bool there = p < a.parts && p != part;
        const __amdgpu_buffer_rsrc_t r = make_rsrc(a.part_sums + (size_t)(there ? p * a.shared + tile : 0) * (kPart / 4), there ? kPart : 0u);
#pragma unroll
        for (int q = 0; q < 2 * NK; ++q) v[p][q] = __builtin_amdgcn_raw_buffer_load_b128(r, (int)(at + (uint32_t)q * (kMidNT * 16u)), 0, kAuxDeviceScope);
    }
#pragma unroll
    for (int q = 0; q < 2 * NK; ++q) {
        floatx4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int p = 0; p < kMidMaxParts; ++p)
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] += p == part ? own[q][e] : __int_as_float(v[p][q][e]);
        store_four<BM>(a, m0, n0, wave, lane, q / NK, q % NK, sum);
    }
}

// Token tiles of a band, where the column is longer than 20 of them: an XCD holds 32 tiles at a time, and a panel of 64 tokens
// is 4 to 8 times as heavy as one of codes, so that 4 x 8 of them (3 x 10 with taller tiles) read the least.
// 2048 tokens, 11008 -> 1024, 2 bit: 76 us in columns, 53 in bands; 1536 tokens 65 and 47; 2048 tokens, 5504 -> 2560: 80 and 70.  With
// shorter columns the codes, which two XCDs then fetch, weigh more: 300 tokens, 4096 -> 8192 30 us in columns, 33 in bands.
inline int band_of(int tiles_m, int bm)
{
    if (tiles_m <= 20) return 0;
    const int most = bm == 64 ? 4 : 3, bands = (tiles_m + most - 1) / most;
    return (tiles_m + bands - 1) / bands;                             // of equal height
}

}  // namespace eqat
