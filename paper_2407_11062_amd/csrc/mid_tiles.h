// Tiles of the kernels for few output tiles (gemm_mid.hip: forward, gemm_mid_dx.hip: dX): a workgroup of eight waves, 2 (64 weight rows each) x 4
// (a quarter of every K step each), computes 128 weight rows for a tile of tokens.
#pragma once
#include "common.h"

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
    float *pairs;                        // the launch of a prepared layer leaves the (s, z) pairs here; NULL: does not
};

constexpr int kMidBN = 128, kMidKG = 4, kMidNT = 512;

// Every XCD gets a contiguous range of tiles, token tiles of one weight tile next to each other: the codes are fetched into one
// L2 only.  With many token tiles that has every XCD read all of X for a weight tile or two: they are walked in bands instead.
__device__ __forceinline__ void tile_of(const MidArgs &a, int bm, uint32_t bid, uint32_t nb, int &m0, int &n0)
{
    const uint32_t xcd = bid & 7, rem = nb & 7;
    uint32_t pid = xcd * (nb >> 3) + (xcd < rem ? xcd : rem) + (bid >> 3), first = 0, rows = (uint32_t)a.tiles_m;
    if (a.band > 0) {
        const uint32_t band = (uint32_t)a.band, width = band * (uint32_t)a.tiles_n, which = pid / width;
        pid -= which * width;
        first = which * band;
        rows = rows - first < band ? rows - first : band;
    }
    m0 = (int)(first + pid % rows) * bm;
    n0 = (int)(pid / rows) * kMidBN;
}

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
// adds the four K quarters, in order, for the kg-th quarter of the tokens and stores 64 bytes of a row per 8 lanes.
template <int BM, uint32_t TOTAL>
__device__ __forceinline__ void store_sums(const MidArgs &a, const floatx16 (&acc)[2][BM / 32], unsigned char *smem_raw, int m0, int n0, int wave, int lane)
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
