// LDS tiles of the fwd / dX GEMMs and the fragments read from them: what the tile kernels and the split-contraction kernel share.
#pragma once
#include "common.h"

namespace eqat {

constexpr int kPadKC = 8;    // bf16 elements
constexpr int kPadKM = 32;
constexpr uint32_t kStoreStageBytes = 2048;   // per wave: one 32 x 32 bf16 block of the result on its way out

// ---- fragment reads ---------------------------------------------------------------------------------
// KC tile: lane l supplies row (l % 32), k = kk*16 + (l / 32) * 8 .. + 8
template <int LD>
__device__ __forceinline__ bf16x8 frag_kc(const bf16_t *tile, int row0, int kk, int lane)
{
    return *reinterpret_cast<const bf16x8 *>(tile + (row0 + (lane & 31)) * LD + kk * 16 + (lane >> 5) * 8);
}
// KM tile [k][n] (dX: What with K = O as the slow axis), rows padded by kPadKM.  The producer writes one 16-byte chunk
// per lane and instruction; the 8 (or 4) lanes that fill one row sit 64 bytes apart.  A 128-bit LDS store is served 8
// lanes per cycle over 32 four-byte banks (the model that reproduces the SQ_LDS_BANK_CONFLICT readings of every layout
// tried here: 24 extra cycles per store unswizzled, 8 with a swizzle that only separated lanes 4 apart, 0 for the
// forward kernel's [n][k] tile), so lanes 128 bytes apart in one row share their banks.  The four chunks of every
// 32-column block are therefore XOR-permuted with km_chunk_swz(k, block): blocks two apart, and the blocks that a
// second row of the same store cycle puts on the same banks, get different chunk positions.
__device__ __forceinline__ int km_chunk_swz(int k, int colblock) { return ((colblock >> 1) + 2 * (k & 1)) & 3; }

// The transpose read hands lane i (of each 16-lane block) four k-consecutive values of column i, gathered from the lanes
// that addressed rows k..k+3.  Block b = lane/16: columns 16*(b&1).., k half b>>1.
template <int LD>
__device__ __forceinline__ bf16x8 frag_km(const bf16_t *tile, int col0, int kk, int lane)
{
    const int i = lane & 15, b = lane >> 4;
    const int k = kk * 16 + (b >> 1) * 8 + (i >> 2), col = col0 + (b & 1) * 16 + (i & 3) * 4;
    const int pcol = (col & ~31) | ((((col >> 3) & 3) ^ km_chunk_swz(k, col >> 5)) << 3) | (col & 7);
    const bf16_t *p = tile + k * LD + pcol;
    typedef short4v __attribute__((address_space(3))) * lds_p;
    const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(p));
    const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(p + 4 * LD));      // (k + 4) & 3 == k & 3: same permutation
    typedef short short8v __attribute__((ext_vector_type(8)));
    short8v r = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, r);
}

// ---- KC tile filled by buffer loads that write LDS directly ----------------------------------------------
// Such a load puts the 16 bytes of lane j at (wave-uniform LDS base) + 16*j, so one instruction fills 8 rows of
// a [rows][64] bf16 tile and no padding can be placed inside it.  Bank conflicts of the fragment reads are
// avoided by a swizzle instead: the 16-byte chunk c of row r lives at position c ^ ((r >> 1) & 7); the
// permutation is applied on the global-address side, which is free.
__device__ __forceinline__ int kc_swz(int row, int chunk) { return chunk ^ ((row >> 1) & 7); }

__device__ __forceinline__ bf16x8 frag_kc_swz(const bf16_t *tile, int row0, int kk, int lane)
{
    const int r = row0 + (lane & 31);
    return *reinterpret_cast<const bf16x8 *>(tile + r * 64 + kc_swz(r, kk * 2 + (lane >> 5)) * 8);
}

constexpr int kAuxOnce = 2;              // "nt": past the caches
constexpr int kAuxDeviceScope = 16;      // "sc1" of the raw buffer intrinsics on gfx940 and later

}  // namespace eqat
