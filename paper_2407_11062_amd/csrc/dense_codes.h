// Codes of the dense stream as MFMA operands: what the forward kernels that read the caller's packed arrays share.
#pragma once
#include "common.h"

namespace eqat {

// code index (0..31, within a segment) that sits in contraction slot m (0..7) of MFMA t (0..3) of the lane owning the segment
template <int BITS> __host__ __device__ constexpr int slot_code(int t, int m)
{
    if (BITS == 2) return 8 * t + 4 * (m % 2) + m / 2;
    return 8 * t + m;
}

// inverse of slot_code: position (8 t + m) of code c in the slot order of its segment
template <int BITS> __host__ __device__ constexpr int code_slot(int c)
{
    if (BITS == 2) { const int k = c % 8; return c - k + 2 * (k % 4) + k / 4; }
    return c;
}

template <int BITS> constexpr bool slot_maps_are_inverse()
{
    for (int c = 0; c < 32; ++c) {
        const int sl = code_slot<BITS>(c);
        if (sl < 0 || sl >= 32 || slot_code<BITS>(sl / 8, sl % 8) != c) return false;
    }
    return true;
}
static_assert(slot_maps_are_inverse<2>() && slot_maps_are_inverse<3>() && slot_maps_are_inverse<4>(), "slot order");

// twelve bits, i.e. four codes, of a 3-bit segment from bit BIT on
template <int BIT> __device__ __forceinline__ uint32_t twelve_at(const CodeWords<3> &c)
{
    constexpr int wi = BIT / 32, sh = BIT % 32;
    if constexpr (sh <= 20) return (c.w[wi] >> sh) & 0xFFFu;
    else return __builtin_amdgcn_alignbit(c.w[wi + 1], c.w[wi], sh) & 0xFFFu;
}
// four 3-bit codes to the four bytes of a register
__device__ __forceinline__ uint32_t spread_3bit(uint32_t x)
{
    const uint32_t pairs = (x | (x << 10)) & 0x003F003Fu;
    return (pairs | (pairs << 5)) & 0x07070707u;
}

// How 4-bit codes become floats: a field extract and a conversion per code; the masked words kept as words, a conversion per code (see WhatTable::four); or
// kept and converted two at a time (two_codes), fewest instructions and the fastest where arithmetic bounds a kernel.
enum CodeForm { kFields, kWords, kTwoCodes };
// the 8 weights of MFMA t of a segment, in slot order
template <int BITS, int T4, int CODES = kTwoCodes>
__device__ __forceinline__ bf16x8 eight_of(const WhatTable<BITS> &tab, const CodeWords<BITS> &c)
{
    uintx4 u;
    if constexpr (BITS == 2) {
        const uint32_t w = c.w[T4 / 2];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            uint32_t d0, d1;                       // the lookup of a word is shared by its two MFMAs
            tab.four((w >> (2 * k)) & 0x03030303u, d0, d1);
            u[k] = T4 % 2 ? d1 : d0;
        }
    } else if constexpr (BITS == 4) {
        uint32_t even = c.w[T4] & 0x0F0F0F0Fu, odd = (c.w[T4] >> 4) & 0x0F0F0F0Fu;
        if constexpr (CODES != kFields) {
            asm("" : "+v"(even));
            asm("" : "+v"(odd));
        }
        float e[4], o[4];
        if constexpr (CODES == kTwoCodes) {
            const floatx2 e01 = two_codes<false>(even), e23 = two_codes<true>(even), o01 = two_codes<false>(odd), o23 = two_codes<true>(odd);
            e[0] = e01[0]; e[1] = e01[1]; e[2] = e23[0]; e[3] = e23[1];
            o[0] = o01[0]; o[1] = o01[1]; o[2] = o23[0]; o[3] = o23[1];
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) { e[k] = byte_to_float(even, k); o[k] = byte_to_float(odd, k); }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            bf16x2 p;
            p[0] = (bf16_t)__builtin_fmaf(e[k], tab.s, tab.b);
            p[1] = (bf16_t)__builtin_fmaf(o[k], tab.s, tab.b);
            u[k] = __builtin_bit_cast(uint32_t, p);
        }
    } else {
        // four codes are 12 bits: pairs to the halves of a register, then codes to its bytes, five instructions in the place of
        // a field extract and an insert per code (one token, 3 bit: 5120 x 13824 18.3 -> 15.6 us, 28672 x 8192 31 -> 27 us)
        const uint32_t t0 = spread_3bit(twelve_at<24 * T4>(c)), t1 = spread_3bit(twelve_at<24 * T4 + 12>(c));
        uint32_t d0, d1;
        tab.four(t0, d0, d1); u[0] = d0; u[1] = d1;
        tab.four(t1, d0, d1); u[2] = d0; u[3] = d1;
    }
    return __builtin_bit_cast(bf16x8, u);
}

// Where the weights come from: the caller's dense stream with packed or with float zero points, or the working layout with
// (s, z) pairs that a workspace holds, or (a prepared layer) with step sizes and zero points as two arrays.  The contraction
// runs in the same order for all four, so the forward of a layer is bitwise the same whichever of them a call has.
constexpr int kPackedZ = 0, kFloatZ = 1, kWorking = 2, kPrepared = 3;
template <int SRC> constexpr bool kRelaid = SRC == kWorking || SRC == kPrepared;          // codes in the working layout
template <int SRC> constexpr bool kTwoFloats = SRC == kFloatZ || SRC == kPrepared;        // step sizes and zero points: an array of floats each

// eight consecutive values in slot order
template <int BITS> __device__ __forceinline__ bf16x8 slots_of(bf16x8 v)
{
    bf16x8 w;
#pragma unroll
    for (int m = 0; m < 8; ++m) w[m] = v[slot_code<BITS>(0, m)];
    return w;
}

// slot order back to eight consecutive values
template <int BITS> __device__ __forceinline__ bf16x8 unslot_of(bf16x8 v)
{
    bf16x8 w;
#pragma unroll
    for (int c = 0; c < 8; ++c) w[c] = v[code_slot<BITS>(c)];
    return w;
}

}  // namespace eqat
